// 3x3x3 convolution for the tensors the bf16 matrix-core kernels do not take -- fp32, and bf16 with
// channel counts that are no multiple of 16 -- on v_mfma_f32_16x16x4_f32: forward, backward-data and
// backward-weight for any channel counts, fp32 products and fp32 accumulation.
//
// Bound: a 16x16x4 instruction occupies the matrix core for 32 clocks and needs one 4-byte
// operand word per lane and side, so neither LDS nor L2 can be the limit; what counts is that
// every CU has several workgroups and that staging overlaps the multiplication.  The
// thread-per-output kernels these replace needed two loads per multiply-add and ran at 1.5 TFLOP/s.
#include "common.h"
#include "conv_internal.h"
#include "index_math.h"
#include "quad_io.h"

#include <type_traits>

namespace k3 {

// voxel offsets inside a tile: with descriptors its span is below 2 GiB, without them it may be anything
template <bool BUF> using TileOff = std::conditional_t<BUF, int, int64_t>;

template <typename T>
struct GenConv {
    const T *src1, *src2, *mask;   // mask: ReLU mask of src1 (backward-data; then there is no src2)
    int c1, c2;                        // contraction channels per source
    const T *w;                        // canonical [27][cin][cout]
    const float *bias;
    int relu;
    T *dst1, *dst2;
    const T *omask;                   // optional: dst1 is zeroed where omask <= 0
    int cd1, cd2;                      // output channels per destination
    int N, D, H, W;
    int ntd, nth, ntw, ncb;            // tiles per axis, output-channel groups
    int64_t total, per_xcd;
    bool vout;                         // outputs (and omask) are accessed as quads
};

// Four consecutive channels ch .. ch+3 of voxel v of the concatenation [p1 | p2]; zero beyond it.
template <typename T>
__device__ __forceinline__ f32x4 load_quad(const T *p1, const T *p2, int c1, int c2, int64_t v, int ch)
{
    f32x4 q;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int c = ch + j;
        q[j] = c < c1 ? elem<T>::ld(p1 + v * c1 + c) : c < c1 + c2 ? elem<T>::ld(p2 + v * c2 + (c - c1)) : 0.f;
    }
    return q;
}

// The same for channel counts in whole quads, through descriptors that start at the first voxel of
// a tile: vo = the voxel's offset from there, or negative where it lies outside the volume (the load
// then returns zeros: no branch, no select).  ch0: first channel of the chunk, span its width, q
// the lane's quad of it.  A chunk that straddles the two sources is read from both, each lane from one.
struct QuadSrc { __amdgpu_buffer_rsrc_t r1, r2; };
template <typename T>
__device__ __forceinline__ f32x4 load_quad_buf(const QuadSrc &s, int c1, int c2, int vo, int ch0, int span, int q)
{
    const int ch = ch0 + q * 4;
    if (ch0 + span <= c1 || c2 == 0) return buf<T>::quad(s.r1, vo < 0 || ch >= c1 ? -1 : vo * c1 + ch, 0);
    f32x4 v = buf<T>::quad(s.r2, vo < 0 || ch < c1 || ch >= c1 + c2 ? -1 : vo * c2 + ch - c1, 0);
    if (ch0 < c1)
        v = __builtin_bit_cast(f32x4, __builtin_bit_cast(u32x4_t, v) |
                                      __builtin_bit_cast(u32x4_t, buf<T>::quad(s.r1, vo < 0 || ch >= c1 ? -1 : vo * c1 + ch, 0)));
    return v;
}

// GEMM D[output channel][voxel] = sum over (tap, channel); A = weights, B = activations.  A lane
// group of 16 lanes carries one 16-byte slot (4 channels of one tap) of a step, and the step's four
// matrix instructions take channel 0..3 of the slot: the contraction order is permuted alike on
// both sides.  S = slots per voxel and chunk (4: 16 channels and a step is a tap; 2 and 1: the 8 or
// 4 channels of a narrow layer, and a step covers two or four taps, so narrow inputs cost no
// padding).  The halo tile of a chunk sits in LDS (pitch of an odd number of slots at S = 4: the 16
// lanes of a group then hit 16 different bank quads), the next chunk's in registers; weights come
// straight from global memory (L2: a step multiplies for 128 clocks or more per fragment).
// WN waves share the tile's voxels, the other factor of 4 splits the steps: volumes too small to
// give each CU a 128-voxel tile take 32-voxel tiles whose four waves split the contraction and add
// their sums through LDS in a fixed order.
// One output block takes 128 registers, so that four workgroups share a CU: 16 -> 16 channels at 48^3
// (864 workgroups, of which 768 fitted before and the rest ran alone) 27.2 -> 24.5 us.
// BUF: tensors and weights are read through buffer descriptors (channel counts in whole quads on quad
// boundaries, a tile's span below 2 GiB); else element by element.
template <typename T, int TD, int TH, int TW, int WN, int S, int MB, bool BWD, bool BUF>
__global__ __launch_bounds__(256, !BUF ? 2 : MB == 1 ? 4 : 3) void conv_general_kernel(GenConv<T> p)
{
    constexpr int HD = TD + 2, HH = TH + 2, HW = TW + 2, NHALO = HD * HH * HW;
    constexpr int PITCH = S == 4 ? 20 : S == 2 ? 12 : 4;        // floats per halo voxel
    constexpr int WK = 4 / WN, NBLK = TD * TH * TW / 16, NB = NBLK / WN;
    constexpr int NSTEP = (27 * S + 3) / 4, ITEMS = (NHALO * S + 255) / 256;
    constexpr int RED = WK > 1 ? 4 * NBLK * MB * 256 : 0;
    __shared__ __attribute__((aligned(16))) float xs[NHALO * PITCH > RED ? NHALO * PITCH : RED];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int wn = wv % WN, wk = wv / WN;
    const int K = p.c1 + p.c2, M = p.cd1 + p.cd2;

    // consecutive workgroup ids go round the 8 XCDs: give each XCD a contiguous run of the logical
    // order, in which the channel groups of a tile are neighbours (they share its halo in the L2)
    const int64_t logical = (int64_t)(blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (logical >= p.total) return;
    const int cb = (int)(logical % p.ncb);
    int64_t t = logical / p.ncb;
    const int w0 = (int)(t % p.ntw) * TW;
    t /= p.ntw;
    const int h0 = (int)(t % p.nth) * TH;
    t /= p.nth;
    const int d0 = (int)(t % p.ntd) * TD;
    const int n = (int)(t / p.ntd);
    const int m0 = cb * 16 * MB;

    // the lane's halo items: (voxel, quad) i = tid + 256 k; offset of the voxel from the halo tile's
    // first one, negative outside the volume
    TileOff<BUF> vo[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int vox = (tid + k * 256) / S;
        const int lw = vox % HW, lh = (vox / HW) % HH, ld = vox / (HW * HH);
        const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
        vo[k] = vox < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W ? tile_offset<TileOff<BUF>>(ld, lh, lw, p.H, p.W) : -1;
    }
    const int64_t halo0 = (((int64_t)n * p.D + d0 - 1) * p.H + h0 - 1) * p.W + w0 - 1;
    const QuadSrc xsrc = {rsrc_of(p.src1 + halo0 * p.c1, 0x7ffffff0), rsrc_of((p.src2 ? p.src2 : p.src1) + halo0 * p.c2, 0x7ffffff0)};
    const QuadSrc msrc = {rsrc_of((p.mask ? p.mask : p.src1) + halo0 * p.c1, 0x7ffffff0), xsrc.r2};

    f32x4 st[ITEMS];
    auto fetch = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int q = (tid + k * 256) % S;
            if constexpr (BUF) {
                st[k] = load_quad_buf<T>(xsrc, p.c1, p.c2, vo[k], c * 4 * S, 4 * S, q);
                if (p.mask) st[k] = keep_positive(st[k], load_quad_buf<T>(msrc, p.c1, 0, vo[k], c * 4 * S, 4 * S, q));
            } else {
                st[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (vo[k] >= 0) {
                    const int ch = c * 4 * S + q * 4;
                    st[k] = load_quad(p.src1, p.src2, p.c1, p.c2, halo0 + vo[k], ch);
                    if (p.mask) st[k] = keep_positive(st[k], load_quad<T>(p.mask, nullptr, p.c1, 0, halo0 + vo[k], ch));
                }
            }
        }
    };
    // Weights of step s: the lane (row ln, slot kg) takes the four channels of its slot.  Rows and
    // channels beyond the layer's get a lane offset outside the descriptor's range and read as zero, as
    // do taps where a lane's offset holds the tap; where the tap is in the scalar offset it is clamped
    // (without a descriptor: all are read from a clamped place and replaced).
    const __amdgpu_buffer_rsrc_t wrsrc = rsrc_of(p.w, BUF ? 27 * K * M * (int)sizeof(T) : 0);
    int lo[MB][4];               // element offset inside a tap, per chunk
    bool keep[MB][4];
    auto weights_chunk = [&](int c, int ln, int kg) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + mb * 16 + ln, mc = m < M ? m : M - 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = c * 4 * S + (S == 4 ? kg : kg % S) * 4 + j, kc = k < K ? k : K - 1;
                keep[mb][j] = m < M && k < K;
                lo[mb][j] = BUF && !keep[mb][j] ? -1 : BWD ? mc * K + kc : kc * M + mc;
            }
        }
    };
    auto weights = [&](int s, float (&a)[MB][4]) __attribute__((always_inline)) {
        const int tap = general_tap(S, s, kg);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if constexpr (BUF) {
                // a step that is one tap has a wave-uniform offset, else the lane's own is added
                const int toff = (BWD ? 26 - tap : tap) * K * M;
                const int soff = general_weight_soff<int>(S, s, BWD, K, M, (int)sizeof(T));
                auto at = [&](int o) __attribute__((always_inline)) { return S == 4 ? o : o < 0 || tap > 26 ? -1 : o + toff; };
                if constexpr (BWD) {   // the contraction runs along the fastest axis: one load
                    const f32x4 v = buf<T>::quad(wrsrc, at(lo[mb][0]), soff);
                    a[mb][0] = v[0]; a[mb][1] = v[1]; a[mb][2] = v[2]; a[mb][3] = v[3];
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) a[mb][j] = buf<T>::one(wrsrc, at(lo[mb][j]), soff);
                }
            } else {
                const int tc = tap < 27 ? tap : 26;
                const T *wt = p.w + (int64_t)(BWD ? 26 - tc : tc) * K * M;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float v = elem<T>::ld(wt + lo[mb][j]);
                    a[mb][j] = keep[mb][j] && tap < 27 ? v : 0.f;
                }
            }
        }
    };
    int vb[NB];   // LDS index of the lane's voxel in each 16-voxel block, tap (0,0,0)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int i = (wn * NB + b) * 16 + ln;
        vb[b] = (((i / (TW * TH)) * HH + (i / TW) % TH) * HW + i % TW) * PITCH;
    }
    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[b][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int nchunk = (K + 4 * S - 1) / (4 * S);
    constexpr int MYSTEPS = (NSTEP + WK - 1) / WK, AHEAD = 2;   // weights travel this many steps ahead
    fetch(0);
    for (int c = 0; c < nchunk; ++c) {
        if (c > 0) __syncthreads();   // every wave is done with the chunk before
        int tl = tid;
        asm("" : "+v"(tl));           // addresses are worked out anew for each chunk: kept across the steps they cost the occupancy
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int i = tl + k * 256;
            if (i < NHALO * S) *reinterpret_cast<f32x4 *>(xs + (i / S) * PITCH + (i % S) * 4) = st[k];
        }
        float a[AHEAD + 1][MB][4];
        weights_chunk(c, tl & 15, (tl & 63) >> 4);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) weights(i * WK + wk, a[i]);
        if (c + 1 < nchunk) fetch(c + 1);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < MYSTEPS; ++i) {
            const int s = i * WK + wk;
            if (NSTEP % WK != 0 && i == MYSTEPS - 1 && s >= NSTEP) break;      // wave-uniform
            if (i + AHEAD < MYSTEPS) weights(s + AHEAD * WK, a[(i + AHEAD) % (AHEAD + 1)]);
            const int q = 4 * s + kg, tap = S == 4 ? s : (q / S < 27 ? q / S : 26), sl = S == 4 ? kg : q % S;
            const int off = ((tap / 9) * HH + (tap / 3) % 3) * HW * PITCH + (tap % 3) * PITCH + sl * 4;
            f32x4 x[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                x[b] = *reinterpret_cast<const f32x4 *>(xs + vb[b] + off);
                // slots behind the last tap: zeros on both sides, or an infinite input would make them NaN
                if (S < 4 && i == MYSTEPS - 1 && q >= 27 * S) x[b] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[b][mb] = mfma_f32(a[i % (AHEAD + 1)][mb][j], x[b][j], acc[b][mb]);
            __builtin_amdgcn_sched_barrier(0);   // no further ahead: hoisted loads cost the occupancy
        }
    }

    // a lane holds output channels m .. m+3 of one voxel of a block
    auto emit = [&](int blk, int mb, f32x4 v) __attribute__((always_inline)) {
        const int i = blk * 16 + ln;
        const int gd = d0 + i / (TW * TH), gh = h0 + (i / TW) % TH, gw = w0 + i % TW;
        const int m = m0 + mb * 16 + kg * 4;
        if (gd >= p.D || gh >= p.H || gw >= p.W || m >= M) return;
        const int64_t vox = (((int64_t)n * p.D + gd) * p.H + gh) * p.W + gw;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float x = v[r] + (p.bias && m + r < M ? p.bias[m + r] : 0.f);
            v[r] = (p.relu && !(x > 0.f)) ? 0.f : x;
        }
        if (p.vout) {
            const bool d1 = m < p.cd1;
            const int64_t o = d1 ? vox * p.cd1 + m : vox * p.cd2 + (m - p.cd1);
            if (d1 && p.omask) v = keep_positive(v, buf<T>::ld4(p.omask + o));
            buf<T>::st4((d1 ? p.dst1 : p.dst2) + o, v);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int mm = m + r;
                if (mm < p.cd1) {
                    const int64_t o = vox * p.cd1 + mm;
                    elem<T>::st(p.dst1 + o, p.omask && !(elem<T>::ld(p.omask + o) > 0.f) ? 0.f : v[r]);
                } else if (mm < M) {
                    elem<T>::st(p.dst2 + vox * p.cd2 + (mm - p.cd1), v[r]);
                }
            }
        }
    };
    if constexpr (WK == 1) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) emit(wn * NB + b, mb, acc[b][mb]);
    } else {
        static_assert(WN == 1 || WK == 1, "the waves split either the voxels or the contraction");
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4 *>(xs + (((wv * NBLK + b) * MB + mb) * 64 + lane) * 4) = acc[b][mb];
        __syncthreads();
        for (int q = wv; q < NBLK * MB; q += 4) {
            f32x4 s = *reinterpret_cast<const f32x4 *>(xs + (q * 64 + lane) * 4);
#pragma unroll
            for (int k = 1; k < 4; ++k) s += *reinterpret_cast<const f32x4 *>(xs + ((k * NBLK * MB + q) * 64 + lane) * 4);
            emit(q / MB, q % MB, s);
        }
    }
}

template <typename T, int TD, int TH, int TW, int WN, int S, int MB, bool BWD, bool BUF>
static int launch_general(GenConv<T> p, hipStream_t st)
{
    p.ntd = (p.D + TD - 1) / TD;
    p.nth = (p.H + TH - 1) / TH;
    p.ntw = (p.W + TW - 1) / TW;
    p.ncb = (p.cd1 + p.cd2 + 16 * MB - 1) / (16 * MB);
    p.total = (int64_t)p.N * p.ntd * p.nth * p.ntw * p.ncb;
    p.per_xcd = (p.total + 7) / 8;
    if (p.per_xcd * 8 > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    conv_general_kernel<T, TD, TH, TW, WN, S, MB, BWD, BUF><<<dim3((unsigned)(p.per_xcd * 8)), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

static uintptr_t bits(const void *p) { return (uintptr_t)p; }

// 128-voxel tiles with two output blocks per workgroup where that gives every CU one, else with
// one, else 32-voxel tiles (16 -> 16 channels at 12^3: 27 workgroups of the large kind)
template <typename T, int S, bool BWD>
static int launch_general_size(GenConv<T> p, hipStream_t st)
{
    const int64_t M = p.cd1 + p.cd2, K = p.c1 + p.c2, C = K > M ? K : M;
    const int64_t big = (int64_t)p.N * ((p.D + 3) / 4) * ((p.H + 3) / 4) * ((p.W + 7) / 8);
    // (of the weights only backward-data reads quads)
    const bool buf = whole_quads(p.c1 | p.c2, bits(p.src1) | bits(p.src2) | bits(p.mask) | (BWD ? bits(p.w) : 0), sizeof(T)) &&
                     6 * (int64_t)(p.H + 1) * p.W * C * 4 < 0x7fffffffLL && 27 * K * M * 4 < 0x7fffffffLL;
    p.vout = whole_quads(p.cd1 | p.cd2, bits(p.dst1) | bits(p.dst2) | bits(p.omask), sizeof(T));
    if (!buf) return launch_general<T, 4, 4, 8, 4, S, 1, BWD, false>(p, st);
    if (M > 16 && big * ((M + 31) / 32) >= 256) return launch_general<T, 4, 4, 8, 4, S, 2, BWD, true>(p, st);
    if (big * ((M + 15) / 16) >= 256) return launch_general<T, 4, 4, 8, 4, S, 1, BWD, true>(p, st);
    return launch_general<T, 2, 4, 4, 1, S, 1, BWD, true>(p, st);
}

template <typename T, bool BWD>
static int launch_general_any(const GenConv<T> &p, hipStream_t st)
{
    const int K = p.c1 + p.c2;
    if (K <= 4) return launch_general_size<T, 1, BWD>(p, st);
    if (K <= 8) return launch_general_size<T, 2, BWD>(p, st);
    return launch_general_size<T, 4, BWD>(p, st);
}

template <typename T>
static int fwd_general_t(const ConvArgs &a, hipStream_t st)
{
    GenConv<T> p{};
    p.src1 = (const T *)a.x; p.src2 = (const T *)a.x2;
    p.c1 = (int)a.c1; p.c2 = (int)a.c2;
    p.w = (const T *)a.w; p.bias = a.bias; p.relu = a.relu;
    p.dst1 = (T *)a.y; p.cd1 = (int)a.cout;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    return launch_general_any<T, false>(p, st);
}
int conv_fwd_general(const ConvArgs &a, hipStream_t st) { return a.dtype == K3_F32 ? fwd_general_t<float>(a, st) : fwd_general_t<bf16_t>(a, st); }

template <typename T>
static int dgrad_general_t(const ConvArgs &a, hipStream_t st)
{
    GenConv<T> p{};
    p.src1 = (const T *)a.dy; p.mask = (const T *)a.ymask;
    p.c1 = (int)a.cout;
    p.w = (const T *)a.w;
    p.dst1 = (T *)a.dx; p.dst2 = (T *)a.dx2; p.omask = (const T *)a.omask;
    p.cd1 = (int)a.c1; p.cd2 = (int)a.c2;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    return launch_general_any<T, true>(p, st);
}
int conv_dgrad_general(const ConvArgs &a, hipStream_t st) { return a.dtype == K3_F32 ? dgrad_general_t<float>(a, st) : dgrad_general_t<bf16_t>(a, st); }

// ---------------------------------------------------------------------------- weight gradient
// dW[tap][ci][co] = sum over voxels of x[v + tap][ci] * g[v][co]: rows = 16 input channels, columns
// = 16 output channels, the contraction runs over 4 neighbouring voxels of a row per instruction.
// Channel-fastest tiles in LDS are read conflict-free as they lie (16 channels x 4 voxels = 64
// consecutive words).  The four waves split the 27 taps 7/7/7/6 and share each tile; the spare
// slot multiplies ones, which gives the bias gradient.  A workgroup takes every nsplit-th tile,
// the next tile's loads in flight, and writes one set of partial sums.
template <typename T>
struct GenWgrad {
    const T *x1, *x2;
    int c1, c2;
    const T *g, *mask;
    int cout;
    float *ws;
    int N, D, H, W, ntd, nth, ntw;
    int tiles, nsplit, ncb;   // ncb: 16-channel blocks of cout
    int64_t per_split;
};

template <typename T, int TD, int TH, int TW, bool BUF>
__global__ __launch_bounds__(256, 3) void conv_general_wgrad_kernel(GenWgrad<T> p)
{
    constexpr int HD = TD + 2, HH = TH + 2, HW = TW + 2, NHALO = HD * HH * HW, NV = TD * TH * TW;
    constexpr int XI = (NHALO * 4 + 255) / 256, GI = (NV * 4 + 255) / 256;
    __shared__ __attribute__((aligned(16))) float xs[NHALO * 16];
    __shared__ __attribute__((aligned(16))) float gs[NV * 16];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int cin = p.c1 + p.c2;
    const int split = (int)(blockIdx.x % (unsigned)p.nsplit), blk = (int)(blockIdx.x / (unsigned)p.nsplit);
    const int ci0 = (blk / p.ncb) * 16, co0 = (blk % p.ncb) * 16;
    // offset of the lane's voxel in each item (tid + 256 k: voxel and quad) from the tile's first one
    TileOff<BUF> hx[XI], hg[GI];
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int vox = (tid + k * 256) >> 2;
        hx[k] = tile_offset<TileOff<BUF>>(vox / (HW * HH), (vox / HW) % HH, vox % HW, p.H, p.W);
    }
#pragma unroll
    for (int k = 0; k < GI; ++k) {
        const int vox = (tid + k * 256) >> 2;
        hg[k] = tile_offset<TileOff<BUF>>(vox / (TW * TH), (vox / TW) % TH, vox % TW, p.H, p.W);
    }
    f32x4 sx[XI], sg[GI];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        int t = tile;
        const int w0 = (t % p.ntw) * TW;
        t /= p.ntw;
        const int h0 = (t % p.nth) * TH;
        t /= p.nth;
        const int d0 = (t % p.ntd) * TD;
        const int n = t / p.ntd;
        const int64_t g0 = (((int64_t)n * p.D + d0) * p.H + h0) * p.W + w0, x0 = g0 - ((int64_t)p.H * p.W + p.W + 1);
        const QuadSrc xsrc = {rsrc_of(p.x1 + x0 * p.c1, 0x7ffffff0), rsrc_of((p.x2 ? p.x2 : p.x1) + x0 * p.c2, 0x7ffffff0)};
        const QuadSrc gsrc = {rsrc_of(p.g + g0 * p.cout, 0x7ffffff0), xsrc.r2};
        const QuadSrc msrc = {rsrc_of((p.mask ? p.mask : p.g) + g0 * p.cout, 0x7ffffff0), xsrc.r2};
#pragma unroll
        for (int k = 0; k < XI; ++k) {
            const int i = tid + k * 256, vox = i >> 2, q = i & 3;
            const unsigned gd = d0 + vox / (HW * HH) - 1, gh = h0 + (vox / HW) % HH - 1, gw = w0 + vox % HW - 1;
            const bool in = vox < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W;
            if constexpr (BUF) sx[k] = load_quad_buf<T>(xsrc, p.c1, p.c2, in ? hx[k] : -1, ci0, 16, q);
            else sx[k] = in ? load_quad(p.x1, p.x2, p.c1, p.c2, x0 + hx[k], ci0 + q * 4) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int k = 0; k < GI; ++k) {
            const int i = tid + k * 256, vox = i >> 2, q = i & 3;
            const bool in = vox < NV && d0 + vox / (TW * TH) < p.D && h0 + (vox / TW) % TH < p.H && w0 + vox % TW < p.W;
            if constexpr (BUF) {
                sg[k] = load_quad_buf<T>(gsrc, p.cout, 0, in ? hg[k] : -1, co0, 16, q);
                if (p.mask) sg[k] = keep_positive(sg[k], load_quad_buf<T>(msrc, p.cout, 0, in ? hg[k] : -1, co0, 16, q));
            } else {
                sg[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (in) {
                    sg[k] = load_quad<T>(p.g, nullptr, p.cout, 0, g0 + hg[k], co0 + q * 4);
                    if (p.mask) sg[k] = keep_positive(sg[k], load_quad<T>(p.mask, nullptr, p.cout, 0, g0 + hg[k], co0 + q * 4));
                }
            }
        }
    };
    // LDS index of the lane's operand for each of the wave's taps, first voxel group
    int xo[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int tap = wv * 7 + j < 27 ? wv * 7 + j : 26;
        xo[j] = (((tap / 9) * HH + (tap / 3) % 3) * HW + tap % 3 + kg) * 16 + ln;
    }
    const int go = kg * 16 + ln;
    const bool ones = wv == 3;
    f32x4 acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    int tile = split;
    fetch(tile);
    while (true) {
#pragma unroll
        for (int k = 0; k < XI; ++k) {
            const int i = tid + k * 256;
            if (i < NHALO * 4) *reinterpret_cast<f32x4 *>(xs + i * 4) = sx[k];
        }
#pragma unroll
        for (int k = 0; k < GI; ++k) {
            const int i = tid + k * 256;
            if (i < NV * 4) *reinterpret_cast<f32x4 *>(gs + i * 4) = sg[k];
        }
        __syncthreads();
        const int next = tile + p.nsplit;
        if (next < p.tiles) fetch(next);
#pragma unroll
        for (int q = 0; q < NV / 4; ++q) {
            constexpr int R = TW / 4;   // groups of 4 voxels per row
            const int row = q / R, off = (((row / TH) * HH + row % TH) * HW + (q % R) * 4) * 16;
            const float b = gs[go + q * 64];
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                float a = xs[xo[j] + off];
                if (j == 6 && ones) a = 1.f;
                acc[j] = mfma_f32(a, b, acc[j]);
            }
        }
        tile = next;
        if (tile >= p.tiles) break;
        __syncthreads();
    }
    float *out = p.ws + (int64_t)split * p.per_split;
    const int co = co0 + ln;
    if (co >= p.cout) return;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int tap = wv * 7 + j;
        if (tap < 27) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ci = ci0 + kg * 4 + r;
                if (ci < cin) out[((int64_t)tap * cin + ci) * p.cout + co] = acc[j][r];
            }
        } else if (ci0 == 0 && kg == 0) {
            out[(int64_t)27 * cin * p.cout + co] = acc[j][0];   // every row holds the sum of g
        }
    }
}

struct GenWgradPlan { bool small; int64_t tiles, nsplit; };
// A 128-voxel tile per workgroup and more where that fills the chip, else 64-voxel tiles; about
// 512 workgroups in all (two per CU cover each other's staging), each with a whole number of tiles.
static GenWgradPlan general_wgrad_plan(int64_t N, int64_t D, int64_t H, int64_t W, int64_t cin, int64_t cout)
{
    const int64_t blocks = ((cin + 15) / 16) * ((cout + 15) / 16), hw = ((H + 3) / 4) * ((W + 7) / 8);
    GenWgradPlan q;
    q.tiles = N * ((D + 3) / 4) * hw;
    q.small = q.tiles * blocks < 256;
    if (q.small) q.tiles = N * ((D + 1) / 2) * hw;
    int64_t want = 512 / blocks;
    if (want < 1) want = 1;
    const int64_t each = (q.tiles + want - 1) / want;
    q.nsplit = (q.tiles + each - 1) / each;
    return q;
}

// The query promises at least one set of partial sums per 256 voxels, at most 1024 (more than the plan
// takes for all but the smallest volumes): the size callers have allocated, and been refused by, so far.
int64_t conv_wgrad_general_sets(int64_t N, int64_t D, int64_t H, int64_t W, int64_t cin, int64_t cout)
{
    int64_t sets = N * D * H * W / 256;
    if (sets > 1024) sets = 1024;
    const int64_t need = general_wgrad_plan(N, D, H, W, cin, cout).nsplit;
    return sets > need ? sets : need;
}
size_t conv_wgrad_general_ws_bytes(int64_t N, int64_t D, int64_t H, int64_t W, int64_t cin, int64_t cout)
{
    return (size_t)conv_wgrad_general_sets(N, D, H, W, cin, cout) * (size_t)(27 * cin * cout + cout) * sizeof(float);
}

template <typename T>
static int wgrad_general_t(const ConvArgs &a, float *dW, float *db, float *ws, hipStream_t st)
{
    const int64_t cin = a.c1 + a.c2;
    const GenWgradPlan q = general_wgrad_plan(a.N, a.D, a.H, a.W, cin, a.cout);
    const int64_t blocks = ((cin + 15) / 16) * ((a.cout + 15) / 16);
    if (q.nsplit * blocks > 0x7fffffffLL || q.tiles > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    GenWgrad<T> p{};
    p.x1 = (const T *)a.x; p.x2 = (const T *)a.x2;
    p.c1 = (int)a.c1; p.c2 = (int)a.c2;
    p.g = (const T *)a.dy; p.mask = (const T *)a.ymask;
    p.cout = (int)a.cout;
    p.ws = ws;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    p.ntd = q.small ? (p.D + 1) / 2 : (p.D + 3) / 4;
    p.nth = (p.H + 3) / 4;
    p.ntw = (p.W + 7) / 8;
    p.tiles = (int)q.tiles;
    p.nsplit = (int)q.nsplit;
    p.ncb = (int)((a.cout + 15) / 16);
    p.per_split = 27 * cin * a.cout + a.cout;
    const dim3 grid((unsigned)(q.nsplit * blocks));
    const int64_t span = 6 * (int64_t)(p.H + 1) * p.W * (cin > a.cout ? cin : a.cout) * 4;
    const bool buf = whole_quads(p.c1 | p.c2 | p.cout, bits(p.x1) | bits(p.x2) | bits(p.g) | bits(p.mask), sizeof(T)) && span < 0x7fffffffLL;
    if (q.small && buf) conv_general_wgrad_kernel<T, 2, 4, 8, true><<<grid, 256, 0, st>>>(p);
    else if (q.small) conv_general_wgrad_kernel<T, 2, 4, 8, false><<<grid, 256, 0, st>>>(p);
    else if (buf) conv_general_wgrad_kernel<T, 4, 4, 8, true><<<grid, 256, 0, st>>>(p);
    else conv_general_wgrad_kernel<T, 4, 4, 8, false><<<grid, 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return launch_reduce_partials(ws, dW, db, 27 * cin * a.cout, p.per_split, (int)q.nsplit, st);
}
int conv_wgrad_general(const ConvArgs &a, float *dW, float *db, float *ws, hipStream_t st)
{
    return a.dtype == K3_F32 ? wgrad_general_t<float>(a, dW, db, ws, st) : wgrad_general_t<bf16_t>(a, dW, db, ws, st);
}

}  // namespace k3

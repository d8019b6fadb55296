// 3x3x3 convolution for the tensors the bf16 matrix-core kernels do not take -- fp32, and bf16 with
// channel counts that are no multiple of 16 or tensors off their alignment -- on
// v_mfma_f32_16x16x4_f32: forward and backward-data for any channel counts, backward-weight of bf16
// tensors (of fp32 ones: wgrad_ordered.hip), fp32 products and fp32 accumulation.
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

// GEMM D[output channel][voxel] = sum over (tap, channel); A = weights, B = activations.  One instruction
// multiplies four neighbouring channels of one tap (lane group kg carries channel kg of them), and an
// accumulator starts from the bias and takes the taps in the order of the definition and the channels
// of a tap in theirs.  The instruction is a chain of four fused multiply-adds in lane-group order
// (measured: equal to the bit over 65536 sums of four magnitudes, subnormal ones too), so every sum is the
// plain loop over the definition with one rounding per term.  That order is kept on purpose: in fp32
// networks any other one moves a few ReLU signs and pooling maxima out of millions, and with them whole
// gradient elements (of the fp32 U-Net at 48^3 in one batch of six by more than 4e-5 of the norm).  So
// neither the waves nor the workgroups split a sum: the waves of a workgroup take different
// voxels (WN of them) and output channels, and all channels of the halo tile are in LDS at once.  Bound:
// the chain of 27 K / 4 instructions of 32 clocks where a volume gives the chip only a wave or so per
// SIMD, else the matrix core.  A step is U instructions on 4 U channels of a tap: U = 4 for channels in
// whole 16s; U = 1 for any, padded to whole fours with zeros on both sides (which change no sum).  SPT:
// steps a tap where that is known at compile time, else 0.  S: quads of a voxel that neighbouring threads
// stage (1: at most 4 channels).  QUAD: activations are read through buffer descriptors (channel counts in
// whole quads on quad boundaries, a tile's span below 2 GiB); else element by element.  LDS false: more
// channels than LDS holds, or weights of 2 GiB and more: all operands come from memory one by one.
template <int TD_, int TH_, int TW_, int WN_, int MB_>
struct GenTile {
    static constexpr int TD = TD_, TH = TH_, TW = TW_, WN = WN_, MB = MB_, WM = 4 / WN, NB = TD * TH * TW / 16 / WN, CO = 16 * MB * WM;
    static constexpr int HD = TD + 2, HH = TH + 2, HW = TW + 2, NHALO = HD * HH * HW;
};

template <typename T, class C, int S, int U, int SPT, bool BWD, bool QUAD, bool LDS>
__global__ __launch_bounds__(256, LDS ? 4 : 2) void conv_general_kernel(GenConv<T> p)
{
    constexpr int TH = C::TH, TW = C::TW, HH = C::HH, HW = C::HW, NHALO = C::NHALO, NB = C::NB, MB = C::MB;
    constexpr int ITEMS = (NHALO * S + 255) / 256, RING = U * NB * MB >= 16 ? 3 : 9, AHEAD = RING - 1;
    constexpr int XRING = LDS ? 3 : RING, XAHEAD = XRING - 1;
    static_assert(27 % RING == 0 && (U == 1 || QUAD), "whole turns of the ring; steps of 16 channels read quads");
    extern __shared__ __attribute__((aligned(16))) float xs[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int wn = wv % C::WN, wm = wv / C::WN;
    const int K = p.c1 + p.c2, M = p.cd1 + p.cd2, KP = (K + 3) & ~3, pitch = general_pitch(K);

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
    const int d0 = (int)(t % p.ntd) * C::TD;
    const int n = (int)(t / p.ntd);
    const int m0 = (cb * C::WM + wm) * 16 * MB;

    if constexpr (LDS) {
        // the lane's halo items: (voxel, quad) i = tid + 256 k; offset of the voxel from the halo tile's
        // first one, negative outside the volume
        TileOff<QUAD> vo[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int vox = (tid + k * 256) / S;
            const int lw = vox % HW, lh = (vox / HW) % HH, ld = vox / (HW * HH);
            const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
            vo[k] = vox < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W ? tile_offset<TileOff<QUAD>>(ld, lh, lw, p.H, p.W) : -1;
        }
        const int64_t halo0 = (((int64_t)n * p.D + d0 - 1) * p.H + h0 - 1) * p.W + w0 - 1;
        const QuadSrc xsrc = {rsrc_of(p.src1 + halo0 * p.c1, 0x7ffffff0), rsrc_of((p.src2 ? p.src2 : p.src1) + halo0 * p.c2, 0x7ffffff0)};
        const QuadSrc msrc = {rsrc_of((p.mask ? p.mask : p.src1) + halo0 * p.c1, 0x7ffffff0), xsrc.r2};
        constexpr int ROUND = ITEMS > 4 ? 2 : ITEMS > 2 ? 3 : 6;     // chunks in flight at once
        f32x4 st[ROUND][ITEMS];
        auto fetch = [&](int c, f32x4 (&to)[ITEMS]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int q = (tid + k * 256) % S;
                if constexpr (QUAD) {
                    to[k] = load_quad_buf<T>(xsrc, p.c1, p.c2, vo[k], c * 4 * S, 4 * S, q);
                    if (p.mask) to[k] = keep_positive(to[k], load_quad_buf<T>(msrc, p.c1, 0, vo[k], c * 4 * S, 4 * S, q));
                } else {
                    to[k] = f32x4{0.f, 0.f, 0.f, 0.f};
                    if (vo[k] >= 0) {
                        const int ch = c * 4 * S + q * 4;
                        to[k] = load_quad(p.src1, p.src2, p.c1, p.c2, halo0 + vo[k], ch);
                        if (p.mask) to[k] = keep_positive(to[k], load_quad<T>(p.mask, nullptr, p.c1, 0, halo0 + vo[k], ch));
                    }
                }
            }
        };
        const int nchunk = (K + 4 * S - 1) / (4 * S);
        for (int c = 0; c < nchunk; c += ROUND) {
#pragma unroll
            for (int r = 0; r < ROUND; ++r)
                if (c + r < nchunk) fetch(c + r, st[r]);
#pragma unroll
            for (int r = 0; r < ROUND; ++r)
#pragma unroll
                for (int k = 0; k < ITEMS; ++k) {
                    const int i = tid + k * 256, ch = (c + r) * 4 * S + (i % S) * 4;
                    if (i < NHALO * S && ch < KP) *reinterpret_cast<f32x4 *>(xs + (i / S) * pitch + ch) = st[r][k];
                }
        }
        __syncthreads();
    }
    if (m0 >= M) return;

    // Weights of (tap, four U channels from c on): the lane (row ln, lane group kg) takes channel kg of each
    // four.  Rows beyond the layer's, and channels beyond it, get a lane offset outside the descriptor's range
    // and read as zero (without a descriptor: both are read from a clamped place and replaced).
    const __amdgpu_buffer_rsrc_t wrsrc = rsrc_of(p.w, LDS ? 27 * K * M * (int)sizeof(T) : 0);
    int lo[MB][U];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int m = m0 + mb * 16 + ln;
            lo[mb][j] = m >= M || (S == 1 && kg >= K) ? -1 : BWD ? m * K + kg * U + j : (4 * j + kg) * M + m;
        }
    auto weights = [&](int tap, int c, float (&a)[MB][U]) __attribute__((always_inline)) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int j = 0; j < U; ++j) {
                if constexpr (BWD && U == 4) {
                    // a row's 16 channels lie together: the lane reads four and spread() deals them out (16 loads
                    // of 16 bytes instead of 64 of 4: 16 -> 16 at 48^3 58 -> 25 us)
                    if (j == 0) {
                        const f32x4 v = buf<T>::quad(wrsrc, lo[mb][0], general_weight<int>(BWD, tap, c, K, M) * (int)sizeof(T));
                        a[mb][0] = v[0]; a[mb][1] = v[1]; a[mb][2] = v[2]; a[mb][3] = v[3];
                    }
                } else if constexpr (LDS) {
                    const int o = !QUAD && S > 1 && c + kg >= K ? -1 : lo[mb][j];
                    a[mb][j] = buf<T>::one(wrsrc, o, general_weight<int>(BWD, tap, c, K, M) * (int)sizeof(T));
                } else {
                    const int m = m0 + mb * 16 + ln, ch = c + kg, mc = m < M ? m : M - 1, kc = ch < K ? ch : K - 1;
                    const float v = elem<T>::ld(p.w + general_weight<int64_t>(BWD, tap, BWD ? 0 : kc, K, M) + (BWD ? (int64_t)mc * K + kc : mc));
                    a[mb][j] = m < M && ch < K ? v : 0.f;
                }
            }
    };
    struct Place {      // in the sum: tap and first channel
        int tap, c;
    };
    auto advance = [&](Place &q) __attribute__((always_inline)) { general_next(q.tap, q.c, 4 * U, KP); };
    int vb[NB];   // LDS index of the lane's voxel and channel in each 16-voxel block, halo position (0,0,0)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int i = (wn * NB + b) * 16 + ln;
        vb[b] = (((i / (TW * TH)) * HH + (i / TW) % TH) * HW + i % TW) * pitch + kg;
    }
    auto inputs = [&](const Place &q, float (&x)[NB][U]) __attribute__((always_inline)) {
        const int c = q.c, pos = BWD ? 26 - q.tap : q.tap;     // place of the tap's voxel in the halo
        if constexpr (LDS) {
            const int off = (((pos / 9) * HH + (pos / 3) % 3) * HW + pos % 3) * pitch + c;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int j = 0; j < U; ++j) x[b][j] = xs[vb[b] + off + 4 * j];
        } else {
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int i = (wn * NB + b) * 16 + ln, ch = c + kg;
                const unsigned gd = d0 + i / (TW * TH) + pos / 9 - 1, gh = h0 + (i / TW) % TH + (pos / 3) % 3 - 1, gw = w0 + i % TW + pos % 3 - 1;
                x[b][0] = 0.f;
                if (gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W && ch < K) {
                    const int64_t v = (((int64_t)n * p.D + gd) * p.H + gh) * p.W + gw;
                    x[b][0] = ch < p.c1 ? elem<T>::ld(p.src1 + v * p.c1 + ch) : elem<T>::ld(p.src2 + v * p.c2 + (ch - p.c1));
                    if (p.mask && !(elem<T>::ld(p.mask + v * p.c1 + ch) > 0.f)) x[b][0] = 0.f;
                }
            }
        }
    };
    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + mb * 16 + kg * 4 + r;
                acc[b][mb][r] = p.bias && m < M ? p.bias[m] : 0.f;
            }

    auto multiply = [&](float (&as)[MB][U], float (&xr)[NB][U]) __attribute__((always_inline)) {
        if constexpr (BWD && U == 4) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) spread(as[mb]);
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) acc[b][mb] = mfma_f32(as[mb][j], xr[b][j], acc[b][mb]);
    };
    if constexpr (SPT > 0) {
        // SPT steps a tap, known at compile time (4 U SPT channels): a turn is one row of taps (the three rows of a
        // plane where a row is only a few steps), everything inside it at constant offsets.  A wave alone on
        // its SIMD pays four clocks for every instruction, and the counting of the other form cost more
        // than the matrix instructions (64 -> 64 at 12^3: 14.5 us against 20, 16 -> 16 at 48^3 24.6 against 29.3).
        constexpr int ROWS = SPT <= (U == 1 ? 2 : 1) ? 3 : 1, ST = 3 * SPT * ROWS, PT = general_pitch(4 * U * SPT);
        constexpr int R = U * NB * MB >= 16 ? 3 : ST % 9 == 0 ? 9 : SPT == 2 ? 6 : 12, A = R - 1 < 8 ? R - 1 : 8;
        float a[R][MB][U], x[3][NB][U];
        auto row = [&](int g) __attribute__((always_inline)) {      // LDS offset of the turn's first row of taps
            const int q = BWD ? (ROWS == 3 ? 2 : 8) - g : g;
            return (ROWS == 3 ? q * HH : (q / 3) * HH + q % 3) * HW * PT;
        };
        auto load_w = [&](int g, int st, float (&as)[MB][U]) __attribute__((always_inline)) {
            weights(g * 3 * ROWS + st / SPT, (st % SPT) * 4 * U, as);
        };
        auto load_x = [&](int at, int st, float (&xr)[NB][U]) __attribute__((always_inline)) {
            const int r = st / (3 * SPT), w = (st / SPT) % 3;
            const int off = ((ROWS == 3 ? (BWD ? 2 - r : r) * HW : 0) + (BWD ? 2 - w : w)) * PT + (st % SPT) * 4 * U;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int j = 0; j < U; ++j) xr[b][j] = xs[vb[b] + at + off + 4 * j];
        };
        int at = row(0);
#pragma unroll
        for (int i = 0; i < A; ++i) load_w(0, i, a[i]);
        load_x(at, 0, x[0]);
        load_x(at, 1, x[1]);
        for (int g = 0; g < 9 / ROWS; ++g) {
            const int gn = g + 1 < 9 / ROWS ? g + 1 : g, next = row(gn);     // (behind the last turn it is read again)
#pragma unroll
            for (int i = 0; i < ST; ++i) {
                load_w(i + A < ST ? g : gn, (i + A) % ST, a[(i + A) % R]);
                load_x(i + 2 < ST ? at : next, (i + 2) % ST, x[(i + 2) % 3]);
                multiply(a[i % R], x[i % 3]);
                __builtin_amdgcn_sched_barrier(0);   // no further ahead: hoisted loads cost the occupancy
            }
            at = next;
        }
    } else {
        float a[RING][MB][U], x[XRING][NB][U];
        Place pa = {0, 0}, px = {0, 0};
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            weights(pa.tap, pa.c, a[i]);
            advance(pa);
            if (i < XAHEAD) {
                inputs(px, x[i]);
                advance(px);
            }
        }
        const int steps = 27 * (KP / (4 * U));
        for (int s = 0; s < steps; s += RING) {
#pragma unroll
            for (int i = 0; i < RING; ++i) {
                weights(pa.tap, pa.c, a[(i + AHEAD) % RING]);
                advance(pa);
                inputs(px, x[(i + XAHEAD) % XRING]);
                advance(px);
                multiply(a[i], x[i % XRING]);
                __builtin_amdgcn_sched_barrier(0);   // no further ahead: hoisted loads cost the occupancy
            }
        }
    }

    // a lane holds output channels m .. m+3 of one voxel of a block
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int i = (wn * NB + b) * 16 + ln;
        const int gd = d0 + i / (TW * TH), gh = h0 + (i / TW) % TH, gw = w0 + i % TW;
        if (gd >= p.D || gh >= p.H || gw >= p.W) continue;
        const int64_t vox = (((int64_t)n * p.D + gd) * p.H + gh) * p.W + gw;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + mb * 16 + kg * 4;
            if (m >= M) continue;
            f32x4 v = acc[b][mb];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = (p.relu && !(v[r] > 0.f)) ? 0.f : v[r];
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
        }
    }
}

template <typename T, class C, int S, int U, int SPT, bool BWD, bool QUAD, bool LDS = true>
static int launch_general(GenConv<T> p, hipStream_t st)
{
    p.ntd = (p.D + C::TD - 1) / C::TD;
    p.nth = (p.H + C::TH - 1) / C::TH;
    p.ntw = (p.W + C::TW - 1) / C::TW;
    p.ncb = (p.cd1 + p.cd2 + C::CO - 1) / C::CO;
    p.total = (int64_t)p.N * p.ntd * p.nth * p.ntw * p.ncb;
    p.per_xcd = (p.total + 7) / 8;
    if (p.per_xcd * 8 > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    const int lds = LDS ? C::NHALO * general_pitch(p.c1 + p.c2) * (int)sizeof(float) : 0;
    if (lds > 64 * 1024) {
        static bool attr_done = false;  // raising the dynamic LDS limit is idempotent
        if (!attr_done) {
            K3_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&conv_general_kernel<T, C, S, U, SPT, BWD, QUAD, LDS>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
            attr_done = true;
        }
    }
    conv_general_kernel<T, C, S, U, SPT, BWD, QUAD, LDS><<<dim3((unsigned)(p.per_xcd * 8)), 256, lds, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

static uintptr_t bits(const void *p) { return (uintptr_t)p; }

// The largest tile that gives every CU a workgroup, with two output blocks a wave where that still does;
// its halo must fit LDS twice (a workgroup then stages while another multiplies), the smallest tile's
// once.  Volumes too small for that: 32 voxels x 32 channels a workgroup (64 x 16 of a 16-channel layer).
template <typename T, int S, int U, int SPT, bool BWD, bool QUAD>
static int launch_general_size(const GenConv<T> &p, hipStream_t st)
{
    const int64_t M = p.cd1 + p.cd2;
    auto groups = [&](int td, int th, int tw, int co) {
        return (int64_t)p.N * ((p.D + td - 1) / td) * ((p.H + th - 1) / th) * ((p.W + tw - 1) / tw) * ((M + co - 1) / co);
    };
    const int64_t voxel = general_pitch(p.c1 + p.c2) * (int64_t)sizeof(float), half = 80 * 1024;
    typedef GenTile<4, 4, 8, 4, 1> T1;
    typedef GenTile<2, 4, 8, 4, 1> T2;
    typedef GenTile<2, 4, 4, 2, 1> T3;
    typedef GenTile<2, 2, 4, 1, 1> T4;
    if constexpr (U * SPT < 16) {        // (a tile that 4 U SPT channels never fit, or never need, is not built)
        if (T1::NHALO * voxel <= half) {
            if constexpr (QUAD)
                if (M > 16 && groups(4, 4, 8, 32) >= 256) return launch_general<T, GenTile<4, 4, 8, 4, 2>, S, U, SPT, BWD, QUAD>(p, st);
            if (groups(4, 4, 8, 16) >= 256) return launch_general<T, T1, S, U, SPT, BWD, QUAD>(p, st);
        }
    }
    if constexpr (U * SPT < 32) {
        if (T2::NHALO * voxel <= half) {
            if constexpr (QUAD)
                if (M > 16 && groups(2, 4, 8, 32) >= 256) return launch_general<T, GenTile<2, 4, 8, 4, 2>, S, U, SPT, BWD, QUAD>(p, st);
            if (M <= 16 || groups(2, 4, 8, 16) >= 256) return launch_general<T, T2, S, U, SPT, BWD, QUAD>(p, st);
        }
    }
    if (T3::NHALO * voxel <= half) return launch_general<T, T3, S, U, SPT, BWD, QUAD>(p, st);
    if constexpr (S == 4 && SPT == 0)
        if (T4::NHALO * voxel <= 160 * 1024) return launch_general<T, T4, S, U, SPT, BWD, QUAD>(p, st);
    if constexpr (SPT > 0) return K3_E_UNSUPPORTED;       // (not reached: up to 128 channels the third tile fits)
    else return launch_general<T, T4, 4, 1, 0, BWD, false, false>(p, st);
}

template <typename T, bool BWD>
static int launch_general_any(GenConv<T> p, hipStream_t st)
{
    const int64_t M = p.cd1 + p.cd2, K = p.c1 + p.c2, C = K > M ? K : M;
    const bool quad = whole_quads(p.c1 | p.c2, bits(p.src1) | bits(p.src2) | bits(p.mask), sizeof(T)) &&
                      6 * (int64_t)(p.H + 1) * p.W * C * 4 < 0x7fffffffLL;
    p.vout = whole_quads(p.cd1 | p.cd2, bits(p.dst1) | bits(p.dst2) | bits(p.omask), sizeof(T));
    if (27 * K * M * 4 >= 0x7fffffffLL) return launch_general<T, GenTile<2, 2, 4, 1, 1>, 4, 1, 0, BWD, false, false>(p, st);
    if (!quad && K <= 4) return launch_general_size<T, 1, 1, 1, BWD, false>(p, st);
    if (!quad) return launch_general_size<T, 4, 1, 0, BWD, false>(p, st);
    if (K == 4) return launch_general_size<T, 1, 1, 1, BWD, true>(p, st);
    if (K == 8) return launch_general_size<T, 4, 1, 2, BWD, true>(p, st);
    if (K % 16 || (BWD && !whole_quads(0, bits(p.w), sizeof(T)))) return launch_general_size<T, 4, 1, 0, BWD, true>(p, st);
    if constexpr (sizeof(T) == 4) {      // (bf16 tensors of these get here by their alignment alone)
        if (K == 16) return launch_general_size<T, 4, 4, 1, BWD, true>(p, st);
        if (K == 32) return launch_general_size<T, 4, 4, 2, BWD, true>(p, st);
        if (K == 64) return launch_general_size<T, 4, 4, 4, BWD, true>(p, st);
        if (K == 128) return launch_general_size<T, 4, 4, 8, BWD, true>(p, st);
    }
    return launch_general_size<T, 4, 4, 0, BWD, true>(p, st);
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

// What the query promises, and no call takes more than: a set of partial sums per 256 voxels, at most 1024.
int64_t conv_wgrad_general_sets(int64_t N, int64_t D, int64_t H, int64_t W)
{
    const int64_t sets = N * D * H * W / 256;
    return sets < 1 ? 1 : sets > 1024 ? 1024 : sets;
}
size_t conv_wgrad_general_ws_bytes(int64_t N, int64_t D, int64_t H, int64_t W, int64_t cin, int64_t cout)
{
    return (size_t)conv_wgrad_general_sets(N, D, H, W) * (size_t)(27 * cin * cout + cout) * sizeof(float);
}

template <typename T>
static int wgrad_general_t(const ConvArgs &a, float *dW, float *db, float *ws, hipStream_t st)
{
    const int64_t cin = a.c1 + a.c2;
    GenWgradPlan q = general_wgrad_plan(a.N, a.D, a.H, a.W, cin, a.cout);
    const int64_t most = conv_wgrad_general_sets(a.N, a.D, a.H, a.W);
    if (q.nsplit > most) q.nsplit = most;
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
    return a.dtype == K3_F32 ? conv_wgrad_ordered(a, dW, db, ws, st) : wgrad_general_t<bf16_t>(a, dW, db, ws, st);
}

}  // namespace k3

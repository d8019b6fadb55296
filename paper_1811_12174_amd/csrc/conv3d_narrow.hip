// bf16 3x3x3 convolution for channel counts in whole 16s that are no whole 32s (the levels of a
// 16-filter network, both ends of 16 <-> 32): forward, backward-data and backward-weight on
// v_mfma_f32_16x16x32_bf16, straight from the canonical weights.
//
// Bound: at 16 -> 16 channels a voxel needs 64 bytes of traffic and 14 matrix instructions per 16
// voxels, so both pass in a few microseconds at the sizes such networks run at and what counts is the
// length of one workgroup's chain (halo from memory, LDS, 14 steps, store) and that the LDS reads of
// four resident workgroups per CU overlap it.  The general kernels these replace multiply in fp32, at
// a sixteenth of the rate, and left the ReLU bit masks to passes of their own.  2 x 40x48x56, before ->
// after: 16 -> 16 forward 46 (51 with its bits) -> 11 - 12 us, backward-data 46 (54) -> 14, backward-weight
// 50 -> 19 with its reduction; 32 -> 16 forward 79 (84) -> 19, backward-data 78 -> 20, backward-weight 78 -> 23.
#include "common.h"
#include "conv_internal.h"
#include "conv_mfma.h"

namespace k3 {

struct NarrowParams : MfmaParams {
    const bf16_t *w;   // canonical [27][cin][cout]
};

// A step = two taps of a 16-channel chunk (lane groups 0, 1: the halves of one tap, 2, 3: of the next);
// the 28th tap of a chunk is zeros on both sides.  TD x TH x 8 voxels per workgroup, two rows of 8 to a
// block; a wave owns whole blocks of one plane.  Halo (32 bytes a voxel) and weights of a chunk are in
// LDS, the halo of the next one in registers.
template <int TD, int TH, int MB, bool BWD>
__global__ __launch_bounds__(256, MB == 1 ? 4 : 3) void conv_narrow_kernel(NarrowParams p)
{
    constexpr int HH = TH + 2, HW = 10, NHALO = (TD + 2) * HH * HW, NB = TD * TH / 8, BPP = TH / 2;   // blocks per wave, per plane
    constexpr int XI = (NHALO * 2 + 255) / 256, ROWS = 16 * MB, WITEMS = 27 * ROWS * 2, WI = (WITEMS + 255) / 256;
    static_assert(NB <= BPP, "one plane per wave");
    __shared__ __attribute__((aligned(16))) unsigned char xs[(NHALO + 1) * 32];   // the last voxel is zeros
    __shared__ __attribute__((aligned(16))) unsigned char wsm[28 * ROWS * 32];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15, half = kg & 1, second = kg >> 1;
    const int K = p.c1 + p.c2, M = p.cd1 + p.cd2, nchunk = K / 16;

    // a contiguous run of the logical order per XCD; the channel groups of a tile are neighbours
    const int64_t logical = (int64_t)(blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (logical >= p.total) return;
    const int m0 = (int)(logical % p.ncg) * ROWS;
    int64_t t = logical / p.ncg;
    const int w0 = (int)(t % p.ntw) * 8;
    t /= p.ntw;
    const int h0 = (int)(t % p.nth) * TH;
    t /= p.nth;
    const int d0 = (int)(t % p.ntd) * TD;
    const int n = (int)(t / p.ntd);

    // the lane's halo items (voxel, 8 channels): offset of the voxel from the halo's first one, -1 outside
    int vo[XI];
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int v = (tid + k * 256) >> 1;
        const int lw = v % HW, lh = (v / HW) % HH, ld = v / (HW * HH);
        const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
        vo[k] = v < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W ? (ld * p.H + lh) * p.W + lw : -1;
    }
    const int64_t halo0 = (((int64_t)n * p.D + d0 - 1) * p.H + h0 - 1) * p.W + w0 - 1;
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.src1 + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.src2 ? p.src2 : p.src1) + halo0 * p.c2), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.mask ? p.mask : p.src1) + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    u32v4 sx[XI], sw[WI];
    auto fetch = [&](int c) __attribute__((always_inline)) {
        const int ch = c * 16 + (tid & 1) * 8;
        const bool first = c * 16 < p.c1;     // a chunk lies in one source
#pragma unroll
        for (int k = 0; k < XI; ++k) {
            if (first) sx[k] = __builtin_amdgcn_raw_buffer_load_b128(r1, vo[k] < 0 ? -1 : (vo[k] * p.c1 + ch) * 2, 0, 0);
            else sx[k] = __builtin_amdgcn_raw_buffer_load_b128(r2, vo[k] < 0 ? -1 : (vo[k] * p.c2 + ch - p.c1) * 2, 0, 0);
            if (p.mask) {                     // backward-data: one source
                const u32v4 m = __builtin_amdgcn_raw_buffer_load_b128(rm, vo[k] < 0 ? -1 : (vo[k] * p.c1 + ch) * 2, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) sx[k][j] = mask_pair_to(sx[k][j], m[j], MASK_NUMBERS);
            }
        }
    };
    auto fetch_weights = [&](int c) __attribute__((always_inline)) {
        int tl = tid;
        asm("" : "+v"(tl));     // addresses are worked out anew for each chunk: kept across the steps they spill
#pragma unroll
        for (int k = 0; k < WI; ++k) {
            const int i = tl + k * 256;
            sw[k] = u32v4{0, 0, 0, 0};
            if constexpr (BWD) {              // eight contraction channels of a row lie together
                const int tap = i / (2 * ROWS), row = (i >> 1) % ROWS;
                if (i < WITEMS && m0 + row < M)
                    sw[k] = *reinterpret_cast<const u32x4_pk *>(p.w + ((int64_t)(26 - tap) * M + m0 + row) * K + c * 16 + (i & 1) * 8);
            } else {                          // eight rows of a contraction channel do
                const int tap = i / (2 * ROWS), oct = (i >> 4) % (2 * MB), k0 = i & 15;
                if (i < WITEMS && m0 + oct * 8 < M)
                    sw[k] = *reinterpret_cast<const u32x4_pk *>(p.w + ((int64_t)tap * K + c * 16 + k0) * M + m0 + oct * 8);
            }
        }
    };
    const int plane = wv * NB / BPP, row0 = (wv * NB % BPP) * 2;
    const unsigned char *x = xs + ((plane * HH + row0 + (ln >> 3)) * HW + (ln & 7)) * 32 + half * 16;
    const unsigned char *a0 = wsm + (second * ROWS + ln) * 32 + half * 16;
    f32x4 acc[NB][MB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[b][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    fetch(0);
    fetch_weights(0);
    if (tid < 2) *reinterpret_cast<u32v4 *>(xs + NHALO * 32 + tid * 16) = u32v4{0, 0, 0, 0};
    if (tid < 2 * ROWS) *reinterpret_cast<u32v4 *>(wsm + 27 * ROWS * 32 + tid * 16) = u32v4{0, 0, 0, 0};
    for (int c = 0; c < nchunk; ++c) {
        if (c > 0) __syncthreads();           // every wave is done with the chunk before
        int tl = tid;
        asm("" : "+v"(tl));
#pragma unroll
        for (int k = 0; k < XI; ++k)
            if (tl + k * 256 < NHALO * 2) *reinterpret_cast<u32v4 *>(xs + (tl + k * 256) * 16) = sx[k];
#pragma unroll
        for (int k = 0; k < WI; ++k) {
            const int i = tl + k * 256;
            if (i >= WITEMS) continue;
            if constexpr (BWD) {
                *reinterpret_cast<u32v4 *>(wsm + i * 16) = sw[k];
            } else {
                const int tap = i / (2 * ROWS), oct = (i >> 4) % (2 * MB), k0 = i & 15;
                bf16_t *o = reinterpret_cast<bf16_t *>(wsm) + (tap * ROWS + oct * 8) * 16 + k0;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e * 16] = (bf16_t)(sw[k][e >> 1] >> (16 * (e & 1)));
            }
        }
        __syncthreads();
        if (c + 1 < nchunk) fetch(c + 1);
        bf16x8 a[2][MB], b[2][NB];            // the next step's operands are read while one is multiplied
        auto operands = [&](int s, bf16x8 (&as)[MB], bf16x8 (&bs)[NB]) __attribute__((always_inline)) {
            auto off = [](int tap) { return (((tap / 9) * HH + (tap / 3) % 3) * HW + tap % 3) * 32; };
            const unsigned char *xt = x + (second ? off(2 * s + 1) : off(2 * s));
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) as[mb] = *reinterpret_cast<const bf16x8 *>(a0 + s * 2 * ROWS * 32 + mb * 512);
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const unsigned char *q = xt + k * 2 * HW * 32;
                if (s == 13) q = second ? xs + NHALO * 32 + half * 16 : q;
                bs[k] = *reinterpret_cast<const bf16x8 *>(q);
            }
        };
        operands(0, a[0], b[0]);
#pragma unroll
        for (int s = 0; s < 14; ++s) {
            if (s < 13) operands(s + 1, a[(s + 1) & 1], b[(s + 1) & 1]);
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
                    acc[k][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[s & 1][mb], b[s & 1][k], acc[k][mb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (c + 1 < nchunk) fetch_weights(c + 1);   // from the L2; not held in registers across the steps
    }
#pragma unroll
    for (int k = 0; k < NB; ++k) {
        const int d = d0 + plane, h = h0 + row0 + 2 * k + (ln >> 3), w = w0 + (ln & 7);
        const bool in = d < p.D && h < p.H && w < p.W;
        const int64_t vox = (((int64_t)n * p.D + d) * p.H + h) * p.W + w;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            if (m0 + mb * 16 < M) store_block16(p, acc[k][mb], in, vox, m0 + mb * 16, kg);
    }
}

// dW[tap][ci][co] = sum over voxels of x[v + tap][ci] * g[v][co] for one 16-channel block of each: the
// contraction runs over 32 voxels (four rows of 8) per instruction, operands through the transposing LDS
// read (lane j of 16 supplies the address of 4 channels of voxel j / 4, lane i receives channel i of the
// 4 voxels).  The waves split the taps 7/7/7/6, the spare slot multiplies ones: the bias gradient.  A
// workgroup takes every nsplit-th tile, the next one's loads in flight, and writes one set of partial sums.
struct NarrowWgrad {
    const bf16_t *x1, *x2, *g, *mask;
    unsigned mask_top;        // MASK_NUMBERS; in place of the kernel for whole 32s MASK_SIGN, as there
    int c1, c2, cout;
    float *outW, *outB;       // first set of partial sums and its bias part, or the gradients themselves (outB may be null)
    int64_t per_split;
    int N, D, H, W, ntd, nth, ntw, tiles, nsplit, ncb;   // ncb: 16-channel blocks of cout
};

__device__ __forceinline__ bf16x8 tr8(const unsigned char *p)     // 8 voxels, 32 bytes each
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * 32));
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

template <int TD>
__global__ __launch_bounds__(256, 3) void conv_narrow_wgrad_kernel(NarrowWgrad p)
{
    constexpr int TH = 8, TW = 8, HH = TH + 2, HW = TW + 2, NHALO = (TD + 2) * HH * HW, NV = TD * TH * TW;
    constexpr int XI = (NHALO * 2 + 255) / 256, GI = NV * 2 / 256;
    static_assert(NV * 2 % 256 == 0, "whole items");
    __shared__ __attribute__((aligned(16))) unsigned char xs[NHALO * 32];
    __shared__ __attribute__((aligned(16))) unsigned char gs[NV * 32];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int cin = p.c1 + p.c2;
    const int split = (int)(blockIdx.x % (unsigned)p.nsplit), blk = (int)(blockIdx.x / (unsigned)p.nsplit);
    const int ci0 = (blk / p.ncb) * 16, co0 = (blk % p.ncb) * 16;
    const bool first = ci0 < p.c1;
    const bf16_t *src = first ? p.x1 + ci0 : p.x2 + (ci0 - p.c1);
    const int cx = first ? p.c1 : p.c2;
    u32v4 sx[XI], sg[GI];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        int t = tile;
        const int w0 = (t % p.ntw) * TW;
        t /= p.ntw;
        const int h0 = (t % p.nth) * TH;
        t /= p.nth;
        const int d0 = (t % p.ntd) * TD;
        const int n = t / p.ntd;
        const int64_t g0 = (((int64_t)n * p.D + d0) * p.H + h0) * p.W + w0, x0 = g0 - ((int64_t)p.H * p.W + p.W + 1);
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(src + x0 * cx), 0, 0x7ffffff0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.g + g0 * p.cout + co0), 0, 0x7ffffff0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.mask ? p.mask : p.g) + g0 * p.cout + co0), 0, 0x7ffffff0, 0x00020000);
#pragma unroll
        for (int k = 0; k < XI; ++k) {
            const int v = (tid + k * 256) >> 1, lw = v % HW, lh = (v / HW) % HH, ld = v / (HW * HH);
            const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
            const bool in = v < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W;
            sx[k] = __builtin_amdgcn_raw_buffer_load_b128(rx, in ? (((ld * p.H + lh) * p.W + lw) * cx + (tid & 1) * 8) * 2 : -1, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < GI; ++k) {
            const int v = (tid + k * 256) >> 1, lw = v % TW, lh = (v / TW) % TH, ld = v / (TW * TH);
            const bool in = d0 + ld < p.D && h0 + lh < p.H && w0 + lw < p.W;
            const int o = in ? (((ld * p.H + lh) * p.W + lw) * p.cout + (tid & 1) * 8) * 2 : -1;
            sg[k] = __builtin_amdgcn_raw_buffer_load_b128(rg, o, 0, 0);
            if (p.mask) {
                const u32v4 m = __builtin_amdgcn_raw_buffer_load_b128(rm, o, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) sg[k][j] = mask_pair_to(sg[k][j], m[j], p.mask_top);
            }
        }
    };
    const unsigned char *xa[7];       // the lane's address for each tap of the wave, first plane
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int tap = wv * 7 + j < 27 ? wv * 7 + j : 26;
        xa[j] = xs + ((((tap / 9) * HH + (tap / 3) % 3 + kg) * HW) + tap % 3 + (ln >> 2)) * 32 + (ln & 3) * 8;
    }
    const unsigned char *ga = gs + (kg * TW + (ln >> 2)) * 32 + (ln & 3) * 8;
    const bool ones = wv == 3;
    bf16x8 one;
#pragma unroll
    for (int i = 0; i < 8; ++i) one[i] = (__bf16)1.0f;
    f32x4 acc[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    int tile = split;
    fetch(tile);
    while (true) {
#pragma unroll
        for (int k = 0; k < XI; ++k)
            if (tid + k * 256 < NHALO * 2) *reinterpret_cast<u32v4 *>(xs + (tid + k * 256) * 16) = sx[k];
#pragma unroll
        for (int k = 0; k < GI; ++k) *reinterpret_cast<u32v4 *>(gs + (tid + k * 256) * 16) = sg[k];
        __syncthreads();
        const int next = tile + p.nsplit;
        if (next < p.tiles) fetch(next);
#pragma unroll
        for (int q = 0; q < NV / 32; ++q) {
            const bf16x8 b = tr8(ga + q * 4 * TW * 32);
            const int off = ((q >> 1) * HH + (q & 1) * 4) * HW * 32;
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                bf16x8 a = tr8(xa[j] + off);
                if (j == 6 && ones) a = one;
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[j], 0, 0, 0);
            }
        }
        tile = next;
        if (tile >= p.tiles) break;
        __syncthreads();
    }
    float *out = p.outW + split * p.per_split + co0 + ln;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int tap = wv * 7 + j;
        if (tap < 27) {
#pragma unroll
            for (int r = 0; r < 4; ++r) out[((int64_t)tap * cin + ci0 + kg * 4 + r) * p.cout] = acc[j][r];
        } else if (ci0 == 0 && kg == 0 && p.outB) {
            p.outB[split * p.per_split + co0 + ln] = acc[j][0];   // every row holds the sum of g
        }
    }
}

// The first layer of a 16-filter network, one input channel: the 27 taps are the contraction (forward:
// one matrix instruction per 16 voxels, padded to 32) or the rows (backward-weight: two blocks of 16, row
// 27 multiplies ones, the bias gradient).  4 x 8 x 16-voxel tiles; a lane gathers its operand from the
// bf16 halo tile in LDS with 2-byte reads.  Replaces the thread-per-channel kernels at 16 channels:
// 2 x 40x48x56 forward with bits 16 -> 12 us, backward-weight 45 -> 14 us with its reduction.
namespace first16 {
constexpr int TD = 4, TH = 8, TW = 16, HH = TH + 2, HW = TW + 2, NHALO = (TD + 2) * HH * HW, NV = TD * TH * TW;
constexpr int XI = (NHALO + 255) / 256;
__device__ __forceinline__ int tap_offset(int tap) { return ((tap / 9) * HH + (tap / 3) % 3) * HW + tap % 3; }

__device__ __forceinline__ void fetch_x(const bf16_t *x, int n, int d0, int h0, int w0, int D, int H, int W, bf16_t (&r)[XI])
{
#pragma unroll
    for (int k = 0; k < XI; ++k) {
        const int v = threadIdx.x + k * 256, lw = v % HW, lh = (v / HW) % HH, ld = v / (HW * HH);
        const int gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
        r[k] = 0;
        if (v < NHALO && gd >= 0 && gd < D && gh >= 0 && gh < H && gw >= 0 && gw < W) r[k] = x[(((int64_t)n * D + gd) * H + gh) * W + gw];
    }
}
}  // namespace first16

__global__ __launch_bounds__(256) void conv_first16_fwd_kernel(NarrowParams p)
{
    using namespace first16;
    __shared__ bf16_t xs[NHALO + 8];      // values beyond the tile: zeros, what the padding taps read
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    unsigned t = blockIdx.x;
    const int w0 = (int)(t % (unsigned)p.ntw) * TW;
    t /= (unsigned)p.ntw;
    const int h0 = (int)(t % (unsigned)p.nth) * TH;
    t /= (unsigned)p.nth;
    const int d0 = (int)(t % (unsigned)p.ntd) * TD;
    const int n = (int)(t / (unsigned)p.ntd);
    bf16_t r[XI];
    fetch_x(p.src1, n, d0, h0, w0, p.D, p.H, p.W, r);
    typedef __attribute__((ext_vector_type(8))) unsigned short u16x8;
    u16x8 wr;
#pragma unroll
    for (int e = 0; e < 8; ++e) wr[e] = kg * 8 + e < 27 ? p.w[(kg * 8 + e) * 16 + ln] : (unsigned short)0;
    const bf16x8 a = __builtin_bit_cast(bf16x8, wr);
#pragma unroll
    for (int k = 0; k < XI; ++k)
        if (tid + k * 256 < NHALO) xs[tid + k * 256] = r[k];
    if (tid < 8) xs[NHALO + tid] = 0;
    __syncthreads();
    const int d = d0 + wv;                // a wave's blocks are the rows of one plane
#pragma unroll
    for (int b = 0; b < TH; ++b) {
        u16x8 xr;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int tap = kg * 8 + e;
            xr[e] = xs[tap < 27 ? (wv * HH + b) * HW + ln + tap_offset(tap) : NHALO];
        }
        const f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, xr), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        const int h = h0 + b, w = w0 + ln;
        store_block16(p, acc, d < p.D && h < p.H && w < p.W, (((int64_t)n * p.D + d) * p.H + h) * p.W + w, 0, kg);
    }
}

__global__ __launch_bounds__(256) void conv_first16_wgrad_kernel(NarrowWgrad p)
{
    using namespace first16;
    constexpr int GI = NV * 2 / 256;
    __shared__ bf16_t xs[NHALO];
    __shared__ __attribute__((aligned(16))) unsigned char gs[NV * 32];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    bf16_t rx[XI];
    u32v4 sg[GI];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        int t = tile;
        const int w0 = (t % p.ntw) * TW;
        t /= p.ntw;
        const int h0 = (t % p.nth) * TH;
        t /= p.nth;
        const int d0 = (t % p.ntd) * TD;
        const int n = t / p.ntd;
        fetch_x(p.x1, n, d0, h0, w0, p.D, p.H, p.W, rx);
#pragma unroll
        for (int k = 0; k < GI; ++k) {
            const int v = (tid + k * 256) >> 1, d = d0 + v / (TW * TH), h = h0 + (v / TW) % TH, w = w0 + v % TW;
            const int64_t o = ((((int64_t)n * p.D + d) * p.H + h) * p.W + w) * 16 + (tid & 1) * 8;
            sg[k] = u32v4{0, 0, 0, 0};
            if (d < p.D && h < p.H && w < p.W) {
                sg[k] = *reinterpret_cast<const u32v4 *>(p.g + o);
                if (p.mask) {
                    const u32v4 m = *reinterpret_cast<const u32v4 *>(p.mask + o);
#pragma unroll
                    for (int j = 0; j < 4; ++j) sg[k][j] = mask_pair_to(sg[k][j], m[j], MASK_NUMBERS);
                }
            }
        }
    };
    // rows ln and 16 + ln of the result are taps; row 27 is the ones row, rows beyond are not kept
    const int t0 = tap_offset(ln), t1 = tap_offset(ln < 11 ? 16 + ln : 26);
    const int xl = (kg >> 1) * HW + (kg & 1) * 8;      // the lane group's eight voxels of a step: half of one of its two rows
    const unsigned char *ga = gs + ((kg >> 1) * TW + (kg & 1) * 8 + (ln >> 2)) * 32 + (ln & 3) * 8;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    typedef __attribute__((ext_vector_type(8))) unsigned short u16x8;
    int tile = blockIdx.x;
    fetch(tile);
    while (true) {
#pragma unroll
        for (int k = 0; k < XI; ++k)
            if (tid + k * 256 < NHALO) xs[tid + k * 256] = rx[k];
#pragma unroll
        for (int k = 0; k < GI; ++k) *reinterpret_cast<u32v4 *>(gs + (tid + k * 256) * 16) = sg[k];
        __syncthreads();
        const int next = tile + p.nsplit;
        if (next < p.tiles) fetch(next);
#pragma unroll
        for (int q = 0; q < 4; ++q) {                   // the wave's plane, two rows a step
            const bf16_t *x = xs + (wv * HH + 2 * q) * HW + xl;
            u16x8 a0, a1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                a0[e] = x[t0 + e];
                a1[e] = x[t1 + e];
            }
            if (ln == 11) a1 = u16x8{0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80, 0x3f80};
            const bf16x8 b = tr8(ga + (wv * TH + 2 * q) * TW * 32);
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), b, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), b, acc[1], 0, 0, 0);
        }
        __syncthreads();
        tile = next;
        if (tile >= p.tiles) break;
    }
    float *red = reinterpret_cast<float *>(gs);         // the waves' sums, added in wave order
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv * 512 + (i * 16 + kg * 4 + r) * 16 + ln] = acc[i][r];
    __syncthreads();
    float *out = p.outW + blockIdx.x * p.per_split;
    for (int i = tid; i < 28 * 16; i += 256) out[i] = ((red[i] + red[512 + i]) + red[1024 + i]) + red[1536 + i];
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// 16 output channels of one input channel; tiles are counted in 31 bits by conv_first_ok's callers
bool conv_first16_ok(const ConvArgs &a) { return a.cout == 16 && aligned16(a.y) && aligned16(a.dy) && aligned16(a.ymask); }

int conv_first16_fwd(const ConvArgs &a, int ntd, int nth, int ntw, int64_t tiles, hipStream_t st)
{
    NarrowParams p{};
    p.src1 = (const bf16_t *)a.x; p.w = (const bf16_t *)a.w; p.bias = a.bias; p.relu = a.relu;
    p.dst1 = (bf16_t *)a.y; p.cd1 = 16; p.bits_out = (unsigned short *)a.ybits;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    p.ntd = ntd; p.nth = nth; p.ntw = ntw;
    conv_first16_fwd_kernel<<<dim3((unsigned)tiles), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

int conv_first16_wgrad(const ConvArgs &a, float *dW, float *db, float *ws, int ntd, int nth, int ntw, int64_t tiles, hipStream_t st)
{
    NarrowWgrad p{};
    p.x1 = (const bf16_t *)a.x; p.g = (const bf16_t *)a.dy; p.mask = (const bf16_t *)a.ymask;
    p.outW = ws; p.per_split = 28 * 16;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    p.ntd = ntd; p.nth = nth; p.ntw = ntw;
    p.tiles = (int)tiles;
    p.nsplit = (int)(tiles < 512 ? tiles : 512);        // two workgroups per CU cover each other's loads
    conv_first16_wgrad_kernel<<<dim3((unsigned)p.nsplit), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return launch_reduce_partials(ws, dW, db, 27 * 16, p.per_split, p.nsplit, st);
}

bool conv_narrow_ok(const ConvArgs &a)
{
    if (a.dtype != K3_BF16 || a.c1 % 16 || a.c2 % 16 || a.cout % 16) return false;
    const int64_t c = a.c1 + a.c2 > a.cout ? a.c1 + a.c2 : a.cout;
    if (c > 4096 || 6 * (a.H + 1) * a.W * c * 2 >= 0x7fffffffLL) return false;   // 32-bit offsets inside a tile
    for (const void *p : {a.x, a.x2, (const void *)a.y, a.dy, a.ymask, (const void *)a.dx, (const void *)a.dx2, a.omask})
        if (!aligned16(p)) return false;
    return true;
}

template <int TD, int TH, int MB, bool BWD>
static int launch_narrow(NarrowParams p, hipStream_t st)
{
    p.ntd = (p.D + TD - 1) / TD;
    p.nth = (p.H + TH - 1) / TH;
    p.ntw = (p.W + 7) / 8;
    p.ncg = (p.cd1 + p.cd2 + 16 * MB - 1) / (16 * MB);
    p.total = (int64_t)p.N * p.ntd * p.nth * p.ntw * p.ncg;
    p.per_xcd = (p.total + 7) / 8;
    if (p.per_xcd * 8 > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    conv_narrow_kernel<TD, TH, MB, BWD><<<dim3((unsigned)(p.per_xcd * 8)), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

// 256-voxel tiles where they give every CU a workgroup, else 64-voxel ones; two output blocks per
// workgroup where that still does
template <bool BWD>
static int launch_narrow_size(const NarrowParams &p, hipStream_t st)
{
    const int64_t M = p.cd1 + p.cd2, big = (int64_t)p.N * ((p.D + 3) / 4) * ((p.H + 7) / 8) * ((p.W + 7) / 8);
    if (M > 16 && big * ((M + 31) / 32) >= 256) return launch_narrow<4, 8, 2, BWD>(p, st);
    if (big * (M / 16) >= 256) return launch_narrow<4, 8, 1, BWD>(p, st);
    return launch_narrow<2, 4, 1, BWD>(p, st);
}

int conv_fwd_narrow(const ConvArgs &a, hipStream_t st)
{
    NarrowParams p{};
    p.src1 = (const bf16_t *)a.x; p.src2 = (const bf16_t *)a.x2;
    p.c1 = (int)a.c1; p.c2 = (int)a.c2;
    p.w = (const bf16_t *)a.w; p.bias = a.bias; p.relu = a.relu;
    p.dst1 = (bf16_t *)a.y; p.cd1 = (int)a.cout; p.bits_out = (unsigned short *)a.ybits;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    return launch_narrow_size<false>(p, st);
}

int conv_dgrad_narrow(const ConvArgs &a, hipStream_t st)
{
    NarrowParams p{};
    p.src1 = (const bf16_t *)a.dy; p.mask = (const bf16_t *)a.ymask;
    p.c1 = (int)a.cout;
    p.w = (const bf16_t *)a.w;
    p.dst1 = (bf16_t *)a.dx; p.dst2 = (bf16_t *)a.dx2;
    p.omask = (const bf16_t *)a.omask; p.omask_bits = (const unsigned short *)a.omask_bits;
    p.cd1 = (int)a.c1; p.cd2 = (int)a.c2;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    return launch_narrow_size<true>(p, st);
}

// 256-voxel tiles where every CU gets one, else 128-voxel ones; about 512 workgroups in all, each with
// a whole number of tiles, and no more sets of partial sums than the workspace query promises.  One
// workgroup per block of channels that walks all tiles and writes the gradient itself saves the sets
// and the reduction's launch: a 256-voxel tile after another costs 2.4 us, the reduction 3.4 us and
// 0.02 us for each workgroup's set (8^3 128->128 with 4 sets 10.4 us, direct 8.2; 2x8^3 64->64 8.5, direct 12.7).
int conv_wgrad_narrow(const ConvArgs &a, float *dW, float *db, float *ws, int64_t max_sets, hipStream_t st)
{
    NarrowWgrad p{};
    const int64_t cin = a.c1 + a.c2, blocks = cin / 16 * (a.cout / 16), hw = ((a.H + 7) / 8) * ((a.W + 7) / 8);
    const int64_t big = a.N * ((a.D + 3) / 4) * hw;
    bool small = big * blocks < 256;
    int64_t tiles = small ? a.N * ((a.D + 1) / 2) * hw : big;
    int64_t want = 512 / blocks;
    if (want > max_sets) want = max_sets;
    if (want < 1) want = 1;
    const int64_t each = (tiles + want - 1) / want;
    int64_t nsplit = (tiles + each - 1) / each;
    if (120 * (big - each + 1) < 170 + nsplit * blocks) nsplit = 1;
    if (nsplit == 1 && small) {
        small = false;
        tiles = big;
    }
    if (tiles > 0x7fffffffLL || nsplit * blocks > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    p.x1 = (const bf16_t *)a.x; p.x2 = (const bf16_t *)a.x2;
    p.g = (const bf16_t *)a.dy; p.mask = (const bf16_t *)a.ymask;
    p.mask_top = mfma_ok(K3_BF16, a.c1, a.c2, a.cout) ? MASK_SIGN : MASK_NUMBERS;
    p.c1 = (int)a.c1; p.c2 = (int)a.c2; p.cout = (int)a.cout;
    p.per_split = 27 * cin * a.cout + a.cout;
    p.outW = nsplit > 1 ? ws : dW;
    p.outB = nsplit > 1 ? ws + 27 * cin * a.cout : db;
    p.N = (int)a.N; p.D = (int)a.D; p.H = (int)a.H; p.W = (int)a.W;
    p.ntd = small ? (p.D + 1) / 2 : (p.D + 3) / 4;
    p.nth = (p.H + 7) / 8;
    p.ntw = (p.W + 7) / 8;
    p.tiles = (int)tiles;
    p.nsplit = (int)nsplit;
    p.ncb = (int)(a.cout / 16);
    const dim3 grid((unsigned)(nsplit * blocks));
    if (small) conv_narrow_wgrad_kernel<2><<<grid, 256, 0, st>>>(p);
    else conv_narrow_wgrad_kernel<4><<<grid, 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    if (nsplit == 1) return K3_OK;
    return launch_reduce_partials(ws, dW, db, 27 * cin * a.cout, p.per_split, (int)nsplit, st);
}

}  // namespace k3

// bf16 3x3x3 convolution (forward and backward-data) for volumes that do not fill the chip with the
// tiles of conv3d_mfma.hip: the deep levels of a network and training on small blocks.
//
// Bound: latency.  With a dozen tiles there is one short chain per workgroup -- halo and weights
// from L2, some hundred matrix instructions, store -- and what counts is its length.  So the work is
// cut fine (64 or 128 voxels x 16 or 32 output channels per workgroup), the four waves of a workgroup
// split the contraction (taps x channels) and add their sums through LDS, the weights go from the
// packed buffer straight into registers several steps ahead, and all of a channel group's halo
// loads are in flight at once.  The kernel this replaces walked 16-channel chunks one after the
// other in 512-voxel tiles, two barriers and one exposed load latency per chunk and tap group.
#include "common.h"
#include "conv_internal.h"
#include "conv_mfma.h"
#include "index_math.h"

namespace k3 {

// 16x16x32 matrix instruction: rows = 16 output channels, columns = 16 voxels, contraction = 32
// channels of one tap (lane group kg = lane / 16 carries channels 8 kg .. 8 kg + 7).  A tile is
// 4 x 4 x 4 voxels = 4 blocks of one 4x4 (h, w) plane; MB output blocks of 16 channels.  One chunk of
// 32 input channels is in LDS (pitch 80 bytes per voxel: the lanes of a read fall on different bank
// quads), the next one's halo in registers.  Wave w takes taps w, w + 4, ...; the weights of its seven
// steps of a chunk are requested while the chunk before is multiplied.
template <int MB>
__global__ __launch_bounds__(256, MB == 1 ? 3 : 2) void conv_small_kernel(MfmaParams p)
{
    constexpr int NHALO = 216, PITCH = 80;
    constexpr int ITEMS = (NHALO * 4 + 255) / 256;
    constexpr int RED = 4 * 4 * MB * 1024;
    __shared__ __attribute__((aligned(16))) unsigned char smem[NHALO * PITCH > RED ? NHALO * PITCH : RED];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int K = p.c1 + p.c2, M = p.cd1 + p.cd2, nkc = K / 16, nck = (K + 31) / 32;

    // a contiguous run of the logical order per XCD; the channel groups of a tile are neighbours
    const int64_t logical = (int64_t)(blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (logical >= p.total) return;
    const int m0 = (int)(logical % p.ncg) * 16 * MB;
    int64_t t = logical / p.ncg;
    const int w0 = (int)(t % p.ntw) * 4;
    t /= p.ntw;
    const int h0 = (int)(t % p.nth) * 4;
    t /= p.nth;
    const int d0 = (int)(t % p.ntd) * 4;
    const int n = (int)(t / p.ntd);

    // weights of (tap j of the wave, chunk c): row ln of the block <-> packed row, slot kg <-> (half chunk, lane half)
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(p.packed) + packed_block(m0 >> 5, nkc) / 2, 0, 0x7ffffff0, 0x00020000);   // (the blocks of a workgroup lie in one)
    const unsigned wlane = (unsigned)((kg >> 1) * 1024 + ((kg & 1) * 32 + (ln >> 2) * 8 + (ln & 3)) * 16);
    auto weights = [&](int c, int j, bf16x8 (&a)[MB]) __attribute__((always_inline)) {
        const bool there = 2 * c + (kg >> 1) < nkc;     // an odd number of 16-channel steps ends in half a chunk
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = m0 + mb * 16;
            const unsigned soff = packed_step(wv + 4 * j, nkc, 2 * c) + ((m >> 4) & 1) * 64;
            a[mb] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, there && m < M ? wlane : 0xffffffffu, soff, 0));
        }
    };
    const int ntap = wv < 3 ? 7 : 6;                     // taps of this wave
    int toff[7];                                         // LDS offset of each
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int tap = wv + 4 * j;
        toff[j] = (((tap / 9) * 6 + (tap / 3) % 3) * 6 + tap % 3) * PITCH;
    }

    // the lane's halo items of a chunk: (voxel, 8 channels)
    const int64_t halo0 = (((int64_t)n * p.D + d0 - 1) * p.H + h0 - 1) * p.W + w0 - 1;
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.src1 + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.src2 ? p.src2 : p.src1) + halo0 * p.c2), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.mask ? p.mask : p.src1) + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    u32v4 st[ITEMS];
    auto fetch = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int i = tid + k * 256, v = i >> 2, q = i & 3;
            const int lw = v % 6, lh = (v / 6) % 6, ld = v / 36;
            const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
            const int ch = c * 32 + q * 8;
            const bool in = v < NHALO && ch < K && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W;
            const int vo = (ld * p.H + lh) * p.W + lw;
            const bool first = ch < p.c1;
            const int o1 = in && first ? (vo * p.c1 + ch) * 2 : -1;
            st[k] = __builtin_amdgcn_raw_buffer_load_b128(r1, o1, 0, 0);
            if (p.c2 > 0) {
                const int o2 = in && !first ? (vo * p.c2 + ch - p.c1) * 2 : -1;
                st[k] |= __builtin_amdgcn_raw_buffer_load_b128(r2, o2, 0, 0);
            }
            if (p.mask) {
                const u32v4 m = __builtin_amdgcn_raw_buffer_load_b128(rm, o1, 0, 0);
#pragma unroll
                for (int j = 0; j < 4; ++j) st[k][j] = mask_pair(st[k][j], m[j]);
            }
        }
    };
    // LDS address of the lane's voxel in plane 0
    const unsigned char *x = smem + ((ln >> 2) * 6 + (ln & 3)) * PITCH + kg * 16;
    f32x4 acc[4][MB];
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[d][mb] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 a[7][MB];
#pragma unroll
    for (int j = 0; j < 7; ++j)
        if (j < ntap) weights(0, j, a[j]);
    fetch(0);
    for (int c = 0; c < nck; ++c) {
        if (c > 0) __syncthreads();     // every wave is done with the chunk before
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) {
            const int i = tid + k * 256;
            if (i < NHALO * 4) *reinterpret_cast<u32v4 *>(smem + (i >> 2) * PITCH + (i & 3) * 16) = st[k];
        }
        __syncthreads();
        const bool more = c + 1 < nck;
        if (more) fetch(c + 1);
        bf16x8 b[2][4];
#pragma unroll
        for (int d = 0; d < 4; ++d) b[0][d] = *reinterpret_cast<const bf16x8 *>(x + toff[0] + d * 36 * PITCH);
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            if (j < 6 || ntap == 7) {              // wave-uniform
                if (j < 5 || (j == 5 && ntap == 7)) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) b[(j + 1) & 1][d] = *reinterpret_cast<const bf16x8 *>(x + toff[j + 1] + d * 36 * PITCH);
                }
#pragma unroll
                for (int d = 0; d < 4; ++d)
#pragma unroll
                    for (int mb = 0; mb < MB; ++mb) acc[d][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j][mb], b[j & 1][d], acc[d][mb], 0, 0, 0);
                if (more) weights(c + 1, j, a[j]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // the waves' sums, added in wave order; wave wv finishes (plane, output block) wv, wv + 4, ...
    __syncthreads();
#pragma unroll
    for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) *reinterpret_cast<f32x4 *>(smem + (((wv * 4 + d) * MB + mb) * 64 + lane) * 16) = acc[d][mb];
    __syncthreads();
    for (int qm = wv; qm < 4 * MB; qm += 4) {
        const int d = qm / MB, mb = qm % MB, h = ln >> 2, w = ln & 3;
        f32x4 s = *reinterpret_cast<const f32x4 *>(smem + (qm * 64 + lane) * 16);
#pragma unroll
        for (int k = 1; k < 4; ++k) s += *reinterpret_cast<const f32x4 *>(smem + ((k * 4 * MB + qm) * 64 + lane) * 16);
        if (m0 + mb * 16 >= M) continue;                       // wave-uniform
        const bool in = d0 + d < p.D && h0 + h < p.H && w0 + w < p.W;
        const int64_t vox = (((int64_t)n * p.D + d0 + d) * p.H + h0 + h) * p.W + w0 + w;
        store_block16(p, s, in, vox, m0 + mb * 16, kg);
    }
}

template <int MB>
static int launch_small_t(MfmaParams p, hipStream_t st)
{
    p.ntd = (p.D + 3) / 4;
    p.nth = (p.H + 3) / 4;
    p.ntw = (p.W + 3) / 4;
    p.ncg = (p.cd1 + p.cd2 + 16 * MB - 1) / (16 * MB);
    p.total = (int64_t)p.N * p.ntd * p.nth * p.ntw * p.ncg;
    p.per_xcd = (p.total + 7) / 8;
    if (p.per_xcd * 8 > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    conv_small_kernel<MB><<<dim3((unsigned)(p.per_xcd * 8)), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

// One 16-channel block per workgroup while that gives no more than one per CU (8^3 256->256: 13.5 us
// against 15.9 with two), else two (16^3 128->128: 10.5 against 12.1).
int launch_conv_small(MfmaParams p, hipStream_t st)
{
    const int64_t tiles = (int64_t)p.N * ((p.D + 3) / 4) * ((p.H + 3) / 4) * ((p.W + 3) / 4);
    if (tiles * ((p.cd1 + p.cd2) / 16) <= 256) return launch_small_t<1>(p, st);
    return launch_small_t<2>(p, st);
}

}  // namespace k3

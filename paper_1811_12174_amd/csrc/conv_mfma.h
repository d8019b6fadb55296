// What the bf16 matrix-core forward / backward-data kernels share: launch parameters, the packed
// weight order, the ReLU mask on packed pairs.
#pragma once
#include "common.h"

namespace k3 {

// acc index i of lane half hb maps to MFMA row (i/4)*8 + hb*4 + i%4; row r therefore
// carries channel (r/4%2)*16 + (r/8)*4 + r%4 of its 32-channel block.
__host__ __device__ static inline int row_to_channel(int r) { return ((r >> 2) & 1) * 16 + (r >> 3) * 4 + (r & 3); }

struct MfmaParams {
    const bf16_t *src1, *src2, *mask;  // mask applies to src1 (src2 is null whenever mask is set)
    int c1, c2;                        // contraction channels per source
    const bf16_t *packed;              // [mblk][27][nkc][64][8]
    const float *bias;
    int relu;
    bf16_t *dst1, *dst2;
    const bf16_t *omask;               // optional: dst1 is zeroed where omask (same shape) is <= 0
    const unsigned short *omask_bits;  // the same mask as one bit per element (word j of a voxel: channels 16j..16j+15)
    unsigned short *bits_out;          // optional: receives that bit mask of dst1 (set where the stored value is > 0)
    bf16_t *pool_out;                  // optional (plane-streaming kernel, ReLU on): receives the 2x2x2 max-pool of dst1
    int cd1, cd2;                      // output channels per destination
    int N, D, H, W;
    int ntd, nth, ntw;                 // tiles per axis
    int ncg;                           // output-channel groups (of 32*MB)
    int64_t total, per_xcd;            // logical blocks, and blocks per XCD slice
};

__device__ __forceinline__ uint32_t mask_pair(uint32_t v, uint32_t m)
{
    // keep each bf16 half of v where the matching half of m is > 0 (sign clear and nonzero)
    uint32_t lo = ((m & 0x8000u) == 0 && (m & 0x7fffu) != 0) ? 0x0000ffffu : 0u;
    uint32_t hi = ((m & 0x80000000u) == 0 && (m & 0x7fff0000u) != 0) ? 0xffff0000u : 0u;
    return v & (lo | hi);
}

// The same with the bf16 values 1 .. top of m, as integers, counting as positive: MASK_NUMBERS keeps only what
// compares > 0, MASK_SIGN also a NaN whose sign is clear, like mask_pair.
constexpr unsigned MASK_NUMBERS = 0x7f80u, MASK_SIGN = 0x7fffu;
__device__ __forceinline__ uint32_t mask_pair_to(uint32_t v, uint32_t m, unsigned top)
{
    const uint32_t lo = (m & 0xffffu) - 1u < top ? 0x0000ffffu : 0u;
    const uint32_t hi = (m >> 16) - 1u < top ? 0xffff0000u : 0u;
    return v & (lo | hi);
}

typedef __attribute__((ext_vector_type(4))) unsigned u32v4;
typedef __attribute__((ext_vector_type(2))) unsigned u32v2;

// Ends a 16x16 result block: the lane holds output channels mblk + 4 kg .. + 3 of voxel vox (its lane
// group's 16 voxels; in: the voxel exists).  Bias, ReLU, rounding, the output masks and the bit mask.
__device__ __forceinline__ void store_block16(const MfmaParams &p, f32x4 s, bool in, int64_t vox, int mblk, int kg)
{
    const int m = mblk + kg * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float v = s[r] + (p.bias ? p.bias[m + r] : 0.f);
        s[r] = p.relu && !(v > 0.f) ? 0.f : v;
    }
    u32v2 o = {pack2bf(s[0], s[1]), pack2bf(s[2], s[3])};
    const bool d1 = mblk < p.cd1;                          // a 16-channel block lies in one destination
    const int64_t eo = d1 ? vox * p.cd1 + m : vox * p.cd2 + (m - p.cd1);
    if (in && d1 && p.omask) {
        const u32v2 k = *reinterpret_cast<const u32v2 *>(p.omask + eo);
        o[0] = mask_pair_to(o[0], k[0], MASK_NUMBERS);
        o[1] = mask_pair_to(o[1], k[1], MASK_NUMBERS);
    }
    if (in && d1 && p.omask_bits) {
        const unsigned k = p.omask_bits[vox * (p.cd1 / 16) + mblk / 16] >> (kg * 4);
        o[0] &= (k & 1u ? 0xffffu : 0u) | (k & 2u ? 0xffff0000u : 0u);
        o[1] &= (k & 4u ? 0xffffu : 0u) | (k & 8u ? 0xffff0000u : 0u);
    }
    if (in) *reinterpret_cast<u32v2 *>((d1 ? p.dst1 : p.dst2) + eo) = o;
    if (p.bits_out) {   // (forward: one destination) the four lane groups hold four bits each of the voxel's word
        const unsigned z0 = mask_pair_to(0x00010001u, o[0], MASK_NUMBERS), z1 = mask_pair_to(0x00010001u, o[1], MASK_NUMBERS);
        unsigned z = (z0 & 1u) | ((z0 >> 15) & 2u) | ((z1 & 1u) << 2) | ((z1 >> 13) & 8u);
        z <<= kg * 4;
        z |= __shfl_xor(z, 16);
        z |= __shfl_xor(z, 32);
        if (in && kg == 0) p.bits_out[vox * (p.cd1 / 16) + mblk / 16] = (unsigned short)z;
    }
}

// Weight packing (weights_pack.hip): one canonical tensor and where its packed forms go.
typedef __attribute__((ext_vector_type(4), aligned(2))) unsigned u32x4_pk;   // 16 bytes at any bf16 address
struct PackJob {
    const bf16_t *w;
    bf16_t *packed;
    int cin, cout, taps;   // taps: 27 (3x3x3) or 8 (transposed)
};
constexpr int PACK_JOBS = 48;
int launch_pack(const PackJob *jobs, int n, hipStream_t st);

// Small volumes (conv3d_small.hip).
int launch_conv_small(MfmaParams p, hipStream_t st);

}  // namespace k3

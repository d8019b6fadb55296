// bf16 3x3x3 convolution (forward and backward-data) for volumes that do not fill the chip with the
// tiles of conv3d_mfma.hip: the deep levels of a network and training on small blocks.
//
// Bound: latency.  With a dozen tiles there is one short chain per wave -- halo from memory, 27 K / 16
// matrix instructions that depend on each other, store -- and what counts is its length: so a wave takes
// no more than 32 voxels x 32 channels, the halo loads of up to 128 channels are all in flight at once,
// and the weights go from the packed buffer straight into registers, a whole step of 27 ahead.  The chain is
// not cut into parts that are added at the end: a sum is taken in the order, and with the instruction,
// of the kernels that serve larger volumes (16 channels after 16, all taps of each), so that all of them
// round alike.  Taps split over four waves were shorter (8^3 256->256 12.2 us, here 16.3, on the first
// matrix kernel 127; 16^3 128->128 9.5, 10.6, on the pipelined kernel 14.7), but differences in their
// last bits move ReLU signs and pooling maxima, and one training step on 16^3 blocks differed from that
// of the other kernels by 7.5e-3 in the norm; with one order it is 1.1e-4 (medians of 100 batches).
#include "common.h"
#include "conv_internal.h"
#include "conv_mfma.h"
#include "index_math.h"

namespace k3 {

// 32x32x16 matrix instruction: rows = 32 output channels in packed order, columns = 32 voxels, contraction =
// 16 channels of one tap.  A workgroup takes 4 x 4 x 4 voxels x 32 channels, each of its two waves two
// planes (two waves and not four, so that a few compute units need not carry all of the weights).  128
// channels of the halo are in LDS at a time (pitch of an odd number of 16-byte slots), the next 128 on
// their way into registers meanwhile.
__global__ __launch_bounds__(128, 1) void conv_small_kernel(MfmaParams p, int bias_last)
{
    constexpr int NHALO = 216, G = 128, PITCH = 2 * G + 16, ITEMS = (NHALO * 4 + 127) / 128;
    extern __shared__ __attribute__((aligned(16))) unsigned char xs[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hb = lane >> 5, vl = lane & 31;
    const int K = p.c1 + p.c2, nkc = K / 16;

    // a contiguous run of the logical order per XCD; the channel groups of a tile are neighbours
    const int64_t logical = (int64_t)(blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (logical >= p.total) return;
    const int m0 = (int)(logical % p.ncg) * 32;
    int64_t t = logical / p.ncg;
    const int w0 = (int)(t % p.ntw) * 4;
    t /= p.ntw;
    const int h0 = (int)(t % p.nth) * 4;
    t /= p.nth;
    const int d0 = (int)(t % p.ntd) * 4;
    const int n = (int)(t / p.ntd);

    // the lane's halo items of 32 channels: (voxel, 8 channels); offset of the voxel from the halo's first one
    int vo[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
        const int v = (tid + k * 128) >> 2, lw = v % 6, lh = (v / 6) % 6, ld = v / 36;
        const unsigned gd = d0 + ld - 1, gh = h0 + lh - 1, gw = w0 + lw - 1;
        vo[k] = v < NHALO && gd < (unsigned)p.D && gh < (unsigned)p.H && gw < (unsigned)p.W ? (ld * p.H + lh) * p.W + lw : -1;
    }
    const int64_t halo0 = (((int64_t)n * p.D + d0 - 1) * p.H + h0 - 1) * p.W + w0 - 1;
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(p.src1 + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.src2 ? p.src2 : p.src1) + halo0 * p.c2), 0, 0x7ffffff0, 0x00020000);
    const __amdgpu_buffer_rsrc_t rm = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>((p.mask ? p.mask : p.src1) + halo0 * p.c1), 0, 0x7ffffff0, 0x00020000);
    u32v4 st[G / 32][ITEMS];
    auto fetch = [&](int g0) __attribute__((always_inline)) {        // channels g0 .. g0 + 127
#pragma unroll
        for (int s = 0; s < G / 32; ++s) {
            const int c0 = g0 + s * 32;
            if (c0 >= K) break;                                      // wave-uniform
            const bool first = c0 < p.c1;                            // 32 channels lie in one source
            const int ch = (first ? c0 : c0 - p.c1) + (tid & 3) * 8, c = first ? p.c1 : p.c2;
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int o = vo[k] < 0 ? -1 : (vo[k] * c + ch) * 2;
                if (first) st[s][k] = __builtin_amdgcn_raw_buffer_load_b128(r1, o, 0, 0);
                else st[s][k] = __builtin_amdgcn_raw_buffer_load_b128(r2, o, 0, 0);
                if (p.mask) {                                        // backward-data: one source
                    const u32v4 m = __builtin_amdgcn_raw_buffer_load_b128(rm, o, 0, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j) st[s][k][j] = mask_pair(st[s][k][j], m[j]);
                }
            }
        }
    };
    auto stage = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < G / 32; ++s) {
            if (g0 + s * 32 >= K) break;
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int i = tid + k * 128;
                if (i < NHALO * 4) *reinterpret_cast<u32v4 *>(xs + (i >> 2) * PITCH + s * 64 + (i & 3) * 16) = st[s][k];
            }
        }
    };

    // weights of (tap, 16-channel step): the lane's 16 bytes of the fragment
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(p.packed) + packed_block(m0 >> 5, nkc) / 2, 0, 0x7ffffff0, 0x00020000);
    auto weights = [&](int tap, int kc) __attribute__((always_inline)) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, lane * 16, packed_step(tap, nkc, kc), 0));
    };
    // the lane's voxel of the wave's two planes, and where its operand lies for tap (0, 0, 0)
    const int vd = wv * 2 + (vl >> 4), vh = (vl >> 2) & 3, vw = vl & 3;
    const unsigned char *x = xs + ((vd * 6 + vh) * 6 + vw) * PITCH + hb * 16;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = p.bias && !bias_last ? p.bias[m0 + hb * 16 + i] : 0.f;

    fetch(0);
    bf16x8 a[27];
#pragma unroll
    for (int i = 0; i < 27; ++i) a[i] = weights(i, 0);
    for (int g0 = 0; g0 < K; g0 += G) {
        if (g0 > 0) __syncthreads();                                 // every wave is done with the channels before
        stage(g0);
        __syncthreads();
        if (g0 + G < K) fetch(g0 + G);
        const int end = K - g0 < G ? (K - g0) / 16 : G / 16;
        for (int c = 0; c < end; ++c) {
            const int kc = g0 / 16 + c, next = kc + 1 < nkc ? kc + 1 : kc;   // (behind the last step it is read again)
            const unsigned char *xc = x + c * 32;
            auto input = [&](int tap) __attribute__((always_inline)) {
                return *reinterpret_cast<const bf16x8 *>(xc + (((tap / 9) * 6 + (tap / 3) % 3) * 6 + tap % 3) * PITCH);
            };
            bf16x8 b[3];
            b[0] = input(0);
            b[1] = input(1);
#pragma unroll
            for (int tap = 0; tap < 27; ++tap) {
                if (tap + 2 < 27) b[(tap + 2) % 3] = input(tap + 2);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[tap], b[tap % 3], acc, 0, 0, 0);
                a[tap] = weights(tap, next);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // a lane holds 16 consecutive output channels of its voxel
    const int gd = d0 + vd, gh = h0 + vh, gw = w0 + vw, co = m0 + hb * 16;
    if (gd >= p.D || gh >= p.H || gw >= p.W) return;
    const int64_t vox = (((int64_t)n * p.D + gd) * p.H + gh) * p.W + gw;
    uint32_t o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float v0 = acc[2 * i], v1 = acc[2 * i + 1];
        if (p.bias && bias_last) {
            v0 += p.bias[co + 2 * i];
            v1 += p.bias[co + 2 * i + 1];
        }
        if (p.relu) {
            v0 = v0 > 0.f ? v0 : 0.f;
            v1 = v1 > 0.f ? v1 : 0.f;
        }
        o[i] = pack2bf(v0, v1);
    }
    const bool d1 = co < p.cd1;                            // a block of 32 lies in one destination
    const int64_t eo = d1 ? vox * p.cd1 + co : vox * p.cd2 + (co - p.cd1);
    if (d1 && p.omask) {
        const uint4 *mp = reinterpret_cast<const uint4 *>(p.omask + eo);
        const uint4 k0 = mp[0], k1 = mp[1];
        const uint32_t k[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = mask_pair(o[i], k[i]);
    }
    if (d1 && p.omask_bits) apply_bits16(o, p.omask_bits[vox * (p.cd1 / 16) + co / 16]);
    uint4 *dst = reinterpret_cast<uint4 *>((d1 ? p.dst1 : p.dst2) + eo);
    dst[0] = make_uint4(o[0], o[1], o[2], o[3]);
    dst[1] = make_uint4(o[4], o[5], o[6], o[7]);
    if (p.bits_out) {                                      // (forward: one destination)
        if (bias_last) {                                   // in place of the first kernel, whose bits a pass of their own wrote
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = mask_pair_to(o[i], o[i], MASK_NUMBERS);
        }
        p.bits_out[vox * (p.cd1 / 16) + co / 16] = (unsigned short)relu_bits16(o);
    }
}

int launch_conv_small(MfmaParams p, hipStream_t st)
{
    constexpr int LDS = 216 * (2 * 128 + 16);
    // the pipelined kernel starts its sums from the bias, the first one, which takes masked inputs and fewer than
    // 48 tiles of 4x8x8 voxels x 32 channels, adds it at the end
    const int64_t small = (int64_t)p.N * ((p.D + 3) / 4) * ((p.H + 7) / 8) * ((p.W + 7) / 8);
    const int bias_last = p.mask || small * ((p.cd1 + p.cd2) / 32) < 48;
    p.ntd = (p.D + 3) / 4;
    p.nth = (p.H + 3) / 4;
    p.ntw = (p.W + 3) / 4;
    p.ncg = (p.cd1 + p.cd2) / 32;
    p.total = (int64_t)p.N * p.ntd * p.nth * p.ntw * p.ncg;
    p.per_xcd = (p.total + 7) / 8;
    if (p.per_xcd * 8 > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    conv_small_kernel<<<dim3((unsigned)(p.per_xcd * 8)), 128, LDS, st>>>(p, bias_last);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

}  // namespace k3

// Packed weight forms of the bf16 matrix-core kernels: MFMA A-fragment order, one form for the
// forward pass and one (channel roles swapped, 3x3x3 taps mirrored) for backward-data.
//   3x3x3:      fwd[cob][tap][kc][lane][j] = W[tap][kc*16 + (lane/32)*8 + j][cob*32 + r2c(lane%32)]
//               bwd[cib][tap][kc][lane][j] = W[26-tap][cib*32 + r2c(lane%32)][kc*16 + (lane/32)*8 + j]
//   transposed: fwd[tap][cob][kc][lane][j] = W[tap][kc*16 + (lane/32)*8 + j][cob*32 + r2c(lane%32)]
//               bwd[cib][tap][kc][lane][j] = W[tap][cib*32 + r2c(lane%32)][kc*16 + (lane/32)*8 + j]
// A thread makes one lane's 16 bytes (j = 0..7).  A launch takes a list of tensors: re-packing a
// network after an update is then one launch instead of one of a few microseconds per layer.
#include "common.h"
#include "conv_internal.h"
#include "conv_mfma.h"
#include "index_math.h"

namespace k3 {

struct PackList {
    PackJob job[PACK_JOBS];
    unsigned first[PACK_JOBS];   // first workgroup of each job
    int n;
};

__global__ __launch_bounds__(256) void pack_weights_kernel(PackList p)
{
    int k = 0;
    while (k + 1 < p.n && blockIdx.x >= p.first[k + 1]) ++k;
    const PackJob q = p.job[k];
    const unsigned per = (unsigned)pack_fragments(q.taps, q.cin, q.cout);    // lane fragments of one form: both fit 31 bits
    unsigned r = (blockIdx.x - p.first[k]) * 256 + threadIdx.x;
    if (r >= 2 * per) return;
    const bool bwd = r >= per;
    u32x4_pk *out = reinterpret_cast<u32x4_pk *>(q.packed) + r;
    if (bwd) r -= per;
    const int lane = (int)(r & 63);
    unsigned f = r >> 6;
    const unsigned nkc = (unsigned)(bwd ? q.cout : q.cin) / 16;
    const int kch = (int)(f % nkc) * 16 + (lane >> 5) * 8;
    f /= nkc;
    int tap, blk;
    if (q.taps == 8 && !bwd) {
        const unsigned ncob = (unsigned)q.cout / 32;
        blk = (int)(f % ncob);
        tap = (int)(f / ncob);
    } else {
        tap = (int)(f % (unsigned)q.taps);
        blk = (int)(f / (unsigned)q.taps);
    }
    if (q.taps == 27 && bwd) tap = 26 - tap;
    const int mch = blk * 32 + row_to_channel(lane & 31);
    if (bwd) {
        *out = *reinterpret_cast<const u32x4_pk *>(q.w + ((int64_t)tap * q.cin + mch) * q.cout + kch);
    } else {
        const bf16_t *s = q.w + ((int64_t)tap * q.cin + kch) * q.cout + mch;
        unsigned v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = s[(int64_t)j * q.cout];
        *out = u32x4_pk{v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16};
    }
}

int launch_pack(const PackJob *jobs, int n, hipStream_t st)
{
    for (int at = 0; at < n; at += PACK_JOBS) {
        PackList p{};
        p.n = n - at < PACK_JOBS ? n - at : PACK_JOBS;
        int64_t blocks = 0;
        for (int k = 0; k < p.n; ++k) {
            p.job[k] = jobs[at + k];
            p.first[k] = (unsigned)blocks;
            const int64_t frags = 2 * pack_fragments(p.job[k].taps, p.job[k].cin, p.job[k].cout);
            if (frags > 0x7fffffffLL) return K3_E_UNSUPPORTED;
            blocks += (frags + 255) / 256;
        }
        if (blocks > 0x7fffffffLL) return K3_E_UNSUPPORTED;
        pack_weights_kernel<<<dim3((unsigned)blocks), 256, 0, st>>>(p);
        K3_LAUNCH_CHECK();
    }
    return K3_OK;
}

}  // namespace k3

// Index arithmetic of the kernels in a form that a host compiler can check too: no HIP types.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#define K3_HD __host__ __device__ __forceinline__
#else
#define K3_HD inline
#endif

namespace k3 {

// General 3x3x3 kernel.  Floats of a halo voxel in LDS: whole fours, and an odd number of them, so that
// the 16 voxels of a block fall on different banks.
K3_HD constexpr int general_pitch(int K) { return 4 * (((K + 3) / 4) | 1); }

// Element of the weights [27][cin][cout] that (tap, contraction channel k, row 0) is; K contraction channels,
// M rows.  Forward contracts over cin, backward-data over cout.  The kernel adds this as a scalar offset,
// which is no part of a descriptor's range check, so it has to lie inside the tensor by itself.
template <typename I>
K3_HD I general_weight(bool bwd, int tap, int k, I K, I M) { return bwd ? (I)tap * M * K + k : ((I)tap * K + k) * M; }

// The next place in the sum over (tap, channel): `step` channels on, KP in all (whole steps).  Behind the
// last step it stays at the last tap, where a wave that looks ahead reads operands it does not use.
K3_HD void general_next(int &tap, int &c, int step, int KP)
{
    c += step;
    if (c >= KP) {
        c = 0;
        tap = tap < 26 ? tap + 1 : 26;
    }
}

// Offset of voxel (d, h, w) of a tile from the tile's first voxel.  I: 32 bits where a tile's span is
// known to be small, else 64.
template <typename I>
K3_HD I tile_offset(int d, int h, int w, int H, int W) { return ((I)d * H + h) * W + w; }

// 16-byte lane fragments of one packed form of a weight tensor.
K3_HD int64_t pack_fragments(int taps, int cin, int cout) { return (int64_t)taps * cin * cout / 8; }

// Packed 3x3x3 weights, [32-channel block][27][nkc][1 KB]: bytes to a block of output channels, and from
// there to (tap, 16-channel step).  A block alone stays below 2 GiB where small_weights_fit says so.
K3_HD int64_t packed_block(int block, int nkc) { return (int64_t)block * 27 * nkc * 1024; }
K3_HD unsigned packed_step(int tap, int nkc, int kc) { return (unsigned)((tap * nkc + kc) * 1024); }
K3_HD bool small_weights_fit(int64_t K) { return 27 * (K / 16) * 1024 < 0x7ffffff0LL; }

// Whether four channels at a time are one aligned access: the channel counts and the base addresses
// (each or-ed together; null addresses do not count), and the bytes of an element.
K3_HD bool whole_quads(int64_t channels, uintptr_t at, int size)
{
    return channels % 4 == 0 && (at & (uintptr_t)(4 * size - 1)) == 0;
}

}  // namespace k3

// Index arithmetic of the kernels in a form that a host compiler can check too: no HIP types.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#define K3_HD __host__ __device__ __forceinline__
#else
#define K3_HD inline
#endif

namespace k3 {

// General 3x3x3 kernel: the tap a lane group's slot of step s belongs to (S slots per voxel and chunk;
// the last step may hold slots that belong to none, and a wave may look ahead past the last step).
K3_HD int general_tap(int S, int s, int kg) { return S == 4 ? s : (4 * s + kg) / S; }

// Byte offset a wave adds to a step's weight loads, the same for all its lanes (S = 4: a step is one tap).
// A wave that looks ahead past the last tap reads the last one again: a scalar offset is no part of
// a descriptor's range check, so it has to lie inside the tensor by itself.
template <typename I>
K3_HD I general_weight_soff(int S, int s, bool bwd, I K, I M, int size)
{
    const int tap = general_tap(S, s, 0) < 26 ? general_tap(S, s, 0) : 26;
    return S == 4 ? (bwd ? 26 - tap : tap) * K * M * size : 0;
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

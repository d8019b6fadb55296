"""The kernels' index arithmetic (csrc/index_math.h), compiled for the host: every offset a kernel can
form lies inside its tensor, also where 32 bits would not hold it."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include "index_math.h"
using namespace k3;
extern "C" {
int64_t weight(int bwd, int tap, int k, int64_t K, int64_t M) { return general_weight<int64_t>(bwd, tap, k, K, M); }
int next_tap(int tap, int c, int step, int K) { general_next(tap, c, step, K); return tap; }
int next_c(int c, int step, int K) { int tap = 0; general_next(tap, c, step, K); return c; }
int pitch(int K) { return general_pitch(K); }
int64_t block(int b, int nkc) { return packed_block(b, nkc); }
int64_t step(int tap, int nkc, int kc) { return packed_step(tap, nkc, kc); }
int fit(int64_t K) { return small_weights_fit(K); }
int quads(int64_t channels, uint64_t at, int size) { return whole_quads(channels, at, size); }
int64_t fragments(int taps, int cin, int cout) { return pack_fragments(taps, cin, cout); }
int64_t offset64(int d, int h, int w, int H, int W) { return tile_offset<int64_t>(d, h, w, H, W); }
int64_t offset32(int d, int h, int w, int H, int W) { return tile_offset<int>(d, h, w, H, W); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("index_math")
    cpp, so = str(d / "index_math.cpp"), str(d / "index_math.so")
    with open(cpp, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-fsanitize=undefined", "-fno-sanitize-recover", "-static-libubsan",
                           "-I" + os.path.join(ROOT, "paper_1811_12174_amd", "csrc"), "-o", so, cpp])
    L = ctypes.CDLL(so)
    q, i = ctypes.c_int64, ctypes.c_int
    L.weight.restype, L.weight.argtypes = q, [i, i, i, q, q]
    L.next_tap.restype, L.next_tap.argtypes = i, [i, i, i, i]
    L.next_c.restype, L.next_c.argtypes = i, [i, i, i]
    L.pitch.restype, L.pitch.argtypes = i, [i]
    L.block.restype, L.block.argtypes = q, [i, i]
    L.step.restype, L.step.argtypes = q, [i, i, i]
    L.fit.restype, L.fit.argtypes = i, [q]
    L.quads.restype, L.quads.argtypes = i, [q, ctypes.c_uint64, i]
    L.fragments.restype, L.fragments.argtypes = q, [i, i, i]
    for f in (L.offset32, L.offset64):
        f.restype, f.argtypes = q, [i, i, i, i, i]
    return L


@pytest.mark.parametrize("U", [1, 4])            # instructions of four channels a step
@pytest.mark.parametrize("bwd", [0, 1])
def test_general_kernel_asks_for_no_weights_outside_the_tensor(lib, U, bwd):
    M = 24
    for K in (4, 16, 20, 48) if U == 1 else (16, 48):
        for tap in range(27):
            for c in range(0, K, 4):
                base = lib.weight(bwd, tap, c, K, M)
                for m in (0, M - 1):
                    for kg in range(4):
                        at = base + (m * K + kg if bwd else kg * M + m)
                        assert at == ((tap * M + m) * K + c + kg if bwd else (tap * K + c + kg) * M + m)
                        assert 0 <= base <= at < 27 * K * M
        # (tap, c) as the kernel steps through them, two or eight steps ahead: behind the last tap it stays there
        tap, c = 0, 0
        for _ in range(27 * K // (4 * U) + 9):
            assert 0 <= lib.weight(bwd, tap, c + 4 * (U - 1), K, M) <= 27 * K * M - (4 if bwd else 4 * M)
            tap, c = lib.next_tap(tap, c, 4 * U, K), lib.next_c(c, 4 * U, K)
            assert tap <= 26


@pytest.mark.parametrize("K", [1, 3, 4, 5, 8, 16, 20, 64, 128, 256, 400])
def test_halo_voxels_lie_on_different_banks(lib, K):
    pitch = lib.pitch(K)
    assert pitch >= K and pitch % 4 == 0
    for kg in range(4):      # 16 neighbouring voxels, one word each, and the four channels of an instruction
        assert len({(v * pitch + kg) % 64 for v in range(16)}) == 16
    assert len({(v * pitch + kg) % 64 for v in range(16) for kg in range(4)}) == 64


def test_offsets_inside_a_tile_of_wide_planes(lib):
    # without descriptors: five planes of 21000 x 21000 voxels pass 2^31
    for H, W in ((3, 5), (21000, 21000), (2 ** 31 - 1, 7), (1, 2 ** 31 - 1)):
        for d, h, w in ((0, 0, 0), (5, 5, 9), (5, 0, 0), (1, 3, 2)):
            assert lib.offset64(d, h, w, H, W) == (d * H + h) * W + w
    # with them a tile spans less than 2 GiB: 6 (H + 1) W elements of 4 bytes
    H, W = 9000, 9000
    assert 6 * (H + 1) * W * 4 < 2 ** 31
    assert lib.offset32(5, 5, 9, H, W) == (5 * H + 5) * W + 9


@pytest.mark.parametrize("taps,cin,cout", [(27, 32, 64), (27, 8928, 8928), (27, 17824, 17824), (8, 16416, 16416), (8, 32768, 32768)])
def test_fragments_of_large_weight_tensors(lib, taps, cin, cout):
    # the launch refuses 2^31 fragments of the two forms; 2^31 weights (a quarter as many fragments) it takes
    assert lib.fragments(taps, cin, cout) == taps * cin * cout // 8


@pytest.mark.parametrize("K", [16, 256, 38912, 1 << 20, 1242736])
def test_packed_weights_of_the_small_volume_kernel(lib, K):
    # 1024 output channels: 32 blocks, whose packed form passes 2 GiB from 38912 input channels on
    assert lib.fit(K)
    nkc = K // 16
    for b in (0, 1, 31):
        for tap in (0, 13, 26):
            for kc in (0, nkc - 1):
                assert 0 <= lib.step(tap, nkc, kc) < 2 ** 31 - 1024
                assert lib.block(b, nkc) + lib.step(tap, nkc, kc) == ((b * 27 + tap) * nkc + kc) * 1024
    assert not lib.fit(1242784)


@pytest.mark.parametrize("size", [2, 4])
def test_quads_lie_on_their_own_boundary(lib, size):
    a, b = 0x7F0000001000, 0x7F0000A00200
    assert lib.quads(8 | 16 | 0, a | b | 0, size)
    for shift in (1, 2, 3):
        assert not lib.quads(8 | 16, a | (b + shift * size), size)
        assert not lib.quads(8 | (16 + shift), a | b, size)
    assert lib.quads(8, (a + 4 * size) | b, size)

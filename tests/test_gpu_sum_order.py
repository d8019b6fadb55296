"""The bf16 kernel of small volumes sums in the order of those of larger ones (last test here).
The general kernels (fp32, and bf16 with odd channel counts) sum in the order of the definition: bias,
then tap after tap, the channels of a tap in order, one fused multiply-add per term; the fp32 weight
gradients in sets, chains and groups that depend on the sizes alone.  All passes of the 3x3x3 and the
transposed convolution are held to those loops bit for bit, at sizes that reach every tile and form of
their dispatch; only the sign of a zero is left open (padding terms add zeros)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SRC = r"""
#include <math.h>
// y[v][m] = bias[m] + sum over (t, k) x[v shifted by tap t][k] * w(t, k, m); back: mirrored shifts, w = [27][m][k]
extern "C" void conv(const float *x, const float *w, const float *b, float *y, long N, long D, long H, long W, long K, long M, int back)
{
    for (long n = 0; n < N; ++n) for (long d = 0; d < D; ++d) for (long h = 0; h < H; ++h) for (long v = 0; v < W; ++v)
        for (long m = 0; m < M; ++m) {
            float s = b ? b[m] : 0.f;
            for (int t = 0; t < 27; ++t) {
                const int pos = back ? 26 - t : t;
                const long zd = d + pos / 9 - 1, zh = h + pos / 3 % 3 - 1, zw = v + pos % 3 - 1;
                if (zd < 0 || zd >= D || zh < 0 || zh >= H || zw < 0 || zw >= W) continue;
                const float *xp = x + (((n * D + zd) * H + zh) * W + zw) * K;
                if (back) for (long k = 0; k < K; ++k) s = fmaf(xp[k], w[(t * M + m) * K + k], s);
                else for (long k = 0; k < K; ++k) s = fmaf(xp[k], w[(t * K + k) * M + m], s);
            }
            y[(((n * D + d) * H + h) * W + v) * M + m] = s;
        }
}
static long at(long o, int t, long D, long H, long W)      // voxel under tap t of input voxel o
{
    const long w = o % W, h = o / W % H, d = o / (W * H) % D, n = o / (W * H * D);
    return ((n * 2 * D + 2 * d + (t >> 2)) * 2 * H + 2 * h + ((t >> 1) & 1)) * 2 * W + 2 * w + (t & 1);
}
extern "C" void up_fwd(const float *x, const float *w, const float *b, float *y, long N, long D, long H, long W, long K, long M)
{
    for (long o = 0; o < N * D * H * W; ++o) for (int t = 0; t < 8; ++t) for (long m = 0; m < M; ++m) {
        float s = b[m];
        for (long k = 0; k < K; ++k) s = fmaf(x[o * K + k], w[(t * K + k) * M + m], s);
        y[at(o, t, D, H, W) * M + m] = s;
    }
}
extern "C" void up_back(const float *g, const float *w, float *dx, long N, long D, long H, long W, long K, long M)
{
    for (long o = 0; o < N * D * H * W; ++o) for (long k = 0; k < K; ++k) {
        float s = 0.f;
        for (int t = 0; t < 8; ++t) for (long m = 0; m < M; ++m) s = fmaf(g[at(o, t, D, H, W) * M + m], w[(t * K + k) * M + m], s);
        dx[o * K + k] = s;
    }
}
// Weight gradient of taps T (27, or 8: transposed).  Sets of at least 256 voxels, 256 / cout interleaved
// chains each, chains added in order; then the sets, in 16 groups (4 where quads do not fit) of two chains.
extern "C" void wgrad(const float *x, const float *g, float *dW, float *db, long N, long D, long H, long W, long K, long M, int T)
{
    const long V = N * D * H * W, want = V / 256, S = want < 1 ? 1 : want > 1024 ? 1024 : want, slab = (V + S - 1) / S;
    const long CH = 256 / (M < 256 ? M : 256), countW = T * K * M, count = countW + M;
    float *ws = new float[S * count];
    for (long s = 0; s < S; ++s) {
        const long v0 = s * slab, v1 = v0 + slab < V ? v0 + slab : V;
        for (long e = 0; e < count; ++e) {
            const long m = e < countW ? e % M : e - countW, k = e / M % K;
            const int t = e < countW ? e / (M * K) : -1;
            float tot = 0.f;
            for (long c = 0; c < CH; ++c) {
                float acc = 0.f;
                for (long v = v0 + c; v < v1; v += CH) {
                    if (T == 8) {
                        if (t >= 0) acc = fmaf(x[v * K + k], g[at(v, t, D, H, W) * M + m], acc);
                        else for (int u = 0; u < 8; ++u) acc += g[at(v, u, D, H, W) * M + m];
                    } else if (t < 0) {
                        acc += g[v * M + m];
                    } else {
                        const long w = v % W + t % 3 - 1, h = v / W % H + t / 3 % 3 - 1, d = v / (W * H) % D + t / 9 - 1, n = v / (W * H * D);
                        if (w < 0 || w >= W || h < 0 || h >= H || d < 0 || d >= D) continue;
                        acc = fmaf(x[(((n * D + d) * H + h) * W + w) * K + k], g[v * M + m], acc);
                    }
                }
                tot += acc;
            }
            ws[s * count + e] = tot;
        }
    }
    const long G = count % 4 == 0 && countW % 4 == 0 ? 16 : 4;
    for (long e = 0; e < count; ++e) {
        float sum = 0.f;
        for (long q = 0; q < G; ++q) {
            float s0 = 0.f, s1 = 0.f;
            for (long k = q; k < S; k += 2 * G) {
                s0 += ws[k * count + e];
                if (k + G < S) s1 += ws[(k + G) * count + e];
            }
            sum = q ? sum + (s0 + s1) : s0 + s1;
        }
        (e < countW ? dW[e] : db[e - countW]) = sum;
    }
    delete[] ws;
}
"""


@pytest.fixture(scope="module")
def loops(tmp_path_factory):
    d = tmp_path_factory.mktemp("loops")
    cpp, so = str(d / "loops.cpp"), str(d / "loops.so")
    with open(cpp, "w") as f:
        f.write(SRC)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-fPIC", "-shared", "-o", so, cpp])
    return ctypes.CDLL(so)


def run(fn, *args):
    fn(*[a.ctypes.data_as(ctypes.c_void_p) if isinstance(a, np.ndarray) else a if a is None else
         (ctypes.c_int(a[0]) if isinstance(a, tuple) else ctypes.c_long(a)) for a in args])


def same(got, want, dt):
    import torch
    w = torch.from_numpy(want)
    return torch.equal(got.cpu(), w.bfloat16() if dt == "bf16" else w)      # (-0 equals 0)


# (N, D, H, W), c1, c2, cout, dtype; forward contracts over c1 + c2, backward-data over cout
CONV = [
    ((1, 3, 5, 9), 1, 0, 8, "f32"),          # elements, at most 4 channels
    ((2, 24, 28, 33), 1, 0, 16, "f32"),      # the same on 128-voxel tiles
    ((1, 3, 5, 9), 4, 0, 20, "f32"),         # one quad a voxel, several output blocks
    ((1, 33, 28, 39), 4, 0, 40, "f32"),      # 128-voxel tiles, two output blocks, the second one partial
    ((1, 5, 6, 7), 4, 4, 12, "f32"),         # two sources in one step
    ((1, 25, 28, 33), 3, 0, 8, "f32"),       # 8 channels backward on 128-voxel tiles
    ((1, 33, 28, 39), 8, 0, 40, "f32"),      # 8 channels, two output blocks
    ((1, 28, 29, 33), 16, 0, 16, "f32"),     # whole 16s, 128-voxel tiles
    ((1, 28, 28, 31), 16, 16, 32, "f32"),    # 64-voxel tiles
    ((1, 12, 12, 12), 32, 0, 32, "f32"),     # 32-voxel tiles
    ((1, 20, 32, 32), 64, 0, 32, "f32"),     # 64 channels: 64-voxel tiles, two output blocks
    ((1, 3, 5, 5), 64, 64, 48, "f32"),       # 128 channels: 32-voxel tiles
    ((1, 2, 3, 5), 256, 0, 80, "f32"),       # 16-voxel tiles
    ((1, 1, 3, 4), 400, 0, 20, "f32"),       # the most LDS takes
    ((1, 2, 3, 5), 300, 132, 17, "f32"),     # more: from memory
    ((1, 3, 3, 3), 5, 0, 431, "f32"),        # the same element by element, in the backward pass
    ((1, 5, 6, 9), 12, 8, 23, "f32"),
    ((1, 12, 11, 10), 40, 0, 24, "bf16"),
    ((1, 30, 31, 34), 6, 0, 20, "bf16"),
]


@pytest.mark.parametrize("case", CONV, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
def test_convolution(loops, case):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import empty, to_dev
    sp, c1, c2, co, dt = case
    ci = c1 + c2
    x, w, g = synth.activations(640, sp + (ci,), dt), synth.conv_weights(641, ci, co, dt), synth.activations(642, sp + (co,), dt)
    ym, om = synth.activations(643, sp + (co,), dt), synth.activations(644, sp + (c1,), dt)
    b = (synth.normal(synth.SEED, 645, (co,), np.float64) * 0.5).astype(np.float32)
    xd, wd, gd = to_dev(x, dt), to_dev(w, dt), to_dev(g, dt)
    x1, x2 = xd[..., :c1].contiguous(), xd[..., c1:].contiguous() if c2 else None
    y, dx, dx2 = empty(sp + (co,), dt), empty(sp + (c1,), dt), empty(sp + (c2,), dt) if c2 else None
    k3.conv3d_fwd(x1, wd, None, torch.from_numpy(b).cuda(), 1, y, x2=x2)
    k3.conv3d_bwd_data(gd, to_dev(ym, dt), wd, None, dx, dx2=dx2, dx_mask=to_dev(om, dt))
    torch.cuda.synchronize()
    x, w, g = (np.ascontiguousarray(t, dtype=np.float32) for t in (x, w, g))
    want = np.empty(sp + (co,), np.float32)
    run(loops.conv, x, w, b, want, *sp, ci, co, (0,))
    assert same(y, np.maximum(want, 0), dt)
    want = np.empty(sp + (ci,), np.float32)
    run(loops.conv, np.where(ym > 0, g, np.float32(0)), w, None, want, *sp, co, ci, (1,))
    assert same(dx, np.where(om > 0, want[..., :c1], np.float32(0)), dt)
    if c2:
        assert same(dx2, np.ascontiguousarray(want[..., c1:]), dt)


# (N, D, H, W) before the up-sampling, cin, cout, dtype
UP = [((1, 1, 1, 1), 1, 1, "f32"), ((2, 3, 5, 7), 16, 8, "f32"), ((1, 6, 6, 6), 32, 16, "f32"), ((1, 4, 5, 6), 128, 64, "f32"),
      ((1, 2, 3, 5), 37, 23, "f32"), ((1, 3, 4, 5), 32, 16, "bf16"), ((1, 3, 4, 5), 6, 20, "bf16")]


@pytest.mark.parametrize("case", UP, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
def test_transposed_convolution(loops, case):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import empty, to_dev
    sp, ci, co, dt = case
    big = (sp[0], 2 * sp[1], 2 * sp[2], 2 * sp[3])
    x, g, om = synth.activations(650, sp + (ci,), dt), synth.activations(651, big + (co,), dt), synth.activations(652, sp + (ci,), dt)
    w = synth.upconv_weights(653, ci, co, dt)
    b = (synth.normal(synth.SEED, 654, (co,), np.float64) * 0.5).astype(np.float32)
    y, dx = empty(big + (co,), dt), empty(sp + (ci,), dt)
    k3.upconv3d_fwd(to_dev(x, dt), to_dev(w, dt), None, torch.from_numpy(b).cuda(), y)
    k3.upconv3d_bwd_data(to_dev(g, dt), to_dev(w, dt), None, dx, dx_mask=to_dev(om, dt))
    torch.cuda.synchronize()
    x, w, g = (np.ascontiguousarray(t, dtype=np.float32) for t in (x, w, g))
    want = np.empty(big + (co,), np.float32)
    run(loops.up_fwd, x, w, b, want, *sp, ci, co)
    assert same(y, want, dt)
    want = np.empty(sp + (ci,), np.float32)
    run(loops.up_back, g, w, want, *sp, ci, co)
    assert same(dx, np.where(om > 0, want, np.float32(0)), dt)


# 3x3x3: (N, D, H, W), c1, c2, cout
WGRAD = [((1, 3, 4, 5), 4, 0, 8), ((1, 16, 16, 16), 4, 0, 8),              # one set, 16 sets: two taps a wave
         ((1, 2, 3, 5), 20, 0, 36), ((2, 9, 10, 11), 1, 0, 3),             # sets whose last one is partial, chains of unequal length
         ((1, 24, 24, 24), 16, 0, 32), ((1, 12, 12, 12), 32, 32, 64),      # seven taps a wave, two sources
         ((1, 23, 24, 26), 5, 3, 16), ((1, 8, 9, 10), 12, 8, 17),          # a block of channels that straddles two sources
         ((1, 5, 6, 7), 3, 0, 300), ((1, 40, 41, 42), 6, 0, 1),            # more outputs than chains, a chain a voxel
         ((1, 130, 130, 131), 1, 0, 2)]                                     # sets beyond the table in LDS


@pytest.mark.parametrize("case", WGRAD, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
@pytest.mark.parametrize("masked", [0, 1])
def test_weight_gradient(loops, case, masked):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev
    sp, c1, c2, co = case
    ci = c1 + c2
    x, g, ym = synth.activations(660, sp + (ci,), "f32"), synth.activations(661, sp + (co,), "f32"), synth.activations(662, sp + (co,), "f32")
    xd, gd, md = to_dev(x, "f32"), to_dev(g, "f32"), to_dev(ym, "f32") if masked else None
    x1, x2 = xd[..., :c1].contiguous(), xd[..., c1:].contiguous() if c2 else None
    dW, db = torch.full((3, 3, 3, ci, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x1, gd, x2=x2), device="cuda", dtype=torch.uint8)
    k3.conv3d_bwd_weight(x1, gd, md, dW, db, ws, x2=x2)
    dW2 = torch.full_like(dW, float("nan"))
    k3.conv3d_bwd_weight(x1, gd, md, dW2, None, ws, x2=x2)      # no bias gradient wanted
    torch.cuda.synchronize()
    x, g = np.ascontiguousarray(x, dtype=np.float32), np.ascontiguousarray(np.where(ym > 0, g, 0) if masked else g, dtype=np.float32)
    wantW, wantb = np.empty((3, 3, 3, ci, co), np.float32), np.empty((co,), np.float32)
    run(loops.wgrad, x, g, wantW, wantb, *sp, ci, co, (27,))
    assert same(dW, wantW, "f32") and same(db, wantb, "f32") and torch.equal(dW, dW2)


# transposed: (N, D, H, W) before the up-sampling, cin, cout
@pytest.mark.parametrize("case", [((1, 1, 1, 1), 1, 1), ((2, 3, 5, 7), 16, 8), ((1, 12, 12, 12), 64, 32), ((1, 13, 24, 23), 32, 16),
                                  ((1, 5, 6, 9), 37, 23), ((1, 4, 5, 6), 20, 260)], ids=lambda c: "x".join(map(str, c[0] + c[1:])))
def test_weight_gradient_of_the_transposed_convolution(loops, case):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev
    sp, ci, co = case
    x, g = synth.activations(670, sp + (ci,), "f32"), synth.activations(671, (sp[0], 2 * sp[1], 2 * sp[2], 2 * sp[3], co), "f32")
    xd, gd = to_dev(x, "f32"), to_dev(g, "f32")
    dW, db = torch.full((2, 2, 2, ci, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.upconv3d_bwd_weight_workspace_bytes(xd, gd), device="cuda", dtype=torch.uint8)
    k3.upconv3d_bwd_weight(xd, gd, dW, db, ws)
    torch.cuda.synchronize()
    wantW, wantb = np.empty((2, 2, 2, ci, co), np.float32), np.empty((co,), np.float32)
    run(loops.wgrad, np.ascontiguousarray(x, dtype=np.float32), np.ascontiguousarray(g, dtype=np.float32), wantW, wantb, *sp, ci, co, (8,))
    assert same(dW, wantW, "f32") and same(db, wantb, "f32")


# (D, H, W), c1, c2, cout
SMALL = [
    ((1, 2, 3), 32, 0, 32),
    ((4, 4, 4), 128, 0, 128),
    ((5, 6, 9), 32, 96, 64),
    ((8, 8, 8), 256, 0, 64),
    ((16, 16, 16), 32, 0, 128),     # 64 tiles of 4x8x8 voxels x 32 channels: sums start from the bias
]


@pytest.mark.parametrize("case", SMALL, ids=lambda c: "x".join(map(str, c)))
def test_bf16_sums_do_not_depend_on_the_batch(case):
    """A sample alone goes to the small-volume kernel, as one of many to the kernels of larger volumes;
    all of them add in the same order, so the sample's results are the same to the bit.  Fewer than
    48 tiles add the bias at the end, as the first matrix kernel does: there the bias is zero."""
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, empty, packed_for
    (D, H, W), c1, c2, co = case
    sp, cin = (D, H, W), c1 + c2
    cubes = -(-D // 4) * -(-H // 4) * -(-W // 4)
    small = -(-D // 4) * -(-H // 8) * -(-W // 8)
    many = 512 // (cubes * min(cin, co) // 32) + 1
    assert cubes * max(cin, co) // 32 <= 512 < many * cubes * min(cin, co) // 32
    x = to_dev(synth.activations(700, (1,) + sp + (cin,), "bf16"), "bf16")
    w = to_dev(synth.conv_weights(701, cin, co, "bf16"), "bf16")
    dy, ym = (to_dev(synth.activations(s, (1,) + sp + (co,), "bf16"), "bf16") for s in (702, 703))
    b = torch.from_numpy(synth.normal(synth.SEED, 704, (co,), np.float32)).cuda()
    if small * co // 32 < 48:
        b.zero_()
    pk = packed_for(w)

    def run_all(n):
        rep = lambda t: t.expand((n,) + t.shape[1:]).contiguous()
        y = empty((n,) + sp + (co,), "bf16")
        k3.conv3d_fwd(rep(x[..., :c1]), w, pk, b, 0, y, x2=rep(x[..., c1:]) if c2 else None)
        out = [y[-1]]
        for mask in (None, rep(ym)):
            dx = empty((n,) + sp + (c1,), "bf16")
            dx2 = empty((n,) + sp + (c2,), "bf16") if c2 else None
            k3.conv3d_bwd_data(rep(dy), mask, w, pk, dx, dx2=dx2)
            out += [dx[-1]] + ([dx2[-1]] if c2 else [])
        torch.cuda.synchronize()
        return out
    for one, of_many in zip(run_all(1), run_all(many)):
        assert torch.equal(one, of_many)

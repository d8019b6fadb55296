"""The general 3x3x3 kernels (fp32, and bf16 with odd channel counts) against the fp64 oracle at the
sizes where their dispatch and their tiles change: 4, 8 and 16 contraction channels and one more
than each, 128-voxel tiles with one and two output blocks, the smaller tiles, edges one short of and
one past a tile, channel quads and widths that are none."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# (N, D, H, W, c1, c2, cout, dtype)
CASES = [
    (1, 1, 1, 1, 1, 0, 1, "f32"),          # one voxel
    (1, 2, 4, 4, 4, 0, 16, "f32"),         # exactly one 32-voxel tile, one quad per voxel
    (1, 3, 5, 5, 8, 0, 17, "f32"),         # one past a tile on every axis, two quads, one row past a block
    (1, 4, 7, 9, 5, 0, 8, "f32"),          # channels that are no quad
    (1, 5, 6, 7, 4, 4, 12, "f32"),         # two sources in 8 channels
    (1, 6, 5, 7, 12, 8, 20, "f32"),        # two sources in 16 staged channels, and a partial step
    (1, 28, 29, 33, 16, 0, 16, "f32"),     # 280 128-voxel tiles, one output block, one past a tile
    (1, 28, 28, 31, 16, 16, 32, "f32"),    # 196 tiles: smaller ones, two sources
    (2, 24, 28, 40, 20, 0, 36, "f32"),     # 128-voxel tiles with two output blocks, the second one partial
    (1, 33, 28, 39, 4, 0, 40, "f32"),      # the same at one quad per voxel
    (1, 12, 11, 10, 40, 0, 24, "bf16"),    # bf16, quads
    (1, 30, 31, 34, 6, 0, 20, "bf16"),     # bf16, no quads, 128-voxel tiles
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
@pytest.mark.parametrize("masked", [0, 1])
def test_general_kernels(orc, case, masked):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, empty, rel_l2
    N, D, H, W, c1, c2, co, dt = case
    # fp32: at most 27 * 40 products per sum, fp32 accumulation: 1e-5 covers it with room (the sums over
    # voxels of the weight gradient too); bf16 results carry one rounding of relative size 2^-9
    tol = 1e-5 if dt == "f32" else 4e-3
    sp = (N, D, H, W)
    x, w = synth.activations(610, sp + (c1 + c2,), dt), synth.conv_weights(611, c1 + c2, co, dt)
    b = (synth.normal(synth.SEED, 612, (co,), np.float64) * 0.5).astype(np.float32)
    dy = synth.activations(613, sp + (co,), dt)
    ym, om = synth.activations(614, sp + (co,), dt), synth.activations(615, sp + (c1,), dt)
    xd = to_dev(x, dt)
    x1, x2 = xd[..., :c1].contiguous(), xd[..., c1:].contiguous() if c2 else None
    wd, dyd, bd = to_dev(w, dt), to_dev(dy, dt), torch.from_numpy(b).cuda()
    ymd, omd = (to_dev(ym, dt), to_dev(om, dt)) if masked else (None, None)

    y = empty(sp + (co,), dt).fill_(float("nan"))
    k3.conv3d_fwd(x1, wd, None, bd, masked, y, x2=x2)
    dx, dx2 = empty(sp + (c1,), dt).fill_(float("nan")), empty(sp + (c2,), dt).fill_(float("nan")) if c2 else None
    k3.conv3d_bwd_data(dyd, ymd, wd, None, dx, dx2=dx2, dx_mask=omd)
    dW, db = torch.full((3, 3, 3, c1 + c2, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x1, dyd, x2=x2), device="cuda", dtype=torch.uint8)
    k3.conv3d_bwd_weight(x1, dyd, ymd, dW, db, ws, x2=x2)
    torch.cuda.synchronize()

    x64, w64, g64 = x.astype(np.float64), w.astype(np.float64), dy.astype(np.float64)
    if masked:
        g64 = orc.relu_bwd(g64, ym.astype(np.float64))
    assert rel_l2(to_f64(y), orc.conv3d_fwd(x64, w64, b.astype(np.float64), relu=bool(masked))) < tol
    rdx = orc.conv3d_bwd_data(g64, w64)
    r1 = orc.relu_bwd(rdx[..., :c1].copy(), om.astype(np.float64)) if masked else rdx[..., :c1]
    assert rel_l2(to_f64(dx), r1) < tol
    if c2:
        assert rel_l2(to_f64(dx2), rdx[..., c1:]) < tol
    rW, rb = orc.conv3d_bwd_weight(x64, g64)
    assert rel_l2(to_f64(dW), rW) < 1e-5
    assert rel_l2(to_f64(db), rb) < 1e-5


# channel counts in whole quads on tensors one element past a quad's boundary: each of them alone and all
# (N, D, H, W), c1, c2, cout, dtype; the second size takes 128-voxel tiles
SHIFTED = [((1, 5, 6, 9), 8, 0, 12, "f32"), ((1, 5, 6, 9), 8, 8, 20, "bf16"), ((1, 28, 29, 33), 16, 0, 16, "f32"), ((1, 6, 7, 9), 16, 16, 32, "bf16")]


@pytest.mark.parametrize("case", SHIFTED, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
@pytest.mark.parametrize("which", ["x", "w", "dy", "masks", "out", "all"])
def test_tensors_off_the_quad_boundary(orc, case, which):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, empty, rel_l2
    sp, c1, c2, co, dt = case
    tol = 1e-5 if dt == "f32" else 4e-3      # as above

    def put(t, kind):
        if which not in (kind, "all"):
            return t
        flat = torch.empty(t.numel() + 1, device=t.device, dtype=t.dtype)
        flat[1:].copy_(t.reshape(-1))
        return flat[1:].view(t.shape)

    def new(c):
        return put(empty(sp + (c,), dt).fill_(float("nan")), "out")
    x, w, dy = synth.activations(620, sp + (c1 + c2,), dt), synth.conv_weights(621, c1 + c2, co, dt), synth.activations(622, sp + (co,), dt)
    ym, om = synth.activations(623, sp + (co,), dt), synth.activations(624, sp + (c1,), dt)
    xd = to_dev(x, dt)
    x1, x2 = put(xd[..., :c1].contiguous(), "x"), put(xd[..., c1:].contiguous(), "x") if c2 else None
    wd, dyd, ymd, omd = put(to_dev(w, dt), "w"), put(to_dev(dy, dt), "dy"), put(to_dev(ym, dt), "masks"), put(to_dev(om, dt), "masks")

    y, dx, dx2 = new(co), new(c1), new(c2) if c2 else None
    k3.conv3d_fwd(x1, wd, None, None, 1, y, x2=x2)
    k3.conv3d_bwd_data(dyd, ymd, wd, None, dx, dx2=dx2, dx_mask=omd)
    dW, db = torch.full((3, 3, 3, c1 + c2, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x1, dyd, x2=x2), device="cuda", dtype=torch.uint8)
    k3.conv3d_bwd_weight(x1, dyd, ymd, dW, db, ws, x2=x2)
    torch.cuda.synchronize()

    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    g64 = orc.relu_bwd(dy.astype(np.float64), ym.astype(np.float64))
    assert rel_l2(to_f64(y), orc.conv3d_fwd(x64, w64, np.zeros(co), relu=True)) < tol
    rdx = orc.conv3d_bwd_data(g64, w64)
    assert rel_l2(to_f64(dx), orc.relu_bwd(rdx[..., :c1].copy(), om.astype(np.float64))) < tol
    if c2:
        assert rel_l2(to_f64(dx2), rdx[..., c1:]) < tol
    rW, rb = orc.conv3d_bwd_weight(x64, g64)
    assert rel_l2(to_f64(dW), rW) < 1e-5
    assert rel_l2(to_f64(db), rb) < 1e-5


def test_weight_gradient_of_more_blocks_than_a_grid_axis_has():
    # 65537 blocks of 16 x 16 channels; two voxels along w, so three taps meet a voxel: dW = x g by hand
    import torch
    from paper_1811_12174_amd import k3
    co = 16 * 65536 + 3
    g = torch.arange(2 * co, device="cuda", dtype=torch.float32).remainder_(251.0).view(1, 1, 1, 2, co)
    x = torch.tensor([3.0, -2.0], device="cuda").view(1, 1, 1, 2, 1)
    dW, db = torch.full((3, 3, 3, 1, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x, g), device="cuda", dtype=torch.uint8)
    k3.conv3d_bwd_weight(x, g, None, dW, db, ws)
    want = torch.zeros_like(dW)      # whole numbers below 2^24: exact
    g0, g1 = g[0, 0, 0, 0], g[0, 0, 0, 1]
    want[1, 1, 0, 0], want[1, 1, 1, 0], want[1, 1, 2, 0] = 3.0 * g1, 3.0 * g0 - 2.0 * g1, -2.0 * g0
    assert torch.equal(dW, want) and torch.equal(db, g0 + g1)


@pytest.mark.parametrize("ch", [1, 4, 5, 8])      # one and two quads a voxel, whole and partial
@pytest.mark.parametrize("size", [(4, 4, 8), (33, 28, 39)])      # small and 128-voxel tiles
def test_an_infinite_input_stays_infinite(orc, ch, size):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, empty
    sp = (1,) + size
    for v in (np.inf, -np.inf):
        x, w = synth.activations(630, sp + (ch,), "f32"), synth.conv_weights(631, ch, 8, "f32")
        x[0, 2, 1, 3, ch - 1] = v
        y = empty(sp + (8,), "f32")
        k3.conv3d_fwd(to_dev(x, "f32"), to_dev(w, "f32"), None, None, 0, y)
        g, wb = synth.activations(632, sp + (ch,), "f32"), synth.conv_weights(633, 8, ch, "f32")
        g[0, 1, 2, 5, 0] = v
        dx = empty(sp + (8,), "f32")
        k3.conv3d_bwd_data(to_dev(g, "f32"), None, to_dev(wb, "f32"), None, dx)
        torch.cuda.synchronize()
        for got, ref in ((to_f64(y), orc.conv3d_fwd(x.astype(np.float64), w.astype(np.float64), np.zeros(8), relu=False)),
                         (to_f64(dx), orc.conv3d_bwd_data(g.astype(np.float64), wb.astype(np.float64)))):
            inf = np.isinf(ref)
            assert inf.sum() == 27 * 8 and not np.isnan(ref).any()
            assert np.array_equal(got[inf], ref[inf]) and np.isfinite(got[~inf]).all()

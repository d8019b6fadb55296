"""bf16 3x3x3 convolution with channel counts in whole 16s that are no whole 32s, and the first layer at
16 channels, against the fp64 oracle where the dispatch and the tiles change: 256- and 64-voxel tiles,
one and two output blocks, the second one partial, edges one short of and one past a tile, two
sources, several chunks, bit masks, tensors off the 16-byte grid (the general kernels)."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# (N, D, H, W), c1, c2, cout, elements the tensors are shifted by
CASES = [
    ((1, 1, 1, 1), 16, 0, 16, 0),          # one voxel
    ((1, 2, 4, 8), 16, 0, 16, 0),          # exactly one 64-voxel tile
    ((1, 3, 5, 9), 16, 0, 48, 0),          # one past it on every axis, three output blocks
    ((2, 4, 8, 7), 16, 16, 16, 0),         # two sources: two chunks
    ((1, 5, 9, 9), 48, 0, 16, 0),          # three chunks
    ((1, 28, 30, 41), 16, 0, 16, 0),       # 256-voxel tiles, ragged
    ((1, 25, 33, 40), 16, 16, 16, 0),      # the same, two sources / destinations
    ((1, 28, 30, 41), 16, 0, 32, 0),       # 168 tiles: 256-voxel tiles are too few for two blocks at once
    ((2, 29, 31, 39), 16, 0, 48, 0),       # two output blocks, the second group half empty
    ((1, 9, 8, 10), 16, 0, 16, 4),         # tensors between two 16-byte boundaries
    ((1, 3, 7, 15), 1, 0, 16, 0),          # first layer, inside one tile
    ((2, 5, 9, 17), 1, 0, 16, 0),          # one past it on every axis
    ((1, 41, 64, 65), 1, 0, 16, 0),        # 440 tiles
    ((1, 64, 72, 65), 1, 0, 16, 0),        # 720: some workgroups of the weight gradient take two
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
@pytest.mark.parametrize("masked", [0, 1])
def test_narrow_kernels(orc, case, masked):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, empty, rel_l2
    sp, c1, c2, co, shift = case
    tol = 4e-3        # one rounding of the result, 2^-9 relative

    def shifted(t):
        if not shift or t is None:
            return t
        flat = torch.empty(t.numel() + shift, device=t.device, dtype=t.dtype)
        flat[shift:].copy_(t.reshape(-1))
        return flat[shift:].view(t.shape)

    def new(c):
        return shifted(empty(sp + (c,), "bf16").fill_(float("nan")))
    x, w = synth.activations(710, sp + (c1 + c2,), "bf16"), synth.conv_weights(711, c1 + c2, co, "bf16")
    b = (synth.normal(synth.SEED, 712, (co,), np.float64) * 0.5).astype(np.float32)
    dy, ym = synth.activations(713, sp + (co,), "bf16"), synth.activations(714, sp + (co,), "bf16")
    om = synth.activations(715, sp + (c1,), "bf16")
    xd = to_dev(x, "bf16")
    x1, x2 = shifted(xd[..., :c1].contiguous()), shifted(xd[..., c1:].contiguous()) if c2 else None
    wd, dyd, bd = to_dev(w, "bf16"), shifted(to_dev(dy, "bf16")), torch.from_numpy(b).cuda()
    ymd, omd = (shifted(to_dev(ym, "bf16")), shifted(to_dev(om, "bf16"))) if masked else (None, None)

    y, yb = new(co), new(co)
    k3.conv3d_fwd(x1, wd, None, bd, masked, y, x2=x2)
    bits = torch.empty(k3.relu_bits_bytes(yb) // 2, device="cuda", dtype=torch.int16)
    k3.conv3d_fwd_bits(x1, wd, None, bd, masked, yb, bits, x2=x2)
    dW, db = torch.full((3, 3, 3, c1 + c2, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x1, dyd, x2=x2), device="cuda", dtype=torch.uint8)
    k3.conv3d_bwd_weight(x1, dyd, ymd, dW, db, ws, x2=x2)
    dx, dx2, dxb, dxb2 = new(c1), new(c2) if c2 else None, new(c1), new(c2) if c2 else None
    if c1 > 1:
        k3.conv3d_bwd_data(dyd, ymd, wd, None, dx, dx2=dx2, dx_mask=omd)
        # the same mask as bits: the words of 16 channels, lowest first
        words = (om.reshape(-1, 16) > 0).astype(np.uint32) @ (1 << np.arange(16, dtype=np.uint32))
        mb = torch.from_numpy(words.astype(np.uint16).view(np.int16)).cuda()
        k3.conv3d_bwd_data_bits(dyd, ymd, wd, None, dxb, mb, dx2=dxb2)
    torch.cuda.synchronize()

    x64, w64, g64 = x.astype(np.float64), w.astype(np.float64), dy.astype(np.float64)
    if masked:
        g64 = orc.relu_bwd(g64, ym.astype(np.float64))
    assert rel_l2(to_f64(y), orc.conv3d_fwd(x64, w64, b.astype(np.float64), relu=bool(masked))) < tol
    assert torch.equal(y.view(torch.int16), yb.view(torch.int16))
    want = (to_f64(yb).reshape(-1, 16) > 0).astype(np.uint32) @ (1 << np.arange(16, dtype=np.uint32))
    assert np.array_equal(bits.cpu().numpy().view(np.uint16), want.astype(np.uint16))
    rW, rb = orc.conv3d_bwd_weight(x64, g64)
    assert rel_l2(to_f64(dW), rW) < 1e-5      # exact products, fp32 sums
    assert rel_l2(to_f64(db), rb) < 1e-5
    if c1 > 1:
        rdx = orc.conv3d_bwd_data(g64, w64)
        r1 = rdx[..., :c1].copy()
        assert rel_l2(to_f64(dx), orc.relu_bwd(r1, om.astype(np.float64)) if masked else r1) < tol
        assert rel_l2(to_f64(dxb), orc.relu_bwd(r1, om.astype(np.float64))) < tol
        if c2:
            assert rel_l2(to_f64(dx2), rdx[..., c1:]) < tol
            assert torch.equal(dx2.view(torch.int16), dxb2.view(torch.int16))


# (N, D, H, W), cin, cout: weight gradients of small volumes on the 16-channel blocks: a single set of
# partial sums written straight to the gradient, several sets, both sides of the rules that choose
SMALL = [((1, 4, 8, 8), 32, 32), ((1, 8, 8, 8), 128, 128), ((1, 8, 8, 8), 32, 32), ((2, 7, 8, 9), 64, 64),
         ((1, 5, 9, 17), 96, 32), ((1, 4, 4, 4), 256, 256), ((2, 9, 16, 16), 32, 64),
         ((1, 3, 3, 3), 512, 512)]


@pytest.mark.parametrize("case", SMALL, ids=lambda c: "x".join(map(str, c[0] + c[1:])))
@pytest.mark.parametrize("masked", [0, 1])
def test_weight_gradient_of_small_volumes(orc, case, masked):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, rel_l2
    sp, ci, co = case
    x, dy = synth.activations(720, sp + (ci,), "bf16"), synth.activations(721, sp + (co,), "bf16")
    ym = synth.activations(722, sp + (co,), "bf16")
    xd, dyd, ymd = to_dev(x, "bf16"), to_dev(dy, "bf16"), to_dev(ym, "bf16") if masked else None
    ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(xd, dyd), device="cuda", dtype=torch.uint8)
    dW, db = torch.full((3, 3, 3, ci, co), float("nan"), device="cuda"), torch.full((co,), float("nan"), device="cuda")
    k3.conv3d_bwd_weight(xd, dyd, ymd, dW, db, ws)
    dW2 = torch.full_like(dW, float("nan"))
    k3.conv3d_bwd_weight(xd, dyd, ymd, dW2, None, ws)      # no bias gradient wanted
    torch.cuda.synchronize()
    g64 = dy.astype(np.float64)
    if masked:
        g64 = orc.relu_bwd(g64, ym.astype(np.float64))
    rW, rb = orc.conv3d_bwd_weight(x.astype(np.float64), g64)
    assert rel_l2(to_f64(dW), rW) < 1e-5
    assert rel_l2(to_f64(db), rb) < 1e-5
    assert torch.equal(dW, dW2)


@pytest.mark.parametrize("case", [((1, 5, 6, 9), 16, 16), ((1, 3, 5, 17), 1, 16), ((1, 4, 4, 4), 32, 32)],
                         ids=["16-16", "1-16", "32-32"])
def test_a_mask_that_is_not_a_number_is_not_positive(case):
    """Masks are > 0 as values: +NaN and -NaN count like zero (weight gradients of channels in whole 32s
    go by the sign instead: there +NaN counts like one), +Inf like any positive number."""
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, empty, packed_for
    sp, ci, co = case
    x, dy = (to_dev(synth.activations(s, sp + (c,), "bf16"), "bf16") for s, c in ((730, ci), (731, co)))
    w = to_dev(synth.conv_weights(732, ci, co, "bf16"), "bf16")
    pk = packed_for(w)
    odd = torch.tensor([0x7fc0, 0x7f81, -64, -127, 0x7f80, -128, 0, -0x8000, 0x3f80], dtype=torch.int32)   # NaNs, infinities, zeros, one

    def masks(c, seed):
        m = synth.activations(seed, sp + (c,), "bf16")
        m = to_dev(m, "bf16").cpu().view(torch.int16)
        pick = torch.arange(m.numel()) % 3 == 0
        m.view(-1)[pick] = odd.to(torch.int16).repeat(m.numel() // 27 + 1)[:int(pick.sum())]
        m = m.view(torch.bfloat16)
        zero, one = m.clone(), m.clone()
        zero[m.isnan()] = 0
        one[m.isnan() & (m.view(torch.int16) > 0)] = 1
        return m.cuda(), zero.cuda(), one.cuda()
    ym, ym0, ym1 = masks(co, 733)
    om, om0, _ = masks(ci, 734)

    def wgrad(mask):
        ws = torch.empty(k3.conv3d_bwd_weight_workspace_bytes(x, dy), device="cuda", dtype=torch.uint8)
        dW, db = torch.empty((3, 3, 3, ci, co), device="cuda"), torch.empty(co, device="cuda")
        k3.conv3d_bwd_weight(x, dy, mask, dW, db, ws)
        return torch.cat([dW.flatten(), db])
    assert torch.equal(wgrad(ym), wgrad(ym1 if ci % 32 == 0 else ym0))
    if ci == 16:
        def dgrad(mask, omask):
            dx = empty(sp + (ci,), "bf16")
            k3.conv3d_bwd_data(dy, mask, w, pk, dx, dx_mask=omask)
            return dx
        assert torch.equal(dgrad(ym, om), dgrad(ym0, om0))
    # bits of an output that holds NaN (no ReLU): of channels whose bias is one
    b = torch.zeros(co, device="cuda")
    b[::5] = float("nan")
    y = empty(sp + (co,), "bf16")
    bits = torch.empty(k3.relu_bits_bytes(y) // 2, device="cuda", dtype=torch.int16)
    k3.conv3d_fwd_bits(x, w, pk, b, 0, y, bits)
    words = (y.float().cpu().numpy().reshape(-1, 16) > 0).astype(np.uint32) @ (1 << np.arange(16, dtype=np.uint32))
    assert bool(y.isnan().any()) and np.array_equal(bits.cpu().numpy().view(np.uint16), words.astype(np.uint16))

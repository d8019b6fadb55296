"""The small-volume bf16 kernel (forward and backward-data) against the fp64 oracle where it can go
wrong: one voxel, one 4x4x4 tile and one voxel more on every axis, one and several 32-channel chunks,
one and several output blocks, more channels than LDS holds at a time, two sources and destinations, input masks, output
masks as tensor and as bits; and the masked first kernel just past the small kernel's range."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# (N, D, H, W, c1, c2, cout)
CASES = [
    (1, 1, 1, 1, 32, 0, 32),
    (1, 4, 4, 4, 32, 0, 32),          # exactly one tile, one chunk
    (1, 5, 5, 5, 32, 0, 64),          # one past a tile on every axis
    (2, 3, 7, 6, 96, 0, 32),          # three chunks
    (1, 4, 5, 3, 32, 64, 96),         # sources of unequal width, three output blocks of 32
    (1, 16, 16, 16, 64, 0, 64),
    (1, 16, 16, 17, 64, 0, 64),
    (1, 16, 16, 32, 128, 128, 128),   # 512 workgroups forward: the last of the range; two loads of 128 channels
    (2, 20, 24, 24, 64, 0, 64),       # past the range: pipelined kernels, and the first kernel for masked inputs
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_small_volumes(orc, case):
    import torch
    from paper_1811_12174_amd import k3
    from gpu_util import to_dev, to_f64, empty, packed_for, rel_l2
    N, D, H, W, c1, c2, co = case
    sp, cin = (N, D, H, W), c1 + c2
    x, w = synth.activations(620, sp + (cin,), "bf16"), synth.conv_weights(621, cin, co, "bf16")
    b = (synth.normal(synth.SEED, 622, (co,), np.float64) * 0.5).astype(np.float32)
    dy, ym = synth.activations(623, sp + (co,), "bf16"), synth.activations(624, sp + (co,), "bf16")
    om = synth.activations(625, sp + (c1,), "bf16")
    xd, wd, dyd, ymd, omd = (to_dev(t, "bf16") for t in (x, w, dy, ym, om))
    x1, x2 = xd[..., :c1].contiguous(), xd[..., c1:].contiguous() if c2 else None
    pk = packed_for(wd)
    y = empty(sp + (co,), "bf16").fill_(float("nan"))
    bits = torch.zeros(k3.relu_bits_bytes(y) // 2, device="cuda", dtype=torch.int16)
    k3.conv3d_fwd_bits(x1, wd, pk, torch.from_numpy(b).cuda(), 1, y, bits, x2=x2)
    x64, w64, g64 = x.astype(np.float64), w.astype(np.float64), dy.astype(np.float64)
    # one bf16 rounding (relative 2^-9 at most, about 1.7e-3 in the norm) of an fp32 sum
    assert rel_l2(to_f64(y), orc.conv3d_fwd(x64, w64, b.astype(np.float64), relu=True)) < 4e-3
    want = (to_f64(y) > 0).reshape(-1, 16) @ (1 << np.arange(16))
    assert np.array_equal(bits.cpu().numpy().astype(np.int64) & 0xffff, want.astype(np.int64))

    def dgrad(mask_in, mask_out):
        dx = empty(sp + (c1,), "bf16").fill_(float("nan"))
        dx2 = empty(sp + (c2,), "bf16").fill_(float("nan")) if c2 else None
        if mask_out == "bits":
            ob = torch.from_numpy(((om > 0).reshape(-1, 16) @ (1 << np.arange(16))).astype(np.uint16).view(np.int16)).cuda()
            k3.conv3d_bwd_data_bits(dyd, ymd if mask_in else None, wd, pk, dx, ob, dx2=dx2)
        else:
            k3.conv3d_bwd_data(dyd, ymd if mask_in else None, wd, pk, dx, dx2=dx2, dx_mask=omd if mask_out else None)
        torch.cuda.synchronize()
        return dx, dx2
    for mask_in in (False, True):
        r = orc.conv3d_bwd_data(orc.relu_bwd(g64.copy(), ym.astype(np.float64)) if mask_in else g64, w64)
        r1 = orc.relu_bwd(r[..., :c1].copy(), om.astype(np.float64))
        dx, dx2 = dgrad(mask_in, "tensor")
        assert rel_l2(to_f64(dx), r1) < 4e-3
        if c2:
            assert rel_l2(to_f64(dx2), r[..., c1:]) < 4e-3
        dxb, dx2b = dgrad(mask_in, "bits")
        assert torch.equal(dx, dxb) and (not c2 or torch.equal(dx2, dx2b))

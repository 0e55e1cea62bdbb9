"""PAR of up to 64 channels in one launch, on every remainder of the 8x8 tiling and at the
channel counts where lanes mirror the last channel, against the oracle with PAR's bar;
and the anchor update from the transform's own values on both reconstruction paths,
whose anchor slots must be bit-identical to the same fp32 additions; and the gate inline
and launched on both sides of the grid where the launch takes over."""
import numpy as np
import pytest
import torch

from oracle import par as OP
from test_gpu_parity import PAR_REL_RMS, rel_rms

pytestmark = pytest.mark.gpu


def _run(cast_lib, n, Hg, Wg, D, anchors, acc, upd, seed):
    rng = np.random.default_rng(seed)
    base = rng.standard_normal((Hg, Wg, D))
    resid = np.zeros((n, Hg, Wg, D), np.float32)
    for j, a in enumerate(anchors):
        resid[a] = np.roll(base, (j, -j), axis=(0, 1)) + 0.3 * rng.standard_normal((Hg, Wg, D))
    x0 = rng.standard_normal(resid.shape).astype(np.float32)
    out = torch.from_numpy(x0).cuda()
    prm = cast_lib.cast_par_params_default(accumulate=int(acc), update_anchors=int(upd))
    cast_lib.cast_par_reconstruct(torch.from_numpy(resid).cuda(), anchors, prm, out=out)
    got = out.cpu().numpy()
    skip = [t for t in range(n) if t not in anchors]
    ref = OP.par_reconstruct_targets(resid.astype(np.float64), anchors, skip, OP.ParParams())
    ref = np.stack([ref[t] for t in skip]) if isinstance(ref, dict) else np.asarray(ref)
    assert rel_rms(got[skip].astype(np.float64), ref + (x0[skip].astype(np.float64) if acc else 0.0)) <= PAR_REL_RMS
    for a in anchors:
        want = (x0[a] + resid[a] if acc else resid[a]) if upd else x0[a]
        np.testing.assert_array_equal(got[a], want)


@pytest.mark.parametrize("acc,upd", [(False, False), (True, False), (False, True), (True, True)])
@pytest.mark.parametrize("Hg,Wg", [(8, 8), (1, 1), (9, 15), (18, 12), (11, 21), (12, 10), (13, 27), (30, 22), (7, 7)])
def test_one_launch_remainders(cast_lib, Hg, Wg, acc, upd):
    _run(cast_lib, 9, Hg, Wg, 24, (1, 3, 7), acc, upd, 10 * Hg + Wg)


@pytest.mark.parametrize("D", [1, 2, 31, 63, 64, 65, 130])
def test_one_launch_channel_edges(cast_lib, D):
    """64 channels are one wave (one launch), 65 two channel blocks (two launches)."""
    for acc in (False, True):
        _run(cast_lib, 6, 13, 17, D, (0, 4), acc, True, D)


@pytest.mark.parametrize("acc", [False, True])
@pytest.mark.parametrize("tiles_x,blocks", [(8, 28), (9, 25), (8, 32), (9, 29)])
def test_gate_inline_up_to_what_the_chip_holds(cast_lib, tiles_x, blocks, acc):
    """Grids of 1792, 1800, 2048 and 2088 reconstruction blocks, around seven and eight per
    compute unit of 256: the call agrees with the one whose gate is launched (conf_out asked
    for) to the rounding of the channel sums' order."""
    n, Hg, D, anchors = 4, 64, 64 * blocks, (0, 3)
    g = torch.Generator(device="cuda")
    g.manual_seed(blocks)
    base = torch.randn((Hg, 8 * tiles_x, D), generator=g, device="cuda")
    resid = torch.zeros((n, Hg, 8 * tiles_x, D), device="cuda")
    for j, a in enumerate(anchors):
        resid[a] = torch.roll(base, (j, -j), dims=(0, 1)) + 0.3 * torch.randn(base.shape, generator=g, device="cuda")
    prm = cast_lib.cast_par_params_default(accumulate=int(acc))
    conf = torch.zeros(cast_lib.par_debug_shapes(2, Hg, 8 * tiles_x, prm)[1], device="cuda")
    outs = [cast_lib.cast_par_reconstruct(resid, anchors, prm, out=torch.ones_like(resid), conf_out=c)
            for c in (None, conf)]
    a, b = ((o - float(acc))[1:3].double() for o in outs)
    assert float((a - b).norm() / b.norm()) <= 1e-5

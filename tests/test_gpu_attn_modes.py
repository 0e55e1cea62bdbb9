"""Attention at the edges of its copy modes and schedules: a current segment before
chunks of >= 64 rows (segment tiles, the tile that holds the segment's end, history tiles
over one or two chunks), the wide schedule of dh = 32 and 64 and the key split with few
tiles, against the oracle with the bars of test_gpu_parity."""
import math

import numpy as np
import pytest
import torch

from test_gpu_parity import check_attn

pytestmark = pytest.mark.gpu


def _inputs(n_a, S, H, dh, M, Bv, k_eff, n0, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    idx = np.random.default_rng(seed).integers(0, M, size=(n_a, H, k_eff))
    return (r(n_a, S, H, dh), r(M, Bv, H, dh), r(M, Bv, H, dh), torch.tensor(idx, dtype=torch.int32, device="cuda"),
            r(n0, H, dh) if n0 else None, r(n0, H, dh) if n0 else None)


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("n0", [1, 63, 64, 65, 128, 200])
@pytest.mark.parametrize("Bv,k_eff", [(64, 3), (65, 2), (100, 5), (64, 1), (128, 0)])
def test_current_segment_before_long_chunks(cast_lib, dh, n0, Bv, k_eff):
    q, k, v, idx, kc, vc = _inputs(2, 70, 2, dh, 6, Bv, k_eff, n0, 1000 * n0 + Bv + dh)
    for split in (True, False):
        check_attn(cast_lib, q, k, v, idx, k_eff, 1 / math.sqrt(dh), kc=kc, vc=vc, split=split,
                   label=f"current dh{dh} n0 {n0} Bv{Bv} k{k_eff} split {split}")


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("S", [1, 33, 256, 257, 300])
@pytest.mark.parametrize("Bv,k_eff,n0", [(64, 4, 0), (64, 5, 70), (90, 7, 0), (20, 17, 0), (20, 9, 33)])
def test_few_tiles_whole_and_split(cast_lib, dh, S, Bv, k_eff, n0):
    q, k, v, idx, kc, vc = _inputs(1, S, 3, dh, 20, Bv, k_eff, n0, S + Bv + dh)
    for split in (True, False):
        check_attn(cast_lib, q, k, v, idx, k_eff, 1 / math.sqrt(dh), kc=kc, vc=vc, split=split,
                   label=f"few tiles dh{dh} S{S} Bv{Bv} n0 {n0} split {split}")


@pytest.mark.parametrize("dh", [32, 64])
def test_scores_formed_again(cast_lib, dh):
    """Key tiles whose logits rise by far more than the running max's slack take the wide
    schedule's exact path, which forms the tile's scores a second time."""
    q, k, v, idx, kc, vc = _inputs(1, 100, 2, dh, 8, 96, 8, 50, dh)
    idx[:] = torch.arange(8, device="cuda", dtype=torch.int32)
    k *= torch.tensor([0.05, 4, 0.5, 8, 1, 12, 0.1, 6], device="cuda")[:, None, None, None].to(torch.bfloat16)
    check_attn(cast_lib, q, k, v, idx, 8, 1 / math.sqrt(dh), kc=kc, vc=vc, label=f"exact path dh{dh}")


@pytest.mark.parametrize("dh", [32, 64])
@pytest.mark.parametrize("n_a,S,H,M,Bv,k_eff,n0", [
    (2, 40, 138, 40, 64, 34, 0),     # 256 whole units of one tile, 20 in pieces, aligned chunks
    (2, 300, 67, 12, 200, 11, 90),   # two tiles each, 12 units in pieces, a segment, ragged tails
])
def test_whole_units_beside_pieces(cast_lib, dh, n_a, S, H, M, Bv, k_eff, n0):
    """Whole units on every compute unit and the few past them split along the keys, in
    one launch: sampled queries of the first, middle and last (anchor, head) pairs."""
    assert cast_lib.cast_anchor_attn_workspace_bytes(n_a, S, H, dh, k_eff, n0, Bv) > 0
    q, k, v, idx, kc, vc = _inputs(n_a, S, H, dh, M, Bv, k_eff, n0, S + dh)
    rows = [(i, h, s) for i, h in ((0, 0), (0, H // 2), (0, H - 1), (1, 0), (1, H - 20), (1, H - 6), (1, H - 2), (1, H - 1))
            for s in (0, 31, S // 2, S - 1)]
    outs = [check_attn(cast_lib, q, k, v, idx, k_eff, 1 / math.sqrt(dh), kc=kc, vc=vc, rows=rows, split=split,
                       label=f"whole + pieces dh{dh} S{S} split {split}") for split in (True, False)]
    d = (outs[0].float() - outs[1].float()).abs().max().item()
    assert d <= 2.0 ** -7 * max(1.0, outs[1].float().abs().max().item())


@pytest.mark.parametrize("dh", [32, 64, 128])
def test_longest_historys_workspace_serves_shorter_ones(cast_lib, dh):
    """A loop that allocates once for its longest history: every shorter call is accepted
    and is bit-identical to the same call with a workspace of its own size."""
    n_a, S, H, Bv = 2, 256, 8, 64
    q, k, v, idx, _, _ = _inputs(n_a, S, H, dh, 64, Bv, 64, 0, dh)
    ws = torch.empty(cast_lib.cast_anchor_attn_workspace_bytes(n_a, S, H, dh, 64, 0, Bv), dtype=torch.uint8, device="cuda")
    for k_eff in range(64, 0, -1):
        sub = idx[:, :, :k_eff].contiguous()
        a, _ = cast_lib.cast_anchor_attn(q, k, v, sub, k_eff, 0.1, workspace=ws)
        b, _ = cast_lib.cast_anchor_attn(q, k, v, sub, k_eff, 0.1)
        assert torch.equal(a, b), k_eff

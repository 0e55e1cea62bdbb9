"""Coupled routing at the edges of its solvers (one wave up to 128 chunks, four to 512,
eight above; 1, 2, 4 or 8 chunks per lane; u staged in LDS or read from memory) and of
the omission launch (32, 64 and 128 chunks per workgroup), with the checker and the bars
of test_gpu_coupled: u against float64, masks exact on heads with a decision margin."""
import numpy as np
import pytest
import torch

from gen import workloads as W
import gen
from test_gpu_coupled import U_REL_RMS, compare_masks, oracle_means, oracle_u, run_case
from test_gpu_parity import np64

pytestmark = pytest.mark.gpu


def _workload(H, dh, anchors):
    return W.Workload(**{**gen.get(W.TINY).__dict__, "H": H, "dh": dh, "anchors": tuple(anchors)})


@pytest.mark.parametrize("M", [1, 2, 40, 41, 63, 64, 65, 127, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096])
def test_solver_edges(cast_lib, M):
    w = _workload(2, 32, (1, 4, 6))
    (exact, loose), idx = run_case(cast_lib, w, w.anchors, 9, max(1, M // 6), M=M, Bv=2, seed=M)
    assert exact + loose == w.H
    assert (idx[..., 1:] > idx[..., :-1]).all() and int(idx.max()) < M and int(idx.min()) >= 0


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("M", [31, 33, 97, 130])
def test_omission_edges(cast_lib, dh, M):
    w = _workload(3, dh, (0, 2, 3, 5, 8))
    (exact, loose), _ = run_case(cast_lib, w, w.anchors, 11, max(1, M // 4), M=M, Bv=5, seed=dh + M)
    assert exact + loose == w.H


def test_many_anchors(cast_lib):
    """512 anchors of 13 chunks: the masks' LDS at its largest beside the staged u."""
    anchors = tuple(range(1, 1025, 2))
    w = _workload(1, 32, anchors)
    (exact, loose), _ = run_case(cast_lib, w, anchors, 1026, 3, M=13, Bv=2)
    assert exact + loose == w.H


@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("M,lo,hi", [(65, 64, 65), (130, 64, 128), (130, 128, 130), (200, 0, 64), (200, 60, 200)])
def test_chunks_of_minus_infinite_score(cast_lib, dh, M, lo, hi):
    """Chunks lo .. hi - 1, which fill whole score tiles of 64, score -inf for every
    anchor: their pi and u are 0 and the others are those of a softmax without them."""
    w = _workload(2, dh, (1, 4, 6))
    q, k, v, _, _ = gen.attn_inputs(w, seed=M + lo, device="cuda", M=M, Bv=3)
    q[..., 0] = 1.0
    k[lo:hi, ..., 0] = -float("inf")
    w_o = gen.wo_weight(w.D, seed=7, device="cuda")
    topk = (M - (hi - lo)) // 4
    idx, k_eff, u = cast_lib.cast_route_coupled(q, k, v, cast_lib.cast_wo_gram(w_o, w.H, dh), w.anchors, 9, topk,
                                                w.scale, want_u=True)
    qb, kb, vb = oracle_means(q, torch.where(torch.isinf(k), torch.zeros_like(k), k), v)
    kb[lo:hi, :, 0] = -1e30          # (finite, and as far below every other score)
    u_or = oracle_u(qb, kb, vb, w_o, w.scale, dh)
    assert np.all(u_or[..., lo:hi] == 0.0)
    got = np64(u)
    assert np.all(got[..., lo:hi] == 0.0)
    assert np.linalg.norm(got - u_or) <= U_REL_RMS * np.linalg.norm(u_or)
    assert k_eff == topk
    exact, loose = compare_masks(idx, u_or, w.anchors, 9, topk, f"-inf dh{dh} M{M} {lo}..{hi}")
    assert exact + loose == w.H

"""TopK selection of cast_route_kv at the edges of its kernels (ranks up to 40 chunks; 64, 256 and
512 in one launch by keys per lane, 1024, 2048 and 4096 in two): one token per frame and chunk
with small integer channels makes every score an exact integer in fp32, so the selection
has many exact ties and must equal the order (score descending, index ascending) with no
tolerance."""
import numpy as np
import pytest

import oracle.route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 7, 8, 9, 40, 41, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1024, 1025, 2048, 2049, 4095, 4096])
@pytest.mark.parametrize("dh,H,n_a", [(32, 3, 1), (64, 2, 5), (128, 1, 4)])
def test_selection_at_kernel_edges(cast_lib, dh, H, n_a, M):
    import torch
    rng = np.random.default_rng(1000 * dh + M)
    q = rng.integers(-2, 3, size=(n_a, 1, H, dh)).astype(np.float32)
    k = rng.integers(-2, 3, size=(M, 1, H, dh)).astype(np.float32)
    q[0, 0, 0] = 0.0                     # every score of this pair is +-0: all tied
    want = np.einsum("ishd,mshd->ihm", q.astype(np.float64), k.astype(np.float64))
    tq = torch.from_numpy(q).to(torch.bfloat16).cuda()
    tk = torch.from_numpy(k).to(torch.bfloat16).cuda()
    for topk in sorted({1, max(1, M // 5), max(1, M - 1), M}):
        idx, k_eff, scores = cast_lib.cast_route_kv(tq, tk, topk, 1.0, want_scores=True)
        assert k_eff == topk
        np.testing.assert_array_equal(scores.cpu().numpy(), want)
        got = idx.cpu().numpy()
        for i in range(n_a):
            for h in range(H):
                assert got[i, h].tolist() == oracle.route.topk_select(want[i, h], topk), (i, h, topk)


@pytest.mark.parametrize("M", [20, 60, 200, 400, 600])
def test_selection_with_infinite_scores(cast_lib, M):
    """Scores of +-inf order like any other value, ties among them by index."""
    import torch
    rng = np.random.default_rng(M)
    q = np.ones((1, 1, 1, 32), np.float32)
    k = rng.integers(-3, 4, size=(M, 1, 1, 32)).astype(np.float32)
    k[rng.random(M) < 0.2, 0, 0, 3] = np.inf
    k[(rng.random(M) < 0.2) & np.isfinite(k[:, 0, 0, 3]), 0, 0, 5] = -np.inf
    want = k.sum(axis=(1, 2, 3)).astype(np.float64)
    idx, _, _ = cast_lib.cast_route_kv(torch.from_numpy(q).to(torch.bfloat16).cuda(),
                                       torch.from_numpy(k).to(torch.bfloat16).cuda(), M // 3, 1.0)
    order = np.lexsort((np.arange(M), -want))[: M // 3]
    assert idx.cpu().numpy()[0, 0].tolist() == sorted(order.tolist())

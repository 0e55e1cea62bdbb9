"""Frame selection at the edges of its selection paths (one wave up to 64 frames, ranks
to 512, counting in all waves above, four frames per lane at 4096), with the checker and the bars of
test_gpu_frame_select, and its order on scores that are not numbers."""
import numpy as np
import pytest
import torch

from test_gpu_frame_select import one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 32, 33, 40, 41, 63, 64, 65, 128, 131, 511, 512, 513, 1024, 1025, 4096])
@pytest.mark.parametrize("branches", [0, 1, 2])
def test_edges(cast_lib, n, branches):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + branches)
    mag = 0.3 + 2.5 * torch.rand((2, n, 1, 1), generator=g, device="cuda")
    x = torch.randn((2, n, 5, 24), generator=g, device="cuda") * mag
    cam, act = (x[0] if branches > 0 else None), (x[1] if branches > 1 else None)
    ages = torch.randint(0, 5, (n,), generator=g, device="cuda", dtype=torch.int32)
    h = [int(a) for a in ages.cpu()]
    for k_f in sorted({1, (n + 2) // 3, n}):
        one_step(cast_lib, cam, act, [0] if n < 3 else [0, n // 2, n - 1], k_f, ages.clone(), np.array(h),
                 f"n{n} k{k_f} b{branches}", n_cur=n)


@pytest.mark.parametrize("n", [12, 100, 600])
def test_nan_scores_are_chosen_first_come(cast_lib, n):
    """A NaN score is neither beaten nor beats: the frames that hold one are chosen with
    the K_f best of the others, and the first K_f of all chosen are written."""
    x = torch.ones((n, 2, 8), device="cuda") * torch.arange(1, n + 1, device="cuda")[:, None, None]
    x[[3, n - 2]] = float("nan")
    ages = torch.zeros(n, dtype=torch.int32, device="cuda")
    k_f = 4
    score = torch.empty(n, device="cuda")
    got = cast_lib.cast_frame_select(x, None, [0], k_f, ages, score_out=score).cpu().numpy()
    s = score.cpu().numpy()
    assert np.isnan(s[[3, n - 2]]).all() and np.isfinite(np.delete(s, [3, n - 2])).all()
    best = sorted((i for i in range(n) if not np.isnan(s[i])), key=lambda i: (-s[i], i))[:k_f]
    assert got.tolist() == sorted(best + [3, n - 2])[:k_f]

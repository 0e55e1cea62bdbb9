"""Token means with one and with two chunks per workgroup: chunk sizes and grid lengths on
both sides of the rule (up to 64 tokens, 2048 segments x 128-channel groups), odd numbers
of chunks, tokens that do not fill the waves, against float64 means."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bv", [1, 3, 31, 64, 65])
@pytest.mark.parametrize("H,dh,M", [(24, 128, 85), (24, 128, 86), (5, 32, 1023), (5, 32, 1024), (5, 32, 1025), (3, 64, 1365)])
def test_means_on_both_sides_of_the_rule(cast_lib, Bv, H, dh, M):
    g = torch.Generator(device="cuda")
    g.manual_seed(Bv + M)
    q = torch.zeros((1, 2, H, dh), device="cuda")
    q[..., 0] = 1.0                      # a score is the mean of its head's first channel
    k = (torch.randn((M, Bv, H, dh), generator=g, device="cuda") + 2.0).to(torch.bfloat16)
    _, _, scores = cast_lib.cast_route_kv(q.to(torch.bfloat16), k, 3, 1.0, want_scores=True)
    want = k[..., 0].double().mean(dim=1).t().cpu().numpy()
    # Bv fp32 additions of values below 8 in any order, then one division
    assert np.abs(scores[0].cpu().numpy() - want).max() <= (Bv + 2) * 2.0 ** -24 * 8

"""The importance formed beside the similarity pass: the step's scores are those of its parts, bit for bit."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu


def _keys(P, H, N, clusters, seed):
    """Copies at distances of their own around a few centroids, so that another partner than the newest gives another sum."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cent = torch.randn((P, H, clusters, 128), generator=gen, device="cuda")
    which = torch.randint(0, clusters, (P, H, N, 1), generator=gen, device="cuda")
    noise = 0.05 + 0.85 * torch.rand((P, H, N, 1), generator=gen, device="cuda")
    k = torch.gather(cent, 2, which.expand(-1, -1, -1, 128))
    return (k + noise * torch.randn(k.shape, generator=gen, device="cuda")).bfloat16(), gen


@pytest.mark.parametrize("P,H,G,n,T", [
    pytest.param(1, 2, 4, 376, 0.5, id="one tile a workgroup"),
    pytest.param(3, 8, 5, 1023, 0.5, id="column parts"),
    pytest.param(32, 8, 1, 1025, 0.5, id="as many heads as compute units, one candidate in a second workgroup"),
    pytest.param(25, 8, 4, 1029, 0.95, id="full scan"),
    pytest.param(25, 8, 2, 2400, 0.5, id="listed rows"),
    pytest.param(1, 4, 8, 4099, 0.5, id="long, an odd end"),
    pytest.param(1, 1, 1, 130, 0.5, id="windows cut at both ends"),
    pytest.param(33, 8, 4, 300, 0.5, id="more heads than compute units: formed by the finalize kernel"),
])
def test_scores_of_the_step_are_those_of_its_parts(P, H, G, n, T):
    print(f"[gpu-case] importance beside the similarity pass P={P} H={H} G={G} n={n} T={T}", flush=True)
    N = n + 8
    k, gen = _keys(P, H, N, 40, n)
    q = torch.randn((P, H * G, 8, 128), generator=gen, device="cuda").bfloat16()
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H * G, n_tokens=N, budget=max(16, N - 100), sim_threshold=T, lam=0.5)
    _, _, _, kept, score = rkv.rkv_compress(shape, q, k, k, want_score=True)
    importance = rkv.rkv_score_importance(shape, q, k)
    redundancy = rkv.rkv_score_redundancy(shape, k)
    kept2, score2 = rkv.rkv_select_topk(shape, importance, redundancy, want_score=True)
    assert torch.equal(score, score2) and torch.equal(kept, kept2)

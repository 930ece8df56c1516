"""Few heads: a workgroup takes 128 rows against one column tile."""
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


@pytest.mark.parametrize("P,H,n,clusters,T,page", [
    pytest.param(1, 1, 129, 5, 0.45, 0, id="two tiles, the newest one key"),
    pytest.param(1, 2, 256, 400, 0.45, 0, id="two whole tiles, hardly a partner"),
    pytest.param(3, 3, 385, 9, 0.0, 0, id="heads no multiple of eight, T = 0"),
    pytest.param(1, 8, 1000, 60, 0.45, 16, id="paged"),
    pytest.param(8, 8, 640, 20, 0.95, 0, id="1600 workgroups, T above 0.9"),
    pytest.param(1, 6, 2048, 300, 0.45, 0, id="sixteen tiles"),
    pytest.param(1, 8, 1800, 1, 0.45, 0, id="every row a partner of every other"),
    pytest.param(33, 4, 384, 30, 0.45, 0, id="132 heads: in the step, not in the pass alone"),
])
def test_one_tile_a_workgroup(P, H, n, clusters, T, page):
    print(f"[gpu-case] few heads P={P} H={H} n={n} clusters={clusters} T={T} page={page}", flush=True)
    N = n + 8
    k, gen = _keys(P, H, N, clusters, n)
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 64, sim_threshold=T, lam=0.5)
    stored = k
    if page:
        per = -(-N // page)
        table = torch.randperm(P * per, generator=gen, device="cuda").int().reshape(P, per)
        rows = torch.zeros((P, H, per * page, 128), dtype=torch.bfloat16, device="cuda")
        rows[:, :, :N] = k
        stored = torch.empty((P * per, H, page, 128), dtype=torch.bfloat16, device="cuda")
        stored[table.reshape(-1).long()] = rows.view(P, H, per, page, 128).transpose(1, 2).reshape(P * per, H, page, 128)
        shape.page_size, shape.block_table = page, table
    q = torch.randn((P, H, 8, 128), generator=gen, device="cuda").bfloat16()
    _, _, _, kept, score = rkv.rkv_compress(shape, q, stored, stored, want_score=True)
    red, mean = rkv.rkv_score_redundancy(shape, stored, want_mean_sim=True)
    kept2, score2 = rkv.rkv_select_topk(shape, rkv.rkv_score_importance(shape, q, stored), red, want_score=True)
    assert torch.equal(score, score2) and torch.equal(kept, kept2)
    shape.flags = rkv.RKV_FLAG_SKIP_SATURATED             # row blocks of 256 rows, the same products in the same order
    assert torch.equal(mean, rkv.rkv_score_redundancy(shape, stored, want_mean_sim=True)[1])
    unit = torch.nn.functional.normalize(k[P - 1, H - 1, :n].double(), dim=-1)
    sim = unit @ unit.t()
    sim.fill_diagonal_(0.0)
    newest = ((sim > T) * torch.arange(1, n + 1, device="cuda")).amax(-1)
    forgiven = torch.where(newest > 0, sim.gather(-1, (newest - 1).clamp_min(0)[:, None])[:, 0], 0.0)
    firm = ((sim - T).abs() > 1e-5).all(-1)
    # products of 128 exact terms summed in 32 bits: 2^-22 of a row sum of at most n; a wrong partner changes a mean by far more
    assert ((mean[P - 1, H - 1].double() - (sim.sum(-1) - forgiven) / n).abs()[firm] <= 2.0 ** -20).all()

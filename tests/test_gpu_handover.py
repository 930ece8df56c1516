"""Row blocks leave the similarity pass with their last open rows, which the block itself takes against the older keys, or
(where all blocks together would read more than 500 MB) a second kernel in groups of 128: mean similarities against float64 and
against the schedule without hand-over, at sizes where a block leaves with no rows, few, as many as it may, or not at all,
and where a workgroup of the second kernel takes no group, one, or several."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu

CASES = [
    # problems, kv heads, candidates n, clusters, page size
    pytest.param(75, 4, 129, 8, 0, id="two tiles, the second one key"),
    pytest.param(75, 4, 257, 4, 0, id="three tiles, hardly a row left"),
    pytest.param(75, 4, 292, 40, 0, id="more heads than compute units"),
    pytest.param(25, 4, 1024, 60, 0, id="whole tiles, last row block of 256"),
    pytest.param(10, 4, 2500, 60, 0, id="few rows left"),
    pytest.param(10, 4, 2500, 400, 0, id="many rows left"),
    pytest.param(4, 4, 8200, 1000, 0, id="long scan, several looks"),
    pytest.param(10, 4, 2500, 2500, 0, id="few rows ever meet a partner"),
    pytest.param(10, 4, 2500, 60, 16, id="paged"),
]


def _reference(k, T):
    """Mean similarity in float64 and the rows that no pair within 1e-5 of T leaves open to rounding."""
    unit = torch.nn.functional.normalize(k.double(), dim=-1)
    sim = unit @ unit.t()
    sim.fill_diagonal_(0.0)
    n = sim.shape[0]
    newest = ((sim > T) * torch.arange(1, n + 1, device=k.device)).amax(-1)
    forgiven = torch.where(newest > 0, sim.gather(-1, (newest - 1).clamp_min(0)[:, None])[:, 0], 0.0)
    return (sim.sum(-1) - forgiven) / n, ((sim - T).abs() > 1e-5).all(-1)


@pytest.mark.parametrize("P,H,n,clusters,page", CASES)
def test_rows_left_open_by_the_scan(P, H, n, clusters, page):
    print(f"[gpu-case] handover P={P} H={H} n={n} clusters={clusters} page={page}", flush=True)
    T, N = 0.45, n + 8
    gen = torch.Generator(device="cuda").manual_seed(n + clusters)
    # copies at distances of their own, so that another partner than the newest gives another sum
    cent = torch.randn((P, H, clusters, 128), generator=gen, device="cuda")
    which = torch.randint(0, clusters, (P, H, N, 1), generator=gen, device="cuda")
    noise = 0.05 + 0.85 * torch.rand((P, H, N, 1), generator=gen, device="cuda")
    k = torch.gather(cent, 2, which.expand(-1, -1, -1, 128))
    k = (k + noise * torch.randn(k.shape, generator=gen, device="cuda")).bfloat16()
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 64, sim_threshold=T)
    stored = k
    if page:
        per = -(-N // page)
        table = torch.randperm(P * per, generator=gen, device="cuda").int().reshape(P, per)
        stored = torch.zeros((P * per, H, page, 128), dtype=torch.bfloat16, device="cuda")
        rows = torch.zeros((P, H, per * page, 128), dtype=torch.bfloat16, device="cuda")
        rows[:, :, :N] = k
        stored[table.reshape(-1).long()] = rows.view(P, H, per, page, 128).transpose(1, 2).reshape(P * per, H, page, 128)
        shape.page_size, shape.block_table = page, table
    _, mean = rkv.rkv_score_redundancy(shape, stored, want_mean_sim=True)
    _, again = rkv.rkv_score_redundancy(shape, stored, want_mean_sim=True)
    assert torch.equal(mean, again)
    for p, h in {(0, 0), (P // 2, 1), (P - 1, H - 1)}:
        want, firm = _reference(k[p, h, :n], T)
        assert firm.float().mean() > 0.5
        # 0.02 / n: a partner that is missed changes a mean by at least T / n, a wrong one by 0.1 / n on
        # average; rounding is 2^-22 of a row sum of at most n / clusters + 30, below 0.001
        assert ((mean[p, h].double() - want).abs()[firm] <= 0.02 / n).all()


def _segments(P, H, n, segments, clusters, lone, gen):
    """Keys whose partners lie inside their own one of `segments` stretches, `lone` of them without any; the newest
    stretch of every other head holds no partners at all, so its row blocks stay in the scan to the end."""
    part = torch.arange(n, device="cuda") * segments // n
    cent = torch.randn((P, H, segments * clusters, 128), generator=gen, device="cuda")
    which = part * clusters + torch.randint(0, clusters, (P, H, n), generator=gen, device="cuda")
    k = torch.gather(cent, 2, which[..., None].expand(-1, -1, -1, 128))
    k = k + (0.05 + 0.85 * torch.rand((P, H, n, 1), generator=gen, device="cuda")) * torch.randn(k.shape, generator=gen, device="cuda")
    alone = torch.rand((P, H, n), generator=gen, device="cuda") < lone
    alone[:, ::2] |= part == segments - 1
    return torch.where(alone[..., None], torch.randn(k.shape, generator=gen, device="cuda"), k).bfloat16()


@pytest.mark.parametrize("P,H,n,segments,clusters,lone", [
    pytest.param(40, 8, 1144, 8, 8, 0.2, id="three blocks, leaving one after another"),
    pytest.param(40, 8, 1144, 1, 8, 0.25, id="a quarter of the rows alone: some blocks leave and some stay"),
    pytest.param(12, 8, 4300, 8, 12, 0.2, id="twelve blocks, lists of several groups"),
    pytest.param(70, 8, 2300, 2, 4, 0.22, id="more heads than compute units, several groups for one workgroup"),
    pytest.param(3, 4, 9000, 3, 40, 0.1, id="few heads, long scans"),
])
def test_row_blocks_that_leave_at_different_points(P, H, n, segments, clusters, lone):
    print(f"[gpu-case] handover mixed P={P} H={H} n={n} segments={segments} lone={lone}", flush=True)
    T, N = 0.45, n + 8
    gen = torch.Generator(device="cuda").manual_seed(n + segments)
    k = _segments(P, H, N, segments, clusters, lone, gen)
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 64, sim_threshold=T)
    _, mean = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)
    _, again = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)
    assert torch.equal(mean, again)
    for p, h in {(0, 0), (P // 2, 1), (P - 1, H - 1)}:
        want, firm = _reference(k[p, h, :n], T)
        assert firm.float().mean() > 0.5
        # as above: a row sum is at most n / clusters + 30
        assert ((mean[p, h].double() - want).abs()[firm] <= 0.02 / n).all()


@pytest.mark.parametrize("P,H,n,segments,clusters,lone", [
    pytest.param(70, 4, 128, 1, 8, 0.1, id="one tile: nothing to leave"),
    pytest.param(70, 4, 129, 1, 8, 0.1, id="the newest tile holds one key"),
    pytest.param(70, 4, 256, 1, 6, 0.24, id="two whole tiles"),
    pytest.param(140, 4, 390, 2, 4, 0.2, id="second block of six rows"),
    pytest.param(70, 4, 642, 1, 4, 0.2, id="a wave without rows"),
    pytest.param(70, 4, 642, 1, 400, 0.0, id="hardly a hit: no second look before tile 8"),
    pytest.param(40, 8, 1144, 1, 200, 0.1, id="leaving late"),
    pytest.param(40, 8, 1144, 1, 8, 0.25, id="as many rows left as can be"),
    pytest.param(9, 4, 3457, 4, 8, 0.15, id="few heads, long scan, last tile of one key"),
    pytest.param(12, 8, 4300, 2, 12, 0.2, id="listed"),
])
def test_same_bits_as_the_schedule_without_hand_over(P, H, n, segments, clusters, lone):
    print(f"[gpu-case] handover bits P={P} H={H} n={n} segments={segments} clusters={clusters} lone={lone}", flush=True)
    N = n + 8
    gen = torch.Generator(device="cuda").manual_seed(n + clusters)
    k = _segments(P, H, N, segments, clusters, lone, gen)
    mean = {}
    for flags in (0, rkv.RKV_FLAG_SKIP_SATURATED):
        shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 64, sim_threshold=0.45, flags=flags)
        mean[flags] = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)[1]
    # the flag's kernel keeps every row in its block's scan; both form the same products in the same order
    assert torch.equal(mean[0], mean[rkv.RKV_FLAG_SKIP_SATURATED])


def _heads_of(P, H, n, clusters, T, flags=0, strided=False, seed=3):
    """A cache whose rows left open are few, dense or as the first n + 8 rows of a [P, tokens, H, 128] allocation."""
    N = n + 8
    gen = torch.Generator(device="cuda").manual_seed(seed)
    k = _segments(P, H, N, 2, clusters, 0.1, gen)
    if strided:
        store = torch.randn((P, N + 5, H, 128), generator=gen, device="cuda").bfloat16()
        store[:, :N] = k.transpose(1, 2)
        k = store.transpose(1, 2)[:, :, :N]
    return k, rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 64, sim_threshold=T, flags=flags)


OWN_AND_LISTED = [pytest.param(50, 8, 1000, id="taken by the block"), pytest.param(12, 8, 4300, id="listed")]


@pytest.mark.parametrize("P,H,n", OWN_AND_LISTED)
def test_strided_keys(P, H, n):
    print(f"[gpu-case] handover strided P={P} H={H} n={n}", flush=True)
    k, shape = _heads_of(P, H, n, 10, 0.45, strided=True)
    assert not k.is_contiguous()
    _, mean = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)
    _, dense = rkv.rkv_score_redundancy(shape, k.contiguous(), want_mean_sim=True)
    assert torch.equal(mean, dense)
    want, firm = _reference(k[P - 1, 1, :n], 0.45)
    assert ((mean[P - 1, 1].double() - want).abs()[firm] <= 0.02 / n).all()


@pytest.mark.parametrize("P,H,n", OWN_AND_LISTED)
@pytest.mark.parametrize("kind", ["T = 0", "identical keys", "zero rows"])
def test_degenerate_keys(P, H, n, kind):
    print(f"[gpu-case] handover degenerate P={P} H={H} n={n} {kind}", flush=True)
    k, shape = _heads_of(P, H, n, 10, 0.0 if kind == "T = 0" else 0.45)
    if kind == "identical keys":
        k[:] = k[:, :, :1].clone()
    if kind == "zero rows":
        k[:, :, 5::7] = 0
    _, mean = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)
    shape.flags = rkv.RKV_FLAG_SKIP_SATURATED
    assert torch.equal(mean, rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)[1])
    assert torch.isfinite(mean).all()
    if kind == "identical keys":
        # n - 1 partners of similarity 1, of which one is forgiven
        assert ((mean - (n - 2) / n).abs() <= 1e-5).all()
    if kind == "zero rows":
        # all similarities are 0; the diagonal that is taken off is (1 - eps r)^2 with r = 1 / eps rounded to 2^-24 of itself
        assert (mean[:, :, 5::7].abs() <= 2.0 ** -46 / n).all()


def test_longest_cache_with_row_indices_up_to_its_end():
    P, H, n = 1, 3, 32760                                 # 258 row blocks: the smallest unsplit scan of this length
    print(f"[gpu-case] handover longest n={n}", flush=True)
    k, shape = _heads_of(P, H, n, 40, 0.45)
    _, mean = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)
    shape.flags = rkv.RKV_FLAG_SKIP_SATURATED
    assert torch.equal(mean, rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)[1])
    unit = torch.nn.functional.normalize(k[0, 1, :n].double(), dim=-1)
    later = torch.arange(1, n + 1, device="cuda")
    for first in (0, 16000, n - 2000):                    # 2000 rows of the matrix at a time
        sim = unit[first:first + 2000] @ unit.t()
        sim[torch.arange(2000), torch.arange(first, first + 2000)] = 0.0
        newest = ((sim > 0.45) * later).amax(-1)
        forgiven = torch.where(newest > 0, sim.gather(-1, (newest - 1).clamp_min(0)[:, None])[:, 0], 0.0)
        firm = ((sim - 0.45).abs() > 1e-5).all(-1)
        assert firm.float().mean() > 0.5
        got = mean[0, 1, first:first + 2000].double()
        # a row sum is at most n / 80 + 60 here: rounding of 2^-22 of that, a wrong partner 0.1 / n on average
        assert ((got - (sim.sum(-1) - forgiven) / n).abs()[firm] <= 0.02 / n).all()


@pytest.mark.parametrize("P,H,n", OWN_AND_LISTED)
def test_graph_replays(P, H, n):
    print(f"[gpu-case] handover graph P={P} H={H} n={n}", flush=True)
    caches = [_heads_of(P, H, n, clusters, 0.45, seed=clusters)[0] for clusters in (10, 60, 25)]
    _, shape = _heads_of(P, H, n, 10, 0.45)
    q = torch.randn((P, H, 8, 128), device="cuda").bfloat16()
    ws = rkv.make_workspace(shape)
    eager = [rkv.rkv_compress(shape, q, k, k, ws=ws, want_score=True) for k in caches]
    k = caches[0].clone()
    out = [torch.empty_like(t) for t in eager[0][1:4]]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rkv.rkv_compress(shape, q, k, k, ws=ws, k_out=out[0], v_out=out[1], kept_idx=out[2])
    for i in (1, 0, 2, 1):                                # a list that an earlier replay left behind must not show
        k.copy_(caches[i])
        graph.replay()
        torch.cuda.synchronize()
        for got, want in zip(out, eager[i][1:4]):
            assert torch.equal(got, want)
        again = rkv.rkv_compress(shape, q, caches[i], caches[i], ws=ws)
        assert torch.equal(again[3], eager[i][3])

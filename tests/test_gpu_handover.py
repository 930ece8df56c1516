"""The similarity pass hands its last open rows to a second kernel: mean similarities against float64 at sizes where
the list of handed rows is empty, short, longer than one workgroup takes, and where it is cut short by the scan's end."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu

CASES = [
    # problems, kv heads, candidates n, clusters, page size
    pytest.param(75, 4, 129, 8, 0, id="two tiles, the second one key"),
    pytest.param(75, 4, 257, 4, 0, id="three tiles, hardly a row left"),
    pytest.param(75, 4, 292, 40, 0, id="more heads than compute units: four waves"),
    pytest.param(25, 4, 1024, 60, 0, id="whole tiles, last row block of 256"),
    pytest.param(10, 4, 2500, 60, 0, id="short list"),
    pytest.param(10, 4, 2500, 400, 0, id="list of several workgroups"),
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
    assert torch.equal(mean, again)                       # whatever order the rows were listed in
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

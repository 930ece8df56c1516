"""The gather of kept rows, byte for byte: last blocks of one row and of all but one, caches below and above the size from which they are
read past the last cache, strided and paged, and outputs inside a larger allocation."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,H,N,budget,page,strided", [
    pytest.param(1, 1, 20, 9, 0, False, id="nine rows"),
    pytest.param(3, 5, 300, 16, 0, True, id="one whole block a head, strided"),
    pytest.param(2, 4, 300, 33, 0, False, id="a last block of one row"),
    pytest.param(2, 3, 333, 31, 16, False, id="paged, a last block short of one row"),
    pytest.param(64, 8, 1030, 1000, 0, False, id="258 MB: read past the caches"),
    pytest.param(64, 8, 1030, 17, 64, False, id="paged, read past the caches"),
])
def test_rows_are_the_kept_ones(P, H, N, budget, page, strided):
    print(f"[gpu-case] gather P={P} H={H} N={N} budget={budget} page={page}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(N + budget)
    kv = [torch.randn((P, N, H, 128) if strided else (P, H, N, 128), generator=gen, device="cuda").bfloat16() for _ in range(2)]
    kv = [t.transpose(1, 2) if strided else t for t in kv]
    kept = torch.rand((P, H, N), generator=gen, device="cuda").argsort(-1)[..., :budget].sort(-1)[0].int()
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=budget, alpha=8)
    stored = kv
    if page:
        per = -(-N // page)
        table = torch.randperm(P * per, generator=gen, device="cuda").int().reshape(P, per)
        shape.page_size, shape.block_table = page, table
        stored = []
        for t in kv:
            rows = torch.zeros((P, H, per * page, 128), dtype=torch.bfloat16, device="cuda")
            rows[:, :, :N] = t
            pool = torch.empty((P * per, H, page, 128), dtype=torch.bfloat16, device="cuda")
            pool[table.reshape(-1).long()] = rows.view(P, H, per, page, 128).transpose(1, 2).reshape(P * per, H, page, 128)
            stored.append(pool)
    room = [torch.full((P, H, budget + 3, 128), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    out = rkv.rkv_compact(shape, *stored, kept, k_out=room[0][:, :, :budget], v_out=room[1][:, :, :budget])
    for got, t, r in zip(out, kv, room):
        assert torch.equal(got, torch.gather(t, 2, kept[..., None].long().expand(-1, -1, -1, 128)))
        assert (r[:, :, budget:] == 7.0).all()

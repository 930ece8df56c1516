"""The pre-pass for queries of two row tiles and chunks by the thousand gives the bits of the general one: the same problems in one
call and one by one, at a ragged last chunk, whole chunks, one chunk a head, and a number of heads that leaves shares uneven."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [0, rkv.RKV_FLAG_RECENCY_TRANSPOSED, rkv.RKV_FLAG_TRIANGULAR_SCAN])
@pytest.mark.parametrize("P,H,G,n,strided", [
    pytest.param(1540, 2, 5, 200, False, id="two chunks, the second ragged"),
    pytest.param(3075, 2, 8, 65, False, id="one chunk a head, 64 query rows, an odd number of problems"),
    pytest.param(515, 3, 7, 512, False, id="four whole chunks, heads that are no multiple of eight"),
    pytest.param(769, 2, 5, 513, True, id="a last chunk of one key, strided keys and queries"),
])
def test_same_bits_as_a_call_per_problem(P, H, G, n, strided, flags):
    """The flagged schedules add to words that the pre-pass clears: the workspaces are full of other values before every call."""
    print(f"[gpu-case] prepass dma P={P} H={H} G={G} n={n} strided={strided} flags={flags}", flush=True)
    N, d = n + 8, 128
    assert P * H * -(-n // 128) >= 8 * 768
    gen = torch.Generator(device="cuda").manual_seed(n)
    if strided:
        k = torch.randn((P, N + 1, H, d), generator=gen, device="cuda").bfloat16().transpose(1, 2)[:, :, :N]
        q = torch.randn((P, 8, H * G, d), generator=gen, device="cuda").bfloat16().transpose(1, 2)
    else:
        k = torch.randn((P, H, N, d), generator=gen, device="cuda").bfloat16()
        q = torch.randn((P, H * G, 8, d), generator=gen, device="cuda").bfloat16()
    budget = N - max(1, n // 4)
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H * G, n_tokens=N, budget=budget, sim_threshold=0.2, flags=flags)
    ws = rkv.make_workspace(shape).fill_(0xa5)
    _, _, _, kept, score = rkv.rkv_compress(shape, q, k, k, ws=ws, want_score=True)
    importance = rkv.rkv_score_importance(shape, q, k, ws=ws.fill_(0xa5))
    one = rkv.Shape(num_problems=1, kv_heads=H, q_heads=H * G, n_tokens=N, budget=budget, sim_threshold=0.2, flags=flags)
    ws = rkv.make_workspace(one)
    for p in (0, 1, P // 2, P - 2, P - 1):
        part = slice(p, p + 1)
        _, _, _, kept1, score1 = rkv.rkv_compress(one, q[part], k[part], k[part], ws=ws.fill_(0xa5), want_score=True)
        assert torch.equal(importance[part], rkv.rkv_score_importance(one, q[part], k[part]))
        assert torch.equal(score[part], score1) and torch.equal(kept[part], kept1)

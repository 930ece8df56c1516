"""The finalize kernel with one and with four requests at a time: the step's scores and kept rows are those of its parts (one at a time), bit
for bit, on both sides of the line, where the last batch holds one, two, three and four values, with few heads and with many, and without
the similarity pass."""
import pytest
import torch

from paper_2505_24133_amd import rkv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam", [0.5, 1.0])
@pytest.mark.parametrize("P,H,n", [
    pytest.param(1, 2, 3, id="three candidates"),
    pytest.param(1, 2, 1024, id="one a thread"),
    pytest.param(2, 4, 2048, id="the last size of one at a time"),
    pytest.param(2, 4, 2049, id="three a thread, the third of one"),
    pytest.param(70, 4, 2048, id="more heads than compute units, two a thread"),
    pytest.param(70, 4, 2049, id="more heads than compute units, the third of one"),
    pytest.param(65, 4, 4096, id="whole batches"),
    pytest.param(1, 3, 4097, id="a batch of one"),
    pytest.param(1, 1, 9217, id="three batches, the last of two and one more candidate"),
])
def test_step_and_parts_agree(P, H, n, lam):
    print(f"[gpu-case] finalize batches P={P} H={H} n={n} lam={lam}", flush=True)
    N = n + 8
    gen = torch.Generator(device="cuda").manual_seed(n)
    k = torch.randn((P, H, N, 128), generator=gen, device="cuda").bfloat16()
    k[:, :, n // 2:n] = k[:, :, :n - n // 2].clone()              # partners, and equal scores
    q = torch.randn((P, H * 4, 8, 128), generator=gen, device="cuda").bfloat16()
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H * 4, n_tokens=N, budget=max(9, N // 2), lam=lam)
    _, _, _, kept, score = rkv.rkv_compress(shape, q, k, k, want_score=True)
    importance = rkv.rkv_score_importance(shape, q, k)
    redundancy = rkv.rkv_score_redundancy(shape, k) if lam < 1.0 else torch.zeros_like(importance)
    kept2, score2 = rkv.rkv_select_topk(shape, importance, redundancy, want_score=True)
    assert torch.equal(score, score2) and torch.equal(kept, kept2)

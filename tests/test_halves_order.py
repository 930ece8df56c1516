"""The order in which the scan with beta = 1 keeps a subtile's keys: the kernel's own row arithmetic replayed on the CPU, and on the
GPU its results at T above 0.9, where no row block hands rows over, against the schedule that keeps the plain order."""
import os
import subprocess

import pytest
import torch

from paper_2505_24133_amd import rkv


def test_copies_put_every_key_in_its_place(repo_root, tmp_path):
    exe = str(tmp_path / "halves_order_check")
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-I", os.path.join(repo_root, "paper_2505_24133_amd", "csrc"),
                    "-o", exe, os.path.join(repo_root, "tests", "halves_order_check.cpp")], check=True)
    for n in list(range(1, 261)) + [384, 385, 1144, 1893, 4216, 32760, 32767]:
        r = subprocess.run([exe, str(n)], capture_output=True, text=True)
        assert r.returncode == 0 and r.stdout.startswith("ok "), f"n={n}: {r.stdout}{r.stderr}"


@pytest.mark.gpu
@pytest.mark.parametrize("P,H,n,clusters", [
    pytest.param(70, 4, 100, 30, id="one tile"),
    pytest.param(70, 4, 129, 9, id="the newest tile holds one key"),
    pytest.param(70, 4, 385, 60, id="second block of one row"),
    pytest.param(40, 8, 1144, 300, id="three blocks"),
    pytest.param(12, 8, 4216, 1, id="all rows near-copies"),
])
def test_same_bits_above_the_hand_over(P, H, n, clusters):
    print(f"[gpu-case] halves P={P} H={H} n={n} clusters={clusters}", flush=True)
    N, T = n + 8, 0.95
    gen = torch.Generator(device="cuda").manual_seed(n)
    cent = torch.randn((P, H, clusters, 128), generator=gen, device="cuda")
    which = torch.randint(0, clusters, (P, H, N, 1), generator=gen, device="cuda")
    noise = 0.4 * torch.rand((P, H, N, 1), generator=gen, device="cuda")
    k = torch.gather(cent, 2, which.expand(-1, -1, -1, 128))
    k = (k + noise * torch.randn(k.shape, generator=gen, device="cuda")).bfloat16()
    mean = {}
    for flags in (0, rkv.RKV_FLAG_SKIP_SATURATED):
        shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=N, budget=N - 16, sim_threshold=T, flags=flags)
        mean[flags] = rkv.rkv_score_redundancy(shape, k, want_mean_sim=True)[1]
    assert torch.equal(mean[0], mean[rkv.RKV_FLAG_SKIP_SATURATED])

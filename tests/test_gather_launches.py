"""The launches of the gather of kept rows: none holds more work items than the runtime takes, calls that need more than one are whole, and
a head's rows are moved by one XCD, or by few."""
import os
import subprocess

import pytest
import torch

from paper_2505_24133_amd import build as B
from paper_2505_24133_amd import rkv


@pytest.fixture(scope="module")
def recorder(repo_root, tmp_path_factory):
    if not os.path.exists(B.LIB):
        B.build()
    exe = str(tmp_path_factory.mktemp("launches") / "launch_record")
    subprocess.run(["g++", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(repo_root, "include"), "-I", B.rocm_include(),
                    os.path.join(repo_root, "tests", "launch_record.cpp"), "-o", exe, "-rdynamic", B.LIB, "-L" + os.path.join(os.path.dirname(B.rocm_include()), "lib"), "-lamdhip64",
                    f"-Wl,-rpath,{os.path.dirname(B.LIB)}:{os.path.join(os.path.dirname(B.rocm_include()), 'lib')}"], check=True)
    return exe


@pytest.mark.parametrize("P,H,N,budget,page,launches", [
    pytest.param(1, 2, 40, 16, 0, 1, id="one block a head"),
    pytest.param(1, 1, 40, 17, 16, 1, id="a block of one row"),
    pytest.param(1 << 19, 8, 40, 32, 0, 1, id="a half of what a launch takes"),
    pytest.param(1 << 19, 8, 80, 64, 0, 2, id="one block more than a launch takes"),
    pytest.param(420000, 8, 100, 80, 0, 2, id="3.36 million heads of 80 rows"),
    pytest.param(1 << 19, 8, 80, 64, 16, 2, id="paged"),
    pytest.param(1, 1, 40, (1 << 28) + 1, 0, 2, id="one long list"),
    pytest.param(1 << 18, 8, 600, 448, 0, 4, id="four launches"),
])
def test_every_launch_is_one_the_runtime_takes(recorder, P, H, N, budget, page, launches):
    r = subprocess.run([recorder, *map(str, (P, H, N, budget, page))], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    word = r.stdout.split()
    assert [int(word[1]), int(word[3]), int(word[5])] == [rkv.RKV_OK, launches, -(-P * H * -(-budget // 16) // 8) * 8], r.stdout
    assert int(word[7]) * 256 < 1 << 32


def test_what_was_too_large_stays_refused(recorder):
    r = subprocess.run([recorder, str(1 << 19), "8", "400", "256", "0"], capture_output=True, text=True)
    assert r.stdout.startswith(f"status {rkv.RKV_ERR_HIP} launches 0 "), r.stdout


@pytest.fixture(scope="module")
def order_check(repo_root, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("order") / "gather_order_check")
    subprocess.run(["g++", "-O1", "-Wall", "-I", os.path.join(repo_root, "paper_2505_24133_amd", "csrc"),
                    os.path.join(repo_root, "tests", "gather_order_check.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("heads", [1, 3, 7, 8, 9, 20, 256])
@pytest.mark.parametrize("per", [1, 7, 65, 640, 641, 2024])
@pytest.mark.parametrize("launch", [64, 1 << 24])
@pytest.mark.parametrize("cache_bytes", [0, (256 << 20) - 1, 256 << 20])
def test_every_block_is_taken_once(order_check, heads, per, launch, cache_bytes):
    r = subprocess.run([order_check, *map(str, (heads, per, launch, cache_bytes))], capture_output=True, text=True)
    assert r.stdout == "ok" and r.returncode == 0, r.stdout


@pytest.mark.parametrize("heads,n_tokens,budget,paged,streams", [
    (256, 2048, 2048, 0, 0), (257, 2048, 2048, 0, 1), (256, 2049, 2049, 0, 1),
    (256, 4224, 410, 0, 0), (512, 1152, 576, 0, 0), (256, 2176, 1632, 0, 0), (256, 4224, 2049, 0, 1),
    (256, 2048, 8000, 0, 0), (256, 2049, 8000, 0, 1),
    (256, 2048, 16, 1, 0), (256, 2049, 16, 1, 1), (256, 2176, 2048, 1, 1),
])
def test_rows_read_past_the_caches(order_check, heads, n_tokens, budget, paged, streams):
    r = subprocess.run([order_check, "streams", *map(str, (heads, n_tokens, budget, paged))], capture_output=True, text=True)
    assert r.stdout == str(streams)


@pytest.mark.gpu
@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("P,H", [(1, 1), (3, 3), (2, 8), (3, 4)])
@pytest.mark.parametrize("budget", [17, 385])
def test_rows_of_every_head(P, H, budget, page):
    n_tokens = 400
    print(f"[gpu-case] gather P={P} H={H} budget={budget} page={page}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(4)
    k, v = (torch.randn((P, H, n_tokens, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    kept = torch.randint(0, n_tokens, (P, H, budget), generator=gen, device="cuda", dtype=torch.int32)
    want = [torch.gather(x, 2, kept.long()[..., None].expand(-1, -1, -1, 128)) for x in (k, v)]
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=n_tokens, budget=budget, alpha=1)
    if page:
        per = n_tokens // page
        shape.page_size, shape.block_table = page, torch.randperm(P * per, generator=gen, device="cuda").int().reshape(P, per)
        pools = [torch.empty((P * per, H, page, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        for pool, x in zip(pools, (k, v)):
            pool[shape.block_table.long()] = x.reshape(P, H, per, page, 128).transpose(1, 2)
        k, v = pools
    out = [torch.full((P, H, budget, 128), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    rkv.rkv_compact(shape, k, v, kept, k_out=out[0], v_out=out[1])
    assert torch.equal(out[0], want[0]) and torch.equal(out[1], want[1])


@pytest.mark.gpu
@pytest.mark.parametrize("budget", [10240, 10241, 32700])
def test_rows_of_long_lists(budget):
    """17 heads of 32768 tokens, 272 MiB: below and beyond the length where the order of the blocks changes."""
    heads, n_tokens = 17, 32768
    print(f"[gpu-case] gather heads={heads} n_tokens={n_tokens} budget={budget}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(6)
    k, v = (torch.randn((1, heads, n_tokens, 128), generator=gen, device="cuda").bfloat16() for _ in range(2))
    kept = torch.randint(0, n_tokens, (1, heads, budget), generator=gen, device="cuda", dtype=torch.int32)
    shape = rkv.Shape(num_problems=1, kv_heads=heads, q_heads=heads, n_tokens=n_tokens, budget=budget)
    for x, got in zip((k, v), rkv.rkv_compact(shape, k, v, kept)):
        assert torch.equal(got, torch.gather(x, 2, kept.long()[..., None].expand(-1, -1, -1, 128)))


@pytest.mark.gpu
def test_rows_of_a_second_launch():
    """2^22 heads of 49 rows (four blocks each): 2^24 blocks, one more than a launch takes.  The heads of eight share a page, K and V and the
    two outputs are one buffer each, so that 53 GB suffice; the outputs are compared in pieces."""
    P, H, budget, page = 1 << 19, 8, 49, 64
    rows = P * H * budget
    if torch.cuda.mem_get_info()[0] < rows * 256 + rows * 4 + (12 << 30):
        pytest.skip("needs 66 GB of GPU memory")
    print(f"[gpu-case] gather in two launches P={P} H={H} budget={budget}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(3)
    pool = torch.randn((8, H, page, 128), generator=gen, device="cuda").bfloat16()
    table = torch.randint(0, 8, (P, 1), generator=gen, device="cuda").int()
    shape = rkv.Shape(num_problems=P, kv_heads=H, q_heads=H, n_tokens=page, budget=budget, page_size=page, block_table=table)
    kept = torch.randint(0, page, (P, H, budget), generator=gen, device="cuda", dtype=torch.int32)
    out = torch.empty((P, H, budget, 128), dtype=torch.bfloat16, device="cuda")
    out[0] = 7.0
    out[-2:] = 7.0
    rkv.rkv_compact(shape, pool, pool, kept, k_out=out, v_out=out)
    piece = 1 << 13
    heads = torch.arange(H, device="cuda")[None, :, None]
    for p in (0, P // 2, P - piece):
        part = slice(p, p + piece)
        assert torch.equal(out[part], pool[table[part].long()[:, :, None], heads, kept[part].long()])

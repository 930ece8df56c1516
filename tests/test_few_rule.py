"""Which calls take the similarity pass of few heads: a step up to a round and a half of workgroups, the pass alone not with more than 128
heads, where it was measured to be the slower one."""
import os
import subprocess

import pytest


@pytest.fixture(scope="module")
def rule(repo_root, tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("few") / "few_rule_check")
    subprocess.run(["g++", "-O1", "-Wall", "-Werror", "-I", os.path.join(repo_root, "paper_2505_24133_amd", "csrc"), "-o", exe,
                    os.path.join(repo_root, "tests", "few_rule_check.cpp")], check=True)

    def ask(heads, n, beta=1, beside=True, other=False):
        return subprocess.run([exe, *map(str, (heads, n, beta, int(beside), int(other)))], capture_output=True, text=True, check=True).stdout == "1"
    ask.exe = exe
    return ask


def test_copies_ahead_in_the_prepass(rule):
    """Eight chunks a resident workgroup, whatever the device holds, and rows that 16-byte copies can read."""
    def ask(*args):
        return subprocess.run([rule.exe, *map(str, args)], capture_output=True, text=True, check=True).stdout == "1"
    assert ask(6144, 768, 1) and not ask(6143, 768, 1) and not ask(1 << 24, 768, 0)
    assert ask(2432, 304, 1) and not ask(6144, 1024, 1)


def test_a_step(rule):
    assert rule(1, 2048) and rule(8, 1144) and rule(64, 640) and rule(132, 384) and rule(256, 192)
    assert not rule(8, 2032) and not rule(16, 1632) and not rule(256, 1144)      # more than a round and a half of workgroups


def test_the_pass_alone(rule):
    assert rule(1, 2048, beside=False) and rule(8, 1144, beside=False) and rule(128, 384, beside=False)
    assert not rule(129, 384, beside=False) and not rule(132, 200, beside=False) and not rule(256, 192, beside=False)


def test_never(rule):
    for beside in (False, True):
        assert not rule(2, 128, beside=beside) and not rule(1, 2049, beside=beside)     # one tile, seventeen
        assert not rule(2, 376, beta=2, beside=beside) and not rule(2, 376, other=True, beside=beside)

"""Decode attention waits for K by counting: all but its sixteen loads of V are done when the sixteen of K, which go to LDS, are.  So K's must
be issued first, whichever way the compiler schedules; here attn.hip is compiled as the library is, and by schedulers that prefer other
orders, and the order of the loads is read from the assembly (this runs without a GPU)."""
import os
import re
import subprocess

import pytest

from paper_2602_00182_amd import build

SCHEDULERS = ["", "gcn-iterative-minreg", "ilpmin", "r600"]


def orders(assembly):
    """{kernel: a letter for each vector load up to the wait for all but sixteen: K (to LDS) or r (to registers)}"""
    found, name, seen = {}, None, ""
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        label = re.fullmatch(r"(_Z\w+):", line)
        if label:
            name, seen = label.group(1), ""
        elif re.match(r"(global|buffer|flat)_load", line):
            seen += "K" if "_lds" in line.split()[0] else "r"
        elif re.search(r"s_waitcnt.*vmcnt\(16\)", line) and name and "attn_chunk_kernel" in name:
            found.setdefault(name, seen)
    return found


@pytest.fixture(scope="module")
def assemblies(tmp_path_factory):
    at = tmp_path_factory.mktemp("attn")
    runs = {}
    for s in SCHEDULERS:
        out = at / f"attn_{s}.s"
        cmd = [build._hipcc(), *build.HIPCC_FLAGS, *(["-mllvm", f"-misched={s}"] if s else []), "-S", "--cuda-device-only",
               os.path.join(build.CSRC, "attn.hip"), "-o", str(out)]
        runs[s] = (subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL), out)
    assert all(p.wait() == 0 for p, _ in runs.values())
    return {s: out.read_text() for s, (_, out) in runs.items()}


@pytest.mark.parametrize("scheduler", SCHEDULERS)
def test_loads_of_k_come_before_those_of_v(assemblies, scheduler):
    found = orders(assemblies[scheduler])
    assert len(found) == 8  # 1, 2, 4 and 8 query heads a KV head, with and without a second pass
    for kernel, seen in found.items():
        assert seen.endswith("K" * 16 + "r" * 16), (kernel, seen)

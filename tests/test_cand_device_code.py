"""What the compiled candidate kernels must and must not contain (no GPU needed).

The kernels are compiled to gfx950 assembly, as the library's build compiles
them: an ordering gap between workgroups shows there and not in test results.
"""
import os
import re
import subprocess

import pytest

from paper_2510_18136_amd import build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("cand") / "k_cand.s")
    flags = [f for f in build.COMMON if f != "-fPIC"]
    subprocess.run([build.HIPCC] + flags + ["-x", "hip", "-S", "--cuda-device-only",
                                            os.path.join(build.CSRC, "k_cand.hip"), "-o", out], check=True)
    return open(out).read()


def kernels(assembly, name):
    """{symbol: instructions} of the kernels whose symbol contains `name`."""
    found = {}
    for m in re.finditer(r"^(_ZN\S*%s\S*):.*?\n(.*?)^\.Lfunc_end" % name, assembly, re.S | re.M):
        lines = (line.split(";")[0].strip() for line in m.group(2).splitlines())
        found[m.group(1)] = [line for line in lines if line and not line.startswith(".")]
    return found


def test_every_wave_waits_for_its_keys_before_the_ticket(assembly):
    """Between a workgroup's last store and the barrier before its ticket: write-back and wait, for every wave."""
    ks = kernels(assembly, "k_cand_top")
    assert len(ks) == 5
    for name, code in ks.items():
        tickets = [i for i, c in enumerate(code) if re.match(r"(flat|global)_atomic_(add|inc)\b.* sc0", c)]
        assert tickets, name
        for t in tickets:
            barrier = max(i for i in range(t) if code[i].startswith("s_barrier"))
            store = max(i for i in range(barrier) if re.match(r"(flat|global)_(store|atomic)", code[i]))
            between = code[store + 1:barrier]
            assert any(c.startswith("buffer_wbl2") and "sc1" in c for c in between), name
            assert any(c.startswith("s_waitcnt") and "vmcnt(0)" in c for c in between), name


def lds_bytes(assembly):
    """{kernel: bytes of LDS a workgroup}"""
    out = {}
    for block in re.split(r"\n  - \.a", assembly)[1:]:
        out[re.search(r"\.name:\s+(\S+)", block).group(1)] = int(
            re.search(r"\.group_segment_fixed_size:\s+(\d+)", block).group(1))
    return out


def test_the_batch_kernel_takes_one_workgroup_s_lds(assembly):
    """It holds the code of four sizes; each with LDS of its own, one workgroup filled a CU."""
    lds = {k: v for k, v in lds_bytes(assembly).items() if "k_cand_top" in k}
    assert len(lds) == 5
    assert max(lds.values()) == min(lds.values())


def test_only_the_keys_kept_are_ranked(assembly):
    """Ranking is quadratic: no more than 256 keys of 8 bytes may reach it, however many are tied."""
    for name, size in lds_bytes(assembly).items():
        if "k_cand_top" in name:
            assert size <= 256 * 8 + 64, name

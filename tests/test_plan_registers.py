"""Registers and row reads of compiled search plans (no GPU needed).

Plans are compiled for gfx950 as a program that has imported PyTorch compiles
them, and read back: a register too many costs a workgroup per CU, a spill a
kernel form or a whole batch, and none of it shows in results.
"""
import os
import re
import subprocess
import sys

import pytest

from tests._lib import ensure_built

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin/"
W5 = [1, 2, 4, 8, 16]
W8 = W5 + [32, 64, 100]
W12 = W5 + [32, 64, 128, 256, 512, 1024, 1200]
W13 = [1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 100]

COMPILE = """
import sys; sys.path.insert(0, %r)
import torch, numpy as np
from paper_2510_18136_amd import nsfrb
nsfrb.SearchConfig(64, 64, {nt}, np.linspace(1.311, 1.499, {ns}), np.linspace(0, 4000, {n_dm}), {widths},
                   in_dtype={store!r}, store_dtype={store!r}).plan_source(compile=True)
""" % ROOT


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def compiled(path, lean=0, max_acc=3, **plan):
    """Code object of a plan, compiled in a child process."""
    env = dict(os.environ, NSFRB_DUMP_CODE=str(path), NSFRB_DEBUG_LEAN=str(lean), NSFRB_DEBUG_MAX_ACC=str(max_acc))
    subprocess.run([sys.executable, "-c", COMPILE.format(**plan)], check=True, env=env, timeout=300)
    return str(path)


def registers(code):
    """{kernel: (VGPRs, bytes of scratch a lane)}"""
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", code], capture_output=True, text=True, check=True).stdout
    out = {}
    for block in re.split(r"\n  - \.a", notes)[1:]:
        value = {k: re.search(r"\.%s:\s+(\S+)" % k, block).group(1)
                 for k in ("name", "vgpr_count", "private_segment_fixed_size")}
        out[value["name"]] = (int(value["vgpr_count"]), int(value["private_segment_fixed_size"]))
    return out


def test_fourteen_samples_per_lane_keep_three_workgroups(tmp_path):
    """Three workgroups of eight waves share a CU with at most 80 VGPRs a wave, four with at most 64."""
    r = registers(compiled(tmp_path / "a", store="f16", nt=700, ns=16, n_dm=12, widths=W12[:-2]))
    assert r["nsfrb_search_c14_p1_w8"][0] <= 80
    r = registers(compiled(tmp_path / "b", store="f16", nt=700, ns=16, n_dm=12, widths=W8))
    assert r["nsfrb_search_c14_p1_w8"][0] <= 64


@pytest.mark.parametrize("nt,c", [(150, 3), (400, 7), (700, 11)])
def test_single_reads_of_16_bit_rows_are_not_merged(tmp_path, nt, c):
    """Odd rows of BF16 samples start anywhere: wider reads from such addresses are an order slower than single ones."""
    code = compiled(tmp_path / "a", store="bf16", nt=nt, ns=16, n_dm=12, widths=W5)
    asm = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", code], capture_output=True, text=True,
                         check=True).stdout
    kernel = re.search(r"<nsfrb_search_c%d_p1_w8>:\n(.*?)\n\n" % c, asm, re.S).group(1)
    assert len(re.findall(r"\bds_read_u16", kernel)) >= c


@pytest.mark.parametrize("store,nt,ns,widths,max_acc", [("bf16", 2400, 16, W13, 1), ("bf16", 3000, 16, W8, 3),
                                                        ("f32", 2048, 16, W13, 3), ("f32", 4096, 8, W5, 3)])
def test_leanest_plan_spills_least(tmp_path, store, nt, ns, widths, max_acc):
    """Batch kernels of 16 waves, 128 VGPRs: at most 64 bytes of spill, or the batch is refused."""
    r = registers(compiled(tmp_path / "a", lean=2, max_acc=max_acc, store=store, nt=nt, ns=ns, n_dm=32, widths=widths))
    assert r["nsfrb_batch_kernel_0"][1] <= 64


def test_rows_read_in_halves_hold_one_row(tmp_path):
    r = registers(compiled(tmp_path / "a", store="f32", nt=2176, ns=16, n_dm=32, widths=W5))
    assert r["nsfrb_batch_kernel_0"][1] == 0 and r["nsfrb_persistent_c35_w16_b1"][1] == 0


@pytest.mark.parametrize("store,widths", [("f16", W12), ("bf16", W12), ("f16", W13)])
def test_forms_held_to_128_registers_stand_beside_the_free_ones(tmp_path, store, widths):
    """The persistent kernel keeps its registers (a spill would drop it); two workgroups fit beside that."""
    r = registers(compiled(tmp_path / "a", store=store, nt=2048, ns=16, n_dm=12, widths=widths))
    c = 34 if store == "f16" else 33
    assert r["nsfrb_persistent_c%d_w8_b1" % c][1] == 0
    for name in ("nsfrb_search_c%d_p1_w8" % c, "nsfrb_batch_kernel_0"):
        assert r[name][1] == 0 and r[name + "_v128"][0] <= 128


def test_no_held_form_where_one_workgroup_fills_the_lds(tmp_path):
    r = registers(compiled(tmp_path / "a", store="f32", nt=2048, ns=16, n_dm=12, widths=W12))
    assert r["nsfrb_batch_kernel_0"][1] == 0 and not any(k.endswith("_v128") for k in r)

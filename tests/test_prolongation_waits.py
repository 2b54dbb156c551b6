"""The fused float64 prolongation fetches coarse planes by direct loads into LDS,
every plane into the same slots, and nothing in LDS orders such a load after the
reads of the plane before it: the reads have to be waited for (lgkmcnt(0)) before the
next plane's loads are issued, on every path.  A missing wait there gave batch
members answers that were off by 5e-13 now and then, so it is looked for in the
assembly of the kernel as it is built (hipcc cross-compiles without a GPU)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_05332_amd", "csrc")
SOURCE = """
#include "strip_forms.h"
namespace rkl {
template __global__ void k_tau_strip_pro<double, 2, 4, 4, %PER%, false, false>(
    LevelView<double>, const double*, const double*, const double*, double*, FCoef<double, 2>, int, int, int, int,
    Batch, const int*);
}
"""


def _blocks(lines):
    """Basic blocks of one function: label -> (instructions, successor labels)."""
    blocks, order, cur = {"": []}, [""], ""
    for ln in lines:
        m = re.match(r"^(\.LBB\w+):", ln)
        if m:
            cur = m.group(1)
            blocks[cur] = []
            order.append(cur)
            continue
        ins = ln.split(";")[0].strip()
        if not ins or ins.startswith("."):
            continue
        blocks[cur].append(ins)
        if re.match(r"s_c?branch", ins):  # what follows is a block of its own
            cur = f"{cur}+{len(order)}"
            blocks[cur] = []
            order.append(cur)
    succ = {}
    for k, name in enumerate(order):
        last = blocks[name][-1] if blocks[name] else ""
        nxt = [order[k + 1]] if k + 1 < len(order) else []
        if last.startswith("s_cbranch"):
            succ[name] = nxt + [last.split()[-1]]
        elif last.startswith("s_branch"):
            succ[name] = [last.split()[-1]]
        elif last.startswith("s_endpgm"):
            succ[name] = []
        else:
            succ[name] = nxt
    return blocks, succ


def unwaited_direct_loads(asm):
    """(direct loads, those reachable with LDS reads outstanding)."""
    body = re.search(r"^_ZN\S*k_tau_strip_pro\S*:.*?$(.*?)^\.Lfunc_end", asm, flags=re.M | re.S).group(1)
    blocks, succ = _blocks(body.split("\n"))
    entry = {name: False for name in blocks}  # LDS reads may be outstanding on entry
    bad, total, work = set(), 0, list(blocks)
    while work:
        name = work.pop()
        out = entry[name]
        for q, ins in enumerate(blocks[name]):
            if ins.startswith("ds_read"):
                out = True
            elif ins.startswith("s_waitcnt") and "lgkmcnt(0)" in ins:
                out = False
            elif ins.startswith("global_load_lds") and out:
                bad.add((name, q))
        for s in succ[name]:
            if out and not entry[s]:
                entry[s] = True
                work.append(s)
    total = sum(ins.startswith("global_load_lds") for b in blocks.values() for ins in b)
    return total, bad


@pytest.mark.parametrize("per", ["true", "false"])
def test_reads_of_a_coarse_plane_end_before_the_next_is_loaded(per, tmp_path):
    from paper_2306_05332_amd import build as B
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    src, out = tmp_path / "pro.hip", tmp_path / "pro.s"
    src.write_text(SOURCE.replace("%PER%", per))
    subprocess.run([B.hipcc(), *B.HIPCC_FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(out)], check=True,
                   capture_output=True)
    total, bad = unwaited_direct_loads(out.read_text())
    print(total, "direct loads,", len(bad), "with reads outstanding", flush=True)
    assert total >= 6 and not bad, sorted(bad)


def test_the_check_sees_a_missing_wait():
    """The analysis on hand-made code: a read, a branch round the loads, a wait on one
    path only."""
    text = """_ZN3rkl15k_tau_strip_proX:
	ds_read_b64 v[0:1], v2
	s_cbranch_scc1 .LBB0_2
	s_waitcnt lgkmcnt(0)
.LBB0_2:
	%s
	global_load_lds_dwordx4 v3, s[0:1]
	s_endpgm
.Lfunc_end0:
"""
    assert len(unwaited_direct_loads(text % "s_nop 0")[1]) == 1
    assert not unwaited_direct_loads(text % "s_waitcnt vmcnt(0) lgkmcnt(0)")[1]

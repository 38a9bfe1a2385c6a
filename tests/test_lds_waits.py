"""Every workgroup barrier of the device code finds the wavefront's own LDS writes finished: followed
through the generated assembly over all paths, as the compiler has dropped such waits in loops."""
import os
import re
import subprocess

import pytest

from paper_2506_16235_amd import build as B


def _unfinished(text):
    """(kernel, instruction) of LDS writes that can be in flight at a barrier."""
    found = []
    for m in re.finditer(r"^(_Z\w+):.*\n([\s\S]*?)^\.Lfunc_end", text, re.M):
        ins, label = [], {}
        for line in m.group(2).split("\n"):
            line = line.split(";")[0].strip()
            q = re.match(r"^(\.?\w+):$", line)
            if q:
                label[q.group(1)] = len(ins)
            elif line and not line.startswith("."):
                ins.append(line)
        seen, work = [None] * len(ins), [(0, -1)]
        while work:
            i, last = work.pop()
            while i < len(ins):
                if seen[i] is not None and (seen[i] >= 0 or last < 0):
                    break
                seen[i] = last
                op = ins[i].split()[0]
                if op.startswith("ds_") and re.search(r"write|store|add|sub|min|max|or_|and_|inc|dec", op):
                    last = i
                elif op == "s_waitcnt" and "lgkmcnt(0)" in ins[i]:
                    last = -1
                elif op == "s_barrier" and last >= 0:
                    found.append((m.group(1), ins[last]))
                if op == "s_endpgm":
                    break
                if op == "s_branch":
                    i = label[ins[i].split()[1]]
                    continue
                if op.startswith("s_cbranch"):
                    work.append((label[ins[i].split()[1]], last))
                i += 1
    return found


def test_follows_back_edges():
    body = "_Zk:\n{}\n.Lfunc_end0:\n"
    loop = ".LBB0:\n\ts_barrier\n\tds_add_u32 v1, v2\n{}\ts_cbranch_scc1 .LBB0\n\ts_endpgm"
    assert _unfinished(body.format(loop.format(""))) == [("_Zk", "ds_add_u32 v1, v2")]
    assert _unfinished(body.format(loop.format("\ts_waitcnt lgkmcnt(0)\n"))) == []


def test_no_lds_write_in_flight_at_a_barrier(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "k.s")
    flags = [f for f in B.HIP_FLAGS if f != "-fPIC"]
    subprocess.run([B.HIPCC, *flags, "-I", B.INCLUDE, "--cuda-device-only", "-S",
                    os.path.join(B.CSRC, "nsml_kernels.hip"), "-o", out], check=True, capture_output=True)
    text = open(out).read()
    assert text.count("s_barrier") > 100
    assert _unfinished(text) == []

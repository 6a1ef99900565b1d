"""Order of memory operations that no run shows reliably, read from the compiled
kernels' assembly.  Where one thread of a block publishes what all its waves have
stored (an agent-scope release behind a barrier), its write-back of the L2 covers
the other waves' stores only if these have arrived there: a gfx950 barrier does
not wait for stores in flight, so each wave has to wait for its own before it."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def kernels(name, tmp_path):
    """Assembly of each function of a HIP source, as lists of lines."""
    out = str(tmp_path / (name + ".s"))
    csrc = os.path.join(ROOT, "paper_2101_01160_amd", "csrc")
    subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"),
                    "-I", csrc, "--cuda-device-only", "-S", os.path.join(csrc, name), "-o", out],
                   check=True, capture_output=True)
    funcs, cur = {}, None
    for line in open(out):
        m = re.match(r"^(_Z\w+):", line)
        if m:
            cur = funcs.setdefault(m.group(1), [])
        elif line.startswith(".Lfunc_end"):
            cur = None
        elif cur is not None:
            cur.append(line.split(";")[0].strip())
    return funcs


def released_barriers(lines):
    """For each agent-scope write-back: whether a wait for all stores stands between the last of them (or the last
    label, behind which others may come) and the barrier before the write-back."""
    out = []
    for i, op in enumerate(lines):
        if not op.startswith("buffer_wbl2"):
            continue
        b = max((j for j in range(i) if lines[j].startswith("s_barrier")), default=None)
        if b is None:
            continue
        waits = False
        for j in range(b - 1, -1, -1):
            if lines[j].startswith("s_waitcnt") and "vmcnt(0)" in lines[j]:
                waits = True
                break
            if lines[j].endswith(":") or re.match(r"(global|flat|buffer)_(store|atomic)", lines[j]):
                break
        out.append(waits)
    return out


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_stores_have_arrived_before_a_block_publishes_them(tmp_path):
    funcs = kernels("neq.hip", tmp_path)
    found = {f: released_barriers(lines) for f, lines in funcs.items()}
    event = [w for f, w in found.items() if "k_neq_event" in f]
    assert event and event[0], "k_neq_event no longer hands shares over behind a barrier: this test has nothing to look at"
    for f, waits in found.items():
        assert all(waits), f

"""The kernels for 17 to 1536 rows place the waits for their activation copies by hand: each counts the memory operations that may
still be in flight, the loads of the next tile's packed words among them.  A compiler that drops some of those loads (it has
done so, in an iteration peeled off the loop) makes a wait too short without any other sign, so the generated code is checked."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2505_03803_amd import build


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="needs hipcc")
def test_hand_placed_waits_count_the_loads_that_are_there(tmp_path):
    out = str(tmp_path / "mid.s")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "midbatch.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    kernels = 0
    for m in re.finditer(r"^(_ZN5rwkvq10mid_kernel\S*):", text, re.M):
        # per kernel: groups of activation copies (to LDS), of other loads, and the waits behind them
        ops = []
        for line in text[m.end(): text.index(".Lfunc_end", m.end())].splitlines():
            line = line.strip()
            wait = re.match(r"s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)", line)
            kind = "wait" if wait else "copy" if re.match(r"buffer_load\S* .* lds$", line) else "load" if line.startswith("buffer_load") else None
            if kind == "wait":
                ops.append([kind, int(wait[1])])
            elif kind and ops and ops[-1][0] == kind:
                ops[-1][1] += 1
            elif kind:
                ops.append([kind, 1])
        copies = min(n for i, (k, n) in enumerate(ops) if k == "copy" and i and ops[i - 1][0] == "wait")
        waits = [ops[i][1] for i in range(len(ops) - 1) if ops[i][0] == "wait" and ops[i + 1] == ["copy", copies]]
        ahead = min(waits)                                             # activation copies of later steps in flight at a wait
        assert ahead % copies == 0, m[1]
        for i in range(len(ops) - 2):
            if ops[i] == ["copy", copies] and ops[i + 1][0] == "load" and ops[i + 2][0] == "wait" and ops[i + 2][1]:
                assert ops[i + 2][1] <= ahead + ops[i + 1][1], (m[1], ops[i - 2: i + 4])
        kernels += 1
    assert kernels >= 20

"""RANMAR's table kernel, checked in the compiler's IR (no GPU): a segment runs on
a wavefront of its own, so there are as many as the dispatcher has to place, and
none of them may wait on a counter in global memory."""
import os
import re
import subprocess

from paper_1003_1898_amd.build import CSRC, FLAGS, HIPCC


def test_ranmar_segments_draw_on_no_counter(tmp_path):
    ir = str(tmp_path / "k_table.ll")
    flags = ["-O1" if f == "-O3" else f for f in FLAGS]
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-emit-llvm", os.path.join(CSRC, "k_table.hip"),
                    "-o", ir], check=True, capture_output=True)
    atomics = {}
    for body in open(ir).read().split("\ndefine ")[1:]:
        body = body.split("\n}\n")[0]
        atomics[re.search(r"@(\S+?)\(", body).group(1)] = len(re.findall(r"atomicrmw|cmpxchg", body))
    count = {k: sum(v for name, v in atomics.items() if k in name) for k in ("k_table_lane", "k_table_ranmar")}
    assert count["k_table_lane"] > 0  # its tasks of 64 segments come from a counter
    assert count["k_table_ranmar"] == 0

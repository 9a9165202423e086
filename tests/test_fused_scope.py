"""The in-kernel consumers' histograms, checked in the compiler's IR (no GPU):
where several wavefronts of a workgroup count in one histogram, every count is
an atomic of workgroup scope; an atomic of wavefront scope says that no other
wavefront touches the word."""
import os
import re
import subprocess

import pytest

from paper_1003_1898_amd.build import CSRC, FLAGS, HIPCC


@pytest.fixture(scope="module")
def consumer_atomics(tmp_path_factory):
    """(kernel's mangled name, synchronisation scopes of its LDS additions) of k_fused.hip."""
    ir = str(tmp_path_factory.mktemp("ir") / "k_fused.ll")
    flags = ["-O1" if f == "-O3" else f for f in FLAGS]
    subprocess.run([HIPCC, *flags, "--cuda-device-only", "-S", "-emit-llvm", os.path.join(CSRC, "k_fused.hip"),
                    "-o", ir], check=True, capture_output=True)
    found = {}
    for body in open(ir).read().split("\ndefine ")[1:]:
        body = body.split("\n}\n")[0]
        name = re.search(r"@(\S+?)\(", body).group(1)
        found[name] = re.findall(r'atomicrmw add ptr addrspace\(3\).*syncscope\("([a-z-]+)"\)', body)
    return found


@pytest.mark.parametrize("wavefronts", [4, 16])
def test_shared_histograms_count_at_workgroup_scope(consumer_atomics, wavefronts):
    kernels = {k: v for k, v in consumer_atomics.items() if "k_split_fused" in k and f"ELi{wavefronts}EEEv" in k}
    assert len(kernels) == 5  # GGL, XOR128, RANECU, DRAND48, RANNYU
    for name, scopes in kernels.items():
        assert scopes and set(scopes) == {"workgroup"}, name

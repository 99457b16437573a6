"""Registers of the attention kernels as the compiler reports them (CPU only, the kernels are compiled, not run)."""
import os
import re
import subprocess

from paper_2603_14549_amd import build


def test_attention_keeps_its_accumulators_in_vector_registers(tmp_path):
    """Softmax and rescaling work on the accumulators: in AGPRs, or in scratch, every one of them would be moved to and fro."""
    res = subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(build.CSRC, "asap_attention.hip"), "-o", str(tmp_path / "attention.o")],
                         capture_output=True, text=True, check=True)
    kernels = re.split(r"Function Name: ", res.stderr)[1:]
    forms = [k for k in kernels if "k_attention" in k.split()[0]]
    assert len(forms) == 12                    # two types, two head dimensions, three forms of the workgroup
    for k in forms:
        agprs, scratch = (int(re.search(n + r": (\d+)", k).group(1)) for n in ("AGPRs", r"ScratchSize \[bytes/lane\]"))
        assert (agprs, scratch) == (0, 0), k.split()[0]

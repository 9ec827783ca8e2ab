"""Register spills of the GEMM kernels.  A spill in an epilogue or a product
loop goes unnoticed by every parity test; the compiler reports it in each
kernel's metadata.  The source is compiled for gfx950 to assembly on the CPU
and no kernel may spill a vector register, save one: the resident reverse
kernel of five fp16 streams with the first layer formed in it, whose six
spills stand beside its weights in LDS at two blocks per CU."""
import os
import re
import subprocess

import pytest

from paper_1910_13444_amd import build

KNOWN = {"k_gemm_nt_wrIDF16_Li2ELi2ELi1ELb1ELb0ELb0E": 6}


def test_gemm_kernels_do_not_spill(tmp_path):
    if not os.path.exists(build.hipcc()):
        pytest.skip("hipcc not available")
    out = str(tmp_path / "gemm.s")
    r = subprocess.run([build.hipcc(), *build.common_flags(), "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "gemm.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        meta = f.read().rsplit("amdhsa.kernels:", 1)[1]
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", meta, re.S)
    assert len(kernels) > 100
    for name, spills in kernels:
        allowed = max([n for part, n in KNOWN.items() if part in name], default=0)
        assert int(spills) <= allowed, f"{name} spills {spills} vector registers"

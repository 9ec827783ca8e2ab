"""Properties of the compiled GEMM kernels that every parity test passes over,
checked on the gfx950 assembly of the source, on the CPU.

Register spills: no kernel may spill a vector register, save one: the resident
reverse kernel of five fp16 streams with the first layer formed in it, whose
six spills stand beside its weights in LDS at two blocks per CU.

Roundings: the tiled kernels' epilogues compute in fp32 and round each result to
the storage type when it is stored.  v_fma_mixlo_f16 / v_fma_mixhi_f16 would
round the last operation of a result to 16 bits at once."""
import os
import re
import subprocess

import pytest

from paper_1910_13444_amd import build

KNOWN = {"k_gemm_nt_wrIDF16_Li2ELi2ELi1ELb1ELb0ELb0E": 6}


@pytest.fixture(scope="module")
def asm(tmp_path_factory):
    if not os.path.exists(build.hipcc()):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("isa") / "gemm.s")
    r = subprocess.run([build.hipcc(), *build.common_flags(), "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, "gemm.hip"), "-o", out], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read()


def test_gemm_kernels_do_not_spill(asm):
    meta = asm.rsplit("amdhsa.kernels:", 1)[1]
    kernels = re.findall(r"\.name:\s+(\S+).*?\.vgpr_spill_count:\s+(\d+)", meta, re.S)
    assert len(kernels) > 100
    for name, spills in kernels:
        allowed = max([n for part, n in KNOWN.items() if part in name], default=0)
        assert int(spills) <= allowed, f"{name} spills {spills} vector registers"


def test_tiled_fp16_epilogues_round_when_they_store(asm):
    bodies = {m.group(1): asm[m.end():asm.find(".Lfunc_end", m.end())] for m in re.finditer(r"^(_Z\w+):", asm, re.M)
              if "k_gemm_ntIDF16_" in m.group(1)}
    assert len(bodies) > 20
    for name, body in bodies.items():
        assert not re.search(r"v_fma_mix(lo|hi)_f16", body), name

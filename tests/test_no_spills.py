"""No kernel of the library may spill registers to scratch memory: the streaming GEMMs sit right at their
register budget (two workgroups per CU at 128 VGPRs), and a spill costs tens of percent without failing any
parity test.  Compiles the device code to assembly (no GPU needed) and reads every kernel's descriptor."""
import functools
import os
import re
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@functools.lru_cache(maxsize=None)
def _kernels(src):
    """(name, descriptor) of every kernel of a source file."""
    from paper_2505_01572_amd import build
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        subprocess.run(["hipcc", *flags, "-S", "--offload-device-only", "-o", out, os.path.join(build.CSRC, src)],
                       check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        return re.findall(r"\.amdhsa_kernel (\S+)(.*?)\.end_amdhsa_kernel", open(out).read(), re.S)


@pytest.mark.parametrize("src", ["pv_kernels_matrix.hip", "pv_kernels_attention.hip", "pv_kernels_common.hip", "pv_kernels_vector.hip", "pv_kernels_prefill.hip"])
def test_kernels_use_no_scratch(src):
    kernels = _kernels(src)
    assert kernels, "no kernel descriptors found"
    spilled = [name for name, body in kernels if int(re.search(r"\.amdhsa_private_segment_fixed_size\s+(\d+)", body).group(1)) > 0]
    assert not spilled, f"kernels with scratch (register spills): {spilled}"


def test_two_workgroups_of_the_4_bit_kernel_fit_a_cu():
    """Up to 16 rows, 4-bit weights: eight waves a workgroup at 128 registers and 80 KiB of LDS at most, whatever the strips; sixteen waves are a CU's."""
    found = [(name, [int(re.search(r"\.amdhsa_%s\s+(\d+)" % k, body).group(1)) for k in ("next_free_vgpr", "group_segment_fixed_size")]) for name, body in _kernels("pv_kernels_matrix.hip") if re.match(r"_Z\d+k_gemm_q4I", name)]
    assert len(found) > 30
    assert not [f for f in found if f[1][0] > 128 or f[1][1] > 81920]

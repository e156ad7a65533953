"""The stores of K-slices' sums that go through to memory are written in assembly: an instruction right behind one must not write the
registers that it reads, so a wait state follows in the same block.  Compiles a probe to assembly (no GPU needed)."""
import re
import subprocess

from paper_2505_01572_amd import build

PROBE = """
#include "pv_internal.h"
#include "pv_kernels_common.h"
#include "pv_matrix_common.h"
// the stored registers are written again at once
__global__ void k_probe(float4 *p, f32x4 v, int n)
{
    for (int i = 0; i < n; ++i) { store_through(p + i * 64 + threadIdx.x, v); v = v * 2.f + 1.f; }
}
"""


def test_a_wait_state_follows(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    subprocess.run(["hipcc", *flags, "-S", "--offload-device-only", "-o", str(out), str(src)], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    code = [l.split(";")[0].strip() for l in out.read_text().splitlines() if re.match(r"\s+[a-z]", l)]
    stores = [i for i, l in enumerate(code) if re.match(r"global_store_dwordx4 .* sc1$", l)]
    assert stores
    assert all(re.fullmatch(r"s_nop [1-9]\d*", code[i + 1]) for i in stores), [code[i:i + 3] for i in stores]

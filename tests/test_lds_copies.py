"""The direct global -> LDS copies of the long-prompt kernels take their LDS address from m0, which the compiler
does not know to be written by inline assembly (m0 on a clobber list is ignored): every block that writes it has to save it first and
to put it back last, and the next instruction must not read it (that would need a wait state).  Compiles the device code to assembly (no GPU needed)."""
import os
import re
import subprocess

from paper_2505_01572_amd import build

PROBE = """
#include "pv_kernels_prefill.hip"
// the compiler sets m0 once for its own two copies, with ours in between
__global__ void k_probe(const uint4 *a, const uint4 *b, uint4 *out)
{
    __shared__ uint4 s[128];
    auto own = [&](const uint4 *p) { __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p, (__attribute__((address_space(3))) void *)s, 16, 0, 0); };
    own(a + threadIdx.x);
    dma_tile(lds_addr(s + 64), b, threadIdx.x * 16);
    own(a + 64 + threadIdx.x);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    out[threadIdx.x] = s[threadIdx.x];
}
"""


def test_m0_is_put_back(tmp_path):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(PROBE)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    subprocess.run(["hipcc", *flags, "-S", "--offload-device-only", "-o", str(out), str(src)], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = out.read_text()
    blocks = [(m[1], text[m.end():]) for m in re.finditer(r"#ASMSTART\n(.*?)#ASMEND", text, re.S) if re.search(r"\bm0,", m[1])]
    assert len(blocks) > 100                                  # all kernels', and the probe's
    code = lambda part: [l.split(";")[0].strip() for l in part.splitlines() if re.match(r"\s*[a-z]", l)]  # noqa: E731
    for block, rest in blocks:
        ops = code(block)
        saved = re.fullmatch(r"s_mov_b32 (s\d+), m0", ops[0])
        writes = [o for o in ops if re.match(r"s_mov_b32 m0,", o)]
        assert saved and writes[-1] == ops[-1] == "s_mov_b32 m0, " + saved[1], block
        assert not any(re.match(r"s_\w+ %s," % saved[1], o) for o in ops[1:]), block
        following = code(rest[:2000])[0]
        assert re.fullmatch(r"s_mov_b32 s\d+, m0", following) or not re.search(r"m0|_lds_|movrel|sendmsg|gws|interp|ttrace", following), following

"""The direct global -> LDS copies of the long-prompt kernels and of the attention take their LDS address from m0, which the compiler
does not know to be written by inline assembly (m0 on a clobber list is ignored): every block that writes it has to save it first and
to put it back last, and the next instruction must not read it (that would need a wait state).  Nor does the compiler look into a block for the five wait states between a
vector instruction that writes a scalar register and a memory instruction that reads it (a copy's source).  Compiles the device code to assembly (no GPU needed)."""
import os
import re
import subprocess

import pytest

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


def _sgprs(operand):
    m = re.fullmatch(r"s\[(\d+):(\d+)\]|s(\d+)", operand)
    return set() if m is None else {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def _states_behind_vector_write(before, src):
    """Wait states at the end of `before` since a vector instruction, or one that a jump may have come from, can have written a register of src; 5 if there are as many."""
    states, left = 0, set(src)
    for op in reversed(before):
        name, _, operands = op.partition(" ")
        written = {r for o in operands.split(",")[:2] for r in _sgprs(o.strip())}        # (a vector instruction's carry or mask is its second operand)
        if name.endswith(":") or (name.startswith("v_") and written & left):
            return states
        if name.startswith("s_") and not re.match(r"s_(cmp|bitcmp|cbranch)", name):
            left -= _sgprs(operands.split(",")[0].strip())
        states += int(operands, 0) + 1 if name == "s_nop" else 1
        if states >= 5 or not left:
            return 5
    return states


# copies a block; the attention's: one, two or four (heads of 32, 64 and 128)
@pytest.mark.parametrize("source,copies", [(PROBE, {1}), ('#include "pv_kernels_attention.hip"\n', {1, 2, 4})], ids=["prompts", "attention"])
def test_m0_is_put_back(tmp_path, source, copies):
    src, out = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(source)
    flags = [f for f in build.FLAGS if f not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    subprocess.run(["hipcc", *flags, "-S", "--offload-device-only", "-o", str(out), str(src)], check=True, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
    text = out.read_text()
    blocks = [(m[1], text[m.end():m.end() + 2000], text[max(0, m.start() - 2000):m.start()]) for m in re.finditer(r"#ASMSTART\n(.*?)#ASMEND", text, re.S) if re.search(r"\bm0,", m[1])]
    assert len(blocks) > (100 if copies == {1} else 20)       # all kernels', and the probe's
    code = lambda part: [l.split(";")[0].strip() for l in part.splitlines() if re.match(r"\s*[a-z]|\.LBB", l)]  # noqa: E731
    assert {sum("global_load_lds" in o for o in code(block)) for block, _, _ in blocks} == copies
    for block, rest, before in blocks:
        ops = code(block)
        saved = re.fullmatch(r"s_mov_b32 (s\d+), m0", ops[0])
        writes = [o for o in ops if re.match(r"s_mov_b32 m0,", o)]
        assert saved and writes[-1] == ops[-1] == "s_mov_b32 m0, " + saved[1], block
        assert not any(re.match(r"s_\w+ %s," % saved[1], o) for o in ops[1:]), block
        first = next(i for i, o in enumerate(ops) if o.startswith("global_load_lds"))
        source_regs = {r for o in ops if o.startswith("global_load_lds") for r in _sgprs(o.split(",")[1].split()[0])}
        assert source_regs and _states_behind_vector_write(code(before) + ops[:first], source_regs) == 5, before[-300:] + block
        following = next(o for o in code(rest) if not o.startswith("."))
        assert re.fullmatch(r"s_mov_b32 s\d+, m0", following) or not re.search(r"m0|_lds_|movrel|sendmsg|gws|interp|ttrace", following), following

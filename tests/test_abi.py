"""The C-ABI library loads and exports every symbol include/pipeverify.h declares (no GPU needed)."""
import ctypes
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    src = open(os.path.join(ROOT, "include", "pipeverify.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(pv_[a-z0-9_]+)\s*\(", src)))


def test_header_symbols_are_exported():
    from paper_2505_01572_amd import binding
    names = _declared()
    assert "pv_load_weights" in names and "pv_verify" in names and "pv_rollback" in names
    L = ctypes.CDLL(binding._LIB_PATH)
    missing = [n for n in names if not hasattr(L, n)]
    assert not missing, missing
    assert sorted(binding.EXPORTS) == names


def test_strerror_without_gpu():
    from paper_2505_01572_amd import binding
    L = binding.lib()
    assert L.pv_strerror(0) == b"ok"
    assert b"range" in L.pv_strerror(-3)


def test_config_validation_without_gpu():
    """pv_model_bytes is pure host arithmetic: it validates shapes and sizes the arena."""
    from paper_2505_01572_amd import binding
    L = binding.lib()
    cfg = binding.pv_model_config(2, 256, 4, 4, 64, 688, 1024, 1e-5, 10000.0, binding.PV_F32, 16, 16, 0)
    wb, sb = ctypes.c_size_t(), ctypes.c_size_t()
    assert L.pv_model_bytes(ctypes.byref(cfg), ctypes.byref(wb), ctypes.byref(sb)) == 0
    assert wb.value >= 2_106_624 * 4
    cfg.n_kv_heads = 3
    assert L.pv_model_bytes(ctypes.byref(cfg), ctypes.byref(wb), ctypes.byref(sb)) == -1
    cfg.n_kv_heads = 4; cfg.max_gamma = 65
    assert L.pv_model_bytes(ctypes.byref(cfg), ctypes.byref(wb), ctypes.byref(sb)) == -1
    cfg.max_gamma = 16; cfg.page_tokens = 12
    assert L.pv_model_bytes(ctypes.byref(cfg), ctypes.byref(wb), ctypes.byref(sb)) == -1


def test_prompt_part_of_the_arena_without_gpu():
    """The long prompts' buffers are an optional part behind the weights, once per model."""
    from paper_2505_01572_amd import binding
    from pv_inputs import CONFIGS
    L = binding.lib()

    def sizes(s, rows, dtype=binding.PV_BF16):
        cfg = binding.pv_model_config(s.n_layers, s.d_model, s.n_q_heads, s.n_kv_heads, s.head_dim, s.ffn_dim, s.vocab, s.rms_eps, s.rope_base, dtype, 16, 16, 0)
        wb, sb, pb = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
        assert L.pv_model_bytes(ctypes.byref(cfg), ctypes.byref(wb), ctypes.byref(sb)) == 0
        return L.pv_prompt_bytes(ctypes.byref(cfg), rows, ctypes.byref(pb)), wb.value, pb.value
    s = CONFIGS["8b"]
    rc, wb, pb = sizes(s, 2048)
    assert rc == 0 and 0 <= wb - pb - 2 * s.n_params() < 1 << 20 and pb < 212 << 20
    got = [sizes(s, r)[2] for r in (0, 64, 65, 128, 129, 192, 2000, 2048)]
    assert got[0] == got[1] == 0 and got[2] == got[3] < got[4] == got[5] < got[6] == got[7]
    assert sizes(s, -1)[0] == sizes(s, 2049)[0] == -3
    assert sizes(CONFIGS["tiny"], 2048, binding.PV_F32)[2] == 0

"""The marshalling in C++ lets other threads run Python while it launches, as ctypes does: a library of stand-ins, bound in
place of the real one, answers a status if its caller holds the interpreter's lock.  No kernel runs.  (Allocations
stand in the same scope of marshal.cpp, which this does not show.)"""
import subprocess

import pytest

pytestmark = pytest.mark.gpu

LAUNCHES = ["fwd_causal", "fwd_causal_from_state", "fwd_causal_varlen", "fwd_causal_dkdv", "fwd_bidir", "fwd_bidir_varlen", "fwd_bidir_dkdv",
            "bwd_causal", "bwd_causal_from_state", "bwd_causal_varlen", "bwd_causal_dkdv", "bwd_bidir", "bwd_bidir_varlen", "bwd_bidir_dkdv",
            "step_dkdv", "scale_from_m_varlen", "scale_backward_varlen"]


def test_lock_is_released(tmp_path):
    import torch
    import paper_2409_18747_amd.binding as b
    src, so = tmp_path / "stand_ins.cpp", tmp_path / "stand_ins.so"
    src.write_text('#include <cstddef>\nextern "C" {\nint PyGILState_Check(void);\n'
                   + "size_t cottn_workspace_bytes_dkdv() { return 256; }\n"
                   + "".join("int cottn_%s() { return PyGILState_Check() ? 5 : 0; }\n" % n for n in LAUNCHES) + "}\n")
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    x = torch.zeros(2, 3, 64, 32, device="cuda", dtype=torch.bfloat16)
    t, s, m = x[:, :, 0].contiguous(), torch.ones(3, device="cuda"), torch.zeros(3, device="cuda")
    sb, state = torch.ones(2, 3, device="cuda"), torch.zeros(2, 3, 32, 32, device="cuda")
    n = torch.full((2,), 64, dtype=torch.int32, device="cuda")
    b._marshal.bind(str(so), b.CottnError)
    try:
        b.cottn_fwd_causal(x, x, x, s)
        b.cottn_fwd_bidir(x, x, x, s)
        b.cottn_fwd_causal_varlen(x, x, x, sb, n)
        b.cottn_bwd_causal(x, x, x, s, x)
        b.cottn_bwd_bidir(x, x, x, s, x)
        b.cottn_bwd_causal_varlen(x, x, x, sb, n, x)
        b.cottn_step(t, t, t, s, state)
        b.cottn_scale_from_m_varlen(m, n)
        b.cottn_scale_backward_varlen(m, n, sb)
    finally:
        b._marshal.bind(b.library_path, b.CottnError)

"""Own prefixes formed four steps at a time (narrow rows, up to 256 workgroups): every number of steps before a segment
from none to beyond two sets, ends of a padded batch inside and between the steps of a set, and fp32 values that
send a workgroup through its whole products, against the oracle's linear forms."""
import numpy as np
import pytest

from helpers import TOL, code, draw_dkdv as draw, ds_terms_rss, rel_err, rel_err_ds, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    b.cottn_tune_segments(0)
    yield b
    b.cottn_tune_segments(0)


TINY = 2.0 ** -118   # below what the parts of fp32 values carry


@pytest.mark.parametrize("dtype,B,H,N,dk,dv,scale", [("bf16", 1, 2, 650, 32, 32, 1.0), ("f16", 2, 3, 961, 64, 32, 1.0),
                                                     ("bf16", 3, 5, 1023, 32, 32, 1.0), ("f32", 1, 2, 288, 32, 32, 1.0),
                                                     ("f32", 2, 3, 257, 32, 32, 1.0), ("f32", 1, 2, 288, 32, 32, TINY),
                                                     ("f32", 2, 3, 257, 32, 32, TINY)])
def test_against_oracle(cottn, oracle, dtype, B, H, N, dk, dv, scale):
    c = code(cottn, dtype)
    G = cottn.cottn_segments_dkdv(cottn.OP_BWD_CAUSAL, B, H, N, dk, dv, 0, c)
    assert 8 < G and B * H * G <= 256
    x = draw(B, H, N, dk, dv, dtype, 1200 + N)
    x["V"] *= np.float32(scale)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.profile_start()
    O = cottn.cottn_fwd_causal_dkdv(Q, K, V, s)
    assert list(cottn.profile_stop().values())[0][0] == 1   # no totals launch
    g = cottn.cottn_bwd_causal_dkdv(Q, K, V, s, dO)         # rebuilds the state
    g_ref = oracle.bwd_recurrent(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {"O": rel_err(to_host(O), oracle.fwd_recurrent(x["Q"], x["K"], x["V"], x["s"])[0])}
    errs.update({n: rel_err(to_host(a), r) for n, a, r in zip(("dQ", "dK", "dV"), g, g_ref)})
    errs["ds"] = rel_err_ds(to_host(g[3]), g_ref[3], ds_terms_rss(oracle, x)) if dk == dv else rel_err(to_host(g[3]), g_ref[3])
    print(dtype, B, H, N, dk, dv, scale, {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype,N,step", [("bf16", 900, 64), ("f32", 280, 32)])
def test_padded(cottn, oracle, dtype, N, step):
    import torch
    lens = [N, 0, 4 * step, 4 * step + 1, 5 * step - 1, N - 1]
    x = draw(len(lens), 2, N, 32, 32, dtype, 1300 + N)
    sc = np.linspace(0.5, 1.5, 2 * len(lens), dtype=np.float32).reshape(-1, 2)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s, n = to_device(sc, "f32"), torch.tensor(lens, dtype=torch.int32, device="cuda")
    O = cottn.cottn_fwd_causal_varlen(Q, K, V, s, n)
    g = cottn.cottn_bwd_causal_varlen(Q, K, V, s, n, dO)
    ref = [oracle.fwd_varlen(x["Q"], x["K"], x["V"], sc, lens)[0], *oracle.bwd_varlen(x["Q"], x["K"], x["V"], sc, x["dO"], lens)[:3]]
    for name, a, r in zip(("O", "dQ", "dK", "dV"), (O, *g[:3]), ref):
        e = rel_err(to_host(a), r)
        print(dtype, N, name, "%.2e" % e, flush=True)
        assert e <= TOL[dtype], (name, e)

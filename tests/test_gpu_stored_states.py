"""Workgroups that add the totals of other segments up themselves, several at once: fourteen segments, so that 0 to 13
stored states lie before or behind a segment (none, part of a batch, whole batches and both sizes of batch), against
the oracle's linear forms."""
import pytest

from helpers import TOL, code, draw_dkdv as draw, ds_terms_rss, rel_err, rel_err_ds, to_device, to_host

pytestmark = pytest.mark.gpu

SEGMENTS = 14


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    b.cottn_tune_segments(SEGMENTS)
    yield b
    b.cottn_tune_segments(0)


@pytest.mark.parametrize("dtype,dk,dv", [("bf16", 32, 32), ("f16", 64, 32), ("bf16", 64, 128), ("f16", 128, 64), ("f32", 32, 32),
                                         ("f32", 64, 64), ("f32", 64, 128)])
def test_against_oracle(cottn, oracle, dtype, dk, dv):
    c, B, H, N = code(cottn, dtype), 3, 11, SEGMENTS * 192 - 5
    assert cottn.cottn_segments_dkdv(cottn.OP_BWD_CAUSAL, B, H, N, dk, dv, 0, c) == SEGMENTS
    x = draw(B, H, N, dk, dv, dtype, 1400 + dk + dv)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.profile_start()
    O = cottn.cottn_fwd_causal_dkdv(Q, K, V, s)
    assert sum(n for n, _ in cottn.profile_stop().values()) == 2   # the totals and the scan, no carry between
    g = cottn.cottn_bwd_causal_dkdv(Q, K, V, s, dO)
    g_ref = oracle.bwd_recurrent(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {"O": rel_err(to_host(O), oracle.fwd_recurrent(x["Q"], x["K"], x["V"], x["s"])[0])}
    errs.update({n: rel_err(to_host(a), r) for n, a, r in zip(("dQ", "dK", "dV"), g, g_ref)})
    errs["ds"] = rel_err_ds(to_host(g[3]), g_ref[3], ds_terms_rss(oracle, x)) if dk == dv else rel_err(to_host(g[3]), g_ref[3])
    print(dtype, dk, dv, {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    assert max(errs.values()) <= TOL[dtype], errs

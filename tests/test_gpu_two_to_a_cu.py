"""16-bit causal 128 x 128 calls of more than 256 workgroups, whose scans take 32-row steps: one segment
(no reverse-time totals) and several that start from totals, lengths around the ends of the steps, padded
batches and a sequence continued from a state, against the oracle at the usual tolerance.  (Of two and three
segments, calls with few rows before the last one form its state themselves, in 64-row steps.)"""
import numpy as np
import pytest

from helpers import TOL, ds_terms_rss, rel_err, rel_err_ds, to_device, to_host

pytestmark = pytest.mark.gpu
D = 128


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    yield b
    b.cottn_tune_segments(0)


def check(errs, dtype, what):
    print(what, {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    for name, e in errs.items():
        assert e <= TOL[dtype], (what, name, e)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,N,segments", [(257, 1, 1), (257, 31, 1), (257, 33, 1), (260, 97, 1), (130, 129, 2), (87, 200, 3)])
def test_forward_backward(cottn, oracle, B, N, segments, dtype):
    import torch
    from paper_2409_18747_amd import workloads
    x = workloads.draw(B, 1, N, D, dtype, seed=900 + N)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.cottn_tune_segments(segments)
    state = torch.full((B, 1, D, D), float("nan"), dtype=torch.float32, device="cuda")
    O = cottn.cottn_fwd_causal(Q, K, V, s, state=state)
    g = cottn.cottn_bwd_causal(Q, K, V, s, dO)
    ref, g_ref = oracle.fwd_quadratic(x["Q"], x["K"], x["V"], x["s"]), oracle.bwd_quadratic(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {"O": rel_err(to_host(O), ref), "state": rel_err(to_host(state), oracle.fwd_recurrent(x["Q"], x["K"], x["V"], x["s"])[1])}
    errs.update({n: rel_err(to_host(a), r) for n, a, r in zip(("dQ", "dK", "dV"), g, g_ref)})
    errs["ds"] = rel_err_ds(to_host(g[3]), g_ref[3], ds_terms_rss(oracle, x))
    check(errs, dtype, "B%d N%d seg%d %s" % (B, N, segments, dtype))


@pytest.mark.parametrize("segments", [1, 2])
def test_pieces(cottn, segments):
    """Two pieces, the states handed on both ways, equal one call (which the test above compares)."""
    import torch
    from paper_2409_18747_amd import workloads
    B, N, cut, dtype = 264, 150, 70, "bf16"
    x = workloads.draw(B, 1, N, D, dtype, seed=31)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.cottn_tune_segments(segments)
    O, g = cottn.cottn_fwd_causal(Q, K, V, s), cottn.cottn_bwd_causal(Q, K, V, s, dO)
    parts = [tuple(t[:, :, a:b].contiguous() for t in (Q, K, V, dO)) for a, b in ((0, cut), (cut, N))]
    zero, mid, end, rev = (torch.zeros(B, 1, D, D, device="cuda") for _ in range(4))
    O0 = cottn.cottn_fwd_causal_from_state(*parts[0][:3], s, zero, state=mid)
    O1 = cottn.cottn_fwd_causal_from_state(*parts[1][:3], s, mid, state=end)
    g1 = cottn.cottn_bwd_causal_from_state(*parts[1][:3], s, parts[1][3], state_in=mid, rev_state_out=rev)
    g0 = cottn.cottn_bwd_causal_from_state(*parts[0][:3], s, parts[0][3], state_in=zero, rev_state_in=rev)
    errs = {"O": rel_err(to_host(torch.cat((O0, O1), 2)), to_host(O)), "ds": rel_err(to_host(g0[3] + g1[3]), to_host(g[3]))}
    errs.update({n: rel_err(to_host(torch.cat((a, b), 2)), to_host(c)) for n, a, b, c in zip(("dQ", "dK", "dV"), g0, g1, g)})
    check(errs, dtype, "pieces seg%d" % segments)


def test_padded(cottn, oracle):
    import torch
    from paper_2409_18747_amd import workloads
    B, N, dtype = 300, 70, "bf16"
    x = workloads.draw(B, 1, N, D, dtype, seed=32)
    lens = [(7 * b) % (N + 1) for b in range(B)]
    sc = np.linspace(0.5, 1.5, B, dtype=np.float32).reshape(B, 1)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s, n = to_device(sc, "f32"), torch.tensor(lens, dtype=torch.int32, device="cuda")
    cottn.cottn_tune_segments(0)
    O = to_host(cottn.cottn_fwd_causal_varlen(Q, K, V, s, n))
    g = [to_host(t) for t in cottn.cottn_bwd_causal_varlen(Q, K, V, s, n, dO)]
    ref = [np.zeros_like(O) for _ in range(4)]
    for b, m in enumerate(lens):
        if m:
            a = [x[k][b:b + 1, :, :m] for k in ("Q", "K", "V", "dO")]
            ref[0][b, :, :m] = oracle.fwd_quadratic(*a[:3], sc[b])
            for r, t in zip(ref[1:], oracle.bwd_quadratic(*a[:3], sc[b], a[3])[:3]):
                r[b, :, :m] = t
    check({k: rel_err(t, r) for k, t, r in zip(("O", "dQ", "dK", "dV"), [O] + g[:3], ref)}, dtype, "padded")


# (sequences, rows, segments): more than 256 workgroups and more than 320 rows before the last segment
FROM_TOTALS = [(130, 700, 2), (129, 769, 2), (100, 500, 3)]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("B,N,segments", FROM_TOTALS)
def test_segments_from_totals(cottn, oracle, B, N, segments, dtype):
    import torch
    from paper_2409_18747_amd import workloads
    c = cottn.COTTN_BF16 if dtype == "bf16" else cottn.COTTN_F16
    x = workloads.draw(B, 1, N, D, dtype, seed=920 + N)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.cottn_tune_segments(segments)
    assert cottn.cottn_segments(cottn.OP_FWD_CAUSAL, B, 1, N, D, 0, c) == segments and B * segments > 256
    state = torch.full((B, 1, D, D), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.full((cottn.cottn_workspace_bytes(cottn.OP_FWD_CAUSAL, B, 1, N, D, 0, c),), 255, dtype=torch.uint8, device="cuda")
    cottn.profile_start()
    O = cottn.cottn_fwd_causal(Q, K, V, s, state=state, workspace=ws)
    assert set(cottn.profile_stop()) == {"fwd_segment_state_" + dtype, "fwd_causal_scan_" + dtype}
    ref, S = oracle.fwd_recurrent(x["Q"], x["K"], x["V"], x["s"])
    g_ref = oracle.bwd_recurrent(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {"O": rel_err(to_host(O), ref), "state": rel_err(to_host(state), S)}
    for kept in (ws, None):
        g = cottn.cottn_bwd_causal(Q, K, V, s, dO, fwd_workspace=kept)
        errs.update({n: rel_err(to_host(a), r) for n, a, r in zip(("dQ", "dK", "dV"), g, g_ref)})
        check(errs, dtype, "totals B%d N%d seg%d %s" % (B, N, segments, dtype))
    # from a state, and padded
    cut = N - 200
    zero, mid, end = (torch.zeros(B, 1, D, D, device="cuda") for _ in range(3))
    cottn.cottn_fwd_causal_from_state(*(t[:, :, :200].contiguous() for t in (Q, K, V)), s, zero, state=mid)
    O1 = cottn.cottn_fwd_causal_from_state(*(t[:, :, 200:].contiguous() for t in (Q, K, V)), s, mid, state=end)
    check({"O from state": rel_err(to_host(O1), ref[:, :, 200:]), "state": rel_err(to_host(end), S)}, dtype, "cut %d" % cut)
    lens = np.array([(37 * b) % (N + 1) for b in range(B)])
    P = to_host(cottn.cottn_fwd_causal_varlen(Q, K, V, s.expand(B, 1).contiguous(),
                                              torch.tensor(lens, dtype=torch.int32, device="cuda")))
    rows = np.arange(N)[None, None, :, None] < lens[:, None, None, None]   # (a row sees the rows before it alone)
    assert (P[np.broadcast_to(~rows, P.shape)] == 0).all()
    check({"O padded": rel_err(P, ref * rows)}, dtype, "lengths")

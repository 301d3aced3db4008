"""Short causal calls in segments whose workgroups form the state of the rows before them by themselves: both
sides of the rule's line, by the launches that each call makes, the first and last segment of one step and a ragged one, a given start state, padded
batches with lengths that end before, inside and behind a segment; forward, the states that it leaves to the
backward, and the backward that rebuilds them, against the oracle's linear forms."""
import numpy as np
import pytest

from helpers import TOL, code, draw_dkdv as draw, ds_terms_rss, rel_err, rel_err_ds, to_device, to_host

pytestmark = pytest.mark.gpu
# rows before the last segment: at the line and beyond it, or the shortest that take segments; last, those
# where only the forward does so, and the first ones beyond.  With each, which calls form their states
# themselves: the forward and a backward that rebuilds them, the forward alone, or neither.
SHAPES = [("bf16", 1, 1, 130, 64, 64, "both"), ("f16", 2, 5, 640, 64, 64, "both"),
          ("bf16", 2, 5, 705, 64, 64, "neither"), ("f16", 8, 5, 511, 64, 64, "both"),
          ("bf16", 2, 5, 1023, 32, 32, "both"), ("f16", 10, 10, 513, 32, 32, "neither"),
          ("bf16", 2, 1, 577, 128, 128, "both"), ("bf16", 10, 10, 641, 128, 128, "both"),
          ("f16", 10, 10, 333, 128, 128, "both"), ("bf16", 10, 10, 321, 128, 32, "both"),
          ("f16", 5, 8, 400, 32, 128, "both"), ("bf16", 3, 3, 257, 128, 64, "both"),
          ("f16", 2, 2, 777, 64, 128, "both"), ("bf16", 2, 5, 1023, 64, 32, "both"), ("f32", 1, 1, 65, 32, 32, "both"),
          ("f32", 1, 2, 319, 32, 32, "both"), ("f32", 1, 2, 321, 32, 32, "neither"),
          ("f32", 10, 10, 129, 32, 32, "both"), ("f32", 1, 1, 33, 64, 64, "both"),
          ("f32", 10, 10, 130, 64, 64, "both"), ("f32", 1, 2, 199, 64, 64, "both"),
          ("f32", 10, 10, 101, 128, 128, "both"), ("f32", 10, 10, 255, 64, 128, "both"),
          ("f32", 4, 1, 66, 128, 32, "both"), ("bf16", 10, 10, 385, 64, 64, "forward"),
          ("f16", 10, 15, 399, 128, 64, "forward"), ("bf16", 12, 10, 640, 32, 128, "forward"),
          ("f16", 12, 10, 577, 64, 128, "forward"), ("bf16", 12, 10, 705, 64, 64, "forward"),
          ("bf16", 16, 5, 777, 128, 128, "forward"), ("f16", 6, 10, 769, 128, 128, "forward"),
          ("bf16", 6, 10, 1025, 128, 128, "neither")]


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    b.cottn_tune_segments(0)
    yield b
    b.cottn_tune_segments(0)


@pytest.mark.parametrize("dtype,B,H,N,dk,dv,own", SHAPES)
def test_against_oracle(cottn, oracle, dtype, B, H, N, dk, dv, own):
    import torch
    c = code(cottn, dtype)
    assert cottn.cottn_segments_dkdv(cottn.OP_BWD_CAUSAL, B, H, N, dk, dv, 0, c) > 1
    x = draw(B, H, N, dk, dv, dtype, 1000 + N)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    ws, bws = (torch.full((cottn.cottn_workspace_bytes_dkdv(op, B, H, N, dk, dv, 0, c),), 255, dtype=torch.uint8, device="cuda")
               for op in (cottn.OP_FWD_CAUSAL, cottn.OP_BWD_CAUSAL))   # (NaN wherever nothing is written)
    state = torch.full((B, H, dk, dv), float("nan"), dtype=torch.float32, device="cuda")
    cottn.profile_start()
    O = cottn.cottn_fwd_causal_dkdv(Q, K, V, s, state=state, workspace=ws)
    forward = cottn.profile_stop()
    grads = cottn.cottn_bwd_causal_dkdv(Q, K, V, s, dO, workspace=bws, fwd_workspace=ws)
    cottn.profile_start()
    rebuilt = cottn.cottn_bwd_causal_dkdv(Q, K, V, s, dO, workspace=bws.fill_(255))
    for names, itself in ((forward, own != "neither"), (cottn.profile_stop(), own == "both")):
        assert any(n.startswith("fwd_segment_state") for n in names) != itself, sorted(names)
    assert own == "neither" or len(forward) == 1
    ref, S = oracle.fwd_recurrent(x["Q"], x["K"], x["V"], x["s"])
    g_ref = oracle.bwd_recurrent(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {"O": rel_err(to_host(O), ref), "state": rel_err(to_host(state), S)}
    for kind, g in (("", grads), (" rebuilt", rebuilt)):
        errs.update({n + kind: rel_err(to_host(a), r) for n, a, r in zip(("dQ", "dK", "dV"), g, g_ref)})
        errs["ds" + kind] = rel_err(to_host(g[3]), g_ref[3]) if dk != dv else rel_err_ds(to_host(g[3]), g_ref[3], ds_terms_rss(oracle, x))
    print(dtype, B, H, N, dk, dv, {k: "%.2e" % v for k, v in errs.items()}, flush=True)
    assert max(errs.values()) <= TOL[dtype], errs


@pytest.mark.parametrize("dtype,d,N", [("bf16", 64, 300), ("f32", 32, 200), ("f16", 128, 257)])
def test_padded_and_from_state(cottn, oracle, dtype, d, N):
    import torch
    c, x = code(cottn, dtype), draw(5, 2, N, d, d, dtype, 1100 + N)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    # the second half from the first one's state equals the rows of one call
    h = N // 2
    O, mid, end, whole = cottn.cottn_fwd_causal(Q, K, V, s), *(torch.zeros(5, 2, d, d, device="cuda") for _ in range(3))
    cottn.cottn_fwd_causal(Q, K, V, s, state=whole)
    first, second = (tuple(t[:, :, a:b].contiguous() for t in (Q, K, V)) for a, b in ((0, h), (h, N)))
    cottn.cottn_fwd_causal(*first, s, state=mid)
    O1 = cottn.cottn_fwd_causal_from_state(*second, s, mid, state=end)
    assert rel_err(to_host(O1), to_host(O[:, :, h:])) <= TOL[dtype] and rel_err(to_host(end), to_host(whole)) <= TOL[dtype]
    # lengths
    lens = [N, 0, 1, 64, N - 1]
    sc = np.linspace(0.5, 1.5, 10, dtype=np.float32).reshape(5, 2)
    s, n = to_device(sc, "f32"), torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.full((cottn.cottn_workspace_bytes(cottn.OP_FWD_CAUSAL, 5, 2, N, d, 0, c),), 255, dtype=torch.uint8, device="cuda")
    O = cottn.cottn_fwd_causal_varlen(Q, K, V, s, n, workspace=ws)
    ref = [oracle.fwd_varlen(x["Q"], x["K"], x["V"], sc, lens)[0], *oracle.bwd_varlen(x["Q"], x["K"], x["V"], sc, x["dO"], lens)[:3]]
    for kept in (ws, None):
        g = cottn.cottn_bwd_causal_varlen(Q, K, V, s, n, dO, fwd_workspace=kept)
        for name, a, r in zip(("O", "dQ", "dK", "dV"), (O, *g[:3]), ref):
            e = rel_err(to_host(a), r)
            print(dtype, d, N, kept is not None, name, "%.2e" % e, flush=True)
            assert e <= TOL[dtype], (name, e)

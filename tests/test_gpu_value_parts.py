"""Causal forwards of one segment whose 128 value columns are shared by two or four workgroups: every pair
of widths and type that takes that way, lengths around the steps' ends, padded rows, with and without a
state to start from and one to leave, against the oracle; and the sizes next to the rule's lines."""
import numpy as np
import pytest

from helpers import TOL, rel_err, to_device, to_host

pytestmark = pytest.mark.gpu
DV = 128


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    b.cottn_tune_segments(1)
    yield b
    b.cottn_tune_segments(0)


def draw(B, N, dk, dtype, seed):
    rng = np.random.default_rng(seed)
    from paper_2409_18747_amd import workloads
    wide = workloads.draw(B, 2, max(N, 1), DV, dtype, seed)   # values already representable in the type
    return wide["Q"][:, :, :N, :dk].copy(), wide["K"][:, :, :N, :dk].copy(), wide["V"][:, :, :N], wide["s"], rng


@pytest.mark.parametrize("dtype,dk", [("bf16", 128), ("f16", 128), ("bf16", 64), ("f16", 32), ("f32", 64)])
@pytest.mark.parametrize("B,N", [(1, 1), (1, 5), (3, 31), (3, 32), (2, 33), (64, 63), (2, 64), (2, 65), (64, 129), (65, 40), (128, 40), (129, 40)])
def test_against_oracle(cottn, oracle, B, N, dk, dtype):
    import torch
    Q, K, V, s, _ = draw(B, N, dk, dtype, 700 + N + dk)
    state = torch.full((B, 2, dk, DV), float("nan"), dtype=torch.float32, device="cuda")
    O = torch.full((B, 2, N, DV), float("nan"), dtype=to_device(V, dtype).dtype, device="cuda")
    cottn.cottn_fwd_causal_dkdv(to_device(Q, dtype), to_device(K, dtype), to_device(V, dtype), to_device(s, "f32"), O=O, state=state)
    ref, S = oracle.fwd_recurrent(Q, K, V, s)
    e = {"O": rel_err(to_host(O), ref), "state": rel_err(to_host(state), S)}
    print("B%d N%d %dx%d %s" % (B, N, dk, DV, dtype), {k: "%.2e" % v for k, v in e.items()}, flush=True)
    assert max(e.values()) <= TOL[dtype], e


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("first,N", [(1, 6), (30, 33), (40, 150)])
def test_from_state(cottn, oracle, first, N, dtype):
    import torch
    Q, K, V, s, _ = draw(3, N, 128, dtype, 800 + N)
    x, sd = [to_device(t, dtype) for t in (Q, K, V)], to_device(s, "f32")
    mid, end = (torch.full((3, 2, 128, DV), float("nan"), device="cuda") for _ in range(2))
    zero = torch.zeros_like(mid)
    O0 = cottn.cottn_fwd_causal_from_state(*(t[:, :, :first].contiguous() for t in x), sd, zero, state=mid)
    O1 = cottn.cottn_fwd_causal_from_state(*(t[:, :, first:].contiguous() for t in x), sd, mid, state=end)
    ref, S = oracle.fwd_recurrent(Q, K, V, s)
    e = {"O": rel_err(to_host(torch.cat((O0, O1), 2)), ref), "state": rel_err(to_host(end), S)}
    print(first, N, dtype, e, flush=True)
    assert max(e.values()) <= TOL[dtype], e


@pytest.mark.parametrize("N", [20, 50, 100])
def test_padded(cottn, oracle, N):
    import torch
    lens = [N, 0, 1, N // 2, N - 1]
    Q, K, V, _, rng = draw(5, N, 128, "bf16", 850 + N)
    sc = rng.uniform(0.5, 1.5, (5, 2)).astype(np.float32)
    O = to_host(cottn.cottn_fwd_causal_varlen(*(to_device(t, "bf16") for t in (Q, K, V)), to_device(sc, "f32"),
                                              torch.tensor(lens, dtype=torch.int32, device="cuda")))
    ref = np.zeros_like(O)
    for b, n in enumerate(lens):
        if n:
            ref[b, :, :n] = oracle.fwd_quadratic(Q[b:b + 1, :, :n], K[b:b + 1, :, :n], V[b:b + 1, :, :n], sc[b])
    assert rel_err(O, ref) <= TOL["bf16"] and all((O[b, :, n:] == 0).all() for b, n in enumerate(lens))

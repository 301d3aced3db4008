"""GPU parity of the bidirectional calls on each of the paths they can take, at the shapes where the library
takes it by itself, against the same sums in plain PyTorch fp32: with S = Kh^T V and G = Qh^T dO over the rows
that exist, O = s Qh S, dQh = s dO S^T, dKh = s V G^T, dV = s Kh G, ds = <S, G>, and the chain rule through
the row normalisation.  Bounds are the suite's (helpers.TOL)."""
import pytest

from helpers import TOL

pytestmark = pytest.mark.gpu

CODES = {"f32": 0, "bf16": 1, "f16": 2}


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    yield b
    b.cottn_tune_segments(0)


def reference(Q, K, V, s, dO, lens):
    """Everything in fp32, s per (batch, head); rows at or beyond lens[b] count for nothing."""
    import torch
    N = Q.shape[2]
    exist = (torch.arange(N, device=Q.device)[None, :] < lens[:, None].to(Q.device))[:, None, :, None].float()
    q, k, v, g = (t.float() * exist for t in (Q, K, V, dO))
    rq, rk = (1.0 / t.norm(dim=-1, keepdim=True).clamp_min(1e-6) for t in (q, k))
    qh, kh = rq * q, rk * k
    T = lambda t: t.transpose(-1, -2).contiguous()
    S, G, sc = T(kh) @ v, T(qh) @ g, s[:, :, None, None]
    dqh, dkh = g @ T(S), v @ T(G)
    rho = (qh * dqh).sum(-1)   # its sum over the rows is <S, G>
    return {"O": sc * (qh @ S), "state": S, "dQ": sc * rq * (dqh - qh * rho[..., None]) * exist,
            "dK": sc * rk * (dkh - kh * (kh * dkh).sum(-1, keepdim=True)) * exist, "dV": sc * (kh @ G),
            "ds": rho.double().sum(-1), "ds_terms": (rho.double() ** 2).sum(-1)}


def run(cottn, B, H, N, dk, dv, dtype, seed, lens=None, saved=True, segments=None):
    """One forward and backward through the library's own choice of path; `segments`: how many it must report."""
    import torch
    cottn.cottn_tune_segments(0)
    if segments is not None:
        assert cottn.cottn_segments_dkdv(cottn.OP_FWD_BIDIR, B, H, N, dk, dv, 0, CODES[dtype]) == segments
    t = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    normal = lambda d: torch.randn(B, H, N, d, device="cuda", generator=gen).to(t)
    Q, K, V, dO = normal(dk), normal(dk), normal(dv), normal(dv)
    nan = lambda *shape, dtype=t: torch.full(shape, float("nan"), dtype=dtype, device="cuda")
    out = {"O": nan(B, H, N, dv), "dQ": nan(B, H, N, dk), "dK": nan(B, H, N, dk), "dV": nan(B, H, N, dv),
           "state": nan(B, H, dk, dv, dtype=torch.float32)}
    ws = None
    if saved:
        n = cottn.cottn_workspace_bytes_dkdv(cottn.OP_FWD_BIDIR, B, H, N, dk, dv, 0, CODES[dtype])
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    if lens is None:
        s = 0.5 + torch.rand(H, device="cuda", generator=gen)
        ds = nan(H, dtype=torch.float32)
        cottn.cottn_fwd_bidir_dkdv(Q, K, V, s, O=out["O"], state=out["state"], workspace=ws)
        cottn.cottn_bwd_bidir_dkdv(Q, K, V, s, dO, dQ=out["dQ"], dK=out["dK"], dV=out["dV"], ds=ds, fwd_workspace=ws)
        per_unit, L = s[None, :].expand(B, H), torch.full((B,), N)
    else:
        per_unit = 0.5 + torch.rand(B, H, device="cuda", generator=gen)
        ds = nan(B, H, dtype=torch.float32)
        on_gpu = torch.tensor(lens, dtype=torch.int32, device="cuda")
        cottn.cottn_fwd_bidir_varlen(Q, K, V, per_unit, on_gpu, O=out["O"], state=out["state"], workspace=ws)
        cottn.cottn_bwd_bidir_varlen(Q, K, V, per_unit, on_gpu, dO, dQ=out["dQ"], dK=out["dK"], dV=out["dV"], ds=ds,
                                     fwd_workspace=ws)
        L = torch.tensor(lens).clamp(0, N)
    torch.cuda.synchronize()
    ref = reference(Q, K, V, per_unit, dO, L)
    errs = {n: float((a.float() - ref[n]).abs().max() / ref[n].abs().max()) for n, a in out.items()}
    total, terms = (ref["ds"], ref["ds_terms"]) if lens is not None else (ref["ds"].sum(0), ref["ds_terms"].sum(0))
    errs["ds"] = float((ds.double() - total).abs().max() / max(float(total.abs().max()), float(terms.sqrt().max())))
    print("bidir path %s B%d H%d N%d %dx%d lens %s saved%d: %s" %
          (dtype, B, H, N, dk, dv, lens, saved, {n: "%.2e" % e for n, e in errs.items()}), flush=True)
    if lens is not None:   # rows that do not exist are exactly zero
        for b, n in enumerate(L.tolist()):
            for name in ("O", "dQ", "dK", "dV"):
                assert bool((out[name][b, :, n:] == 0).all()), (name, b)
    for name, e in errs.items():
        assert e <= TOL[dtype], (name, e)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("N,segments", [(1, 1), (64, 1), (65, 1), (129, 1), (300, 1), (1100, 2)])
def test_widest_units_beyond_one_per_compute_unit(cottn, dtype, N, segments):
    """258 units of 128 x 128: the forward as totals and 64-row steps, the backward by unit, or both split."""
    run(cottn, 43, 6, N, 128, 128, dtype, seed=2000 + N, saved=N % 2 == 1, segments=segments)
    if N in (129, 300):
        run(cottn, 43, 6, N, 128, 128, dtype, seed=2100 + N, lens=[(37 * b) % (N + 1) for b in range(43)], segments=1)


@pytest.mark.parametrize("B,H,N,dk,dv,segments", [(43, 8, 2100, 32, 32, 2), (27, 10, 1100, 64, 128, 3), (27, 10, 600, 128, 32, 3),
                                                  (33, 16, 1100, 64, 64, 2), (1, 20, 50000, 32, 32, 23)])
def test_splits_of_many_units_and_of_the_longest(cottn, B, H, N, dk, dv, segments):
    run(cottn, B, H, N, dk, dv, "bf16", seed=2200 + N, segments=segments)

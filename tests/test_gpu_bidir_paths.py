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


def run(cottn, B, H, N, dk, dv, dtype, seed, lens=None, saved=True, segments=None, kernels=()):
    """One forward and backward through the library's own choice of path; `segments`: how many it must
    report, `kernels`: what it must launch (without the element type)."""
    import torch
    cottn.profile_start()
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
    launched = {name.replace("_" + dtype, "") for name in cottn.profile_stop()}
    assert set(kernels) <= launched, (kernels, launched)
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
    kernels = ["fwd_bidir_apply", "bwd_bidir_unit" if segments == 1 else "bwd_bidir_dq"]
    run(cottn, 43, 6, N, 128, 128, dtype, seed=2000 + N, saved=N % 2 == 1, segments=segments, kernels=kernels)
    if N in (129, 300):
        run(cottn, 43, 6, N, 128, 128, dtype, seed=2100 + N, lens=[(37 * b) % (N + 1) for b in range(43)], segments=1,
            kernels=kernels)


@pytest.mark.parametrize("B,H,N,dk,dv,segments", [(43, 8, 2100, 32, 32, 2), (27, 10, 1100, 64, 128, 3), (27, 10, 600, 128, 32, 3),
                                                  (33, 16, 1100, 64, 64, 2), (1, 20, 50000, 32, 32, 23)])
def test_splits_of_many_units_and_of_the_longest(cottn, B, H, N, dk, dv, segments):
    run(cottn, B, H, N, dk, dv, "bf16", seed=2200 + N, segments=segments)


BY_UNIT = ["fwd_bidir_unit", "bwd_bidir_unit"]


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("N", [100, 200, 389])
def test_padded_batches_by_unit(cottn, dtype, d, N):
    """One to four 128-row steps per unit; sequences that are empty, end inside, at and just beyond a step,
    and lengths outside 0 .. N."""
    ends = [0, 1, 127, 128, 129, 255, 256, 257, 384, 385, N - 1, N, N + 9, -4]
    lens = [ends[(5 * b) % len(ends)] for b in range(28)]
    for saved in (True, False):
        run(cottn, 28, 6, N, d, d, dtype, seed=2300 + N + d, lens=[min(n, N + 9) for n in lens], saved=saved, segments=1,
            kernels=BY_UNIT)


@pytest.mark.parametrize("dk,dv", [(32, 128), (128, 32), (64, 128), (128, 64), (128, 128)])
def test_several_steps_by_unit(cottn, dk, dv):
    run(cottn, 27, 6, 389, dk, dv, "bf16", seed=2400 + dk, segments=1, kernels=BY_UNIT)
    run(cottn, 1, 224, 600, dk, dv, "f16", seed=2500 + dv, saved=False, segments=1, kernels=BY_UNIT)   # one batch: ds whole


@pytest.mark.parametrize("dtype,N,d,segments", [("bf16", 6500, 64, 26), ("f16", 6500, 32, 26), ("bf16", 2700, 128, 11),
                                                ("f32", 6500, 64, 34), ("f32", 2700, 128, 15)])
def test_split_so_fine_that_a_launch_combines(cottn, dtype, N, d, segments):
    """The library's own choice for one long sequence: more segments than the kernels add up themselves."""
    for saved in (True, False):
        run(cottn, 1, 1, N, d, d, dtype, seed=2600 + N + d, saved=saved, segments=segments, kernels=["bidir_combine"])
        run(cottn, 1, 1, N, d, d, dtype, seed=2700 + N + d, lens=[N - 700], saved=saved, segments=segments,
            kernels=["bidir_combine"])

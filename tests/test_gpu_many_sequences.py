"""GPU: so many (batch, head) units of one token that a launch of 512-thread workgroups would reach the
2^32 threads a launch may have.  One token has a closed form, so the reference is plain PyTorch in fp32:
with P = qh . kh and A = dO . v, O = s P v, dV = s P dO, dqh = s A kh, dkh = s A qh and ds = sum P A."""
import pytest

from helpers import TOL

pytestmark = pytest.mark.gpu

B, H = 524288, 16   # 8 388 608 units: 2^32 threads at 512 each


@pytest.mark.parametrize("causal,d,memory", [(True, 128, 40e9), (False, 32, 150e9)])
def test_one_token_each(causal, d, memory):
    import torch
    import paper_2409_18747_amd.binding as cottn
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < memory:
        pytest.skip("needs %d GB of device memory" % (memory / 1e9))
    cottn.cottn_tune_segments(0)
    gen = torch.Generator(device="cuda").manual_seed(31)
    Q, K, V, dO = (torch.randn(B, H, 1, d, device="cuda", generator=gen, dtype=torch.bfloat16) for _ in range(4))
    s = 0.5 + torch.rand(H, device="cuda", generator=gen)
    outs = [torch.full_like(Q, float("nan")) for _ in range(4)]
    ds = torch.full((H,), float("nan"), device="cuda")
    if causal:
        # (a forward of 128 x 128 takes 512 threads in any case)
        dQ, dK, dV, _ = cottn.cottn_bwd_causal(Q, K, V, s, dO, dQ=outs[0], dK=outs[1], dV=outs[2], ds=ds)
        got = {"dQ": dQ, "dK": dK, "dV": dV}
    else:
        ws = torch.empty(cottn.cottn_workspace_bytes(cottn.OP_FWD_BIDIR, B, H, 1, d), dtype=torch.uint8, device="cuda")
        O = cottn.cottn_fwd_bidir(Q, K, V, s, O=outs[3], workspace=ws)
        dQ, dK, dV, _ = cottn.cottn_bwd_bidir(Q, K, V, s, dO, dQ=outs[0], dK=outs[1], dV=outs[2], ds=ds, fwd_workspace=ws)
        got = {"O": O, "dQ": dQ, "dK": dK, "dV": dV}
    torch.cuda.synchronize()
    worst, largest = dict.fromkeys(got, 0.0), dict.fromkeys(got, 0.0)
    ds_ref = torch.zeros(H, dtype=torch.float64, device="cuda")
    squares = torch.zeros_like(ds_ref)
    step = 65536
    for b in range(0, B, step):
        q, k, v, g = (t[b:b + step].float().squeeze(2) for t in (Q, K, V, dO))
        rq, rk = (1.0 / t.norm(dim=-1, keepdim=True).clamp_min(1e-6) for t in (q, k))
        qh, kh = rq * q, rk * k
        P, A, sc = (qh * kh).sum(-1, keepdim=True), (g * v).sum(-1, keepdim=True), s[None, :, None]
        ref = {"O": sc * P * v, "dV": sc * P * g, "dQ": sc * A * rq * (kh - qh * P), "dK": sc * A * rk * (qh - kh * P)}
        for name, t in got.items():
            worst[name] = max(worst[name], float((t[b:b + step].float().squeeze(2) - ref[name]).abs().max()))
            largest[name] = max(largest[name], float(ref[name].abs().max()))
        terms = (P * A).double().squeeze(-1)
        ds_ref += terms.sum(0)
        squares += (terms ** 2).sum(0)
    errs = {n: worst[n] / largest[n] for n in got}
    errs["ds"] = float((ds.double() - ds_ref).abs().max() / max(float(ds_ref.abs().max()), float(squares.sqrt().max())))
    del Q, K, V, dO, outs, got
    torch.cuda.empty_cache()
    print("one token each, %s d%d: %s" % ("causal" if causal else "bidir", d, {n: "%.2e" % e for n, e in errs.items()}), flush=True)
    for name, e in errs.items():
        assert e <= TOL["bf16"], (name, e)

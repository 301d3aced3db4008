"""GPU parity: cottn_bwd_causal (through the C ABI) against the CPU oracle's brute-force gradients."""
import numpy as np
import pytest

from helpers import TOL, ds_terms_rss, rel_err, rel_err_ds, to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    yield b
    b.cottn_tune_segments(0)


def run_bwd(cottn, oracle, B, H, N, d, dtype, seed, chunk=0, segments=0, scale=1.0, mutate=None,
            saved=False):
    import torch
    from paper_2409_18747_amd import workloads
    x = workloads.draw(B, H, N, d, dtype, seed, value_scale=scale)
    if mutate:
        mutate(x)
    Q, K, V, dO = (to_device(x[k], dtype) for k in ("Q", "K", "V", "dO"))
    s = to_device(x["s"], "f32")
    cottn.cottn_tune_segments(segments)
    fwd_ws = None
    if saved:
        # the backward takes the forward-time segment states over from the forward's workspace
        code = cottn.COTTN_BF16 if dtype == "bf16" else cottn.COTTN_F32
        need = cottn.cottn_workspace_bytes(cottn.OP_FWD_CAUSAL, B, H, N, d, chunk, code)
        fwd_ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
        cottn.cottn_fwd_causal(Q, K, V, s, workspace=fwd_ws, chunk=chunk)
    dQ, dK, dV, ds = cottn.cottn_bwd_causal(Q, K, V, s, dO, chunk=chunk, fwd_workspace=fwd_ws)
    torch.cuda.synchronize()
    if N <= 1024:
        ref = oracle.bwd_quadratic(x["Q"], x["K"], x["V"], x["s"], x["dO"], causal=True)
    else:
        ref = oracle.bwd_recurrent(x["Q"], x["K"], x["V"], x["s"], x["dO"])
    errs = {}
    for name, got, want in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
        errs[name] = rel_err(to_host(got), want)
    errs["ds"] = rel_err_ds(to_host(ds), ref[3], ds_terms_rss(oracle, x) if N <= 1024 else 0.0)
    errs["ds_plain"] = rel_err(to_host(ds), ref[3])
    print("bwd_causal %s B%d H%d N%d d%d chunk%d seg%d: %s" %
          (dtype, B, H, N, d, chunk, segments, {k: "%.2e" % v for k, v in errs.items()}), flush=True)
    for name, e in errs.items():
        if name != "ds_plain":  # reported; equal to "ds" unless ds cancels below its terms' size
            assert e <= TOL[dtype], (name, e)
    return dQ, dK, dV, ds


@pytest.mark.parametrize("N", [1, 15, 16, 63, 64, 65, 200, 261])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_bf16_one_segment(cottn, oracle, N, d):
    run_bwd(cottn, oracle, 2, 3, N, d, "bf16", seed=200 + N + d, segments=1)


@pytest.mark.parametrize("segments", [2, 3, 5, 64])
@pytest.mark.parametrize("d,N", [(64, 517), (128, 330), (32, 700)])
def test_bf16_segmented(cottn, oracle, segments, d, N):
    run_bwd(cottn, oracle, 2, 2, N, d, "bf16", seed=8, segments=segments)


@pytest.mark.parametrize("chunk,d", [(128, 32), (128, 64), (256, 32), (256, 64)])
def test_bf16_chunk_sizes(cottn, oracle, chunk, d):
    for segments in (1, 3):
        run_bwd(cottn, oracle, 1, 3, 900, d, "bf16", seed=12, chunk=chunk, segments=segments)


@pytest.mark.parametrize("segments", [1, 2, 4, 7])
@pytest.mark.parametrize("d,N", [(64, 517), (128, 330), (32, 700)])
def test_bf16_states_saved_by_forward(cottn, oracle, segments, d, N):
    """With the forward's workspace handed over the gradients meet the same bar and equal, bit
    for bit, those of the backward that rebuilds the states (same kernel, same values)."""
    import torch
    a = run_bwd(cottn, oracle, 2, 2, N, d, "bf16", seed=31, segments=segments, saved=True)
    b = run_bwd(cottn, oracle, 2, 2, N, d, "bf16", seed=31, segments=segments, saved=False)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("segments", [2, 3, 7])
def test_f32_states_saved_by_forward(cottn, oracle, segments):
    """The same for fp32, with totals added in place and (128 x 128 in 7 segments) carried."""
    import torch
    for d in (64, 128):
        a = run_bwd(cottn, oracle, 1, 2, 230, d, "f32", seed=5, segments=segments, saved=True)
        b = run_bwd(cottn, oracle, 1, 2, 230, d, "f32", seed=5, segments=segments, saved=False)
        for x, y in zip(a, b):
            assert torch.equal(x, y)


def test_bf16_default_plan_gpt_shape(cottn, oracle):
    run_bwd(cottn, oracle, 2, 12, 1024, 64, "bf16", seed=1, segments=0)


def test_bf16_zero_rows_and_determinism(cottn, oracle):
    import torch

    def mutate(x):
        x["Q"][:, :, 10] = 0.0
        x["K"][:, :, 20:23] = 0.0
        x["V"][:, :, 20:23] = 0.0

    a = run_bwd(cottn, oracle, 1, 2, 150, 64, "bf16", seed=6, segments=2, mutate=mutate)
    b = run_bwd(cottn, oracle, 1, 2, 150, 64, "bf16", seed=6, segments=2, mutate=mutate)
    for x, y in zip(a, b):
        assert torch.isfinite(x.float()).all()
        assert torch.equal(x, y)


def test_bf16_zero_key_rows_with_values(cottn, oracle):
    """Key rows that are exactly zero while their value rows are not (Sec. 3.2 normalisation
    clamped at eps): they contribute nothing forward, their dK follows the x/eps rule without
    the projection, and nothing becomes NaN or Inf."""
    import torch

    def mutate(x):
        x["K"][:, :, 5] = 0.0
        x["K"][:, :, 70:72] = 0.0
        x["Q"][:, :, 64] = 0.0

    out = run_bwd(cottn, oracle, 2, 2, 200, 64, "bf16", seed=33, segments=2, mutate=mutate)
    for t in out:
        assert torch.isfinite(t.float()).all()

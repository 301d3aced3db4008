"""fp32 keeps its precision over its range: rows of very different magnitudes, every pair of widths the
fp32 kernels are built for in one way or the other, lengths around the ends of their 32-row steps.

Every element is compared with float64 against the size of what was added up for it (the same products
with all signs dropped), so that a small row next to large ones has to be as exact as they are.  A sum
over 32 features or tokens is rounded at most 48 times (six matrix products, each rounding eight times at
most on the way), so c = 48 (dk/32 + dv/32 + rows/32) + 20 roundings of 2^-24 bound the error.  Its root mean
square: roundings of independent sign add up to sqrt(c), and each is relative to a partial sum, which for
min(dk, dv) terms of independent sign is that root of what is added up without signs.  (Operands short of
their third part, 2^-18 off, would be 64 / sqrt(min(dk, dv)) of 2^-24 away.)"""
import numpy as np
import pytest

from helpers import to_device, to_host

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    yield b
    b.cottn_tune_segments(0)


def reference(Q, K, V, s, dO, causal):
    """Results in float64 and, under the same names, what was added up for them without signs."""
    rq, rk = (1.0 / np.linalg.norm(x, axis=-1, keepdims=True) for x in (Q, K))
    qh, kh = Q * rq, K * rk
    M = np.tril(np.ones((Q.shape[2], Q.shape[2]))) if causal else 1.0
    T = lambda x: np.swapaxes(x, -1, -2)
    sc = s[None, :, None, None]
    out = []
    for f in (lambda x: x, np.abs):
        q, k, v, g = f(qh), f(kh), f(V), f(dO)
        P, A = (q @ T(k)) * M, (g @ T(v)) * M
        sign = -1.0 if f(-1.0) < 0 else 1.0
        chain = lambda x, dx, r: sc * r * (dx + sign * x * (x * dx).sum(-1, keepdims=True))
        out.append({"O": sc * (P @ v), "dQ": chain(q, A @ k, rq), "dK": chain(k, T(A) @ q, rk),
                    "dV": sc * (T(P) @ g)})
    return out


@pytest.mark.parametrize("causal,segments", [(True, 1), (True, 3), (False, 2)])
@pytest.mark.parametrize("dk,dv", [(32, 32), (64, 64), (64, 128), (128, 64), (128, 32), (32, 128), (128, 128)])
@pytest.mark.parametrize("N", [31, 65, 97])
def test_rows_of_any_magnitude(cottn, N, dk, dv, causal, segments):
    rng = np.random.default_rng([N, dk, dv, causal])
    B, H = 1, 2
    x = {}
    for name, d in (("Q", dk), ("K", dk), ("V", dv), ("dO", dv)):
        size = 10.0 ** rng.uniform(-9, 9, (B, H, N, 1)) if name in ("V", "dO") else 10.0 ** rng.uniform(-4, 9, (B, H, N, 1))
        x[name] = (rng.standard_normal((B, H, N, d)) * size).astype(np.float32)
    s = rng.uniform(0.5, 1.5, H).astype(np.float32)
    Q, K, V, dO = (to_device(x[n], "f32") for n in ("Q", "K", "V", "dO"))
    sd = to_device(s, "f32")
    fwd, bwd = ((cottn.cottn_fwd_causal_dkdv, cottn.cottn_bwd_causal_dkdv) if causal
                else (cottn.cottn_fwd_bidir_dkdv, cottn.cottn_bwd_bidir_dkdv))
    cottn.cottn_tune_segments(segments)
    got = dict(zip(("O", "dQ", "dK", "dV"), (fwd(Q, K, V, sd),) + tuple(bwd(Q, K, V, sd, dO)[:3])))
    ref, size = reference(*(x[n].astype(np.float64) for n in ("Q", "K", "V")), s.astype(np.float64),
                          x["dO"].astype(np.float64), causal)
    c = 48 * (dk // 32 + dv // 32 + (N + 31) // 32) + 20
    for name in ref:
        e = np.abs(to_host(got[name]) - ref[name]) / size[name] / U
        rms, worst = float(np.sqrt((e ** 2).mean())), float(e.max())
        print("%s N%d %dx%d %s G%d: rms %.2f max %.1f of 2^-24" % (name, N, dk, dv, causal, segments, rms, worst), flush=True)
        assert worst <= c and rms <= (c / min(dk, dv)) ** 0.5, (name, rms, worst)

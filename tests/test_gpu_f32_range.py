"""fp32 keeps its precision over its range: rows of very different magnitudes, every pair of widths the
fp32 kernels are built for in one way or the other, lengths around the ends of their 32-row steps.

Every element is compared with float64 against the size of what was added up for it (the same products
with all signs dropped), so that a small row next to large ones has to be as exact as they are.  A sum
over 32 features or tokens is rounded at most 48 times (six matrix products, each rounding eight times at
most on the way), so c = 48 (dk/32 + dv/32 + rows/32) + 20 roundings of 2^-24 bound the error.  Its root mean
square: roundings of independent sign add up to sqrt(c), and each is relative to a partial sum, which for
min(dk, dv) terms of independent sign is that root of what is added up without signs.  (Operands short of
their third part, 2^-18 off, would be 64 / sqrt(min(dk, dv)) of 2^-24 away.)

Below 2^-110 and at the upper end the products in parts give way to whole ones, whose sums are rounded once
for every four terms: at most 8 times for 32 of them, less than the 48."""
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


WIDTHS = [(32, 32), (32, 64), (64, 64), (64, 128), (128, 64), (128, 32), (32, 128), (128, 128)]


def run(cottn, x, s, causal, segments):
    Q, K, V, dO = (to_device(x[n], "f32") for n in ("Q", "K", "V", "dO"))
    sd = to_device(s, "f32")
    fwd, bwd = ((cottn.cottn_fwd_causal_dkdv, cottn.cottn_bwd_causal_dkdv) if causal
                else (cottn.cottn_fwd_bidir_dkdv, cottn.cottn_bwd_bidir_dkdv))
    cottn.cottn_tune_segments(segments)
    return dict(zip(("O", "dQ", "dK", "dV"), (to_host(t) for t in (fwd(Q, K, V, sd),) + tuple(bwd(Q, K, V, sd, dO)[:3]))))


def compare(got, x, s, causal, what, terms):
    """Every element within the roundings that the docstring counts; terms: that make a sum at the least."""
    B, H, N, dk = x["Q"].shape
    dv = x["V"].shape[-1]
    ref, size = reference(*(x[n].astype(np.float64) for n in ("Q", "K", "V")), s.astype(np.float64), x["dO"].astype(np.float64), causal)
    c = 48 * (dk // 32 + dv // 32 + (N + 31) // 32) + 20
    for name in ref:
        # (a result, and each of the c sums on the way to it, is rounded to a multiple of 2^-149 at the least)
        e = np.abs(got[name] - ref[name]) / (size[name] * U + 2.0 ** -149)
        rms, worst = float(np.sqrt((e ** 2).mean())), float(e.max())
        print("%s %s %dx%d causal %s: rms %.2f max %.1f of 2^-24" % (what, name, dk, dv, causal, rms, worst), flush=True)
        assert worst <= c and rms <= (c / terms) ** 0.5, (name, rms, worst)


def drawn(dk, dv, N, seed):
    rng = np.random.default_rng(seed)
    x = {n: rng.standard_normal((1, 2, N, d)) for n, d in (("Q", dk), ("K", dk), ("V", dv), ("dO", dv))}
    return x, rng.uniform(0.5, 1.5, 2).astype(np.float32)


@pytest.mark.parametrize("causal,segments", [(True, 1), (True, 3), (True, 0), (False, 2)])
@pytest.mark.parametrize("dk,dv", WIDTHS)
def test_small_values(cottn, dk, dv, causal, segments):
    """Values, gradients of the output or one feature of the keys at magnitudes around and below 2^-110, in all rows
    or in one row of the last step."""
    N = 150
    for power in (-104, -109, -113, -118):   # (what a product in between is rounded to, 2^-149, stays below 2^-24 of it)
        for small in ("V", "dO", "K", "one row"):
            x, s = drawn(dk, dv, N, [dk, dv, -power])
            if small == "K":   # and queries that see nothing else
                x["K"][..., 0] *= 2.0 ** power
                x["Q"][..., 1:] = 0.0
            elif small == "one row":
                x["V"][:, :, N - 2] *= 2.0 ** power
            else:
                x[small] *= 2.0 ** power
            x = {k: v.astype(np.float32) for k, v in x.items()}
            compare(run(cottn, x, s, causal, segments), x, s, causal, "2^%d in %s" % (power, small),
                    1 if small == "K" else min(dk, dv))


@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 64), (128, 128)])
def test_small_values_in_even_shares(cottn, dk, dv):
    """Shares that go on into the next unit, small values in one row of each third unit; and padded."""
    import torch
    B, H, N = 8, 11, 333
    rng = np.random.default_rng([dk, dv, 3])
    x = {n: rng.standard_normal((B, H, N, d)) for n, d in (("Q", dk), ("K", dk), ("V", dv), ("dO", dv))}
    x["V"][:, ::3, 200] *= 2.0 ** -115
    x = {k: v.astype(np.float32) for k, v in x.items()}
    s = rng.uniform(0.5, 1.5, H).astype(np.float32)
    got = run(cottn, x, s, True, 0)
    compare(got, x, s, True, "shares", min(dk, dv))
    if dk == dv:
        lens = [333, 0, 200, 201, 1, 64, 32, 300]
        n, per_unit = torch.tensor(lens, dtype=torch.int32, device="cuda"), to_device(np.tile(s, (B, 1)), "f32")
        O = to_host(cottn.cottn_fwd_causal_varlen(*(to_device(x[k], "f32") for k in ("Q", "K", "V")), per_unit, n))
        for b, m in enumerate(lens):   # (a row sees the rows before it: those of the call above)
            assert (O[b, :, m:] == 0).all() and np.abs(O[b, :, :m] - got["O"][b, :, :m]).max(initial=0.0) <= 1e-5


@pytest.mark.parametrize("causal,segments", [(True, 1), (True, 3), (False, 2)])
@pytest.mark.parametrize("dk,dv", WIDTHS)
def test_largest_values(cottn, dk, dv, causal, segments):
    """One value in the last 0.4 % below the largest fp32 number, which no bfloat16 number reaches."""
    x, s = drawn(dk, dv, 150, [dk, dv, 7])
    x["Q"] *= 2.0 ** -6   # raw rows meet the state before their norms divide
    x["dO"] *= 2.0 ** -60
    x["V"][:, :, 70, 5] = 3.3995e38
    x = {k: v.astype(np.float32) for k, v in x.items()}
    s = s * np.float32(0.25)
    compare(run(cottn, x, s, causal, segments), x, s, causal, "largest", 1)   # (one value outweighs all others)


@pytest.mark.parametrize("dk,dv", [(32, 64), (64, 64), (128, 64), (128, 128)])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_infinity_stays_in_its_column(cottn, bad, dk, dv):
    """An infinite value is infinite with the sign of its weight in the 16 rows it sits in and not a number or
    infinite in its column from there on; other columns, and rows of earlier steps, do not see it."""
    N, j, col = 150, 70, 5
    x, s = drawn(dk, dv, N, [dk, dv, 9])
    x["V"][:, :, j, col] = bad
    x = {k: v.astype(np.float32) for k, v in x.items()}
    O = run(cottn, x, s, True, 1)["O"]
    clean = dict(x, V=np.where(np.isfinite(x["V"]), x["V"], 0.0).astype(np.float32))
    ref, size = reference(*(clean[n].astype(np.float64) for n in ("Q", "K", "V")), s.astype(np.float64), x["dO"].astype(np.float64), True)
    others = np.arange(dv) != col
    c = 48 * (dk // 32 + dv // 32 + (N + 31) // 32) + 20
    for rows, cols in ((slice(None), others), (slice(0, 64), slice(None))):
        e = np.abs(O - ref["O"])[:, :, rows][..., cols] / size["O"][:, :, rows][..., cols] / U
        assert e.max() <= c
    assert not np.isfinite(O[:, :, j:, col]).any()
    if np.isinf(bad):
        weight = np.einsum("bhnd,bhd->bhn", x["Q"].astype(np.float64), x["K"][:, :, j].astype(np.float64))[:, :, j:80]
        assert (O[:, :, j:80, col] == np.sign(weight) * bad).all()

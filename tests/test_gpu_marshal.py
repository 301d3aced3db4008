"""The two ways a call is marshalled (binding.py over ctypes, taken where a stream is named, and _marshal): the same kernels
with the same arguments, so the same bits, the same objects handed back, and the same refusals."""
import pytest

pytestmark = pytest.mark.gpu
B, H, N, DK, DV = 3, 2, 70, 64, 32


@pytest.fixture(scope="module")
def cottn():
    import paper_2409_18747_amd.binding as b
    return b


def calls(cottn, torch):
    """name -> (function, positional arguments, shapes of the results it allocates)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)

    def normal(*shape, dtype=torch.bfloat16):
        return torch.randn(*shape, device="cuda", generator=gen).to(dtype)
    Q, K, V, dO = (normal(B, H, N, DK) for _ in range(4))
    v, dv = normal(B, H, N, DV), normal(B, H, N, DV)
    s, su = torch.rand(H, device="cuda") + 0.5, torch.rand(B, H, device="cuda") + 0.5
    lens = torch.tensor([N, 1, 33], dtype=torch.int32, device="cuda")
    m, st = normal(H, dtype=torch.float32), normal(B, H, DK, DK, dtype=torch.float32)
    t = [normal(B, H, DK) for _ in range(3)]
    tv = normal(B, H, DV)
    row, rv = (B, H, N, DK), (B, H, N, DV)
    grads, gv = [row, row, row, (H,)], [row, row, rv, (H,)]
    out = {}
    for kind in ("causal", "bidir"):
        f = lambda name: getattr(cottn, "cottn_%s_%s" % (name, kind))
        out["fwd_" + kind] = f("fwd"), (Q, K, V, s), [row]
        out["bwd_" + kind] = f("bwd"), (Q, K, V, s, dO), grads
        out["fwd_%s_varlen" % kind] = getattr(cottn, "cottn_fwd_%s_varlen" % kind), (Q, K, V, su, lens), [row]
        out["bwd_%s_varlen" % kind] = getattr(cottn, "cottn_bwd_%s_varlen" % kind), (Q, K, V, su, lens, dO), [row, row, row, (B, H)]
        out["fwd_%s_dkdv" % kind] = getattr(cottn, "cottn_fwd_%s_dkdv" % kind), (Q, K, v, s), [rv]
        out["bwd_%s_dkdv" % kind] = getattr(cottn, "cottn_bwd_%s_dkdv" % kind), (Q, K, v, s, dv), gv
    out["fwd_causal_from_state"] = cottn.cottn_fwd_causal_from_state, (Q, K, V, s, st), [row]
    out["bwd_causal_from_state"] = cottn.cottn_bwd_causal_from_state, (Q, K, V, s, dO, st, st), grads
    out["step"] = (lambda q, k, w, x, **o: cottn.cottn_step(q, k, w, x, st.clone(), **o)), (*t, s), [(B, H, DK)]
    out["step_dkdv"] = ((lambda q, k, w, x, **o: cottn.cottn_step_dkdv(q, k, w, x, st[..., :DV].contiguous(), **o)),
                        (t[0], t[1], tv, s), [(B, H, DV)])
    out["scale_from_m_varlen"] = cottn.cottn_scale_from_m_varlen, (m, lens), [(B, H)]
    out["scale_backward_varlen"] = cottn.cottn_scale_backward_varlen, (m, lens, su), [(H,)]
    return out


NAMES = ["%s_%s%s" % (d, k, v) for k in ("causal", "bidir") for d in ("fwd", "bwd") for v in ("", "_varlen", "_dkdv")] + [
    "fwd_causal_from_state", "bwd_causal_from_state", "step", "step_dkdv", "scale_from_m_varlen", "scale_backward_varlen"]


@pytest.mark.parametrize("name", NAMES)
def test_both_ways_give_the_same(cottn, name):
    import torch
    call, args, shapes = calls(cottn, torch)[name]
    tried = []
    marshal = cottn._marshal

    class Watch:
        def __getattr__(self, what):
            def through(*a):
                r = getattr(marshal, what)(*a)
                tried.append(r is not None)
                return r
            return through
    listed = lambda r: list(r) if isinstance(r, tuple) else [r]
    ref = listed(call(*args, stream=torch.cuda.current_stream()))
    cottn._marshal = Watch()
    try:
        got = listed(call(*args))
        assert tried == [True]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            again = listed(call(*args))
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        assert tried == [True, True]
        for a, b, c, shape in zip(ref, got, again, shapes):
            assert a.shape == b.shape == shape and a.dtype == b.dtype
            assert torch.equal(a, b) and torch.equal(a, c)
        # results go where they are asked for
        into = {"fwd": ["O"], "bwd": ["dQ", "dK", "dV", "ds"], "ste": ["o"]}.get(name[:3], ["dm" if "backward" in name else "s"])
        given = [torch.full_like(a, 7) for a in ref]
        for a, b in zip(listed(call(*args, **dict(zip(into, given)))), given):
            assert a is b
        assert all(torch.equal(a, b) for a, b in zip(given, ref))
        # what _marshal does not take is for the other way, which says what is wrong
        with pytest.raises((ValueError, TypeError)):
            call(args[0].double(), *args[1:])
        if "scale" not in name:
            with pytest.raises(ValueError, match="contiguous"):
                call(torch.stack([args[0], args[0]], -1)[..., 0], *args[1:])
            with pytest.raises(cottn.CottnError) as e:
                call(*args, eps=-1.0)
            assert e.value.status == 7 and str(e.value).startswith("cottn_%s:" % name)
    finally:
        cottn._marshal = marshal


def test_modes_and_transforms_go_the_other_way(cottn):
    """A mode that watches torch calls sees the allocation it saw before; a batched tensor is refused as before."""
    import torch
    from torch.overrides import TorchFunctionMode
    call, args, _ = calls(cottn, torch)["fwd_causal"]

    class Count(TorchFunctionMode):
        seen = 0

        def __torch_function__(self, f, types, a=(), kw=None):
            Count.seen += f is torch.empty_like
            return f(*a, **(kw or {}))
    answers, marshal = [], cottn._marshal

    class Watch:
        def fwd(self, *a):
            answers.append(marshal.fwd(*a))
            return answers[-1]
    cottn._marshal = Watch()
    try:
        with Count():
            O = call(*args)
        assert Count.seen == 1 and answers == [None]
        with pytest.raises(RuntimeError, match="data pointer"):
            torch.vmap(lambda q: call(q, *args[1:]))(torch.stack([args[0], args[0]]))
        assert answers == [None, None]
    finally:
        cottn._marshal = marshal
    assert torch.equal(O, call(*args))


@pytest.mark.filterwarnings("ignore:Named tensors")
@pytest.mark.parametrize("name", ["fwd_causal", "bwd_bidir", "step"])
def test_results_keep_dimension_names(cottn, name):
    """Results of a tensor with named dimensions are allocated like it, names and all."""
    import torch
    call, args, shapes = calls(cottn, torch)[name]
    named = args[0].rename(*"BHNd"[:args[0].dim() - 1], "w")
    got, plain = (r if isinstance(r, tuple) else (r,) for r in (call(named, *args[1:]), call(*args)))
    for a, b, shape in zip(got, plain, shapes):
        assert torch.equal(a.rename(None), b) and b.names == (None,) * len(shape)
        assert a.names == (named.names if shape == args[0].shape else b.names)

"""What the C++ marshalling must not take: every tensor argument of every call that it makes, wrong in each way that the
kernels would index beyond (or behind a stride, in another type, in the host's memory).  The kernels take all sizes from the
first argument, and marshal.cpp checks for itself, so each check of it has a case here: it answers None, and binding.py refuses.  (Checks that
tell two GPUs apart are reached by host tensors only as far as the first of them.)

Nothing is launched, also where a check is missing: _marshal is bound to stand-ins that answer a status, and the library that
binding.py calls has only its size queries."""
import subprocess

import pytest

from test_gpu_marshal_threads import LAUNCHES

pytestmark = pytest.mark.gpu
DEVICE, ELSEWHERE = "cuda", "cpu"
B, H, N, DK, DV = 2, 3, 8, 64, 32
TAKEN = 5   # what the stand-ins answer

# shapes of the arguments: rows and tokens in the call's type, numbers in float32, lengths in int32, bytes in uint8
ROW, WIDE, TOKEN, NARROW = ("rows", (B, H, N, DK)), ("rows", (B, H, N, DV)), ("rows", (B, H, DK)), ("rows", (B, H, DV))
PER_HEAD, PER_UNIT, LENGTHS, BYTES = ("floats", (H,)), ("floats", (B, H)), ("lengths", (B,)), ("bytes", (4096,))
STATE, STATE_DKDV = ("floats", (B, H, DK, DK)), ("floats", (B, H, DK, DV))


def calls():
    """name -> (function of _marshal, {argument: kind and shape})"""
    out = {}
    for kind in ("causal", "bidir"):
        for variant, v, s, st in (("", ROW, PER_HEAD, STATE), ("_varlen", ROW, PER_UNIT, STATE), ("_dkdv", WIDE, PER_HEAD, STATE_DKDV)):
            first = {"Q": ROW, "K": ROW, "V": v, "s": s, **({"seq_len": LENGTHS} if variant == "_varlen" else {})}
            out["cottn_fwd_%s%s" % (kind, variant)] = "fwd", {**first, "O": v, "state": st, "workspace": BYTES}
            out["cottn_bwd_%s%s" % (kind, variant)] = "bwd", {**first, "dO": v, "dQ": ROW, "dK": ROW, "dV": v, "ds": s,
                                                              "fwd_workspace": BYTES, "workspace": BYTES}
    out["cottn_fwd_causal_from_state"] = "fwd", {"Q": ROW, "K": ROW, "V": ROW, "s": PER_HEAD, "state_in": STATE, "O": ROW, "state": STATE,
                                                 "workspace": BYTES}
    out["cottn_bwd_causal_from_state"] = "bwd", {"Q": ROW, "K": ROW, "V": ROW, "s": PER_HEAD, "dO": ROW, "state_in": STATE,
                                                 "rev_state_in": STATE, "dQ": ROW, "dK": ROW, "dV": ROW, "ds": PER_HEAD,
                                                 "rev_state_out": STATE, "fwd_workspace": BYTES, "workspace": BYTES}
    out["cottn_step"] = "step", {"q": TOKEN, "k": TOKEN, "v": TOKEN, "s": PER_HEAD, "state": STATE, "o": TOKEN}
    out["cottn_step_dkdv"] = "step", {"q": TOKEN, "k": TOKEN, "v": NARROW, "s": PER_HEAD, "state": STATE_DKDV, "o": NARROW}
    out["cottn_scale_from_m_varlen"] = "scale_varlen", {"m": PER_HEAD, "seq_len": LENGTHS, "s": PER_UNIT}
    out["cottn_scale_backward_varlen"] = "scale_varlen", {"m": PER_HEAD, "seq_len": LENGTHS, "ds": PER_UNIT, "dm": PER_HEAD}
    return out


def good(torch, spec):
    kind, shape = spec
    types = {"rows": torch.bfloat16, "floats": torch.float32, "lengths": torch.int32, "bytes": torch.uint8}
    return torch.ones(shape, device=DEVICE, dtype=types[kind])


def wrongs(torch, call, name, spec):
    """(what is wrong, the argument): each must be refused, next to others that are right."""
    kind, shape = spec
    t = good(torch, spec)
    sizes_given = name in ("Q", "q", "m") or (name in ("V", "v") and call.endswith("_dkdv"))   # the others follow these
    yield "elsewhere", t.to(ELSEWHERE)
    yield "strided", torch.stack([t, t], -1)[..., 0]
    if kind == "bytes":
        return
    yield "wider type", t.to(torch.float64 if kind != "lengths" else torch.int64)
    if not (kind == "rows" and name in ("Q", "q")):   # another type that the call has kernels for: the others must follow
        yield "other type of the same size", t.view({"rows": torch.float16, "floats": torch.int32, "lengths": torch.float32}[kind])
    if kind == "rows":
        yield "rank", t[0] if len(shape) > 3 else t.unsqueeze(0)
        for dim in range(len(shape)):
            if not sizes_given or (name in ("V", "v") and dim < len(shape) - 1):
                yield "shorter in dim %d" % dim, t.narrow(dim, 0, shape[dim] - 1).contiguous()
                yield "longer in dim %d" % dim, torch.cat([t, t], dim)
    elif name != "m" and not (name == "seq_len" and "scale" in call):
        yield "one element less", t.flatten()[1:].clone()
        yield "one element more", torch.cat([t.flatten(), t.flatten()[:1]])


def wrong_alike(torch, call, arguments, specs):
    """(what is wrong, all arguments): wrong ones that match each other."""
    def changed(names, change):
        return {**arguments, **{n: change(arguments[n]) for n in names}}
    yield "all elsewhere", changed(specs, lambda t: t.to(ELSEWHERE))
    rows = [n for n, (kind, _) in specs.items() if kind == "rows"]
    if not rows:
        return
    yield "all rows of a wider type", changed(rows, lambda t: t.double())
    yield "all rows of one dimension less", changed(rows, lambda t: t[0])
    yield "all rows of one dimension more", changed(rows, lambda t: t.unsqueeze(0))
    yield "all rows without the last dimension", changed(rows, lambda t: t[..., 0].contiguous())
    values = [n for n in rows if n in ("V", "O", "dO", "dV", "v", "o")]
    yield "values elsewhere", changed(values, lambda t: t.to(ELSEWHERE))
    yield "values of another type", changed(values, lambda t: t.half())
    yield "values of one dimension less", changed(values, lambda t: t[0])
    yield "values without the last dimension", changed(values, lambda t: t[..., 0].contiguous())
    yield "values of two for one", changed(values, lambda t: torch.stack([t, t], -1))
    for dim in range(arguments[values[0]].dim() - call.endswith("_dkdv")):
        yield "values shorter in dim %d" % dim, changed(values, lambda t: t.narrow(dim, 0, t.shape[dim] - 1).contiguous())
        yield "values longer in dim %d" % dim, changed(values, lambda t: torch.cat([t, t], dim))


@pytest.fixture(scope="module")
def stand_ins(tmp_path_factory):
    where = tmp_path_factory.mktemp("stand_ins")
    src, so = where / "stand_ins.cpp", where / "stand_ins.so"
    src.write_text('#include <cstddef>\nextern "C" {\nsize_t cottn_workspace_bytes_dkdv() { return 256; }\n'
                   + "".join("int cottn_%s() { return %d; }\n" % (n, TAKEN) for n in LAUNCHES) + "}\n")
    subprocess.run(["g++", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    return str(so)


@pytest.fixture
def cottn(stand_ins, monkeypatch):
    import paper_2409_18747_amd.binding as b
    real, marshal = b.lib, b._marshal
    answers = []

    class SizesOnly:
        def __getattr__(self, name):
            if "workspace_bytes" in name or name == "cottn_status_string":
                return getattr(real, name)

            def called(*_):
                raise AssertionError("%s was called" % name)
            return called

    class Watch:
        def __getattr__(self, what):
            def through(*a):
                answers.append(what)
                r = getattr(marshal, what)(*a)
                if r is None:
                    answers.append(None)
                return r
            return through
    monkeypatch.setattr(b, "lib", SizesOnly())
    monkeypatch.setattr(b, "_marshal", Watch())
    b.answers = answers
    marshal.bind(stand_ins, b.CottnError)
    yield b
    marshal.bind(b.library_path, b.CottnError)
    del b.answers


@pytest.mark.parametrize("call", sorted(calls()))
def test_refused(cottn, call):
    import torch
    function, specs = calls()[call]
    arguments = {name: good(torch, spec) for name, spec in specs.items()}
    with pytest.raises(cottn.CottnError) as e:
        getattr(cottn, call)(**arguments)
    assert e.value.status == TAKEN and cottn.answers == [function]   # all right: the C++ half makes the call
    tries = [("%s: %s" % (name, what), {**arguments, name: wrong})
             for name, spec in specs.items() for what, wrong in wrongs(torch, call, name, spec)]
    taken = []
    for what, wrong in tries + list(wrong_alike(torch, call, arguments, specs)):
        del cottn.answers[:]
        try:
            getattr(cottn, call)(**wrong)
        except (ValueError, TypeError):
            if cottn.answers == [function, None]:
                continue
        except (cottn.CottnError, AssertionError):
            pass
        taken.append(what)
    assert not taken

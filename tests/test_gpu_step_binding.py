"""The decode steps through the extension against the same calls through the checks in binding.py: the same bits for every way of
calling (given and new output, another output type, integers of other classes, a stream of one's own or a current one, a
Parameter), taken by the extension or left to the checks as it should be, and an error for every wrong call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
B, Hh, D = 3, 5, 64


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _args(kind):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda") / 8
    x = lambda: r(B, Hh, D).bfloat16()
    state = r(B, Hh, D, D)
    gamma = torch.rand(Hh, generator=gen, device="cuda")
    lam = torch.sigmoid(r(B, Hh, D) * 8 + 2).bfloat16()
    return {"plain": ("lasad_decode_step", dict(q=x(), k=x(), v=x(), gamma=gamma, state=state, grid_h=4, grid_w=6, pos=8)),
            "gated": ("lasad_decode_step_gated", dict(q=x(), lam=lam, v=x(), state=state, grid_h=4, grid_w=6, pos=8, k=x())),
            "layer": ("lasad_decode_step_layer", dict(q_pre=x(), z=x(), v=x(), state=state, grid_h=4, grid_w=6, pos=8,
                                                      norm_weight=r(Hh, D))),
            "rows": ("lasad_decode_step_rows", dict(q=x(), v=x(), state=state, grid_h=4, grid_w=6, k=x(), gamma=gamma,
                                                    pos_rows=torch.tensor([0, 7, 23], dtype=torch.int32, device="cuda")))}[kind]


def _run(lasad, monkeypatch, kind, change, slow):
    """result and new state, or the error; what the extension answered (None: left to the checks); what was returned"""
    import torch
    name, kw = _args(kind)
    answers, step = [], lasad._step
    with monkeypatch.context() as m:
        m.setattr(lasad, "_step", (lambda *a: None) if slow else (lambda *a: answers.append(step(*a)) or answers[-1]))
        change(kw)
        try:
            o = getattr(lasad, name)(**kw)
            torch.cuda.synchronize()
        except Exception as e:                               # noqa: BLE001 (whatever it is, it has to be the same)
            return (type(e), str(e)), answers, None
    assert kw.get("out") is None or o is kw["out"]
    return (o.dtype, o.float().cpu().numpy().tobytes(), kw["state"].cpu().numpy().tobytes()), answers, o


def _set(**new):
    return lambda kw: kw.update({k: f(kw) for k, f in new.items()})


def _first(kw):
    return kw["q"] if "q" in kw else kw["q_pre"]


# calls that the extension takes
FAST = {
    "as it is": _set(),
    "output given": _set(out=lambda kw: _first(kw).clone()),
    "fp32 output given": _set(out=lambda kw: _first(kw).float()),
    "whole query scale": _set(q_scale=lambda kw: 2),
    "stream": _set(stream=lambda kw: (__import__("torch").cuda.synchronize(), __import__("torch").cuda.Stream())[1]),
    "parameter": _set(v=lambda kw: __import__("torch").nn.Parameter(kw["v"], requires_grad=False)),
}
# calls that only the checks take
SLOW = {
    "fp32 output asked for": _set(out_dtype=lambda kw: __import__("torch").float32),
    "numpy integers": _set(grid_w=lambda kw: np.int64(kw["grid_w"])),
}
# wrong calls (the last two reach the library through the extension, which refuses them)
WRONG = {
    "every other row": _set(v=lambda kw: kw["v"].repeat(1, 2, 1)[:, ::2]),
    "other type": _set(v=lambda kw: kw["v"].float()),
    "half": _set(v=lambda kw: kw["v"].half()),
    "short value": _set(v=lambda kw: kw["v"][:2]),
    "flat state": _set(state=lambda kw: kw["state"].view(-1)),
    "bf16 state": _set(state=lambda kw: kw["state"].bfloat16()),
    "value in host memory": _set(v=lambda kw: kw["v"].cpu()),
    "output too small": _set(out=lambda kw: _first(kw)[:1].clone()),
    "output with gaps": _set(out=lambda kw: _first(kw).repeat(1, 1, 2)[..., ::2]),
    "text": _set(grid_w=lambda kw: "6"),
    "rule that is none": _set(boundary_mode=lambda kw: 7),
    "no grid": _set(grid_h=lambda kw: 0),
}
KINDS = ["plain", "gated", "layer", "rows"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("what", list(FAST) + list(SLOW))
def test_same_as_the_checks_in_python(lasad, monkeypatch, kind, what):
    fast, answers, o = _run(lasad, monkeypatch, kind, {**FAST, **SLOW}[what], False)
    slow, _, _ = _run(lasad, monkeypatch, kind, {**FAST, **SLOW}[what], True)
    assert o is not None and fast == slow
    if what in FAST:
        assert answers == [o] or (len(answers) == 1 and answers[0] is o)
    else:
        assert answers in ([], [None])


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("what", list(WRONG))
def test_wrong_calls_are_refused_the_same(lasad, monkeypatch, kind, what):
    fast, answers, o = _run(lasad, monkeypatch, kind, WRONG[what], False)
    slow, _, _ = _run(lasad, monkeypatch, kind, WRONG[what], True)
    assert o is None and fast == slow and issubclass(fast[0], (ValueError, TypeError, RuntimeError, AssertionError, __import__("ctypes").ArgumentError))
    if what in ("rule that is none", "no grid"):
        assert fast[0] is lasad.LasadError
    else:
        assert answers == [None]


@pytest.mark.parametrize("kind", KINDS)
def test_output_of_another_shape(lasad, monkeypatch, kind):
    """The layer's step takes any output with as many elements in a row, through the checks; the others do not."""
    change = _set(out=lambda kw: _first(kw).clone().view(B * Hh, D))
    fast, answers, o = _run(lasad, monkeypatch, kind, change, False)
    assert answers == [None] and fast == _run(lasad, monkeypatch, kind, change, True)[0]
    assert (o is not None) == (kind == "layer") and (o is not None or fast[0] is ValueError)


@pytest.mark.parametrize("kind", KINDS)
def test_the_current_stream_is_used(lasad, kind):
    """Under torch.cuda.stream: the step waits for what that stream does before it, with and without a given output."""
    import torch
    name, kw = _args(kind)
    want = getattr(lasad, name)(**kw)
    want_state = kw["state"].clone()
    for given in (False, True):
        name, kw = _args(kind)
        v = kw["v"]
        kw["v"] = torch.zeros_like(v)
        if given:
            kw["out"] = torch.empty_like(v)
        big = torch.ones(1 << 28, device="cuda")
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(8):                               # (about 2 ms of work)
                big.mul_(1.0)
            kw["v"].copy_(v)
            o = getattr(lasad, name)(**kw)
            after = o.clone()                                # (on the same stream: right without any synchronisation)
        torch.cuda.synchronize()
        assert torch.equal(after, want) and torch.equal(kw["state"], want_state)

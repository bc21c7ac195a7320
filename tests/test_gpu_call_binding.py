"""Forwards and backwards through the extension against the same calls through the checks in binding.py: the same bits for every way
of calling (layouts, given and new output, states, a stream that is current), taken by the extension or left to the checks as it
should be, and the same error for wrong calls."""
import pytest

pytestmark = pytest.mark.gpu
B, Hh, N, D = 2, 3, 1500, 64           # (long enough that the scalar-decay forward takes a workspace)


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _view(x, layout):
    import torch
    if layout == "bhnd":
        return x.transpose(1, 2).contiguous().transpose(1, 2)
    if layout == "rows":                                     # token rows of a larger buffer
        return torch.cat([x[:, :1], x, x[:, :2]], 1)[:, 1:N + 1]
    return x


def _args(kind, layout):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda") / 8
    x = lambda: _view(r(B, N, Hh, D).bfloat16(), layout)
    gamma = torch.rand(Hh, generator=gen, device="cuda") * 0.1 + 0.9
    lam = lambda: _view(torch.sigmoid(r(B, N, Hh, D) * 8 + 2).bfloat16(), layout)
    states = dict(state_in=r(B, Hh, D, D), state_out=torch.zeros((B, Hh, D, D), device="cuda"))
    at = dict(grid_h=50, grid_w=40, start_pos=7)
    return {"forward_chunked": lambda: dict(q=x(), k=x(), v=x(), gamma=gamma, **at, **states),
            "forward_gated": lambda: dict(q=x(), lam=lam(), v=x(), k=x(), **at, **states),
            "forward_layer": lambda: dict(q_pre=x(), z=x(), v=x(), norm_weight=r(Hh, D), **at, **states),
            "backward_chunked": lambda: dict(q=x(), k=x(), v=x(), d_o=x(), gamma=gamma, **at),
            "backward_gated": lambda: dict(q=x(), lam=lam(), v=x(), d_o=x(), **at),
            "backward_layer": lambda: dict(q_pre=x(), z=x(), v=x(), d_out=x(), norm_weight=r(Hh, D), **at)}[kind]()


KINDS = ["forward_chunked", "forward_gated", "forward_layer", "backward_chunked", "backward_gated", "backward_layer"]


def _run(lasad, monkeypatch, kind, kw, slow):
    import torch
    answers, fast = [], lasad._fast
    with monkeypatch.context() as m:
        m.setattr(lasad, "_fast", (lambda *a: None) if slow else (lambda *a: answers.append(fast(*a)) or answers[-1]))
        try:
            got = getattr(lasad, "lasad_" + kind)(**kw)
            torch.cuda.synchronize()
        except Exception as e:                               # noqa: BLE001 (whatever it is, it has to be the same)
            return (type(e), str(e)), answers
    got = list(got) if isinstance(got, tuple) else [got]
    if "state_out" in kw and kw["state_out"] is not None:
        got.append(kw["state_out"])
    return [(t.dtype, t.shape, t.stride(), t.float().cpu().numpy().tobytes()) if t is not None else None for t in got], answers


def _both(lasad, monkeypatch, kind, layout, change):
    out = []
    for slow in (False, True):
        kw = _args(kind, layout)
        change(kw)
        out.append(_run(lasad, monkeypatch, kind, kw, slow))
    assert out[0][0] == out[1][0]
    return out[0]


@pytest.mark.parametrize("layout", ["dense", "bhnd", "rows"])
@pytest.mark.parametrize("kind", KINDS)
def test_taken(lasad, monkeypatch, kind, layout):
    result, answers = _both(lasad, monkeypatch, kind, layout, lambda kw: None)
    assert isinstance(result, list) and answers[0] is not None


@pytest.mark.parametrize("kind", KINDS)
def test_options_taken(lasad, monkeypatch, kind):
    """no states and a given fp32 output; the tied key, no weight gradient"""
    import torch

    def change(kw):
        if kind.startswith("forward"):
            kw.update(state_in=None, state_out=None, out=torch.empty((B, N, Hh, D), device="cuda"))
            kw.pop("k", None) if kind == "forward_gated" else None
        elif kind == "backward_gated":
            kw.update(k=kw["v"].clone())
        elif kind == "backward_layer":
            kw.update(want_dweight=False, norm_weight=None)
    result, answers = _both(lasad, monkeypatch, kind, "dense", change)
    assert isinstance(result, list) and answers[0] is not None


@pytest.mark.parametrize("kind", KINDS)
def test_other_stream_current(lasad, monkeypatch, kind):
    import torch
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        result, answers = _both(lasad, monkeypatch, kind, "dense", lambda kw: None)
    assert isinstance(result, list) and answers[0] is not None


WRONG = {
    "strides differ": lambda kw: kw.update(v=_view(kw["v"], "bhnd")),
    "type differs": lambda kw: kw.update(v=kw["v"].float()),
    "short": lambda kw: kw.update(v=kw["v"][:, 1:]),
    "leaves the grid": lambda kw: kw.update(grid_h=30),
    "no rule": lambda kw: kw.update(boundary_mode=9),
    "text": lambda kw: kw.update(grid_w="40"),
}


@pytest.mark.parametrize("wrong", WRONG)
@pytest.mark.parametrize("kind", KINDS)
def test_wrong_calls(lasad, monkeypatch, kind, wrong):
    result, _ = _both(lasad, monkeypatch, kind, "dense", WRONG[wrong])
    assert isinstance(result, tuple)


def test_without_extension(lasad, monkeypatch):
    """These calls work where the extension is missing."""
    monkeypatch.setattr(lasad, "_steps", None)
    monkeypatch.setattr(lasad, "_has_extension", lambda: False)
    result, answers = _run(lasad, monkeypatch, "forward_chunked", _args("forward_chunked", "dense"), False)
    assert isinstance(result, list) and answers == [None]

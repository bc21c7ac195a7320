"""The decode steps through the extension against the same calls through the checks in binding.py: the same bits for every way of
calling (given and new output, another output type, integers of other classes, a stream of one's own, a Parameter), and the
same error for every wrong call."""
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


def _both(lasad, monkeypatch, kind, change):
    """(result or error, new state) with the extension and without it"""
    import torch
    res = []
    for slow in (False, True):
        name, kw = _args(kind)
        with monkeypatch.context() as m:
            if slow:
                m.setattr(lasad, "_step", lambda *a: None)
            change(kw)
            try:
                o = getattr(lasad, name)(**kw)
                torch.cuda.synchronize()
                res.append((o.dtype, o.float().cpu().numpy().tobytes(), kw["state"].cpu().numpy().tobytes()))
                assert kw.get("out") is None or o is kw["out"]
            except Exception as e:                           # noqa: BLE001 (whatever it is, it has to be the same)
                res.append((type(e), str(e)))
    return res


def _set(**new):
    return lambda kw: kw.update({k: f(kw) for k, f in new.items()})


def _first(kw):
    return kw["q"] if "q" in kw else kw["q_pre"]


CALLS = {
    "as it is": _set(),
    "output given": _set(out=lambda kw: _first(kw).clone()),
    "fp32 output given": _set(out=lambda kw: _first(kw).float()),
    "fp32 output asked for": _set(out_dtype=lambda kw: __import__("torch").float32),
    "numpy integers": _set(grid_w=lambda kw: np.int64(kw["grid_w"])),
    "whole query scale": _set(q_scale=lambda kw: 2),
    "stream": _set(stream=lambda kw: (__import__("torch").cuda.synchronize(), __import__("torch").cuda.Stream())[1]),
    "parameter": _set(v=lambda kw: __import__("torch").nn.Parameter(kw["v"], requires_grad=False)),
    "every other row": _set(v=lambda kw: kw["v"].repeat(1, 2, 1)[:, ::2]),
    "other type": _set(v=lambda kw: kw["v"].float()),
    "half": _set(v=lambda kw: kw["v"].half()),
    "short value": _set(v=lambda kw: kw["v"][:2]),
    "flat state": _set(state=lambda kw: kw["state"].view(-1)),
    "bf16 state": _set(state=lambda kw: kw["state"].bfloat16()),
    "output of another shape": _set(out=lambda kw: _first(kw).view(B * Hh, D)),
    "rule that is none": _set(boundary_mode=lambda kw: 7),
    "no grid": _set(grid_h=lambda kw: 0),
    "text": _set(grid_w=lambda kw: "6"),
}


@pytest.mark.parametrize("kind", ["plain", "gated", "layer", "rows"])
@pytest.mark.parametrize("what", list(CALLS))
def test_same_as_the_checks_in_python(lasad, monkeypatch, kind, what):
    fast, slow = _both(lasad, monkeypatch, kind, CALLS[what])
    assert fast == slow

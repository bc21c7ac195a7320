"""The binding without a GPU: what it loads for which call, and what it refuses before anything is launched."""
import sys

import pytest

from paper_2507_01652_amd import binding


@pytest.fixture
def no_extension(monkeypatch):
    import paper_2507_01652_amd as package
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_steps", None)
    monkeypatch.setitem(sys.modules, "paper_2507_01652_amd._steps", None)      # (its import fails)
    monkeypatch.delattr(package, "_steps", raising=False)


def test_only_the_decode_steps_need_the_extension(no_extension):
    assert binding.version().startswith("lasad")
    assert binding.lasad_backward_gated_workspace_bytes(1, 2, 64, 64) > 0


def test_a_missing_extension_says_how_to_build_it(no_extension):
    import torch
    x = torch.zeros(1, 2, 64)
    with pytest.raises(ImportError, match="paper_2507_01652_amd.build"):
        binding.lasad_decode_step(x, x, x, torch.ones(2), torch.zeros(1, 2, 64, 64), 2, 2, 0)


class _Library:
    """In the place of liblasad: a call that the checks let through is recorded, and nothing is launched."""
    def __init__(self):
        self.called = []

    def __getattr__(self, name):
        return lambda *a: self.called.append(name) or 0


B, Hh, D = 4, 2, 64


def _decode(kind, monkeypatch, pinned, **change):
    import torch
    library = _Library()
    monkeypatch.setattr(binding, "load", lambda: library)
    monkeypatch.setattr(binding, "_step", lambda *a: None)         # (as for everything that the extension does not take)
    if pinned:                                                     # (stands for memory that a kernel can reach)
        monkeypatch.setattr(torch.Tensor, "is_pinned", lambda self: True)
    x, state = torch.zeros(B, Hh, D), torch.zeros(B, Hh, D, D)
    stream = type("Stream", (), {"cuda_stream": 0})()
    kw = dict(state=state, grid_h=4, grid_w=4, stream=stream)
    if kind == "rows":
        kw.update(q=x, v=x, k=x, gamma=torch.ones(Hh), pos_rows=torch.zeros(B, dtype=torch.int32))
    elif kind == "layer":
        kw.update(q_pre=x, z=x, v=x, pos=0, norm_weight=torch.ones(Hh, D))
    elif kind == "gated":
        kw.update(q=x, lam=x, v=x, pos=0)
    else:
        kw.update(q=x, k=x, v=x, gamma=torch.ones(Hh), pos=0)
    kw.update(change)
    name = "lasad_decode_step" + ("" if kind == "plain" else "_" + kind)
    getattr(binding, name)(**kw)
    return library.called


KINDS = ["plain", "gated", "layer", "rows"]


@pytest.mark.parametrize("kind", KINDS)
def test_a_good_call_passes_the_checks_of_the_decode_steps(kind, monkeypatch):
    assert len(_decode(kind, monkeypatch, True)) == 1


@pytest.mark.parametrize("kind", KINDS)
def test_host_memory_is_refused_by_the_decode_steps(kind, monkeypatch):
    with pytest.raises(ValueError, match="GPU"):
        _decode(kind, monkeypatch, False)


def _cases():
    import torch
    few, bf16 = torch.zeros(1, Hh, D), torch.bfloat16
    for kind in KINDS:
        yield kind, dict(out=few)
        yield kind, dict(out=torch.zeros(B, Hh, 2 * D)[:, :, ::2])
    yield "layer", dict(norm_weight=torch.ones(D))
    yield "layer", dict(norm_weight=torch.ones(Hh, D, dtype=bf16))
    yield "layer", dict(norm_weight=torch.ones(D, Hh).t())
    yield "rows", dict(gamma=torch.ones(1))
    yield "rows", dict(gamma=torch.ones(Hh, dtype=bf16))
    yield "rows", dict(gamma=torch.ones(2 * Hh)[::2])


@pytest.mark.parametrize("kind,change", list(_cases()), ids=lambda x: x if isinstance(x, str) else next(iter(x)))
def test_what_a_decode_step_would_read_or_write_out_of_range_is_refused(kind, change, monkeypatch):
    with pytest.raises(ValueError):
        _decode(kind, monkeypatch, True, **change)

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

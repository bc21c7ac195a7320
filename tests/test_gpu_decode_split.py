"""Decode steps on both sides of the rules that give a state one or four wavefronts (256 | 257 and 2999 | 3000 states): every state
the same bits as in calls of 300 states at most and in calls of two, the outputs, whose sums run in another order, within the fp32
tolerance; sampled states against the oracle."""
import numpy as np
import pytest

from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu
D = 64


@pytest.mark.parametrize("n_states", [2, 256, 257, 2999, 3000])
@pytest.mark.parametrize("kind", ["scalar", "layer", "rows"])
def test_split(oracle, n_states, kind):
    import torch
    from paper_2507_01652_amd import binding as lasad
    gen = torch.Generator(device="cuda").manual_seed(n_states)
    r = lambda *s: torch.randn(s, generator=gen, device="cuda")
    q, k, v = (r(n_states, 1, D) / 8 for _ in range(3))
    z, w = r(n_states, 1, D) + 2, r(1, D) * 0.1 + 1
    s0 = r(n_states, 1, D, D) * 0.3
    gamma = torch.tensor([0.93], device="cuda")
    pos = torch.randint(-1, 24, (n_states,), generator=gen, device="cuda", dtype=torch.int32)       # -1: inactive

    def step(lo, hi):
        s = s0[lo:hi].clone()
        a = [x[lo:hi].contiguous() for x in (q, k, v, z)]
        if kind == "scalar":
            return lasad.lasad_decode_step(a[0], a[1], a[2], gamma, s, 4, 6, 8, q_scale=0.7), s
        if kind == "layer":
            return lasad.lasad_decode_step_layer(a[0], a[3], a[2], s, 4, 6, 8, norm_weight=w), s
        return lasad.lasad_decode_step_rows(a[0], a[2], s, pos[lo:hi].contiguous(), 4, 6, k=a[1], gamma=gamma, q_scale=0.7), s
    o, s = step(0, n_states)
    for size in (2, 300):
        for lo in range(0, n_states, size) if size == 300 else (0, n_states - 2):
            o1, s1 = step(lo, min(n_states, lo + size))
            assert torch.equal(s1, s[lo:lo + size])
            assert rel_err(o1.cpu().numpy(), o[lo:lo + size].cpu().numpy()) <= TOL["f32"]
    if kind == "scalar":
        i = [0, n_states // 2, n_states - 1]
        ref = s0[i].cpu().numpy().astype(np.float64)
        lam, _ = oracle.decay_factors(gamma.cpu().numpy(), 4, 6, 8, 1)
        ref_o = oracle.decode_step(*(x[i].cpu().numpy() for x in (q, k, v)), lam[:, 0], ref, q_scale=0.7)
        assert rel_err(o[i].cpu().numpy(), ref_o) <= TOL["f32"] and rel_err(s[i].cpu().numpy(), ref) <= TOL["f32"]

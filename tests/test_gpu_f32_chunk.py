"""The chunked fp32 scalar-decay forward at the edges of its tiles (16 tokens a chunk, 32 a barrier): lengths around one,
two and three of them, narrow and wide grids, a mid-row start and a carried state, strided inputs, all three boundary
rules, and gammas from 0 to 1 (no power of which is ever a reciprocal).  Tolerance: fp32 (helpers.TOL) against the fp64 oracle."""
import numpy as np
import pytest

from helpers import TOL, rel_err

pytestmark = pytest.mark.gpu
D = 64
GAMMA = np.array([0.0, 1e-30, 0.01, 0.5, 0.93, 0.9999, 1.0], dtype=np.float32)


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 97])
@pytest.mark.parametrize("W,mode,start", [(1, 0, 0), (5, 1, 7), (16, 0, 0), (23, 0, 17), (23, 2, 3), (70, 1, 40)])
def test_tile_edges(lasad, oracle, n, W, mode, start):
    import torch
    rng = np.random.default_rng(n + W)
    B, Hh = 2, len(GAMMA)
    x = rng.standard_normal((3, B, n + 2, Hh, D), dtype=np.float32) / 8
    s0 = (rng.standard_normal((B, Hh, D, D)) * 0.3).astype(np.float32)
    dev = torch.from_numpy(x).cuda()[:, :, 1:n + 1]                 # token rows of a larger buffer
    q, k, v = (np.ascontiguousarray(t[:, 1:n + 1]) for t in x)
    H = (start + n + W - 1) // W
    s1 = torch.empty((B, Hh, D, D), dtype=torch.float32, device="cuda")
    o = lasad.lasad_forward_chunked(dev[0], dev[1], dev[2], torch.from_numpy(GAMMA).cuda(), H, W, start_pos=start,
                                    boundary_mode=mode, q_scale=0.7, state_in=torch.from_numpy(s0).cuda(), state_out=s1)
    torch.cuda.synchronize()
    lam, _ = oracle.decay_factors(GAMMA, H, W, start, n, mode)
    ref, s_ref = oracle.forward_fullmask(q, k, v, lam, q_scale=0.7, s0=s0.astype(np.float64), want_state=True)
    assert rel_err(o.cpu().numpy(), ref) <= TOL["f32"]
    assert rel_err(s1.cpu().numpy(), s_ref) <= TOL["f32"]


@pytest.mark.parametrize("n", [1, 4, 5])
@pytest.mark.parametrize("Hh", [64, 65], ids=["128_sequences", "130"])
def test_few_tokens(lasad, oracle, n, Hh):
    """Both sides of the rule that leaves up to four tokens of few sequences to the token-serial kernel."""
    import torch
    rng = np.random.default_rng(n)
    q, k, v = (rng.standard_normal((2, n, Hh, D), dtype=np.float32) / 8 for _ in range(3))
    s0 = (rng.standard_normal((2, Hh, D, D)) * 0.3).astype(np.float32)
    gamma = rng.uniform(0.5, 1.0, Hh).astype(np.float32)
    up = lambda x: torch.from_numpy(x).cuda()
    s1 = torch.empty((2, Hh, D, D), dtype=torch.float32, device="cuda")
    o = lasad.lasad_forward_chunked(up(q), up(k), up(v), up(gamma), 3, 3, start_pos=1, state_in=up(s0), state_out=s1)
    lam, _ = oracle.decay_factors(gamma, 3, 3, 1, n, 0)
    ref, s_ref = oracle.forward_fullmask(q, k, v, lam, s0=s0.astype(np.float64), want_state=True)
    assert rel_err(o.cpu().numpy(), ref) <= TOL["f32"] and rel_err(s1.cpu().numpy(), s_ref) <= TOL["f32"]


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("t", [0, 1, 13, 15, 16, 30, 47])
def test_non_finite_value_stays_causal(lasad, oracle, t, bad):
    """A value that is no number reaches its own and later tokens of its channel only."""
    import torch
    rng = np.random.default_rng(t)
    n, W, Hh, c = 48, 70, 2, 21
    q, k, v = (rng.standard_normal((1, n, Hh, D), dtype=np.float32) / 8 for _ in range(3))
    gamma = np.array([0.9, 0.5], dtype=np.float32)
    lam, _ = oracle.decay_factors(gamma, 1, W, 0, n, 0)
    ref = oracle.forward_fullmask(q, k, v, lam)
    v[0, t, :, c] = bad
    up = lambda x: torch.from_numpy(x).cuda()
    o = lasad.lasad_forward_chunked(up(q), up(k), up(v), up(gamma), 1, W).cpu().numpy()
    assert not np.isfinite(o[0, t:, :, c]).any()
    o[0, t:, :, c] = ref[0, t:, :, c]
    assert rel_err(o, ref) <= TOL["f32"]


@pytest.mark.parametrize("n", [127, 128, 129, 160, 257, 1000])
@pytest.mark.parametrize("Hh", [2, 60, 70, 100, 128])
def test_dealt_to_several_workgroups(lasad, n, Hh):
    """Few sequences are dealt to two to four workgroups each, which form the state before their steps with the same
    operations: the same bits as in a call of so many sequences that each has one workgroup, an infinite value included, and
    with the final state written over the incoming one."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    many, W, start = 260, 19, 7
    x = torch.randn((3, 1, n, many, D), generator=gen, device="cuda") / 8
    x[2, 0, n // 2, 1, 3] = float("inf")
    s0 = torch.randn((1, many, D, D), generator=gen, device="cuda") * 0.3
    gamma = torch.rand(many, generator=gen, device="cuda")

    def call(h, in_place):
        a = x[:, :, :, :h].contiguous()
        si = s0[:, :h].contiguous()
        so = si if in_place else torch.empty_like(si)
        o = lasad.lasad_forward_chunked(a[0], a[1], a[2], gamma[:h].contiguous(), (start + n + W - 1) // W, W, start_pos=start,
                                        q_scale=0.7, state_in=si, state_out=so)
        torch.cuda.synchronize()
        return o, so
    o, s = call(many, False)
    for in_place in (False, True):
        got, st = call(Hh, in_place)
        assert torch.equal(got.view(torch.int32), o[:, :, :Hh].contiguous().view(torch.int32))
        assert torch.equal(st.view(torch.int32), s[:, :Hh].contiguous().view(torch.int32))

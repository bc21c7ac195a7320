"""The scalar-decay forward for few sequences (one to four workgroups each, chunks of 64 tokens): lengths around one, two and three
chunks and their query tiles of 16, counts of sequences on both sides of the rules that split a sequence by value channels, narrow and
wide grids, mid-row starts, carried states, strided inputs; calls long enough for the segment plan, on both sides of its rule; the
passes of a backward, which run reversed and add up the decay gradient.  Tolerance: bf16 (helpers.TOL) against the fp64
oracle; the bf16 output is the rounded fp32 one."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl
from helpers import TOL, both_outputs, rel_err, sample_pairs

pytestmark = pytest.mark.gpu
D = 64


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _draw(rng, *shape, scale=0.125):
    x = (rng.standard_normal(shape) * scale).astype(np.float32)
    return wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(x))


def _forward(lasad, oracle, B, Hh, n, W, start, mode, seed, pad=0, carry=True, lo=0.55):
    import torch
    rng = np.random.default_rng(seed)
    x = _draw(rng, 3, B, n + 2 * pad, Hh, D)
    dev = torch.from_numpy(x).cuda().bfloat16()[:, :, pad:pad + n]          # token rows of a larger buffer
    x = x[:, :, pad:pad + n]
    gamma = rng.uniform(lo, 1.0, Hh).astype(np.float32)
    s0 = (rng.standard_normal((B, Hh, D, D)) * 0.3).astype(np.float32) if carry else None
    s1 = torch.empty((B, Hh, D, D), dtype=torch.float32, device="cuda")
    H = (start + n + W - 1) // W
    o = both_outputs(lasad.lasad_forward_chunked, True, q=dev[0], k=dev[1], v=dev[2], gamma=torch.from_numpy(gamma).cuda(), grid_h=H,
                     grid_w=W, start_pos=start, boundary_mode=mode, q_scale=0.7,
                     state_in=torch.from_numpy(s0).cuda() if carry else None, state_out=s1).cpu().numpy()
    s1 = s1.cpu().numpy()
    for b, h in sample_pairs(B, Hh, 6, seed):
        lam, _ = oracle.decay_factors(gamma[h:h + 1], H, W, start, n, mode)
        one = [np.ascontiguousarray(t[b:b + 1, :, h:h + 1]) for t in x]
        ref, s_ref = oracle.forward_fullmask(*one, lam, q_scale=0.7, want_state=True,
                                             s0=s0[b:b + 1, h:h + 1].astype(np.float64) if carry else None)
        assert rel_err(o[b:b + 1, :, h:h + 1], ref) <= TOL["bf16"]
        assert rel_err(s1[b:b + 1, h:h + 1], s_ref) <= TOL["bf16"]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 63, 64, 65, 127, 128, 129, 200])
@pytest.mark.parametrize("W,mode,start", [(1, 0, 0), (5, 1, 7), (23, 0, 17), (64, 1, 0), (70, 2, 3), (200, 0, 60)])
def test_tile_edges(lasad, oracle, n, W, mode, start):
    _forward(lasad, oracle, 2, 5, n, W, start, mode, seed=n + W, pad=1)


@pytest.mark.parametrize("B,Hh", [(1, 1), (4, 16), (5, 13), (8, 16), (3, 43), (16, 16), (1, 257)])
@pytest.mark.parametrize("n", [70, 192])
def test_split_by_value_channels(lasad, oracle, B, Hh, n):
    """1, 64 | 65, 128 | 129, 256 | 257 sequences: four, two, one workgroup each, and the kernel for more."""
    _forward(lasad, oracle, B, Hh, n, 19, 3, 0, seed=Hh + n)


@pytest.mark.parametrize("B,Hh,n", [(1, 2, 1344), (1, 2, 1345), (4, 4, 1400), (1, 17, 1792), (1, 17, 1793), (5, 17, 1850), (1, 86, 1900), (2, 64, 2817), (3, 43, 1900)])
@pytest.mark.parametrize("carry", [False, True])
def test_segments(lasad, oracle, B, Hh, n, carry):
    """Calls with and without segments, next to the line between them, with a ragged last segment."""
    _forward(lasad, oracle, B, Hh, n, 37, 5, 0, seed=n, carry=carry, lo=0.9)


def test_state_in_place_over_segments(lasad):
    """With the final state written over the incoming one a call is not cut: the same result as with two buffers."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((1, 2000, 3, D), generator=gen, device="cuda").div_(8).bfloat16() for _ in range(3))
    gamma = torch.tensor([0.95, 0.99, 0.999], device="cuda")
    s = torch.randn((1, 3, D, D), generator=gen, device="cuda") * 0.3
    s1 = torch.empty_like(s)
    o = lasad.lasad_forward_chunked(q, k, v, gamma, 50, 40, state_in=s, state_out=s1, out_dtype=torch.float32)
    o2 = lasad.lasad_forward_chunked(q, k, v, gamma, 50, 40, state_in=s, state_out=s, out_dtype=torch.float32)
    assert rel_err(o2.cpu().numpy(), o.cpu().numpy()) <= TOL["bf16"] and rel_err(s.cpu().numpy(), s1.cpu().numpy()) <= TOL["bf16"]


def _backward(lasad, oracle, B, Hh, n, W, start, mode, lo=0.55):
    import torch
    rng = np.random.default_rng(n + Hh)
    q, k, v, g = (_draw(rng, B, n, Hh, D) for _ in range(4))
    gamma = rng.uniform(lo, 1.0, Hh).astype(np.float32)
    up = lambda x: torch.from_numpy(x).cuda().bfloat16()
    H = (start + n + W - 1) // W
    dq, dk, dv, dgam = both_outputs(lasad.lasad_backward_chunked, True, dtype_kw="grad_dtype", q=up(q), k=up(k), v=up(v), d_o=up(g),
                                    gamma=torch.from_numpy(gamma).cuda(), grid_h=H, grid_w=W, start_pos=start, boundary_mode=mode,
                                    q_scale=0.7)
    lam, cum = oracle.decay_factors(gamma, H, W, start, n, mode)
    rq, rk, rv, rlam = oracle.backward(q, k, v, lam, g, q_scale=0.7)
    for got, ref in ((dq, rq), (dk, rk), (dv, rv)):
        assert rel_err(got.cpu().numpy(), ref) <= TOL["bf16"]
    # the decay gradient is a small difference of large sums: their rounding is the floor (as in test_gpu_backward.py)
    rgam = oracle.dgamma(rlam, W, start, mode)
    E = (cum[1:] - cum[0]).astype(np.float64)
    terms = ((np.abs(q * rq).sum(axis=3) + np.abs(k * rk).sum(axis=3)) * E[None, :, None]).sum(axis=(0, 1)).max()
    assert np.abs(dgam.cpu().numpy() - rgam).max() <= TOL["bf16"] * np.abs(rgam).max() + 1e-6 * terms / float(gamma.min())


@pytest.mark.parametrize("B,Hh", [(1, 3), (1, 16), (1, 17), (2, 20), (1, 41), (5, 16), (3, 27), (5, 17), (2, 43), (9, 23)])
@pytest.mark.parametrize("n,W,start,mode", [(1, 5, 2, 0), (65, 9, 4, 1), (130, 17, 0, 0), (257, 33, 12, 2), (192, 33, 0, 0), (193, 30, 7, 1)])
def test_backward_passes(lasad, oracle, B, Hh, n, W, start, mode):
    """Three passes in one launch: 3 to 207 sequences, of four, two, one workgroup a pass (16 | 17, 40 | 41), those of a sequence on
    one XCD or not (80 | 81, 85 | 86), a workgroup walking several (with more than 192 tokens), another kernel; with the decay
    gradient."""
    _backward(lasad, oracle, B, Hh, n, W, start, mode)


@pytest.mark.parametrize("B,Hh", [(5, 16), (9, 23)])
def test_backward_small_gamma(lasad, oracle, B, Hh):
    """Heads for the fp32 recurrence among the others, one and up to three at a time in a workgroup, passes with and without a sum."""
    _backward(lasad, oracle, B, Hh, 200, 23, 3, 0, lo=0.2)


@pytest.mark.parametrize("B,Hh,n,W", [(3, 87, 192, 31), (3, 87, 193, 31), (5, 103, 320, 25), (9, 64, 769, 40)])
@pytest.mark.parametrize("lo", [0.3, 0.6])
def test_several_sequences_a_workgroup(lasad, oracle, B, Hh, n, W, lo):
    """More sequences than workgroups, one after the other with carried states; lo 0.3: among them some for the fp32 recurrence
    (gamma <= 0.5)."""
    _forward(lasad, oracle, B, Hh, n, W, 5, 0, seed=n, lo=lo)


def test_many_sequences_a_workgroup(lasad):
    """More than 64 for each of 256 workgroups: the same results as part by part."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(4)
    q, k, v = (torch.randn((1, 200, 16400, D), generator=gen, device="cuda", dtype=torch.bfloat16).div_(8) for _ in range(3))
    gamma = torch.rand((16400,), generator=gen, device="cuda") * 0.3 + 0.7
    o = lasad.lasad_forward_chunked(q, k, v, gamma, 10, 20)
    for i in (0, 8, 16390):
        part = lasad.lasad_forward_chunked(q[:, :, i:i + 10], k[:, :, i:i + 10], v[:, :, i:i + 10], gamma[i:i + 10].contiguous(), 10, 20)
        assert rel_err(o[:, :, i:i + 10].float().cpu().numpy(), part.float().cpu().numpy()) <= TOL["bf16"]


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("B,Hh", [(11, 9), (32, 16)])
def test_non_finite_values_stay_in_their_sequence(lasad, B, Hh, value):
    """A value of d_o that is not finite, in one sequence: every other sequence's gradients, and every other head's decay gradient, have
    the bits of the call without it (a workgroup walks several sequences and passes, with one accumulator for their sums)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, d_o = (torch.randn((B, 200, Hh, D), generator=gen, device="cuda").div_(8).bfloat16() for _ in range(4))
    gamma = torch.rand((Hh,), generator=gen, device="cuda") * 0.2 + 0.79
    clean = lasad.lasad_backward_chunked(q, k, v, d_o, gamma, 10, 20)
    d_o[0, 70, 0, 5] = value
    got = lasad.lasad_backward_chunked(q, k, v, d_o, gamma, 10, 20)
    assert not torch.isfinite(got[3][0]) and torch.equal(got[3][1:], clean[3][1:])
    for x, y in zip(got[:3], clean[:3]):
        x, y = (t.view(torch.int16).clone() for t in (x, y))
        x[0, :, 0] = y[0, :, 0] = 0
        assert torch.equal(x, y)


@pytest.mark.parametrize("n", [1, 65, 128])
@pytest.mark.parametrize("beyond", [-8, 8])
def test_widest_token_stride(lasad, n, beyond):
    """Token strides on both sides of the widest one whose rows, and the 384 past them that loads are asked for, lie within 2^31 bytes
    (beyond it another kernel takes the call): as with dense tensors."""
    import torch
    Hh = 2
    stride = ((1 << 31) // (n + 384) - 4) // 2 // 8 * 8 + beyond
    gen = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn((3, 1, n, Hh, D), generator=gen, device="cuda").div_(8).bfloat16()
    gamma = torch.tensor([0.9, 0.97], device="cuda")
    rows = torch.full(((n - 1) * stride + 4 * Hh * D,), float("nan"), dtype=torch.bfloat16, device="cuda")    # q, k, v, o: one row
    q, k, v, o = (rows.as_strided((1, n, Hh, D), (n * stride, stride, D, 1), i * Hh * D) for i in range(4))
    for t, y in zip((q, k, v), x):
        t.copy_(y)
    want = lasad.lasad_forward_chunked(*x, gamma, 16, 16)
    lasad.lasad_forward_chunked(q, k, v, gamma, 16, 16, out=o)
    assert rel_err(o.float().cpu().numpy(), want.float().cpu().numpy()) <= TOL["bf16"]
    assert all(torch.equal(t, y) for t, y in zip((q, k, v), x))

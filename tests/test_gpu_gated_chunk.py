"""The chunked vector-decay kernels at the edges of their 32-token tiles: lengths around one, two and three tiles, with
few sequences (a compute unit each: two loader groups) and with more than there are compute units (one loader group),
own key, tied key and fused layer, a mid-row start and a carried state; and a chunk beyond the range of the factorised
form in the first, a middle and the last tile.  Tolerance: the storage type's (helpers.TOL) against the fp64 oracle."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl
from helpers import TOL, both_outputs, gather_pairs, rel_err, sample_pairs

pytestmark = pytest.mark.gpu
D, W = 64, 23


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _check(lasad, oracle, n, B, Hh, form, start, seed, spike=None):
    import torch
    rng = np.random.default_rng(seed)
    draw = lambda scale, shift=0.0: wl.store_round(rng.standard_normal((B, n, Hh, D), dtype=np.float32) * np.float32(scale) + np.float32(shift), "bf16")
    q, v, k = draw(1.0 if form == "layer" else D ** -0.5), draw(D ** -0.5), draw(D ** -0.5)
    z = draw(1.0, 2.0)
    if spike is not None:
        z[:, spike, :, 5] = -90.0 if form == "layer" else -30.0     # a gate of 0 (as good as) in one channel of one token
    lam = wl.store_round(oracle.sigmoid(z).astype(np.float32), "bf16")
    s0 = (rng.standard_normal((B, Hh, D, D)) * 0.3).astype(np.float32)
    H = (start + n + W - 1) // W
    dev = lambda x: lasad.to_device(x, "bf16")
    s1 = torch.empty((B, Hh, D, D), dtype=torch.float32, device="cuda")
    kw = dict(grid_h=H, grid_w=W, start_pos=start, q_scale=0.7, state_in=torch.from_numpy(s0).cuda(), state_out=s1)
    if form == "layer":
        o = both_outputs(lasad.lasad_forward_layer, True, q_pre=dev(q), z=dev(z), v=dev(v), norm_eps=1e-5, **kw)
    else:
        o = both_outputs(lasad.lasad_forward_gated, True, q=dev(q), lam=dev(lam), v=dev(v), k=dev(k) if form == "own" else None, **kw)
    torch.cuda.synchronize()
    pairs = sample_pairs(B, Hh, 4, seed)
    at = lambda x: gather_pairs(x, pairs)
    s0s = np.stack([s0[b, h] for b, h in pairs])[None].astype(np.float64)
    if form == "layer":
        ref, s_ref = oracle.gated_layer(at(q), at(z), at(v), W, eps=1e-5, start_pos=start, q_scale=0.7, s0=s0s, want_state=True)
    else:
        ref, s_ref = oracle.gated_recurrent(at(q), at(lam), at(v), W, k=at(k) if form == "own" else None, start_pos=start,
                                            q_scale=0.7, s0=s0s, want_state=True)
    got_s = s1.cpu().numpy()
    assert rel_err(at(o.cpu().numpy()), ref) <= TOL["bf16"]
    assert rel_err(np.stack([got_s[b, h] for b, h in pairs])[None], s_ref) <= TOL["bf16"]


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 97])
@pytest.mark.parametrize("B,Hh", [(1, 3), (20, 13)], ids=["few", "many"])
@pytest.mark.parametrize("form", ["own", "tied", "layer"])
def test_tile_edges(lasad, oracle, n, B, Hh, form):
    _check(lasad, oracle, n, B, Hh, form, start=17, seed=n + B)


@pytest.mark.parametrize("spike", [3, 22, 40, 95])      # (22: the last token of a row, where the decay is off)
@pytest.mark.parametrize("B,Hh", [(1, 3), (20, 13)], ids=["few", "many"])
@pytest.mark.parametrize("form", ["tied", "layer"])
def test_range_exit(lasad, oracle, spike, B, Hh, form):
    _check(lasad, oracle, 97, B, Hh, form, start=0, seed=spike, spike=spike)


@pytest.mark.parametrize("n,B,Hh", [(768, 2, 3), (800, 1, 5), (929, 3, 4), (1023, 1, 2), (1300, 4, 20)])
@pytest.mark.parametrize("form", ["own", "tied", "layer"])
@pytest.mark.parametrize("spike", [None, 5, 400])
def test_segments(lasad, oracle, n, B, Hh, form, spike):
    """Few, long sequences: segments walked by different workgroups from states formed ahead of the walk."""
    _check(lasad, oracle, n, B, Hh, form, start=30, seed=n, spike=spike)


def _out_view(layout, B, n, Hh, dtype):
    import torch
    if layout == "head_major":
        return torch.full((B, Hh, n, D), 7.0, dtype=dtype, device="cuda").transpose(1, 2), None
    if layout == "padded":                             # rows of a wider buffer, which keeps what stands beside them
        buf = torch.full((B, n, Hh + 1, D + 8), 7.0, dtype=dtype, device="cuda")
        return buf[:, :, :Hh, :D], buf
    return torch.empty((B, n, Hh, D), dtype=dtype, device="cuda"), None


# Lengths that no number of equally long segments fits (1281, 1537: one token in the last chunk), from 4 to 16 segments;
# the incoming states pass through the output's rows, whatever its strides are
@pytest.mark.parametrize("n,Hh", [(1281, 12), (1537, 90), (2116, 24), (3844, 3)])
@pytest.mark.parametrize("layout,dtype", [("dense", "bf16"), ("head_major", "bf16"), ("padded", "bf16"), ("padded", "f32")])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_segment_forms(lasad, oracle, n, Hh, layout, dtype, mode):
    import torch
    rng = np.random.default_rng(n + mode)
    form = ["own", "tied", "layer"][(mode + n) % 3]
    q, k, v, z = (wl.store_round(rng.standard_normal((1, n, Hh, D), dtype=np.float32) * np.float32(s), "bf16")
                  for s in (1.0 if form == "layer" else 0.125, 0.125, 0.125, 1.0))
    lam = wl.store_round(oracle.sigmoid(z + 2.0).astype(np.float32), "bf16")
    s0 = (rng.standard_normal((1, Hh, D, D)) * 0.3).astype(np.float32)
    H, start = (30 + n + W - 1) // W, 30
    dev = lambda x: lasad.to_device(x, "bf16")
    def call(out):                                     # the final state replaces the incoming one
        state = torch.from_numpy(s0).cuda()
        kw = dict(start_pos=start, boundary_mode=mode, q_scale=0.7, state_in=state, state_out=state, out=out)
        if form == "layer":
            lasad.lasad_forward_layer(dev(q), dev(z), dev(v), H, W, norm_eps=1e-5, **kw)
        else:
            lasad.lasad_forward_gated(dev(q), dev(lam), dev(v), H, W, k=dev(k) if form == "own" else None, **kw)
        return out, state
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    view, buf = _out_view(layout, 1, n, Hh, t)
    out, state = call(view)
    out32, state32 = call(torch.empty((1, n, Hh, D), dtype=torch.float32, device="cuda"))
    assert torch.equal(out, out32.to(t)) and torch.equal(state, state32)
    pairs = sample_pairs(1, Hh, 3, n)
    at = lambda x: gather_pairs(x, pairs)
    rk = dict(start_pos=start, mode=mode, q_scale=0.7, s0=np.stack([s0[b, h] for b, h in pairs])[None].astype(np.float64), want_state=True)
    if form == "layer":
        ref, s_ref = oracle.gated_layer(at(q), at(z), at(v), W, eps=1e-5, **rk)
    else:
        ref, s_ref = oracle.gated_recurrent(at(q), at(lam), at(v), W, k=at(k) if form == "own" else None, **rk)
    assert rel_err(at(out32.cpu().numpy()), ref) <= TOL["bf16"]
    got = state.cpu().numpy()
    assert rel_err(np.stack([got[b, h] for b, h in pairs])[None], s_ref) <= TOL["bf16"]
    if buf is not None:
        assert (buf[:, :, Hh] == 7).all() and (buf[..., D:] == 7).all()


@pytest.mark.parametrize("n,B,Hh", [(97, 1, 3), (97, 20, 13), (1023, 1, 2)], ids=["few", "many", "segments"])
@pytest.mark.parametrize("row", [0, 1, -1])
def test_nan_gate_at_a_row_end(lasad, oracle, n, B, Hh, row):
    """Where the decay is off the gate still makes the key: a NaN logit there reaches its own and all later tokens.  (The
    kernels split operands in pairs of channels, so the state's row beside the channel's own may be NaN as well.)"""
    import torch
    rng = np.random.default_rng(n)
    q, z, v = (wl.store_round(rng.standard_normal((B, n, Hh, D), dtype=np.float32), "bf16") for _ in range(3))
    t, c = (row % (n // W)) * W + W - 1, 9
    pairs = sample_pairs(B, Hh, 2, n)
    at = lambda x: gather_pairs(x, pairs)
    ref = oracle.gated_layer(at(q), at(z), at(v), W, eps=1e-5)
    z[:, t, :, c] = np.nan
    dev = lambda x: lasad.to_device(x, "bf16")
    s1 = torch.empty((B, Hh, D, D), dtype=torch.float32, device="cuda")
    o = lasad.lasad_forward_layer(dev(q), dev(z), dev(v), -(-n // W), W, norm_eps=1e-5, state_out=s1, out_dtype=torch.float32)
    o, s1 = o.cpu().numpy(), s1.cpu().numpy()
    assert np.isnan(o[:, t:]).all() and np.isfinite(o[:, :t]).all()
    assert np.isnan(s1[:, :, c]).all() and np.isfinite(np.delete(s1, (c, c ^ 1), axis=2)).all()
    assert rel_err(at(o)[:, :t], ref[:, :t]) <= TOL["bf16"]
    # without the norm nothing but the state carries it into the gradient of the query
    g = lasad.lasad_backward_layer(dev(q), dev(z), dev(v), dev(v), -(-n // W), W, norm_eps=-1.0, grad_dtype=torch.float32)
    dq = g[0].cpu().numpy()
    assert np.isnan(dq[:, t:, :, c]).all() and np.isfinite(np.delete(dq, (c, c ^ 1), axis=3)[:, :t]).all()

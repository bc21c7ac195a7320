"""The two walks of the vector-decay backward (dq, then dv, dk and the decay gradient in reversed order) on both sides of
the rules that choose them: 81 sequences and more (fewer take three passes when they are short, and so do up to 160 of 33 to 64
tokens), segments with a workgroup each up to 128 sequences of 449 tokens and more, parts of a sequence beyond that.  Lengths
around the 32-token tiles, one and two loader groups of the dq walk, row ends on and off the bounds, carried states, all three
key forms, bf16 and fp32 gradients, views and strides of all kinds, and a gate beyond the range of the factorised form (the
token-serial walk of that part, and no states kept by it).  A few sequences of each call against the
fp64 oracle at the storage type's tolerance (helpers.TOL)."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl
from helpers import TOL, both_outputs, rel_err

pytestmark = pytest.mark.gpu
D = 64


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _inputs(n, Hh, seed):
    rng = np.random.default_rng(seed)
    q, v, g, k = (wl.store_round(rng.standard_normal((1, n, Hh, D), dtype=np.float32) / np.float32(8), "bf16") for _ in range(4))
    return rng, q, v, g, k, wl.gate_inputs((1, n, Hh, D), "bf16", seed + 1)


def _check(lasad, oracle, n, Hh, own, W, start=0, spike=None, carried=False):
    import torch
    rng, q, v, g, k, lam = _inputs(n, Hh, 7 * n + Hh)
    pick, c = [0, Hh // 2, Hh - 1], 5
    spikes = [] if spike is None else list(np.atleast_1d(spike))
    for t in spikes:                                         # (several: beyond the range together)
        lam[:, t, Hh // 2, c] = 2.0 ** (-120 if len(spikes) == 1 else -60)
    if not own:
        k = None
    s0, ds = ((rng.standard_normal((1, Hh, D, D)) * 0.3).astype(np.float32) for _ in range(2))
    dev = lambda x: None if x is None else lasad.to_device(x, "bf16")
    sub = lambda x: None if x is None else np.ascontiguousarray(x[:, :, pick])
    H = (start + n + W - 1) // W
    kw = dict(q=dev(q), lam=dev(lam), v=dev(v), d_o=dev(g), grid_h=H, grid_w=W, k=dev(k), start_pos=start, q_scale=0.7)
    if carried:
        up = lambda x: torch.from_numpy(x).cuda()
        got = lasad.lasad_backward_gated_carried(state_in=up(s0), d_state_out=up(ds), grad_dtype=torch.float32, **kw)
        ref = oracle.gated_backward_carried(sub(q), sub(lam), sub(v), sub(g), W, k=sub(k), start_pos=start, q_scale=0.7,
                                            s0=s0[:, pick], d_state=ds[:, pick])
    else:
        got = both_outputs(lasad.lasad_backward_gated, True, dtype_kw="grad_dtype", **kw)      # (bf16: the fp32 ones rounded)
        ref = oracle.gated_backward(sub(q), sub(lam), sub(v), sub(g), W, k=sub(k), start_pos=start, q_scale=0.7)
    state = len(got) - 1 if carried else -1
    for i, (a, r) in enumerate(zip(got, [x for x in ref if x is not None])):
        a = a.float().cpu().numpy()
        a, r = (a[:, pick] if i == state else a[:, :, pick]), np.array(r)
        if i == 1 and spikes:                                # a quotient by the tiny gate, and what it hides of the steps before
            a[:, :spikes[-1] + 1, 1, c] = r[:, :spikes[-1] + 1, 1, c] = 0
        assert rel_err(a, r) <= TOL["bf16"], (i, rel_err(a, r))


@pytest.mark.parametrize("n,Hh", [(1, 81), (31, 81), (33, 81), (64, 81), (97, 81), (449, 81), (513, 100), (545, 129), (600, 129), (640, 257)])
@pytest.mark.parametrize("own", [False, True], ids=["tied", "own"])
def test_walks(lasad, oracle, n, Hh, own):
    _check(lasad, oracle, n, Hh, own, W=16, start=n % 16)


@pytest.mark.parametrize("n,Hh", [(40, 81), (520, 100), (1000, 12), (577, 129)])
@pytest.mark.parametrize("own", [False, True], ids=["tied", "own"])
def test_carried(lasad, oracle, n, Hh, own):
    _check(lasad, oracle, n, Hh, own, W=23, start=5, carried=True)


@pytest.mark.parametrize("n,Hh,spike", [(97, 81, 40), (520, 100, 3), (520, 100, 300), (520, 100, 519), (577, 129, 100), (577, 129, 570)])
@pytest.mark.parametrize("carried", [False, True])
def test_range_exit(lasad, oracle, n, Hh, spike, carried):
    _check(lasad, oracle, n, Hh, True, W=23, spike=spike, carried=carried)


@pytest.mark.parametrize("n,Hh,spike", [(97, 81, [0]), (97, 81, [31, 32]), (520, 100, [0]), (520, 100, [287, 288]), (577, 129, [63, 64])],
                         ids=["dq", "reversed", "dq_of_a_segment", "reversed_of_a_segment", "reversed_with_parts"])
@pytest.mark.parametrize("carried", [False, True])
def test_range_exit_of_one_walk(lasad, oracle, n, Hh, spike, carried):
    """The first token's gate is in no product of the reversed order; two gates on both sides of a tile's bound are in one
    product only there.  What the other walk made is then kept, or (dq) made again."""
    _check(lasad, oracle, n, Hh, True, W=23, spike=spike, carried=carried)


def test_range_exit_takes_no_longer_than_the_passes(lasad):
    """Every gate leaves the range: 96 sequences, on the walks, against 80, whose three passes have a compute unit each (1.8
    times their time; with the token-serial walks one after the other 3.1)."""
    import torch

    def time(Hh, n=256, W=16):
        gen = torch.Generator(device="cuda").manual_seed(Hh)
        x = [torch.randn((1, n, Hh, D), generator=gen, device="cuda").bfloat16() for _ in range(5)]
        lam = torch.sigmoid(x[4].float() - 10).bfloat16()
        best = 1e30
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                lasad.lasad_backward_gated(x[0], lam, x[1], x[2], n // W, W, k=x[3])
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    assert time(96) <= 2.3 * time(80)


# dq's second loader group, up to 256 workgroups; with one, chunks go two at a time, and the second may be empty.
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 97])
@pytest.mark.parametrize("Hh", [256, 257], ids=["two_loader_groups", "one"])
@pytest.mark.parametrize("own", [False, True], ids=["tied", "own"])
def test_loader_groups_of_dq(lasad, oracle, n, Hh, own):
    _check(lasad, oracle, n, Hh, own, W=16, start=n % 16)


@pytest.mark.parametrize("n,spike", [(33, 3), (65, 64), (97, 40), (97, 70), (128, 127)])
@pytest.mark.parametrize("carried", [False, True])
def test_range_exit_with_one_loader_group(lasad, oracle, n, spike, carried):
    _check(lasad, oracle, n, 340, True, W=23, spike=spike, carried=carried)


# two and three segments of two parts each, the states at their bounds and a range left in either segment
@pytest.mark.parametrize("n,Hh,first,last", [(833, 100, 100, 700), (705, 128, 300, 704), (1444, 81, 5, 1300)])
@pytest.mark.parametrize("how", ["whole", "carried", "first", "last", "carried_first", "carried_last"])
def test_segments_with_parts(lasad, oracle, n, Hh, first, last, how):
    spike = first if how.endswith("first") else last if how.endswith("last") else None
    _check(lasad, oracle, n, Hh, True, W=23, start=2, spike=spike, carried=how.startswith("carried"))


def _views(form, B, n, Hh, count, dtype):
    """`count` tensors [B, n, Hh, D] with one set of strides"""
    import torch
    new = lambda *shape: torch.empty(shape, dtype=dtype, device="cuda")
    if form == "projection":                                 # side by side in the rows of one tensor
        return list(new(B, n, count, Hh, D).unbind(2))
    if form == "padded_rows":                                # heads apart, a row longer than its heads
        return [x[..., :Hh, 8:8 + D] for x in (new(B, n, Hh + 1, D + 16) for _ in range(count))]
    return [x.transpose(1, 2) for x in (new(B, Hh, n, D) for _ in range(count))]       # head by head


def _on_views(inputs, B, n, Hh, form, grad_form, n_grads, dtype):
    """the inputs on views of one form, and gradient tensors of another"""
    views = _views(form, B, n, Hh, len(inputs), inputs[0].dtype)
    for x, y in zip(views, inputs):
        x.copy_(y)
    grads = _views(grad_form, B, n, Hh, n_grads, dtype)
    assert grads[0].stride() != inputs[0].stride() and views[0].stride() != inputs[0].stride()
    return views, grads


@pytest.mark.parametrize("B,n,Hh", [(2, 97, 70), (1, 833, 100), (3, 64, 90)], ids=["whole", "segments", "one_loader_group"])
@pytest.mark.parametrize("form,grad_form", [("projection", "heads"), ("heads", "projection"), ("padded_rows", "padded_rows")])
@pytest.mark.parametrize("own", [False, True], ids=["tied", "own"])
def test_views(lasad, B, n, Hh, form, grad_form, own):
    """The same bits as for dense tensors (which the other tests hold to the oracle), in both types of the gradients."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    new = lambda: (torch.randn((B, n, Hh, D), generator=gen, device="cuda") / 8).bfloat16()
    q, v, g, k = new(), new(), new(), new()
    lam = torch.sigmoid(new().float() * 8 + 2).bfloat16()
    W = 16
    kw = dict(grid_h=(n + W) // W + 1, grid_w=W, start_pos=5, q_scale=0.7)
    for dtype in (torch.bfloat16, torch.float32):
        want = lasad.lasad_backward_gated(q, lam, v, g, k=k if own else None, grad_dtype=dtype, **kw)
        ins, grads = _on_views([q, lam, v, g] + ([k] if own else []), B, n, Hh, form, grad_form, len(want), dtype)
        got = lasad.lasad_backward_gated(*ins[:4], k=ins[4] if own else None, grads=tuple(grads), **kw)
        for i, (a, b) in enumerate(zip(got, want)):
            assert torch.equal(a, b), (dtype, i)


@pytest.mark.parametrize("B,n,Hh", [(2, 97, 70), (1, 833, 100)], ids=["whole", "segments"])
@pytest.mark.parametrize("form,grad_form", [("projection", "heads"), ("heads", "padded_rows")])
def test_views_of_the_layer(lasad, B, n, Hh, form, grad_form):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    new = lambda: torch.randn((B, n, Hh, D), generator=gen, device="cuda").bfloat16()
    q, z, v, g = new(), new() + 2, new(), new()
    w = 1 + 0.1 * torch.randn((Hh, D), generator=gen, device="cuda")
    W = 16
    kw = dict(grid_h=(n + W) // W + 1, grid_w=W, start_pos=5, norm_weight=w)
    want = lasad.lasad_backward_layer(q, z, v, g, **kw)
    ins, grads = _on_views([q, z, v], B, n, Hh, form, grad_form, 3, torch.bfloat16)
    d_out = _views(grad_form, B, n, Hh, 1, torch.bfloat16)[0].copy_(g)       # strides of its own
    got = lasad.lasad_backward_layer(*ins, d_out, grads=tuple(grads), **kw)
    for i, (a, b) in enumerate(zip(got, want)):
        assert torch.equal(a, b), i


@pytest.mark.parametrize("n", [65, 97, 129])
@pytest.mark.parametrize("what", ["inputs", "gradients"])
def test_token_strides_that_the_walks_refuse(lasad, oracle, n, what):
    """A lane's offsets in a chunk of the walks are 32 bits; the three passes, with one loader group here, take a token stride of
    2^25 elements, and any of the gradients."""
    import torch
    Hh, W, far = 161, 16, 1 << 25
    rng, q, v, g, k, lam = _inputs(n, Hh, n)
    pick = [0, Hh // 2, Hh - 1]
    sub = lambda x: np.ascontiguousarray(x[:, :, pick])
    ins = [lasad.to_device(x, "bf16") for x in (q, lam, v, g, k)]
    grads = [torch.empty((1, n, Hh, D), device="cuda") for _ in range(4)]
    side = ins if what == "inputs" else grads
    base = torch.empty((n - 1) * far + len(side) * Hh * D, dtype=side[0].dtype, device="cuda")
    apart = [base.as_strided((1, n, Hh, D), (Hh * D, far, D, 1), i * Hh * D) for i in range(len(side))]
    for x, y in zip(apart, side):
        x.copy_(y)
    if what == "inputs":
        ins = apart
    else:
        grads = apart
    got = lasad.lasad_backward_gated(*ins[:4], (n + W - 1) // W, W, k=ins[4], grads=tuple(grads))
    for i, (a, r) in enumerate(zip(got, oracle.gated_backward(sub(q), sub(lam), sub(v), sub(g), W, k=sub(k)))):
        a = a[:, :, pick].cpu().numpy()
        assert rel_err(a, r) <= TOL["bf16"], (i, rel_err(a, r))


# The last call for the three passes and the first for the walks, and the other way round.
@pytest.mark.parametrize("n,Hh", [(32, 128), (33, 128), (33, 129), (64, 128), (65, 128), (640, 33), (641, 33), (704, 24), (705, 24),
                                  (768, 48), (769, 48), (896, 49), (897, 49), (1088, 72), (1089, 72)])
def test_both_sides_of_the_lines(lasad, oracle, n, Hh):
    _check(lasad, oracle, n, Hh, True, W=16, start=3)


@pytest.mark.parametrize("n,Hh", [(32, 128), (32, 129), (64, 160), (64, 161), (40, 256), (40, 257), (33, 321), (97, 128), (97, 129)])
def test_both_sides_of_the_lines_with_carried_states(lasad, oracle, n, Hh):
    _check(lasad, oracle, n, Hh, False, W=16, start=3, carried=True)


def test_the_decay_gradient_is_a_rounded_quotient(lasad):
    """One token that adds nothing to the state: its decay gradient is (lambda s) / lambda, s a power of two, without an error."""
    import torch
    Hh = 200
    zero = torch.zeros((1, 1, Hh, D), dtype=torch.bfloat16, device="cuda")
    lam = (torch.arange(1, Hh * D + 1, device="cuda").reshape(1, 1, Hh, D) / (Hh * D + 1)).bfloat16()
    s0, ds = (torch.zeros((1, Hh, D, D), device="cuda") for _ in range(2))
    s0[..., 0] = 2.0 ** (torch.arange(D, device="cuda") % 7 - 3)
    ds[..., 0] = 1
    dlam = lasad.lasad_backward_gated_carried(zero, lam, zero, zero, 2, 8, k=zero.clone(), state_in=s0, d_state_out=ds,
                                              grad_dtype=torch.float32)[1]
    assert torch.equal(dlam[0, 0], s0[0, :, :, 0])


@pytest.mark.parametrize("n,Hh,mode", [(33, 81, 0), (33, 89, 1), (100, 81, 1), (513, 96, 0), (580, 129, 2), (1000, 12, 1)])
def test_layer(lasad, oracle, n, Hh, mode):
    import torch
    W = 16
    rng, q, v, g, z, _ = _inputs(n, Hh, n + Hh)
    q, z = wl.store_round(q * 8, "bf16"), wl.store_round(z * 8 + 2, "bf16")
    w = (1 + 0.1 * rng.standard_normal((Hh, D))).astype(np.float32)
    pick = [0, Hh // 2, Hh - 1]
    sub = lambda x: np.ascontiguousarray(x[:, :, pick])
    dev = lambda x: lasad.to_device(x, "bf16")
    got = both_outputs(lasad.lasad_backward_layer, True, dtype_kw="grad_dtype", q_pre=dev(q), z=dev(z), v=dev(v), d_out=dev(g),
                       grid_h=(n + W - 1) // W, grid_w=W, norm_weight=torch.from_numpy(w).cuda(), boundary_mode=mode)
    ref = oracle.gated_layer_backward(sub(q), sub(z), sub(v), sub(g), W, mode=mode, norm_weight=w[pick])
    for i in range(3):
        a = got[i].float().cpu().numpy()[:, :, pick]
        assert rel_err(a, ref[i]) <= TOL["bf16"], (i, rel_err(a, ref[i]))
    assert rel_err(got[3].cpu().numpy()[pick], ref[3]) <= TOL["bf16"]


@pytest.mark.parametrize("n,Hh", [(1024, 12), (1024, 81), (2304, 12)])
def test_room_for_fewer_bounds(lasad, oracle, n, Hh):
    """A workspace sized for a longer call may hold fewer bounds: then there are fewer segments, and without any the kernel that
    is fastest so.  Right at every size, and never more than 2.2 times the time (the three passes of 12 long sequences, 1.4 and
    1.9 of the segments'; walks that are not cut take 2.3 and 3.6 times as long)."""
    import torch
    rng, q, v, g, k, lam = _inputs(n, Hh, n + Hh)
    pick, W = [0, Hh // 2, Hh - 1], 16
    sub = lambda x: np.ascontiguousarray(x[:, :, pick])
    dev = lambda x: lasad.to_device(x, "bf16")
    kw = dict(q=dev(q), lam=dev(lam), v=dev(v), d_o=dev(g), grid_h=(n + W - 1) // W, grid_w=W, k=dev(k), grad_dtype=torch.float32)
    ref = oracle.gated_backward(sub(q), sub(lam), sub(v), sub(g), W, k=sub(k))
    full, least = lasad.lasad_backward_gated_workspace_bytes(1, Hh, n, D), 2 * n * Hh * D * 4 + Hh * 8 * D * 4

    def time(ws):
        best = 1e30
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                lasad.lasad_backward_gated(**kw, workspace=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        return best

    whole = time(torch.empty(full, dtype=torch.uint8, device="cuda"))
    for room in (7, 5, 3, 1, 0):
        ws = torch.empty(least + (full - least) * room // 8 // 256 * 256, dtype=torch.uint8, device="cuda")
        for i, (a, r) in enumerate(zip(lasad.lasad_backward_gated(**kw, workspace=ws), ref)):
            a = a.cpu().numpy()[:, :, pick]
            assert rel_err(a, r) <= TOL["bf16"], (room, i, rel_err(a, r))
        assert time(ws) <= 2.2 * whole, room

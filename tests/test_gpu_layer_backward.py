"""GPU parity of the fused layer's backward (lasad_backward_layer: chain rule through the normalisation, the
vector-decay recurrence with the tied key and the two activations of Algorithm 1) against the oracle's
gated_layer_backward, element by element on seeded inputs: fp32 results against the bare tolerance; results
stored as bf16 must be those fp32 results rounded, bit for bit (helpers.both_outputs)."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl
from helpers import TOL, both_outputs, rel_err, sample_pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _inputs(B, n, Hh, d, dtype, seed):
    """Pre-activation query ~ N(0, 1), gate logits ~ N(2, 1), values ~ N(0, 1)/sqrt(d) (the forward layer tests'
    recipe) and an output gradient ~ N(0, 1)/sqrt(d); all rounded to the storage type."""
    rng = np.random.default_rng(seed)
    shape = (B, n, Hh, d)
    q = wl.store_round(rng.standard_normal(shape, dtype=np.float32), dtype)
    z = wl.store_round(rng.standard_normal(shape, dtype=np.float32) + np.float32(2.0), dtype)
    v = wl.store_round(rng.standard_normal(shape, dtype=np.float32) / np.float32(np.sqrt(d)), dtype)
    g = wl.store_round(rng.standard_normal(shape, dtype=np.float32) / np.float32(np.sqrt(d)), dtype)
    return q, z, v, g


def _weight(Hh, d, seed=3):
    return np.random.default_rng(seed).uniform(0.5, 1.5, size=(Hh, d)).astype(np.float32)


def _call(lasad, dtype, tensors, H, W, w, eps, start=0, mode=0, q_scale=1.0, grad_bf16=False):
    """lasad_backward_layer on device tensors -> device results with fp32 gradients; grad_bf16 (bf16 inputs) runs
    the call with bf16 gradients as well: they must be the fp32 gradients rounded, dweight the same."""
    import torch
    q_pre, z, v, d_out = tensors
    res = both_outputs(lasad.lasad_backward_layer, grad_bf16 and dtype == "bf16", dtype_kw="grad_dtype",
                       q_pre=q_pre, z=z, v=v, d_out=d_out, grid_h=H, grid_w=W,
                       norm_weight=None if w is None else torch.from_numpy(w).cuda(),
                       norm_eps=eps, start_pos=start, boundary_mode=mode, q_scale=q_scale)
    torch.cuda.synchronize()
    return res


def _run(lasad, dtype, q, z, v, g, H, W, w, eps, start=0, mode=0, q_scale=1.0, grad_bf16=False):
    dev = lambda x: lasad.to_device(x, dtype)
    res = _call(lasad, dtype, (dev(q), dev(z), dev(v), dev(g)), H, W, w, eps, start, mode, q_scale, grad_bf16)
    return [r.cpu().numpy() for r in res]


def _norm_condition(oracle, q, z, v, g, W, w, eps, okw, d_o_ref):
    """How much more than the recurrence output o the gradient d_o = rstd gw - o rstd^3 mean_c(gw o) may be off,
    both relative to their RMS, when o carries an error delta (rstd = (mean_c(o^2) + eps)^(-1/2), gw = d_out w).
    Differentiating in o and bounding the four terms (|o . delta| <= |o| |delta|, |mean(gw o)| <= |gw| |o| / d,
    rstd^2 |o|^2 / d <= 1) gives, per token, |delta d_o| <= 6 rstd^2 |gw| |delta| / sqrt(d) in Euclidean norms,
    so an element of d_o moves by at most 6 rstd^2 |gw|_2 max|delta|.  With fp32 inputs o is only required to be
    right to TOL x rms(o), which by this bound allows d_o an error of
        TOL x 6 max_t(rstd_t^2 |gw_t|_2) rms(o) / rms(d_o)
    of its RMS: that factor (never below 1) is the condition used for the fp32 tolerance of d_o and of the
    gradients computed from it.  Tokens whose o nearly cancels (large rstd) dominate it."""
    o = oracle.gated_recurrent(oracle.silu(q), oracle.sigmoid(z), v, W, **okw)
    gw = g.astype(np.float64) * (1.0 if w is None else w[None, None])
    rstd2 = 1.0 / (np.mean(o * o, axis=-1) + eps)
    worst = float(np.max(rstd2 * np.sqrt(np.sum(gw * gw, axis=-1))))
    return max(1.0, 6.0 * worst * float(np.sqrt(np.mean(o * o))) / float(np.sqrt(np.mean(d_o_ref * d_o_ref))))


def _tol(nm, dtype, z):
    # dz inherits the quotient by lambda of the decay gradient (see the vector-decay backward's tests)
    lam_min = float(1.0 / (1.0 + np.exp(-np.float64(z.min()))))
    return TOL[dtype] / lam_min if nm == "dz" and dtype == "f32" else TOL[dtype]


def _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, w, eps, dtype="bf16", start=0, mode=0, q_scale=1.0,
                 grad_bf16=False):
    """The whole call against the oracle, and its two parts as calls of their own:
      1. lasad_backward_layer_norm: d_o in fp32 (bare tolerance; the bf16 d_o must be its rounding) and dweight;
      2. the recurrence + activations part (the call without a normalisation) on the oracle's d_o, rounded to the
         storage type (an input like any other).
    The whole call keeps d_o as a bf16 pair between the two parts, so it is held against the UNROUNDED oracle."""
    import torch
    kw = dict(start=start, mode=mode, q_scale=q_scale)
    okw = dict(start_pos=start, mode=mode, q_scale=q_scale)
    wt = None if w is None else torch.from_numpy(w).cuda()
    d_o_ref, dw_ref = oracle.layer_norm_backward(q, z, v, g, W, norm_weight=w, eps=eps, **okw)
    d_o, dw = both_outputs(lasad.lasad_backward_layer_norm, dtype == "bf16", dtype_kw="d_o_dtype",
                           q_pre=dev_in[0], z=dev_in[1], v=dev_in[2], d_out=dev_in[3], grid_h=H, grid_w=W,
                           norm_weight=wt, norm_eps=eps, start_pos=start, boundary_mode=mode, q_scale=q_scale)
    torch.cuda.synchronize()
    cond = _norm_condition(oracle, q, z, v, g, W, w, eps, okw, d_o_ref) if dtype == "f32" else 1.0
    err = rel_err(d_o.cpu().numpy(), d_o_ref)
    assert err <= cond * TOL[dtype], ("d_o", err, cond)
    assert rel_err(dw.cpu().numpy(), dw_ref) <= TOL[dtype], "dweight"
    d_o_in = wl.store_round(d_o_ref.astype(np.float32), dtype)
    got = _call(lasad, dtype, (*dev_in[:3], lasad.to_device(d_o_in, dtype)), H, W, None, -1.0, grad_bf16=grad_bf16, **kw)[:3]
    ref = oracle.layer_core_backward(q, z, v, d_o_in, W, **okw)
    for nm, a, r in zip(("dq_pre", "dz", "dv"), got, ref):
        err = rel_err(a.cpu().numpy(), r)
        assert err <= _tol(nm, dtype, z), (nm, err)
    whole = _call(lasad, dtype, dev_in, H, W, w, eps, grad_bf16=grad_bf16, **kw)
    ref = oracle.gated_layer_backward(q, z, v, g, W, norm_weight=w, eps=eps, **okw)
    for nm, a, r in zip(("dq_pre", "dz", "dv"), whole, ref):
        err = rel_err(a.cpu().numpy(), r)
        assert err <= cond * _tol(nm, dtype, z), (nm, err, cond)
    assert torch.equal(whole[3], dw)


def _check(lasad, oracle, B, Hh, H, W, dtype, seed, norm="weighted", start=0, n=None, mode=0, q_scale=1.0,
           grad_bf16=False):
    n = H * W - start if n is None else n
    q, z, v, g = _inputs(B, n, Hh, 64, dtype, seed)
    w = _weight(Hh, 64) if norm == "weighted" else None
    if norm == "off":
        got = _run(lasad, dtype, q, z, v, g, H, W, None, -1.0, start, mode, q_scale, grad_bf16)
        ref = oracle.layer_core_backward(q, z, v, g, W, start_pos=start, mode=mode, q_scale=q_scale)
        for nm, a, r in zip(("dq_pre", "dz", "dv"), got, ref):
            assert rel_err(a, r) <= _tol(nm, dtype, z), (nm, rel_err(a, r))
        assert not got[3].any()
        return
    dev_in = tuple(lasad.to_device(x, dtype) for x in (q, z, v, g))
    # one token: o is a multiple of v_0 whatever q and z are, so with a tiny eps the layer output does not depend on
    # them at all and dq_pre, dz are nothing but the residue of a total cancellation; an eps of the size of
    # mean(o^2) leaves a gradient to compare
    eps = 1e-5 if n > 1 else 1e-2
    _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, w, eps, dtype, start, mode, q_scale, grad_bf16)


CASES = [
    # name, B, Hh, H, W, dtype
    ("f32_small", 1, 2, 4, 5, "f32"),
    ("f32_batches", 2, 2, 7, 9, "f32"),
    ("bf16_one_chunk", 2, 3, 3, 5, "bf16"),
    ("bf16_chunks_and_tail", 2, 2, 13, 17, "bf16"),
    ("bf16_single_token", 1, 2, 1, 1, "bf16"),
    ("bf16_many_sequences", 70, 4, 3, 5, "bf16"),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("norm", ["weighted", "plain", "off"])
def test_backward_layer_shapes(lasad, oracle, case, mode, norm):
    name, B, Hh, H, W, dtype = case
    _check(lasad, oracle, B, Hh, H, W, dtype, 50 + H + mode, norm=norm, mode=mode, q_scale=0.5)


@pytest.mark.parametrize("start,n", [(5, 100), (17, 64), (16, 3)])
def test_backward_layer_partial_range(lasad, oracle, start, n):
    _check(lasad, oracle, 2, 2, 9, 17, "bf16", 4300 + start, start=start, n=n)


@pytest.mark.parametrize("H,W,start,n,mode", [(1, 36, 35, 1, 0), (10, 22, 196, 7, 2), (16, 16, 0, 65, 0)])
def test_backward_layer_many_short_sequences(lasad, oracle, H, W, start, n, mode):
    """260 sequences of a few tokens: dv of a sequence's last tokens is a multiple of a single row of the gradient that
    enters the recurrence, so that gradient's storage shows in dv element by element, and the more elements there are
    the further out the worst one sits (a seeded sweep over irregular shapes found these; with one bf16 for that
    gradient they read 2.0e-2 to 2.2e-2 of the RMS)."""
    _check(lasad, oracle, 130, 2, H, W, "bf16", 31029 + n, start=start, n=n, mode=mode, q_scale=0.125, grad_bf16=True)


@pytest.mark.parametrize("grad_bf16", [True, False])
def test_backward_layer_grad_types(lasad, oracle, grad_bf16):
    _check(lasad, oracle, 2, 3, 10, 12, "bf16", 79, grad_bf16=grad_bf16)


def test_backward_layer_inputs_cut_from_one_projection(lasad, oracle):
    """q_pre, z, v as slices of one [B, n, 3 Hh d] tensor (token stride 3 Hh d), d_out and the gradients dense:
    the intermediate gradient in the workspace takes the inputs' strides."""
    import torch
    B, Hh, H, W, d = 2, 3, 9, 11, 64
    n = H * W
    q, z, v, g = _inputs(B, n, Hh, d, "bf16", 123)
    w = _weight(Hh, d)
    fused = torch.empty((B, n, 3, Hh, d), dtype=torch.bfloat16, device="cuda")
    for i, x in enumerate((q, z, v)):
        fused[:, :, i] = lasad.to_device(x, "bf16")
    dev_in = (fused[:, :, 0], fused[:, :, 1], fused[:, :, 2], lasad.to_device(g, "bf16"))
    _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, w, 1e-5)


def test_backward_layer_strong_gates_take_the_serial_route(lasad, oracle):
    """Gate logits around -1.5: every chunk leaves the chunked kernels' range, the walks apply the activations."""
    B, Hh, H, W = 1, 2, 6, 11
    q, z, v, g = _inputs(B, H * W, Hh, 64, "bf16", 5)
    z = wl.store_round(z - np.float32(3.5), "bf16")
    dev_in = tuple(lasad.to_device(x, "bf16") for x in (q, z, v, g))
    _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, None, 1e-5)


@pytest.mark.parametrize("name,n_pairs", [("base_prefill_16x16", 8), ("large_prefill_24x24", 8), ("highres_64x64", 3)])
def test_backward_layer_bench_shapes_sampled(lasad, oracle, name, n_pairs):
    """The benchmark shapes in the benchmark's launch configuration; the oracle on sampled sequences (dweight sums
    over the batch: compared for one head over sampled batch rows by linearity is not possible, so for the base shape
    it is compared in full for two heads)."""
    import torch
    w = wl.CONFIGS[name]
    q, z, v, g = _inputs(w.B, w.N, w.Hh, w.d, "bf16", w.seed + 21)
    wt = _weight(w.Hh, w.d)
    got = _run(lasad, "bf16", q, z, v, g, w.grid_h, w.grid_w, wt, 1e-6, grad_bf16=True)
    pairs = sample_pairs(w.B, w.Hh, n_pairs, seed=w.seed)
    ref = [oracle.gated_layer_backward(q[b:b + 1, :, h:h + 1], z[b:b + 1, :, h:h + 1], v[b:b + 1, :, h:h + 1],
                                       g[b:b + 1, :, h:h + 1], w.grid_w, norm_weight=wt[h:h + 1], eps=1e-6)
           for b, h in pairs]
    for i, nm in enumerate(("dq_pre", "dz", "dv")):
        r = np.concatenate([x[i] for x in ref], axis=0)
        a = np.concatenate([got[i][b:b + 1, :, h:h + 1] for b, h in pairs], axis=0)
        assert rel_err(a, r) <= TOL["bf16"], (nm, rel_err(a, r))
    if name == "base_prefill_16x16":
        full = oracle.layer_norm_backward(q[:, :, :2], z[:, :, :2], v[:, :, :2], g[:, :, :2], w.grid_w, norm_weight=wt[:2], eps=1e-6)
        assert rel_err(got[3][:2], full[1]) <= TOL["bf16"]


def test_backward_layer_deterministic_and_workspace_check(lasad):
    import torch
    q, z, v, g = _inputs(2, 256, 12, 64, "bf16", 3)
    dev = lambda x: lasad.to_device(x, "bf16")
    r1 = lasad.lasad_backward_layer(dev(q), dev(z), dev(v), dev(g), 16, 16)
    r2 = lasad.lasad_backward_layer(dev(q), dev(z), dev(v), dev(g), 16, 16)
    torch.cuda.synchronize()
    for a, b in zip(r1, r2):
        assert torch.equal(a, b)
    small = torch.empty((1024,), dtype=torch.uint8, device="cuda")
    with pytest.raises(lasad.LasadError):
        lasad.lasad_backward_layer(dev(q), dev(z), dev(v), dev(g), 16, 16, workspace=small)


def test_backward_layer_empty_call_zeroes_the_weight_gradient(lasad):
    import torch
    B, Hh, d = 2, 3, 64
    e = torch.empty((B, 0, Hh, d), dtype=torch.bfloat16, device="cuda")
    dw = torch.full((Hh, d), 7.0, device="cuda")
    dq, dz, dv, dw2 = lasad.lasad_backward_layer(e, e.clone(), e.clone(), e.clone(), 4, 4, dweight=dw)
    torch.cuda.synchronize()
    assert dw2 is dw and not dw.any()
    assert dq.numel() == 0 and dz.numel() == 0 and dv.numel() == 0


def test_backward_layer_head_major_inputs(lasad, oracle):
    """q_pre, z, v, d_out stored [B, Hh, n, d] (views permuted to the logical [B, n, Hh, d]), gradients token-major."""
    B, Hh, H, W = 2, 3, 7, 13
    q, z, v, g = _inputs(B, H * W, Hh, 64, "bf16", 77)
    w = _weight(Hh, 64)
    to_hm = lambda x: lasad.to_device(np.ascontiguousarray(x.transpose(0, 2, 1, 3)).transpose(0, 2, 1, 3), "bf16")
    dev_in = tuple(to_hm(x) for x in (q, z, v, g))
    assert dev_in[0].stride(1) == 64 and dev_in[0].stride(2) == H * W * 64
    _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, w, 1e-5)


@pytest.mark.parametrize("B,Hh,H,W,gate", [
    (1, 1, 1, 32, None), (2, 2, 1, 33, None), (2, 2, 5, 13, None),     # two loader groups: one, two and three chunks
    (130, 2, 5, 13, None), (130, 2, 1, 32, None),                      # one loader group
    (1, 2, 31, 67, None),                                              # segments, the last one short
    (1, 2, 31, 67, 1500),                                              # ... one of them left to the token-serial walk
    (130, 2, 5, 13, 40), (1, 2, 6, 11, 40),                            # a range left in a later chunk
    (1, 2, 12, 25, None), (1, 2, 7, 43, None), (1, 8, 6, 45, None), (1, 8, 13, 21, None),     # both sides of the rule that leaves it to a kernel of its own
])
def test_backward_layer_norm_in_the_recomputed_forward(lasad, oracle, B, Hh, H, W, gate):
    """The normalisation's backward is the recomputed forward's epilogue: every tile edge of both loader arrangements, a
    sequence cut into segments, and the token-serial walk (gate: strong gates from this token on, for 40 tokens)."""
    q, z, v, g = _inputs(B, H * W, Hh, 64, "bf16", 900 + B + H * W)
    if gate is not None:
        z[:, gate:gate + 40] = wl.store_round(z[:, gate:gate + 40] - np.float32(3.5), "bf16")
    w = _weight(Hh, 64)
    dev_in = tuple(lasad.to_device(x, "bf16") for x in (q, z, v, g))
    _check_parts(lasad, oracle, dev_in, q, z, v, g, H, W, w, 1e-5, q_scale=0.125)

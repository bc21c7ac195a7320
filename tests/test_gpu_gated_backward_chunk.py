"""The chunked vector-decay backward passes at the edges of their 32-token tiles and of the pairs of tiles they are walked
in: lengths around one to four tiles, own and tied key, a mid-row start and carried states, and a chunk beyond the range
of the factorised form in the first, a middle and the last tile.  Tolerance: the storage type's (helpers.TOL) against
the fp64 oracle; where a gate is next to zero the decay gradient, a quotient by it, is left out.

Few long sequences: the finishing kernel's segments start from the states that the passes kept at the bounds."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl
from helpers import TOL, both_outputs, rel_err

pytestmark = pytest.mark.gpu
D, W = 64, 23


@pytest.fixture(scope="module")
def lasad():
    import torch
    assert torch.cuda.is_available()
    from paper_2507_01652_amd import binding
    binding.load()
    return binding


def _check(lasad, oracle, n, own_key, start, seed, spike=None, W=W):
    import torch
    rng = np.random.default_rng(seed)
    B, Hh = 2, 3
    draw = lambda: wl.store_round(rng.standard_normal((B, n, Hh, D), dtype=np.float32) / np.float32(8), "bf16")
    q, v, g = draw(), draw(), draw()
    k = draw() if own_key else None
    lam = wl.gate_inputs((B, n, Hh, D), "bf16", seed + 1)
    if spike is not None:
        lam[:, spike, :, 5] = 2.0 ** -120
    s0, ds = ((rng.standard_normal((B, Hh, D, D)) * 0.3).astype(np.float32) for _ in range(2))
    H = (start + n + W - 1) // W
    dev = lambda x: None if x is None else lasad.to_device(x, "bf16")
    up = lambda x: torch.from_numpy(x).cuda()
    res = both_outputs(lasad.lasad_backward_gated, True, dtype_kw="grad_dtype", q=dev(q), lam=dev(lam), v=dev(v), d_o=dev(g),
                       grid_h=H, grid_w=W, k=dev(k), start_pos=start, q_scale=0.7)
    ref = oracle.gated_backward(q, lam, v, g, W, k=k, start_pos=start, q_scale=0.7)
    car = lasad.lasad_backward_gated_carried(dev(q), dev(lam), dev(v), dev(g), H, W, k=dev(k), start_pos=start, q_scale=0.7,
                                             state_in=up(s0), d_state_out=up(ds), grad_dtype=torch.float32)
    rc = oracle.gated_backward_carried(q, lam, v, g, W, k=k, start_pos=start, q_scale=0.7, s0=s0, d_state=ds)
    torch.cuda.synchronize()
    for got, want in ((res, ref), (car, rc)):
        for i, (a, r) in enumerate(zip(got, want)):
            if a is not None and not (spike is not None and i == 1):
                assert rel_err(a.cpu().numpy(), r) <= TOL["bf16"], (i, rel_err(a.cpu().numpy(), r))


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 128])
@pytest.mark.parametrize("own_key", [False, True], ids=["tied", "own"])
def test_tile_edges(lasad, oracle, n, own_key):
    _check(lasad, oracle, n, own_key, start=17, seed=n)


@pytest.mark.parametrize("spike", [3, 40, 70, 96])
@pytest.mark.parametrize("own_key", [False, True], ids=["tied", "own"])
def test_range_exit(lasad, oracle, spike, own_key):
    _check(lasad, oracle, 97, own_key, start=0, seed=spike, spike=spike)


# bounds on and off row ends; a shorter last segment; lengths that fill no chunk
@pytest.mark.parametrize("n", [512, 513, 543, 544, 1024, 1040, 1056])
@pytest.mark.parametrize("start", [0, 15, 17])
@pytest.mark.parametrize("own_key", [False, True], ids=["tied", "own"])
def test_segment_bounds(lasad, oracle, n, start, own_key):
    _check(lasad, oracle, n, own_key, start, seed=n + start, W=16)


@pytest.mark.parametrize("spike", [3, 300, 1020])
def test_segment_bounds_beside_a_range_exit(lasad, oracle, spike):
    """One sequence goes to the token-serial walk and keeps no states; the channel of its tiny gate is left out."""
    import torch
    n, W, c = 1024, 16, 5
    rng = np.random.default_rng(spike)
    q, v, g, k = (wl.store_round(rng.standard_normal((1, n, 2, D), dtype=np.float32) / np.float32(8), "bf16") for _ in range(4))
    lam = wl.gate_inputs((1, n, 2, D), "bf16", spike + 1)
    lam[:, spike, 1, c] = 2.0 ** -120
    dev = lambda x: lasad.to_device(x, "bf16")
    got = lasad.lasad_backward_gated(dev(q), dev(lam), dev(v), dev(g), n // W, W, k=dev(k), grad_dtype=torch.float32)
    ref = oracle.gated_backward(q, lam, v, g, W, k=k)
    for i, (a, r) in enumerate(zip(got, ref)):
        a, r = a.cpu().numpy(), np.array(r)
        if i == 1:
            a[:, :, 1, c] = r[:, :, 1, c] = 0
        assert rel_err(a, r) <= TOL["bf16"], i


@pytest.mark.parametrize("n", [1, 32, 33, 64, 96, 97, 129])
@pytest.mark.parametrize("Hh", [80, 81], ids=["80_sequences", "81"])
def test_loader_groups(lasad, oracle, n, Hh):
    """80 sequences take the three passes, whose workgroups have two loader groups here (33 to 64 tokens: one); 81 take the passes
    with one loader group for 33 to 64 tokens, else the two walks."""
    import torch
    rng = np.random.default_rng(n)
    q, v, g = (wl.store_round(rng.standard_normal((1, n, Hh, D), dtype=np.float32) / np.float32(8), "bf16") for _ in range(3))
    lam = wl.gate_inputs((1, n, Hh, D), "bf16", n)
    dev = lambda x: lasad.to_device(x, "bf16")
    got = lasad.lasad_backward_gated(dev(q), dev(lam), dev(v), dev(g), (n + W - 1) // W, W, grad_dtype=torch.float32)
    for i, (a, r) in enumerate(zip(got, oracle.gated_backward(q, lam, v, g, W))):
        assert rel_err(a.cpu().numpy(), r) <= TOL["bf16"], i


@pytest.mark.parametrize("carried", [False, True])
@pytest.mark.parametrize("n,longer", [(1536, 1537), (1536, 1552), (1792, 1793)])
def test_workspace_of_a_longer_call(lasad, oracle, n, longer, carried):
    """The states at segment bounds need scratch of their own, and some longer calls have fewer bounds and ask for less: a
    workspace sized for such a call serves the shorter one; a byte less than it cannot do without is refused."""
    import torch
    rng = np.random.default_rng(n)
    Hh = 5
    q, v, g = (wl.store_round(rng.standard_normal((1, n, Hh, D), dtype=np.float32) / np.float32(8), "bf16") for _ in range(3))
    lam = wl.gate_inputs((1, n, Hh, D), "bf16", n)
    size, call, ref = lasad.lasad_backward_gated_workspace_bytes, lasad.lasad_backward_gated, oracle.gated_backward
    if carried:
        size, call = lasad.lasad_backward_gated_carried_workspace_bytes, lasad.lasad_backward_gated_carried
    given = size(1, Hh, longer, D)
    assert given < size(1, Hh, n, D)
    dev = lambda x: lasad.to_device(x, "bf16")
    ws = torch.empty(given, dtype=torch.uint8, device="cuda")
    args = dev(q), dev(lam), dev(v), dev(g), (n + W - 1) // W, W
    got = call(*args, grad_dtype=torch.float32, workspace=ws)
    for i, (a, r) in enumerate(zip(got, ref(q, lam, v, g, W))):
        assert rel_err(a.cpu().numpy(), r) <= TOL["bf16"], i
    least = 2 * n * Hh * D * 4 + Hh * 8 * D * 4 + (3 * Hh * D * D * 4 + Hh * D * 4 if carried else 0)
    call(*args, workspace=ws[:least])
    with pytest.raises(lasad.LasadError):
        call(*args, workspace=ws[:least - 1])
    layer = [lasad.lasad_backward_layer_workspace_bytes(torch.empty((1, m, Hh, D), dtype=torch.bfloat16)) for m in (n, longer)]
    assert layer[0] < layer[1]


@pytest.mark.parametrize("W,start", [(1, 0), (3, 2), (5, 31), (23, 17), (70, 69)])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("n,Hh", [(33, 3), (63, 85), (77, 3), (513, 3)])
def test_reversed_start(lasad, oracle, W, start, mode, n, Hh):
    """The reversed passes start with a chunk of n % 32 tokens: every row rule on grids narrower and wider than what is
    missing from it, with two loader groups (few sequences) and with one (33 to 64 tokens)."""
    import torch
    rng = np.random.default_rng(n + W)
    q, v, g = (wl.store_round(rng.standard_normal((1, n, Hh, D), dtype=np.float32) / np.float32(8), "bf16") for _ in range(3))
    lam = wl.gate_inputs((1, n, Hh, D), "bf16", n)
    dev = lambda x: lasad.to_device(x, "bf16")
    got = lasad.lasad_backward_gated(dev(q), dev(lam), dev(v), dev(g), (start + n + W - 1) // W, W, start_pos=start,
                                     boundary_mode=mode, q_scale=0.7, grad_dtype=torch.float32)
    for i, (a, r) in enumerate(zip(got, oracle.gated_backward(q, lam, v, g, W, start_pos=start, mode=mode, q_scale=0.7))):
        assert rel_err(a.cpu().numpy(), r) <= TOL["bf16"], i

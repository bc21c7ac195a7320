"""The allocation-free entry point (lasad_forward_chunked_static) against lasad_forward_chunked:
same kernels, the segment states in the library's built-in scratch array instead of a caller's
workspace.  Shapes with few, long sequences so that the segment plan (and with it the scratch
array) is really used; two calls in a row, the second with a smaller input, which leaves stale
contents of the first call in the array."""
import numpy as np
import pytest

from paper_2507_01652_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _case(torch, lasad, B, Hh, H, W, seed, start_pos=0, with_state=False):
    w = wl.Workload(f"static_{B}x{Hh}_{H}x{W}", B, Hh, 64, H, W, "bf16", 0.85, 0.999, seed)
    q, k, v, gam = wl.prefill_inputs(w)
    q, k, v = (np.ascontiguousarray(x[:, start_pos:]) for x in (q, k, v))
    n = q.shape[1]
    tq, tk, tv = (lasad.to_device(x, "bf16") for x in (q, k, v))
    tg = torch.from_numpy(gam).cuda()
    s0 = torch.from_numpy(wl.random_state(w, seed + 1)).cuda() if with_state else None
    need = lasad.lasad_forward_workspace_bytes(B, Hh, n, 64, lasad.BF16)
    assert 0 < need <= lasad.lasad_forward_static_scratch_bytes(), "the case must use the segment plan"
    ws = torch.empty((need,), dtype=torch.uint8, device="cuda")
    o_ref = torch.empty_like(tq)
    s_ref = torch.empty((B, Hh, 64, 64), dtype=torch.float32, device="cuda")
    ws.fill_(255)
    lasad.lasad_forward_chunked(tq, tk, tv, tg, H, W, start_pos=start_pos, state_in=s0, state_out=s_ref,
                                out=o_ref, workspace=ws)
    assert (ws[:B * Hh * 64 * 64 * 4] != 255).any(), "no partial state was written: the call was not cut"
    o = torch.full_like(tq, float("nan"))
    s1 = torch.full_like(s_ref, float("nan"))
    lasad.lasad_forward_chunked_static(tq, tk, tv, tg, H, W, o, start_pos=start_pos, state_in=s0, state_out=s1)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), o_ref.view(torch.int16)), "outputs differ"
    assert torch.equal(s1, s_ref), "final states differ"
    # the same with fp32 output (returned for the comparison with the oracle)
    o32_ref = lasad.lasad_forward_chunked(tq, tk, tv, tg, H, W, start_pos=start_pos, state_in=s0, workspace=ws,
                                          out_dtype=torch.float32)
    o32 = torch.full_like(o32_ref, float("nan"))
    lasad.lasad_forward_chunked_static(tq, tk, tv, tg, H, W, o32, start_pos=start_pos, state_in=s0)
    torch.cuda.synchronize()
    assert torch.equal(o32, o32_ref), "fp32 outputs differ"
    return o32, (q, k, v, gam, s0)


def test_static_entry_matches_workspace_entry(oracle):
    import torch
    from paper_2507_01652_amd import binding as lasad
    lasad.load()
    assert lasad.lasad_forward_static_scratch_bytes() == 8 << 20
    # 4 sequences of 36 chunks -> 6 segments and more of the array than the next call takes; then 6 sequences of 24 chunks (ragged
    # tail) -> 4 segments, started mid-row from a carried state
    _case(torch, lasad, 1, 4, 48, 48, 4101)
    o, (q, k, v, gam, s0) = _case(torch, lasad, 2, 3, 40, 38, 4102, start_pos=31, with_state=True)
    # and the second call's fp32 output against the oracle (fp64, full mask), tolerance of bf16 inputs
    from helpers import rel_err
    lam, _ = oracle.decay_factors(gam, 40, 38, 31, q.shape[1])
    ref = oracle.forward_fullmask(q, k, v, lam, s0=s0.cpu().numpy().astype(np.float64))
    assert rel_err(o.cpu().numpy(), ref) <= 2e-2

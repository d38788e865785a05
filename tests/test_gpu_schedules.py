"""How a chunk's schedule reaches the device follows from its size: as kernel arguments (up to 104 forward items, up to 3584
bytes of backward lists) or through device memory, with a workgroup per block (up to 256 blocks, dQ and dK/dV together in the
backward) or with blocks claimed through counters.  Chunks on both sides of every line against the fp64 oracle (2e-2 for O, 5e-2 for the
gradients, as everywhere), twice for the same bits, and the static forward bit for bit."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, TOL_O, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [128, 96, 64, 256])
@pytest.mark.parametrize("n,hq,hk", [
    (16, 8, 8), (17, 8, 8),     # 256 and 272 dQ and dK/dV blocks
    (32, 8, 8), (33, 8, 8),     # 256 and 264 forward blocks
    (36, 4, 4), (37, 4, 4),     # 3552 and 3648 bytes of backward lists
    (104, 2, 1), (105, 2, 1),   # forward items
])
def test_schedules_on_both_sides_of_each_line(oracle_mod, n, hq, hk, d):
    case = synth.ChunkCase(f"schedule{n}", synth.packed_chunk([33 if i % 2 else 40 for i in range(n)]), sum(33 if i % 2 else 40 for i in range(n)),
                           sum(33 if i % 2 else 40 for i in range(n)), hq, hk, d, 70 + n)
    q, k, v, do = make_inputs(case)
    got = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    o, lse, dq, dk, dv = got
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    assert rel_err(o, O) <= TOL_O
    # (head dimensions 64 and 256 sum the probabilities as they are rounded to bf16 for the product with V: each is off by 2^-9 of
    # itself at most, so the sum is, and its logarithm by as much; scores of some ten nats in float32 add 1e-5)
    assert float(abs(lse.double().cpu().numpy() - LSE).max()) <= (2.0 ** -9 + 1e-5 if d in (64, 256) else 1e-4)
    assert max(rel_err(dq, dQ), rel_err(dk, dK), rel_err(dv, dV)) <= TOL_GRAD
    if n <= 64:
        o2, lse2 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
        ca.chunk_attn_fwd_static(ca.make_desc(case.segs, hq, hk, d, case.total_q, case.total_kv, case.scale), q, k, v, o2, lse2)
        assert torch.equal(o, o2) and torch.equal(lse, lse2)

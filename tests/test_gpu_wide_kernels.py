"""The pipelined forward and dQ kernels of head dimension 256 at the edges of its tiles (32 query rows per wave, stages of 32 keys, rings of four
to six stages), with blocks that are taken a second time because a row outgrows its reference maximum, and with more blocks
than workgroups, against the fp64 oracle (2e-2, as everywhere; LSE: float32 sums of unrounded probabilities, 1e-4)."""
import math

import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, TOL_O, kernels, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu


def _check(oracle_mod, case, q, k, v):
    o, lse = run_gpu(case, q, k, v, backward=False)
    O, LSE = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), None, case.scale).forward()
    assert rel_err(o, O) <= TOL_O and float(abs(lse.double().cpu().numpy() - LSE).max()) <= 1e-4 * max(1.0, float(abs(LSE).max()))


def _case(segs, hq, hk):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    return synth.ChunkCase("wide_forward", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, 256, 300 + tq)


@pytest.mark.parametrize("limit", [60.0, -1e30])
@pytest.mark.parametrize("q_len,ctx", [(1, 0), (1, 31), (32, 0), (33, 31), (64, 64), (65, 95), (97, 130), (129, 1)])
@pytest.mark.parametrize("hq,hk", [(4, 1), (6, 2), (3, 3)])  # 4, 1 and 1 heads per workgroup: 32, 128 and 128 rows
def test_tile_edges(oracle_mod, hq, hk, q_len, ctx, limit):
    case = _case([(0, q_len, 2, q_len + ctx), (q_len, 40, q_len + ctx + 2, 40)], hq, hk)
    q, k, v, _ = make_inputs(case)
    once = run_gpu(case, q, k, v, backward=False)
    ca.chunk_attn_test_set_fwd_rescale_limit(limit)  # (a very low one: every block is taken twice)
    try:
        _check(oracle_mod, case, q, k, v)
        got = run_gpu(case, q, k, v, backward=False)
    finally:
        ca.chunk_attn_test_set_fwd_rescale_limit(60.0)
    if q_len + ctx > 2 * 64:  # (rows whose maximum lies past the two stages of the first reference)
        assert torch.equal(once[0], got[0]) == (limit == 60.0)


def test_late_growth_and_more_blocks_than_workgroups(oracle_mod):
    """Some of 288 blocks have scores that grow by more than 2^60 after the first stage."""
    case = _case([(65 * i, 65, 65 * i, 65) for i in range(12)] + [(780, 33, 780, 400)], 16, 16)
    q, k, v, _ = make_inputs(case)
    k[780 + 350:780 + 400] += 3.0
    q[780:] = q[780:].abs() + 1.0
    _check(oracle_mod, case, q, k, v)


@pytest.mark.parametrize("limit", [60.0, -1e30])
@pytest.mark.parametrize("d,mode", [(256, 1), (64, 1), (64, 0)])
def test_rounding_of_the_probabilities_cancels_in_the_quotient(d, mode, limit):
    """V is one everywhere, so that every row of O is one.  All keys but the first have the same probability relative to it, 0.5018, which bf16
    rounds to 0.5: divided by a sum of unrounded probabilities, O would be 0.9964 for many keys, 0.9961 in bf16.  Divided by the sum of what
    is multiplied with V it is one up to float32 sums of a few hundred terms, which is one in bf16.  LSE takes the unrounded sum at 256,
    the rounded one at 64 (2^-9 of it, as the sum's terms)."""
    n, ctx, hq, hk = 70, 300, 4, 2
    q = torch.zeros((n, hq, d), dtype=torch.bfloat16, device="cuda")
    k = torch.zeros((n + ctx, hk, d), dtype=torch.bfloat16, device="cuda")
    q[..., 0], k[1:, :, 0] = 1.0, -1.0
    v = torch.ones_like(k)
    case = synth.ChunkCase("ones", [synth.Seg(0, n, 0, n + ctx)], n, n + ctx, hq, hk, d, 0)
    ca.chunk_attn_test_set_fwd_rescale_limit(limit)
    try:
        with kernels(mode):
            o, lse = run_gpu(case, q, k, v, scale=0.68955, backward=False)
    finally:
        ca.chunk_attn_test_set_fwd_rescale_limit(60.0)
    assert torch.all(o == 1.0)
    want = torch.log(1.0 + torch.arange(ctx, ctx + n, dtype=torch.float64) * math.exp(-0.68955))
    assert float((lse.double().cpu() - want).abs().max()) <= (1e-5 if d == 256 else 2.0 ** -8)


@pytest.mark.parametrize("segs,hq,hk", [
    ([(0, 1, 2, 201)], 4, 1),                                  # one query
    ([(0, 33, 2, 203), (33, 32, 205, 224)], 4, 1),              # a full tile and a tile of one row; walks that end on a stage
    ([(0, 129, 0, 353)], 6, 2),                                # 128-row items, the last of one row
    ([(0, 97, 1, 497), (97, 1, 498, 161)], 3, 3),
    ([(65 * i, 65, 260 * i, 255) for i in range(12)], 16, 16),  # 384 dQ blocks: more than workgroups
])
def test_dq_of_long_walks(oracle_mod, segs, hq, hk):
    """Walks of 5.5 stages or more on average, from where the pipelined dQ kernel runs; the same bits on a second run."""
    case = _case(segs, hq, hk)
    q, k, v, do = make_inputs(case)
    got = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip(got, run_gpu(case, q, k, v, do)))
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    dQ, dK, dV = orc.backward()
    assert max(rel_err(got[2], dQ), rel_err(got[3], dK), rel_err(got[4], dV)) <= TOL_GRAD

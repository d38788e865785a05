"""Chunks with few query rows and long key walks, whose work items the head_dim 128 and 96 kernels cut into pieces:
against the fp64 oracle (2e-2 for O, 5e-2 for the gradients, as everywhere), against the uncut run (a workspace
without room for partial results; both are bf16 roundings of float32 sums in different orders, so they differ by about one
rounding: 2^-7 of the largest value), and bit for bit between the workspace and the static forward."""
import pytest
import torch

import synth
import paper_2509_21275_amd as ca
from gpu_util import TOL_GRAD, TOL_O, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu

CASES = [  # name, segments, query heads, key/value heads
    ("one_query", [(0, 1, 0, 1100)], 8, 2),
    ("ragged_slice", [(0, 203, 0, 1704)], 8, 2),
    ("walk_ends_on_a_stage", [(0, 64, 0, 1024)], 4, 1),
    ("one_key_past_a_stage", [(0, 65, 0, 1025 + 64)], 16, 2),
    ("mha_256_row_items", [(0, 257, 0, 2000)], 3, 3),
    ("causal_from_the_start", [(0, 1900, 0, 1900)], 2, 1),
    ("key_blocks_cut_too", [(0, 700, 0, 1100)], 8, 2),
    ("cut_and_uncut_items", [(0, 130, 3, 1630), (130, 70, 1640, 70), (200, 1, 1710, 900), (201, 300, 2612, 300)], 6, 2),
]


# The second pass sums the probabilities as they are rounded to bf16 for the product with V: each is off by 2^-9 of itself at
# most, so the sum is, and its logarithm by as much; the scores (up to 140 nats in float32) add 1e-4 at most.
TOL_LSE_SECOND_PASS = 2.0 ** -9 + 1e-4


def _lse_err(lse, want):
    return float(abs(lse.double().cpu().numpy() - want).max())


def _case(name, segs, hq, hk, d=128):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    return synth.ChunkCase(name, [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, d, 900 + len(name))


@pytest.mark.parametrize("d", [128, 96])
@pytest.mark.parametrize("name,segs,hq,hk", CASES, ids=[c[0] for c in CASES])
def test_cut_walks(oracle_mod, name, segs, hq, hk, d):
    case = _case(name, segs, hq, hk, d)
    q, k, v, do = make_inputs(case)
    o, lse, dq, dk, dv = run_gpu(case, q, k, v, do)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    assert rel_err(o, O) <= TOL_O and rel_err(lse, LSE) <= 1e-4
    assert max(rel_err(dq, dQ), rel_err(dk, dK), rel_err(dv, dV)) <= TOL_GRAD

    desc = ca.make_desc(case.segs, hq, hk, d, case.total_q, case.total_kv, case.scale)
    o2 = torch.full_like(o, float("nan")); lse2 = torch.full_like(lse, float("nan"))
    ca.chunk_attn_fwd_static(desc, q, k, v, o2, lse2)
    assert torch.equal(o, o2) and torch.equal(lse, lse2)

    # the largest workspace with which nothing is cut: found by halving (calls with less are refused without a launch)
    lo, hi = 0, ca.chunk_attn_workspace_bytes(desc)[0]
    ws = torch.empty(hi, dtype=torch.uint8, device=q.device)
    while hi - lo > 256:
        mid = (lo + hi) // 512 * 256
        try:
            ca.chunk_attn_fwd(desc, q, k, v, o2, lse2, ws[:mid])
            hi = mid
        except ca.ChunkAttnError:
            lo = mid
    o2.fill_(float("nan")); lse2.fill_(float("nan"))
    ca.chunk_attn_fwd(desc, q, k, v, o2, lse2, ws[:hi])
    assert rel_err(o, o2.double().cpu().numpy()) <= 2.0 ** -7 and rel_err(lse, lse2.double().cpu().numpy()) <= 1e-5


@pytest.mark.parametrize("d", [128, 96])
def test_cut_walks_that_take_the_second_pass(oracle_mod, d):
    """Every piece raises its item's flag: the whole items are recomputed, not put together."""
    case = _case(*CASES[7], d)
    q, k, v, _ = make_inputs(case)
    ca.chunk_attn_test_set_fwd_rescale_limit(-1e30)
    try:
        o, lse = run_gpu(case, q, k, v, backward=False)
    finally:
        ca.chunk_attn_test_set_fwd_rescale_limit(60.0)
    O, LSE = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), None, case.scale).forward()
    assert rel_err(o, O) <= TOL_O and _lse_err(lse, LSE) <= TOL_LSE_SECOND_PASS


def test_piece_whose_scores_outgrow_its_first_stage(oracle_mod):
    """Only a later piece's scores grow past the limit: its flag alone sends the item to the second pass."""
    n, case = 1500, _case("late_growth", [(0, 64, 0, 1500)], 8, 2)
    q, k, v, _ = make_inputs(case)
    ramp = torch.zeros(k.shape[0], device=q.device)
    ramp[n - 400: n] = torch.linspace(0.0, 3.0, 400, device=q.device)
    q = torch.full_like(q, 4.0)
    k = (k.float() * 0.05 + ramp.view(-1, 1, 1)).to(torch.bfloat16)
    o, lse = run_gpu(case, q, k, v, backward=False)
    O, LSE = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), None, case.scale).forward()
    assert rel_err(o, O) <= TOL_O and _lse_err(lse, LSE) <= TOL_LSE_SECOND_PASS


@pytest.mark.parametrize("d", [128, 96])
@pytest.mark.parametrize("f32kv", [False, True])
def test_cut_key_blocks_accumulate(oracle_mod, f32kv, d):
    """dK / dV of key blocks whose walks over the queries were cut, added to what the buffers hold; rows outside every key
    range stay as they are; the same bits on a second run."""
    segs = [(0, 1100, 5, 1400), (1100, 77, 1410, 77)]
    case = _case("cut_accumulate", segs, 6, 2, d)
    q, k, v, do = make_inputs(case)
    init = torch.full(k.shape, 3.0, device=q.device, dtype=torch.float32 if f32kv else torch.bfloat16)
    got = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=f32kv)
    again = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=f32kv)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    cov = torch.zeros(case.total_kv, dtype=torch.bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    _, dK, dV = orc.backward()
    for g, w in ((got[3], dK), (got[4], dV)):
        assert torch.all(g.cpu()[~cov] == 3.0) and rel_err(g.cpu()[cov], w[cov.numpy()] + 3.0) <= TOL_GRAD

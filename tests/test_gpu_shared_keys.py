"""Small chunks whose forward and backward divide the walks of 32 rows among the waves of a workgroup (head dimensions 64, 96 and 128), at the edges of tiles,
stages and shares: against the fp64 oracle (2e-2 for O as everywhere; LSE: 1.1e-4 at 96 and 128, a float32 sum of unrounded probabilities, and
2^-9 + 1e-4 at 64, where they are summed as rounded to bf16), the static forward bit for bit, and the same bits on a second run.  Every
case asserts how many heads share a workgroup."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, TOL_O, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu

CASES = [  # head dimension, segments, query heads, key/value heads, heads per workgroup
    (64, [(0, 1, 0, 65)], 1, 1, 1),
    (64, [(0, 33, 0, 33)], 8, 8, 1),                                          # a second tile of one row, two stages for eight waves
    (64, [(0, 256, 3, 256), (256, 257, 260, 257), (513, 31, 520, 288)], 8, 8, 1),
    (64, [(0, 100, 0, 3000)], 32, 8, 1),
    (64, [(0, 65, 0, 513), (65, 64, 513, 576), (129, 1, 1089, 545)], 32, 8, 1),
    (64, [(0, 700, 2, 700), (700, 33, 705, 400)], 32, 8, 2),
    (64, [(0, 165, 0, 166), (165, 11, 166, 11), (176, 33, 177, 34), (209, 2, 211, 462)], 128, 16, 4),
    (128, [(0, 1, 0, 1)], 1, 1, 1),
    (128, [(0, 32, 0, 32)], 4096, 8, 4),
    (128, [(0, 1, 0, 1100)], 8, 2, 1),
    (128, [(0, 257, 0, 2000)], 3, 3, 1),
    (128, [(0, 64, 0, 1024), (64, 65, 1024, 1089)], 16, 2, 1),
    (128, [(0, 203, 0, 1704), (203, 211, 1704, 211), (414, 120, 1915, 120)], 32, 8, 1),
    (128, [(0, 203, 0, 1704), (203, 246, 1704, 246), (449, 145, 1950, 145), (594, 220, 2095, 220)], 32, 8, 2),
    (128, [(0, 500, 3, 500)], 32, 8, 2),
    (128, [(65 * i, 65, 65 * i, 65) for i in range(12)], 32, 8, 4),
    (128, [(0, 600, 0, 600)], 64, 8, 4),
    (96, [(0, 1, 0, 1100)], 8, 2, 1),
    (96, [(0, 64, 0, 1024), (64, 65, 1024, 1089)], 16, 2, 1),
    (96, [(0, 257, 3, 257), (257, 31, 260, 288)], 8, 8, 1),
    (96, [(0, 500, 3, 500)], 32, 8, 2),
    (96, [(65 * i, 65, 65 * i, 65) for i in range(12)], 32, 8, 4),
]


def _case(d, segs, hq, hk):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    return synth.ChunkCase("shared", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, d, 300 + len(segs) + hq)


def _check(oracle_mod, case, q, k, v, o, lse):
    O, LSE = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), None, case.scale).forward()
    assert rel_err(o, O) <= TOL_O
    assert float(abs(lse.double().cpu().numpy() - LSE).max()) <= (2.0 ** -9 + 1e-4 if case.head_dim == 64 else 1.1e-4)


def _desc(case):
    return ca.make_desc(case.segs, case.num_q_heads, case.num_kv_heads, case.head_dim, case.total_q, case.total_kv, case.scale)


@pytest.mark.parametrize("d,segs,hq,hk,heads", CASES)
def test_shared_keys(oracle_mod, d, segs, hq, hk, heads):
    case = _case(d, segs, hq, hk)
    assert ca.chunk_attn_test_shared_heads(_desc(case)) == heads
    q, k, v, _ = make_inputs(case)
    o, lse = run_gpu(case, q, k, v, backward=False)
    again = run_gpu(case, q, k, v, backward=False)
    assert torch.equal(o, again[0]) and torch.equal(lse, again[1])
    _check(oracle_mod, case, q, k, v, o, lse)
    if ca.chunk_attn_workspace_bytes(_desc(case))[0] > 16 << 20:
        return  # too large for the static forward, whatever kernel runs
    o2, lse2 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
    ca.chunk_attn_fwd_static(_desc(case), q, k, v, o2, lse2)
    torch.cuda.synchronize()
    assert torch.equal(o, o2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("d,hq,hk", [(64, 8, 8), (64, 32, 8), (128, 8, 8), (128, 32, 8)])
def test_shares_of_very_different_scores(oracle_mod, d, hq, hk):
    """Scores grow by some hundred nats along the keys, so the references of the shares lie far apart and move many times."""
    n = 450
    case = _case(d, [(0, n, 0, n)], hq, hk)
    assert ca.chunk_attn_test_shared_heads(_desc(case)) > 0
    q, k, v, _ = make_inputs(case)
    ramp = torch.zeros(k.shape[0], device=q.device)
    ramp[:n] = torch.linspace(-2.0, 2.0, n, device=q.device)
    q = torch.full_like(q, 4.0)
    k = (k.float() * 0.05 + ramp.view(-1, 1, 1)).to(torch.bfloat16)
    o, lse = run_gpu(case, q, k, v, backward=False)
    _check(oracle_mod, case, q, k, v, o, lse)


@pytest.mark.parametrize("scale", [3e-38, 1e-38, 1e-44])
@pytest.mark.parametrize("d,hq,hk", [(64, 8, 8), (64, 32, 8), (96, 8, 2), (128, 8, 8), (128, 32, 8)])
def test_smallest_scales(d, hq, hk, scale):
    """Any scale above zero is a valid one.  With these every score is zero in float32 (below 1e-34), so LSE is ln of the number of visible keys, and O
    their mean; a share's reference has to be its maximum all the same, and not the value that stands for "no key yet"."""
    n, ctx = 70, 300
    case = _case(d, [(0, n, 0, ctx + n)], hq, hk)
    assert ca.chunk_attn_test_shared_heads(_desc(case)) > 0
    q, k, v, _ = make_inputs(case)
    o, lse = run_gpu(case, q, k, v, scale=scale, backward=False)
    visible = torch.arange(ctx + 1, ctx + n + 1, dtype=torch.float64)
    assert float((lse.double().cpu() - visible.log()).abs().max()) <= 2.0 ** -19  # (log2 of an exact sum of ones below 2^9: an ulp of 2^-20, times ln 2)
    mean = v[:ctx + n].double().cpu().cumsum(0)[ctx:] / visible.view(-1, 1, 1)
    assert rel_err(o, mean.repeat_interleave(hq // hk, 1).numpy()) <= TOL_O


BWD_CASES = [  # head dimension, segments, query heads, key/value heads, waves per workgroup
    (64, [(0, 1, 0, 40)], 1, 1, 4),
    (64, [(0, 33, 0, 33)], 8, 8, 4),
    (64, [(0, 256, 3, 256), (256, 257, 260, 257), (513, 31, 520, 288)], 8, 8, 4),
    (64, [(0, 596, 0, 596)], 4, 4, 8),
    (64, [(0, 117, 0, 5600)], 4, 1, 8),
    (64, [(0, 365, 2, 513), (365, 64, 515, 576), (429, 1, 1091, 545)], 16, 8, 4),
    (64, [(97 * i, 97, 97 * i, 97) for i in range(10)], 8, 2, 4),
    (64, [(0, 31, 0, 1000), (31, 95, 1003, 127)], 6, 2, 8),
    (64, [(32 * i, 32, 288 * i, 288) for i in range(64)], 1, 1, 4),            # as many segments and tiles as the arguments have room for
    (128, [(32 * i, 32, 288 * i, 288) for i in range(64)], 1, 1, 4),
    (128, [(0, 32, 0, 32)], 4096, 8, 4),                                      # as many heads
    (128, [(0, 1, 0, 40)], 1, 1, 4),
    (128, [(0, 33, 0, 65)], 3, 3, 4),
    (128, [(0, 257, 3, 257), (257, 31, 260, 288)], 8, 8, 4),
    (128, [(0, 65, 0, 513), (65, 64, 515, 576)], 8, 2, 4),
    (128, [(0, 150, 2, 150)], 32, 8, 4),
    (128, [(0, 764, 0, 764)], 8, 8, 4),
    (96, [(0, 1, 0, 40)], 1, 1, 4),
    (96, [(0, 257, 3, 257), (257, 31, 260, 288)], 8, 8, 4),
    (96, [(0, 65, 0, 513), (65, 64, 515, 576)], 8, 2, 4),
]


@pytest.mark.parametrize("f32kv,accumulate", [(False, False), (False, True), (True, False), (True, True)])
@pytest.mark.parametrize("d,segs,hq,hk,waves", BWD_CASES)
def test_shared_walks_of_the_backward(oracle_mod, d, segs, hq, hk, waves, f32kv, accumulate):
    """5e-2 of the oracle as everywhere, the same bits on a second run, rows outside every key range as they were or zero, and the other kernels'
    results up to one bf16 rounding either way (2^-7).  (One query of many keys: with one or two, dS is a small difference of rounded values.)"""
    case = _case(d, segs, hq, hk)
    assert ca.chunk_attn_test_shared_waves(_desc(case)) == waves
    q, k, v, do = make_inputs(case)
    init = torch.full(k.shape, 3.0, device=q.device, dtype=torch.float32 if f32kv else torch.bfloat16)
    run = lambda: run_gpu(case, q, k, v, do, accumulate=accumulate, dk_init=init, dv_init=init, f32kv=f32kv)
    got, again = run(), run()
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    cov = torch.zeros(case.total_kv, dtype=torch.bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    old = 3.0 if accumulate else 0.0
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    dQ, dK, dV = orc.backward()
    assert rel_err(got[2], dQ) <= TOL_GRAD
    for g, w in ((got[3], dK), (got[4], dV)):
        assert torch.all(g.cpu()[~cov] == old) and rel_err(g.cpu()[cov], w[cov.numpy()] + old) <= TOL_GRAD
    ca.chunk_attn_test_set_bwd_mode(1)
    try:
        assert ca.chunk_attn_test_shared_waves(_desc(case)) == 0
        other = run()
    finally:
        ca.chunk_attn_test_set_bwd_mode(0)
    for a, b in zip(got[2:], other[2:]):
        assert rel_err(a, b.double().cpu().numpy()) <= 2.0 ** -7


@pytest.mark.parametrize("place", ["dq over o", "dk over o", "dv over o", "dq over lse"])
@pytest.mark.parametrize("d", [64, 96, 128])
def test_gradients_in_the_place_of_what_they_come_from(d, place):
    """A caller may write a gradient over O or LSE.  The kernels that read both before they write any then run: the bits of buffers apart."""
    n, heads = 257, 8
    case = synth.ChunkCase("in_place", [synth.Seg(0, n, 0, n)], n, n, heads, heads, d, 318)
    desc = _desc(case)
    assert ca.chunk_attn_test_shared_waves(desc) > 0
    q, k, v, do = make_inputs(case)
    ca.chunk_attn_test_set_bwd_mode(1)
    try:
        o, lse, *want = run_gpu(case, q, k, v, do)
    finally:
        ca.chunk_attn_test_set_bwd_mode(0)
    got = {"dq": torch.empty_like(q), "dk": torch.empty_like(k), "dv": torch.empty_like(v)}
    grad, source = place.split(" over ")
    if source == "o":
        got[grad].copy_(o)
        o = got[grad]
    else:
        inside = got[grad].view(-1)[:2 * lse.numel()].view(torch.float32).view(lse.shape)
        inside.copy_(lse)
        lse = inside
    ca.chunk_attn_bwd(desc, q, k, v, o, do, lse, got["dq"], got["dk"], got["dv"], 0, ca.alloc_workspace(desc))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got.values(), want))


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("segs,hq,hk", [
    ([(0, 32, 0, 32), (32, 33, 32, 33), (65, 64, 65, 64), (129, 1, 129, 129), (130, 95, 258, 95)], 2, 2),
    ([(0, 40, 0, 127), (40, 40, 127, 128), (80, 40, 255, 129), (120, 200, 384, 513)], 8, 2),
    ([(0, 65, 0, 193)], 6, 2),
    ([(0, 96, 0, 640), (96, 160, 640, 160)], 16, 2),
])
def test_small_chunks_through_the_other_kernels(oracle_mod, d, segs, hq, hk):
    """The kernels of larger chunks at the edges of their tiles and walks, which only small chunks have."""
    case = _case(d, segs, hq, hk)
    q, k, v, do = make_inputs(case)
    ca.chunk_attn_test_set_bwd_mode(1)
    try:
        assert ca.chunk_attn_test_shared_heads(_desc(case)) == 0 and ca.chunk_attn_test_shared_waves(_desc(case)) == 0
        o, lse, dq, dk, dv = run_gpu(case, q, k, v, do)
    finally:
        ca.chunk_attn_test_set_bwd_mode(0)
    _check(oracle_mod, case, q, k, v, o, lse)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    dQ, dK, dV = orc.backward()
    cov = torch.zeros(case.total_kv, dtype=torch.bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    assert max(rel_err(dq, dQ), rel_err(dk.cpu()[cov], dK[cov.numpy()]), rel_err(dv.cpu()[cov], dV[cov.numpy()])) <= TOL_GRAD

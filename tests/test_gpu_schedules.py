"""How a chunk's schedule reaches the device follows from its size: as kernel arguments (up to 104 forward items, up to 3584
bytes of backward lists) or through device memory, with a workgroup per block (up to 256 blocks, dQ and dK/dV together in the
backward) or with blocks claimed through counters.  Chunks on both sides of every line against the fp64 oracle (2e-2 for O, 5e-2 for the
gradients, as everywhere), twice for the same bits, and the static forward bit for bit.  These are lines of the larger chunks' kernels; the small
chunks', of 104 forward items as well, run where the library chooses them."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, TOL_O, kernels, make_inputs, rel_err, routes, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,mode", [(128, 1), (96, 1), (64, 1), (256, 1), (128, 0), (96, 0), (64, 0)])
@pytest.mark.parametrize("n,hq,hk", [
    (16, 8, 8), (17, 8, 8),     # 256 and 272 dQ and dK/dV blocks
    (32, 8, 8), (33, 8, 8),     # 256 and 264 forward blocks
    (36, 4, 4), (37, 4, 4),     # 3552 and 3648 bytes of backward lists
    (104, 2, 1), (105, 2, 1),   # forward items
])
def test_schedules_on_both_sides_of_each_line(oracle_mod, n, hq, hk, d, mode):
    with kernels(mode):
        _schedules_on_both_sides_of_each_line(oracle_mod, n, hq, hk, d, mode)


def _schedules_on_both_sides_of_each_line(oracle_mod, n, hq, hk, d, mode):
    case = synth.ChunkCase(f"schedule{n}", synth.packed_chunk([33 if i % 2 else 40 for i in range(n)]), sum(33 if i % 2 else 40 for i in range(n)),
                           sum(33 if i % 2 else 40 for i in range(n)), hq, hk, d, 70 + n)
    assert mode == 0 or not routes(case) & (ca.ROUTE_FWD_SHARED | ca.ROUTE_BWD_SHARED)
    q, k, v, do = make_inputs(case)
    got = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    o, lse, dq, dk, dv = got
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    assert rel_err(o, O) <= TOL_O
    # (head dimension 64 sums the probabilities as they are rounded to bf16 for the product with V: each is off by 2^-9 of
    # itself at most, so the sum is, and its logarithm by as much; scores of some ten nats in float32 add 1e-5)
    assert float(abs(lse.double().cpu().numpy() - LSE).max()) <= (2.0 ** -9 + 1e-5 if d == 64 else 1e-4)
    assert max(rel_err(dq, dQ), rel_err(dk, dK), rel_err(dv, dV)) <= TOL_GRAD
    if n <= 64:
        o2, lse2 = torch.full_like(o, float("nan")), torch.full_like(lse, float("nan"))
        ca.chunk_attn_fwd_static(ca.make_desc(case.segs, hq, hk, d, case.total_q, case.total_kv, case.scale), q, k, v, o2, lse2)
        assert torch.equal(o, o2) and torch.equal(lse, lse2)


@pytest.mark.parametrize("d,n,rows,ctx,hq,hk", [
    (256, 10, 200, 0, 4, 4), (256, 11, 200, 0, 4, 4),  # 240 and 264 blocks; 5.5 stages per dQ walk: the pipelined dQ kernel
    (256, 8, 65, 0, 24, 6), (256, 9, 65, 0, 24, 6),    # 240, 270; dQ items of 32 rows and four heads, the last of one row
    (64, 18, 129, 0, 8, 2), (64, 19, 129, 0, 8, 2),    # 252, 266; the same at 64
    (64, 5, 33, 700, 3, 3), (256, 5, 33, 700, 3, 3),   # dQ has the longer walks and goes first
    (64, 40, 129, 0, 8, 8), (64, 1, 1, 0, 1, 1), (256, 1, 1, 0, 1, 1),
])
def test_dq_and_dkv_blocks_in_one_launch(oracle_mod, d, n, rows, ctx, hq, hk):
    """The unpipelined dK/dV kernels of head dimensions 64 and 256 share their launch with dQ; the same bits on a second run."""
    segs = [synth.Seg(rows * i, rows, (rows + ctx) * i, rows + ctx) for i in range(n)]
    case = synth.ChunkCase("joint", segs, n * rows, n * (rows + ctx), hq, hk, d, 90 + n)
    q, k, v, do = make_inputs(case)
    with kernels(1):
        assert not routes(case) & (ca.ROUTE_DQ_PIPELINED | ca.ROUTE_DKV_PIPELINED | ca.ROUTE_BWD_SHARED)
        got = run_gpu(case, q, k, v, do)
        assert all(torch.equal(a, b) for a, b in zip(got, run_gpu(case, q, k, v, do)))
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    dQ, dK, dV = orc.backward()
    assert max(rel_err(got[2], dQ), rel_err(got[3], dK), rel_err(got[4], dV)) <= TOL_GRAD


@pytest.fixture
def kernels_of_larger_chunks():
    with kernels(1):
        yield


@pytest.mark.usefixtures("kernels_of_larger_chunks")
@pytest.mark.parametrize("f32kv", [False, True])
@pytest.mark.parametrize("d,segs,hq,hk", [
    (64, [(0, 1100, 5, 1400), (1100, 77, 1410, 77)], 6, 2),      # pieces of three query heads per tile, a ragged last block
    (64, [(0, 1025, 0, 1025)], 2, 2),                          # a last tile and a last block of one row each
    (256, [(0, 700, 5, 900), (700, 33, 910, 33)], 6, 2),
    (256, [(0, 1025, 0, 1025)], 1, 1),
])
def test_cut_dkv_walks_of_head_dims_64_and_256(oracle_mod, d, segs, hq, hk, f32kv):
    """Against the oracle, with gradients added to what the buffers hold; a workspace without room for the pieces gives the uncut
    walks' results, another float32 order of the same sums, rounded once: 2^-7 of the largest value in bf16, 1e-5 in float32."""
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    case = synth.ChunkCase("cut_dkv", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, d, 40 + d)
    desc = ca.make_desc(case.segs, hq, hk, d, tq, tkv, case.scale)
    assert ca.chunk_attn_test_routes(desc) & (ca.ROUTE_DKV_CUT | ca.ROUTE_DKV_PIPELINED) == ca.ROUTE_DKV_CUT
    q, k, v, do = make_inputs(case)
    init = torch.full(k.shape, 3.0, device=q.device, dtype=torch.float32 if f32kv else torch.bfloat16)
    got = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=f32kv)
    again = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=f32kv)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    cov = torch.zeros(tkv, dtype=torch.bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    orc.forward()
    dQ, dK, dV = orc.backward()
    assert rel_err(got[2], dQ) <= TOL_GRAD
    for g, w in ((got[3], dK), (got[4], dV)):
        assert torch.all(g.cpu()[~cov] == 3.0) and rel_err(g.cpu()[cov], w[cov.numpy()] + 3.0) <= TOL_GRAD

    o, lse = got[:2]
    dq, dk, dv = torch.empty_like(q), init.clone(), init.clone()
    size = ca.chunk_attn_workspace_bytes(desc)[1]
    small = torch.empty(size - 256, dtype=torch.uint8, device=q.device)  # (the pieces take more than that)
    (ca.chunk_attn_bwd_f32kv if f32kv else ca.chunk_attn_bwd)(desc, q, k, v, o, do, lse, dq, dk, dv, 1, small)
    torch.cuda.synchronize()
    assert torch.equal(dq, got[2])
    for a, b in ((dk, got[3]), (dv, got[4])):
        assert rel_err(a, b.double().cpu().numpy()) <= (1e-5 if f32kv else 2.0 ** -7)
        assert not f32kv or not torch.equal(a, b)  # (it did run uncut; bf16 may round both sums alike)

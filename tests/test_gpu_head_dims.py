"""Head dimensions other than the benchmark's 64 and 128: 256 and 96, through the C ABI against the fp64 oracle: scaled replicas of the five workloads, the
slice-by-slice accumulation of a split sequence in bf16 and float32 buffers, untouched / zeroed rows outside the key
ranges, workspace sizes, bit-reproducibility."""
import dataclasses

import numpy as np
import pytest
import torch

import synth
import paper_2509_21275_amd as ca
from gpu_util import TOL_GRAD, TOL_O, kernels, make_inputs, rel_err, routes, run_gpu

pytestmark = pytest.mark.gpu

DIMS = [96, 256]


def _with_dim(case, d):
    return dataclasses.replace(case, name=f"{case.name}_d{d}", head_dim=d)


@pytest.mark.parametrize("d", DIMS)
@pytest.mark.parametrize("idx", [1, 2, 3, 4, 5])
def test_scaled_replicas(oracle_mod, idx, d):
    case = _with_dim(synth.scaled_case(idx, 16 if idx == 1 else 32), d)
    q, k, v, do = make_inputs(case)
    print(case.name, case.total_q, case.total_kv, flush=True)
    o, lse, dq, dk, dv = run_gpu(case, q, k, v, do)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    errs = (rel_err(o, O), rel_err(dq, dQ), rel_err(dk, dK), rel_err(dv, dV), float(np.abs(lse.double().cpu().numpy() - LSE).max()))
    print(case.name, errs, flush=True)
    assert errs[0] <= TOL_O and max(errs[1:4]) <= TOL_GRAD and errs[4] <= 2e-2
    again = run_gpu(case, q, k, v, do)
    for x, y in zip((o, lse, dq, dk, dv), again):
        assert torch.equal(x, y)


@pytest.mark.parametrize("d", DIMS)
@pytest.mark.parametrize("f32kv", [False, True])
def test_split_sequence_accumulates_over_slices(oracle_mod, d, f32kv):
    """Four slices of one sequence, backward in reverse order, adding into shared dK/dV (bf16 or float32)."""
    n_slices, sl, Hq, Hkv = 4, 192, 4, 2
    n = n_slices * sl
    q = synth.normal_bf16(777, 0, (n, Hq, d), "cuda"); k = synth.normal_bf16(777, 1, (n, Hkv, d), "cuda")
    v = synth.normal_bf16(777, 2, (n, Hkv, d), "cuda"); do = synth.normal_bf16(777, 3, (n, Hq, d), "cuda")
    kv_dtype = torch.float32 if f32kv else torch.bfloat16
    dk = torch.zeros_like(k, dtype=kv_dtype); dv = torch.zeros_like(v, dtype=kv_dtype)
    o_all = torch.empty_like(q); dq_all = torch.empty_like(q)
    for i in range(n_slices - 1, -1, -1):
        case = synth.ChunkCase(f"slice{i}_d{d}", synth.split_slice(sl, sl * i), sl, n, Hq, Hkv, d, 0)
        print(case.name, "f32kv" if f32kv else "bf16", flush=True)
        qi = q[i * sl:(i + 1) * sl].contiguous(); doi = do[i * sl:(i + 1) * sl].contiguous()
        o, lse, dq, dk, dv = run_gpu(case, qi, k, v, doi, accumulate=True, dk_init=dk, dv_init=dv, f32kv=f32kv)
        o_all[i * sl:(i + 1) * sl] = o; dq_all[i * sl:(i + 1) * sl] = dq
    whole = oracle_mod.Oracle([(0, n, 0, n)], q.cpu(), k.cpu(), v.cpu(), do.cpu(), d ** -0.5)
    O, _ = whole.forward(); dQ, dK, dV = whole.backward()
    errs = (rel_err(o_all, O), rel_err(dq_all, dQ), rel_err(dk, dK), rel_err(dv, dV))
    print(errs, flush=True)
    assert errs[0] <= TOL_O and max(errs[1:]) <= TOL_GRAD


@pytest.mark.parametrize("d", DIMS)
def test_rows_outside_key_ranges(oracle_mod, d):
    segs = [(0, 100, 10, 150), (100, 60, 200, 60)]
    case = synth.ChunkCase(f"gaps_d{d}", [synth.Seg(*s) for s in segs], 160, 300, 4, 2, d, 31)
    q, k, v, do = make_inputs(case)
    init_k = torch.full_like(k, 3.0); init_v = torch.full_like(v, -2.0)
    _, _, _, dk_acc, dv_acc = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init_k, dv_init=init_v)
    _, _, _, dk_ow, dv_ow = run_gpu(case, q, k, v, do)
    cov = torch.zeros(300, dtype=torch.bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    assert torch.all(dk_acc.cpu()[~cov] == 3.0) and torch.all(dv_acc.cpu()[~cov] == -2.0)
    assert torch.all(dk_ow.cpu()[~cov] == 0) and torch.all(dv_ow.cpu()[~cov] == 0)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    _, dK, dV = orc.backward()
    c = cov.numpy()
    assert rel_err(dk_acc.cpu()[cov], dK[c] + 3.0) <= TOL_GRAD and rel_err(dv_acc.cpu()[cov], dV[c] - 2.0) <= TOL_GRAD


def test_padded_head_needs_a_larger_workspace_and_says_so():
    """The sizes reported for head_dim 96 cover zero-padded copies of the operands, and a
    workspace sized for head_dim 128 alone is refused before anything is launched."""
    segs = synth.packed_chunk([300, 200])
    d96 = ca.make_desc(segs, 8, 2, 96, 500, 500, 96 ** -0.5)
    d128 = ca.make_desc(segs, 8, 2, 128, 500, 500, 128 ** -0.5)
    f96, b96 = ca.chunk_attn_workspace_bytes(d96)
    f128, b128 = ca.chunk_attn_workspace_bytes(d128)
    qb, kb = 500 * 8 * 128 * 2, 500 * 2 * 128 * 2
    assert f96 >= f128 + 2 * qb + 2 * kb and b96 >= b128 + 4 * qb + 2 * kb + 2 * 2 * kb
    q = torch.zeros((500, 8, 96), dtype=torch.bfloat16, device="cuda"); kv = torch.zeros((500, 2, 96), dtype=torch.bfloat16, device="cuda")
    o = torch.empty_like(q); lse = torch.empty((8, 500), dtype=torch.float32, device="cuda")
    ws = torch.empty(f128, dtype=torch.uint8, device="cuda")
    with pytest.raises(ca.ChunkAttnError) as e:
        ca.chunk_attn_fwd(d96, q, kv, kv, o, lse, ws)
    assert e.value.code == ca.WORKSPACE_TOO_SMALL
    torch.cuda.synchronize()


@pytest.mark.parametrize("name,segs,Hq,Hkv", [
    ("tiny_walks", [(0, 32, 0, 32), (32, 33, 32, 33), (65, 64, 65, 64), (129, 1, 129, 129), (130, 95, 258, 95)], 2, 2),
    ("many_contexts", [(0, 40, 0, 127), (40, 40, 127, 128), (80, 40, 255, 129), (120, 200, 384, 513)], 8, 2),
    ("two_way_walks", [(0, 1500, 0, 1500 + 200), (1500, 90, 1700, 90)], 64, 64),
    ("gqa3_odd_group", [(0, 65, 0, 193)], 6, 2),
    ("gqa8", [(0, 96, 0, 640), (96, 160, 640, 160)], 16, 2),
])
def test_pipelined_kernels_of_head_dim_96(oracle_mod, name, segs, Hq, Hkv):
    """Edges of the software-pipelined kernels' head_dim 96 instantiations (walks of one to three stages, key blocks of 127
    to 129 rows, both walk directions, head splits), against the oracle and against head_dim 128 on zero-padded inputs: the
    same sums in the same order up to the order inside a matrix instruction, so two bf16 roundings apart at most."""
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs)
    case = synth.ChunkCase(f"{name}_d96", [synth.Seg(*s) for s in segs], tq, tkv, Hq, Hkv, 96, 500 + len(name))
    q, k, v, do = make_inputs(case)
    with kernels(1):
        assert routes(case) & ALL_PIPELINED == ALL_PIPELINED
        got = run_gpu(case, q, k, v, do)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    errs = [rel_err(a, b) for a, b in zip(got, (O, LSE, dQ, dK, dV))]
    print(case.name, errs, flush=True)
    assert errs[0] <= TOL_O and errs[1] <= 1e-4 and max(errs[2:]) <= TOL_GRAD
    wide = dataclasses.replace(case, head_dim=128)
    with kernels(1):
        ref = run_gpu(wide, *(torch.nn.functional.pad(x, (0, 32)) for x in (q, k, v, do)), scale=case.scale)
    for a, b in zip(got, ref):
        b = b if b.dim() == 2 else b[..., :96]
        assert rel_err(a, b.double().cpu().numpy()) <= 2.0 ** -7


ALL_PIPELINED = ca.ROUTE_FWD_PIPELINED | ca.ROUTE_DQ_PIPELINED | ca.ROUTE_DKV_PIPELINED


@pytest.mark.parametrize("name,segs,Hq,Hkv,want", [
    # many heads: enough blocks for the pipelined kernels of head_dim 64 on short chunks
    ("dkv_ragged", [(0, 1000, 0, 1000), (1000, 33, 1000, 160)], 128, 128, ca.ROUTE_DKV_PIPELINED),
    ("dkv_groups_and_gaps", [(0, 130, 3, 900), (130, 1, 910, 129), (131, 95, 1041, 127)], 512, 256, ca.ROUTE_DKV_PIPELINED),
    ("all_pipelined", [(0, 300, 0, 4000)], 256, 256, ALL_PIPELINED),
    ("all_pipelined_ragged", [(0, 290, 0, 3900), (290, 30, 3903, 70)], 512, 512, ALL_PIPELINED),
    ("all_pipelined_gqa4", [(0, 500, 0, 3600)], 256, 64, ALL_PIPELINED),
    ("all_pipelined_gqa8", [(0, 500, 0, 3700)], 512, 64, ALL_PIPELINED),
])
def test_pipelined_kernels_of_head_dim_64(oracle_mod, name, segs, Hq, Hkv, want):
    """Chunks with enough blocks (and, for forward and dQ, long enough walks) for head_dim 64's pipelined kernels: ragged key
    blocks and query tiles, rows outside key ranges, accumulation; against the oracle on one head group of each end.  (LSE:
    the forward that is not pipelined sums the probabilities as rounded to bf16, 2^-9 of the sum at most.)"""
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 2
    case = synth.ChunkCase(f"{name}_d64", [synth.Seg(*s) for s in segs], tq, tkv, Hq, Hkv, 64, 700 + len(name))
    assert routes(case) == want
    q, k, v, do = make_inputs(case)
    got = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip(got, again))
    init = torch.full_like(k, 3.0)
    acc = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init)
    cov = np.zeros(tkv, dtype=bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    o, lse, dq, dk, dv = got
    assert torch.all(dk.cpu()[~cov] == 0) and torch.all(acc[3].cpu()[~cov] == 3.0) and torch.all(acc[4].cpu()[~cov] == 3.0)
    G = Hq // Hkv
    for h in (0, Hkv - 1):
        qs = slice(h * G, (h + 1) * G)
        orc = oracle_mod.Oracle(case.segs, q[:, qs].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(), v[:, h:h + 1].cpu().contiguous(),
                                do[:, qs].cpu().contiguous(), case.scale)
        O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
        errs = (rel_err(o[:, qs], O), float(np.abs(lse[qs].double().cpu().numpy() - LSE).max()), rel_err(dq[:, qs], dQ), rel_err(dk[:, h:h + 1], dK), rel_err(dv[:, h:h + 1], dV))
        print(case.name, h, errs, flush=True)
        assert errs[0] <= TOL_O and errs[1] <= 2.0 ** -9 + 1e-4 and max(errs[2:]) <= TOL_GRAD
        assert rel_err(acc[3][:, h:h + 1].cpu()[cov], dK[cov] + 3.0) <= TOL_GRAD and rel_err(acc[4][:, h:h + 1].cpu()[cov], dV[cov] + 3.0) <= TOL_GRAD


@pytest.mark.parametrize("d,mode,want", [(64, 1, 0), (256, 1, 0), (64, 0, ca.ROUTE_FWD_SHARED | ca.ROUTE_BWD_SHARED)])
@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 1), (6, 2)])
def test_tile_edges_of_the_kernels_for_short_walks(oracle_mod, d, mode, want, Hq, Hkv):
    """Head dimensions 64 and 256 below the pipelined kernels' sizes, and the small chunks' kernels of 64 (asserted): key counts on both sides of the
    32- and 64-row tiles the forward and dQ kernels read rows and transposed operands from, contexts that are and are not whole tiles, single rows.
    (LSE: that of 64 sums the probabilities as rounded to bf16, 2^-9 of the sum at most.)"""
    lens = [(1, 1), (31, 31), (32, 32), (33, 33), (63, 64), (64, 65), (65, 65), (1, 96), (2, 128), (40, 129), (95, 191), (129, 193)]
    segs, tq, tkv = [], 0, 0
    for n, keys in lens:
        segs.append((tq, n, tkv, keys))
        tq, tkv = tq + n, tkv + keys
    case = synth.ChunkCase(f"tile_edges_d{d}", [synth.Seg(*s) for s in segs], tq, tkv, Hq, Hkv, d, 610 + Hq)
    q, k, v, do = make_inputs(case)
    with kernels(mode):
        assert routes(case) == want
        o, lse, dq, dk, dv = run_gpu(case, q, k, v, do)
    orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
    O, LSE = orc.forward(); dQ, dK, dV = orc.backward()
    assert float(np.abs(lse.double().cpu().numpy() - LSE).max()) <= (2.0 ** -9 + 1e-4 if d == 64 else 1e-4)
    for q0, n, k0, keys in segs:  # per sequence: an error in a short one does not drown in the others
        assert rel_err(o[q0:q0 + n], O[q0:q0 + n]) <= TOL_O
        if keys > 1:  # (one query on one key: its dQ and dK are zero up to rounding)
            assert rel_err(dq[q0:q0 + n], dQ[q0:q0 + n]) <= TOL_GRAD and rel_err(dk[k0:k0 + keys], dK[k0:k0 + keys]) <= TOL_GRAD
        assert rel_err(dv[k0:k0 + keys], dV[k0:k0 + keys]) <= TOL_GRAD


def test_second_pass_of_head_dim_64(oracle_mod):
    """The pipelined forward of head_dim 64 with every block taken twice, the second time with the maximum over all keys: other references than
    with the default limit, so other bits, and LSE as close to the oracle (float32 sums of unrounded probabilities)."""
    case = synth.ChunkCase("redo_d64", [synth.Seg(0, 290, 0, 3900), synth.Seg(290, 30, 3903, 70)], 320, 3973, 512, 512, 64, 77)
    assert routes(case) & ca.ROUTE_FWD_PIPELINED
    q, k, v, _ = make_inputs(case)
    first = run_gpu(case, q, k, v, backward=False)
    ca.chunk_attn_test_set_fwd_rescale_limit(-1e30)
    try:
        o, lse = run_gpu(case, q, k, v, backward=False)
    finally:
        ca.chunk_attn_test_set_fwd_rescale_limit(60.0)
    assert not torch.equal(o, first[0]) and not torch.equal(lse, first[1])
    for h in (5, 511):
        O, LSE = oracle_mod.Oracle(case.segs, q[:, h:h + 1].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(),
                                   v[:, h:h + 1].cpu().contiguous(), None, case.scale).forward()
        assert rel_err(o[:, h:h + 1], O) <= TOL_O and float(np.abs(lse[h:h + 1].double().cpu().numpy() - LSE).max()) <= 1e-4


def test_scores_that_outgrow_their_first_stage_at_head_dim_64(oracle_mod):
    """Half of the heads have keys whose scores grow past the limit late in the walk: their blocks alone are taken again."""
    case = synth.ChunkCase("late_growth_d64", [synth.Seg(0, 300, 0, 4000)], 300, 4000, 256, 256, 64, 78)
    assert routes(case) & ca.ROUTE_FWD_PIPELINED
    q, k, v, _ = make_inputs(case)
    ramp = torch.zeros((4000, 256, 1), device=q.device)
    ramp[3000:3400, :128] = torch.linspace(0.0, 3.0, 400, device=q.device).view(-1, 1, 1)   # up to 96 nats
    q = torch.full_like(q, 4.0)
    k = (k.float() * 0.05 + ramp).to(torch.bfloat16)
    o, lse = run_gpu(case, q, k, v, backward=False)
    for h in (3, 127, 128, 255):
        O, LSE = oracle_mod.Oracle(case.segs, q[:, h:h + 1].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(),
                                   v[:, h:h + 1].cpu().contiguous(), None, case.scale).forward()
        assert rel_err(o[:, h:h + 1], O) <= TOL_O and float(np.abs(lse[h:h + 1].double().cpu().numpy() - LSE).max()) <= 1e-4


@pytest.mark.parametrize("name,segs,Hq,Hkv", [
    # enough 64-key blocks and stages for the pipelined dK/dV kernel of head_dim 256, both walk directions among them
    ("ragged", [(0, 1100, 0, 1100), (1100, 33, 1100, 160)], 64, 64),
    ("groups_and_gaps", [(0, 400, 3, 900), (400, 1, 910, 129), (401, 63, 1041, 127)], 64, 32),
    ("many_context_blocks", [(0, 250, 0, 250 + 70 * 64)], 16, 8),
])
def test_pipelined_dkv_of_head_dim_256(oracle_mod, name, segs, Hq, Hkv):
    """Ragged key blocks and query tiles, walks of one stage upwards, rows outside key ranges, accumulation, float32 buffers;
    against the oracle on one head group of each end."""
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 2
    case = synth.ChunkCase(f"{name}_d256", [synth.Seg(*s) for s in segs], tq, tkv, Hq, Hkv, 256, 800 + len(name))
    assert routes(case) == ca.ROUTE_DKV_PIPELINED
    q, k, v, do = make_inputs(case)
    _, _, _, dk, dv = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert torch.equal(dk, again[3]) and torch.equal(dv, again[4])
    init = torch.full(k.shape, 3.0, device=k.device)
    acc = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=True)
    cov = np.zeros(tkv, dtype=bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    assert torch.all(dk.cpu()[~cov] == 0) and torch.all(dv.cpu()[~cov] == 0)
    assert torch.all(acc[3].cpu()[~cov] == 3.0) and torch.all(acc[4].cpu()[~cov] == 3.0)
    G = Hq // Hkv
    for h in (0, Hkv - 1):
        qs = slice(h * G, (h + 1) * G)
        orc = oracle_mod.Oracle(case.segs, q[:, qs].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(), v[:, h:h + 1].cpu().contiguous(),
                                do[:, qs].cpu().contiguous(), case.scale)
        orc.forward()
        _, dK, dV = orc.backward()
        assert max(rel_err(dk[:, h:h + 1], dK), rel_err(dv[:, h:h + 1], dV)) <= TOL_GRAD
        assert rel_err(acc[3][:, h:h + 1].cpu()[cov], dK[cov] + 3.0) <= TOL_GRAD and rel_err(acc[4][:, h:h + 1].cpu()[cov], dV[cov] + 3.0) <= TOL_GRAD

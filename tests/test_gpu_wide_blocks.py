"""dQ and dK/dV blocks in one launch at head dimensions 256 and 64 (dK/dV blocks of 128 and 256 keys): either kind first, blocks that are assigned by number (no more than
workgroups) and blocks that are claimed, all three gradients against the fp64 oracle; and what a block leaves in LDS."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu


def _case(segs, hq, hk, d, keys):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    case = synth.ChunkCase("wide", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, d, 700 + tq + d)
    assert ca.chunk_attn_test_dkv_keys(ca.make_desc(case.segs, hq, hk, d, tq, tkv, case.scale)) == keys
    return case


def _blocks(segs, hq, hk):
    """Blocks of dQ (units of 32 rows of up to four heads of a group, four to a workgroup) and of dK/dV of 128 keys, and whether the dQ walks are the longer ones."""
    g, per_wg = hq // hk, 1
    while per_wg < 4 and g % (2 * per_wg) == 0:
        per_wg *= 2
    rows, inner = 32 * (4 // per_wg), hk * (g // per_wg)
    return (sum(-(-s[1] // rows) for s in segs) * inner, sum(-(-s[3] // 128) for s in segs) * hk,
            max(-(-s[3] // 32) for s in segs) > max(-(-s[1] // 32) * g for s in segs))


@pytest.mark.parametrize("segs,hq,hk,claimed,dq_first", [
    ([(0, 458, 0, 458), (458, 298, 461, 298), (756, 274, 762, 274)], 16, 16, True, False),
    ([(0, 513, 3, 513), (513, 417, 516, 417), (930, 199, 936, 858)], 16, 8, True, False),
    ([(0, 276, 0, 952), (276, 314, 955, 314), (590, 189, 1269, 189)], 32, 8, True, False),
    ([(0, 223, 0, 223), (223, 414, 226, 414), (637, 123, 643, 925)], 16, 16, True, True),
    ([(0, 277, 0, 4165), (277, 23, 4165, 3768), (300, 243, 7933, 243)], 12, 4, True, True),
    ([(0, 34, 0, 1622), (34, 174, 1625, 1580)], 32, 8, True, True),
    ([(0, 500, 0, 500), (500, 461, 503, 461)], 16, 16, False, False),
    ([(0, 279, 0, 890), (279, 258, 893, 258)], 32, 8, False, False),
    ([(0, 408, 0, 408), (408, 141, 411, 141), (549, 306, 552, 920)], 16, 8, False, True),
    ([(0, 175, 3, 175), (175, 218, 181, 1002)], 32, 8, False, True),
])
def test_both_kinds_of_256_in_one_launch(oracle_mod, segs, hq, hk, claimed, dq_first):
    case = _case(segs, hq, hk, 256, 128)
    dq_blocks, dkv_blocks, first = _blocks(segs, hq, hk)
    assert (dq_blocks + dkv_blocks > 256) == claimed and first == dq_first
    q, k, v, do = make_inputs(case)
    _, _, dq, dk, dv = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again[2:]))
    G = hq // hk
    for h in (0, hk - 1):
        qs = slice(h * G, (h + 1) * G)
        orc = oracle_mod.Oracle(case.segs, q[:, qs].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(), v[:, h:h + 1].cpu().contiguous(),
                                do[:, qs].cpu().contiguous(), case.scale)
        orc.forward()
        dQ, dK, dV = orc.backward()
        assert max(rel_err(dq[:, qs], dQ), rel_err(dk[:, h:h + 1], dK), rel_err(dv[:, h:h + 1], dV)) <= TOL_GRAD


@pytest.mark.parametrize("poisoned", [0, 1])
@pytest.mark.parametrize("d,keys,segs,hq,hk", [
    (256, 128, [(0, 700, 0, 700), (700, 600, 700, 900), (1300, 300, 1600, 300)], 64, 64),
    (256, 128, [(0, 650, 0, 650), (650, 640, 650, 1100), (1290, 300, 1750, 300)], 64, 16),
    (64, 256, [(0, 257, 0, 4001), (257, 255, 4010, 4351), (512, 100, 8361, 2000)], 256, 64),
])
def test_a_block_leaves_nothing_to_the_next(d, keys, segs, hq, hk, poisoned):
    """Queries of one sequence that are not finite, of the one whose dK/dV or whose dQ blocks start first, change the gradients of that sequence alone: a workgroup's LDS is
    written again, or cleared, before a block reads it."""
    case = _case(segs, hq, hk, d, keys)
    q, k, v, do = make_inputs(case)
    want = run_gpu(case, q, k, v, do)
    rows = slice(segs[poisoned][0], segs[poisoned][0] + segs[poisoned][1])
    q[rows], do[rows] = float("inf"), float("nan")
    got = run_gpu(case, q, k, v, do)
    for n, s in enumerate(segs):
        at, keys_at = slice(s[0], s[0] + s[1]), slice(s[2], s[2] + s[3])
        if n == poisoned:
            assert not torch.isfinite(got[3][keys_at]).any()
        else:
            assert torch.equal(want[2][at], got[2][at]) and all(torch.equal(want[x][keys_at], got[x][keys_at]) for x in (3, 4))

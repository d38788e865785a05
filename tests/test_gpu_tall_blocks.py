"""dK/dV blocks of 256 keys (head dimensions 64, 96 and 128): ragged last blocks and query tiles, waves whose keys no query or few queries see, groups of one to
four heads, walks of one step and in both directions, rows outside key ranges, accumulation and float32 buffers, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    ([(0, 545, 0, 545)], 256, 256),                                              # 33 keys in the last block, one row in the last tile
    ([(0, 257, 0, 257), (257, 255, 260, 511)], 128, 128),                         # one key and 255 keys in the last blocks, keys no segment has
    ([(0, 33, 2, 1000)], 512, 256),                                              # two query tiles, context blocks that every query sees
    ([(0, 1025, 0, 1025)], 192, 64),                                             # three heads to a group, walks down and up
    ([(0, 513, 0, 513), (513, 700, 513, 1700), (1213, 31, 2213, 300), (1244, 1, 2513, 1), (1245, 255, 2514, 1000)], 96, 96),
    ([(0, 640, 0, 1153)], 256, 64),                                              # four heads, more blocks than workgroups
]


def _case(segs, hq, hk, d):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    case = synth.ChunkCase("tall", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, d, 900 + tq + d)
    assert ca.chunk_attn_test_dkv_keys(ca.make_desc(case.segs, hq, hk, d, tq, tkv, case.scale)) == 256
    return case


NARROW = [  # of head dimension 64: walks long enough for the pipelined kernels
    ([(0, 640, 0, 4097)], 256, 64),                                              # one key in the last block
    ([(0, 257, 0, 4001), (257, 255, 4010, 4351)], 256, 64),                       # one row in the last tile, keys no segment has, 255 keys in the last block
]


@pytest.mark.parametrize("segs,hq,hk,d", [(*c, d) for c in CASES for d in (128, 96)] + [(*c, 64) for c in NARROW])
def test_edges_of_blocks_and_tiles(oracle_mod, segs, hq, hk, d):
    case = _case(segs, hq, hk, d)
    q, k, v, do = make_inputs(case)
    _, _, dq, dk, dv = run_gpu(case, q, k, v, do)
    again = run_gpu(case, q, k, v, do)
    assert all(torch.equal(a, b) for a, b in zip((dq, dk, dv), again[2:]))
    init = torch.full(k.shape, 3.0, device=k.device)
    acc = run_gpu(case, q, k, v, do, accumulate=True, dk_init=init, dv_init=init, f32kv=True)
    cov = np.zeros(case.total_kv, dtype=bool)
    for s in segs:
        cov[s[2]:s[2] + s[3]] = True
    assert torch.all(dk.cpu()[~cov] == 0) and torch.all(dv.cpu()[~cov] == 0)
    assert torch.all(acc[3].cpu()[~cov] == 3.0) and torch.all(acc[4].cpu()[~cov] == 3.0)
    G = hq // hk
    for h in (0, hk - 1):
        qs = slice(h * G, (h + 1) * G)
        orc = oracle_mod.Oracle(case.segs, q[:, qs].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(), v[:, h:h + 1].cpu().contiguous(),
                                do[:, qs].cpu().contiguous(), case.scale)
        orc.forward()
        dQ, dK, dV = orc.backward()
        assert max(rel_err(dq[:, qs], dQ), rel_err(dk[:, h:h + 1], dK), rel_err(dv[:, h:h + 1], dV)) <= TOL_GRAD
        assert rel_err(acc[3][:, h:h + 1].cpu()[cov], dK[cov] + 3.0) <= TOL_GRAD and rel_err(acc[4][:, h:h + 1].cpu()[cov], dV[cov] + 3.0) <= TOL_GRAD


@pytest.mark.parametrize("d", [128, 96])
def test_a_block_leaves_nothing_to_the_next(d):
    """Queries of one sequence that are not finite change the gradients of that sequence alone: a workgroup's LDS is written again, or cleared, before a
    block reads it."""
    segs = [(300 * i, 300, 300 * i, 300) for i in range(8)]
    case = _case(segs, 64, 64, d)
    q, k, v, do = make_inputs(case)
    want = run_gpu(case, q, k, v, do)
    q[:300], do[:300] = float("inf"), float("nan")
    got = run_gpu(case, q, k, v, do)
    assert not torch.isfinite(got[3][:300]).any()
    assert all(torch.equal(a[300:], b[300:]) for a, b in zip(want[2:], got[2:]))

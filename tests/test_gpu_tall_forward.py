"""The forward of head dimension 256 with 64 query rows per wave: ragged last tiles and stages, walks of one stage, waves without rows, groups of one to four heads, blocks
that are taken a second time because a row outgrows its reference maximum, and the static entry point, against the fp64 oracle (O 2e-2, as everywhere;
LSE: float32 sums of unrounded probabilities, 1e-4)."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_O, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    ([(0, 641, 0, 641)], 128, 32),                                          # four heads to a workgroup, one row in the last tile, one key in the last stage
    ([(0, 1025, 0, 1025)], 192, 64),                                        # three heads to a group: one to a workgroup, tiles of 256 rows
    ([(0, 65, 2, 1022), (65, 7, 1024, 7)], 512, 256),                       # two heads; waves without rows
    ([(0, 700, 0, 731), (700, 1, 740, 1), (701, 33, 741, 64), (734, 97, 805, 1000)], 128, 32),  # a walk of one stage; keys no segment has
    ([(250 * i, 250, 600 * i, 600) for i in range(9)], 96, 96),             # more blocks than workgroups
]


def _case(segs, hq, hk):
    tq, tkv = max(s[0] + s[1] for s in segs), max(s[2] + s[3] for s in segs) + 3
    case = synth.ChunkCase("tall_forward", [synth.Seg(*s) for s in segs], tq, tkv, hq, hk, 256, 500 + tq)
    assert ca.chunk_attn_test_fwd_rows(ca.make_desc(case.segs, hq, hk, 256, tq, tkv, case.scale)) == 64
    return case


def _check(oracle_mod, case, q, k, v, o, lse):
    G = case.num_q_heads // case.num_kv_heads
    for h in (0, case.num_kv_heads - 1):
        qs = slice(h * G, (h + 1) * G)
        O, LSE = oracle_mod.Oracle(case.segs, q[:, qs].cpu().contiguous(), k[:, h:h + 1].cpu().contiguous(), v[:, h:h + 1].cpu().contiguous(), None, case.scale).forward()
        assert rel_err(o[:, qs], O) <= TOL_O and float(abs(lse[qs].double().cpu().numpy() - LSE).max()) <= 1e-4 * max(1.0, float(abs(LSE).max()))


@pytest.mark.parametrize("limit", [60.0, -1e30])
@pytest.mark.parametrize("segs,hq,hk", CASES)
def test_edges_of_tiles_and_stages(oracle_mod, segs, hq, hk, limit):
    case = _case(segs, hq, hk)
    q, k, v, _ = make_inputs(case)
    ca.chunk_attn_test_set_fwd_rescale_limit(limit)  # (a very low one: every block is taken twice)
    try:
        o, lse = run_gpu(case, q, k, v, backward=False)
        o2, lse2 = run_gpu(case, q, k, v, backward=False)
        assert torch.equal(o, o2) and torch.equal(lse, lse2)
        desc = ca.make_desc(case.segs, hq, hk, 256, case.total_q, case.total_kv, case.scale)
        if ca.chunk_attn_workspace_bytes(desc)[0] <= 16 << 20:  # (the first case; its scratch memory is fixed)
            ca.chunk_attn_fwd_static(desc, q, k, v, o2.fill_(float("nan")), lse2.fill_(float("nan")))
            torch.cuda.synchronize()
    finally:
        ca.chunk_attn_test_set_fwd_rescale_limit(60.0)
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    _check(oracle_mod, case, q, k, v, o, lse)


def test_late_growth(oracle_mod):
    """The last sequence's scores grow by more than 2^60 after the first stages; the others' blocks keep their bits."""
    segs = [(300 * i, 300, 300 * i, 300) for i in range(12)]
    case = _case(segs, 128, 32)
    q, k, v, _ = make_inputs(case)
    want = run_gpu(case, q, k, v, backward=False)
    k[3500:3600] += 3.0
    q[3300:] = q[3300:].abs() + 1.0
    o, lse = run_gpu(case, q, k, v, backward=False)
    assert torch.equal(o[:3300], want[0][:3300]) and torch.equal(lse[:, :3300], want[1][:, :3300])
    _check(oracle_mod, case, q, k, v, o, lse)

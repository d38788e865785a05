"""Packed chunks of many short sequences through the pipelined dK/dV blocks: their waves start a block one after the other, and what
one wave clears another one may have copied already (the row values of a block's first stages were lost so, and dK with them)."""
import pytest
import torch

import paper_2509_21275_amd as ca
import synth
from gpu_util import TOL_GRAD, make_inputs, rel_err, run_gpu

pytestmark = pytest.mark.gpu

LENGTHS = (77, 199, 52, 73, 77, 46, 75, 58, 23, 95, 30, 163, 51, 112, 84, 24, 105, 72, 34, 33, 105, 43, 121, 68, 46, 21)


@pytest.mark.parametrize("d,mode", [(128, 1), (96, 1), (128, 2)])
def test_every_run_gives_the_same_gradients(oracle_mod, d, mode):
    segs = [synth.Seg(0, 21, 0, 252)]
    for n in LENGTHS:
        segs.append(synth.Seg(segs[-1].q_start + segs[-1].q_len, n, segs[-1].kv_start + segs[-1].kv_len, n))
    tq, tkv = sum(s.q_len for s in segs), sum(s.kv_len for s in segs)
    for seed in range(4):
        case = synth.ChunkCase("short_walks", segs, tq, tkv, 8, 8, d, 500 + seed)
        q, k, v, do = make_inputs(case)
        ca.chunk_attn_test_set_bwd_mode(mode)
        try:
            runs = [run_gpu(case, q, k, v, do) for _ in range(6)]
        finally:
            ca.chunk_attn_test_set_bwd_mode(0)
        assert all(torch.equal(a, b) for r in runs[1:] for a, b in zip(runs[0], r))
        if seed == 0:
            orc = oracle_mod.Oracle(case.segs, q.cpu(), k.cpu(), v.cpu(), do.cpu(), case.scale)
            orc.forward()
            for g, w in zip(runs[0][2:], orc.backward()):
                assert rel_err(g, w) <= TOL_GRAD

"""Which chunks of head dimensions 64, 96 and 128 run dK/dV blocks of 256 keys, which of 256 the pipelined ones of 128 keys and which the forward of 64 query
rows per wave, and what their steps compile to."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2509_21275_amd as ca
from paper_2509_21275_amd.build import FLAGS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21275_amd", "csrc")


@pytest.mark.parametrize("segs,hq,hk,keys", [
    ([(0, 8192, 0, 32768)], 32, 8, 256),                            # long walks, four blocks to a compute unit
    ([(0, 1024, 0, 32768)], 32, 8, 256),
    ([(0, 16384, 0, 16384)], 64, 8, 256),
    ([(1000 * i, 1000, 1000 * i, 1000) for i in range(64)], 32, 8, 256),
    ([(0, 3193, 0, 8192)], 32, 8, 256),
    ([(0, 4999, 0, 4999)], 32, 8, 128),                              # 160 blocks of 256 keys, the longest twice the even share
    ([(129 * i, 129, 129 * i, 129) for i in range(64)], 32, 8, 128),  # most of a second 128 keys would be empty
    ([(0, 1024, 0, 1024)], 8, 8, 32),                                # a small chunk
])
@pytest.mark.parametrize("d", [96, 128])
def test_blocks_that_end_sooner(d, segs, hq, hk, keys):
    tq, tkv = sum(s[1] for s in segs), segs[-1][2] + segs[-1][3]
    desc = ca.make_desc(segs, hq, hk, d, tq, tkv, d ** -0.5)
    cut = ca.chunk_attn_test_routes(desc) & (ca.ROUTE_DQ_CUT | ca.ROUTE_DKV_CUT)
    assert ca.chunk_attn_test_dkv_keys(desc) == keys and not (cut and keys == 256)


@pytest.mark.parametrize("segs,hq,hk,keys", [
    ([(0, 16384, 0, 16384)], 32, 8, 128),
    ([(1000 * i, 1000, 1000 * i, 1000) for i in range(64)], 32, 8, 128),   # two blocks of 64 keys per compute unit and 14 steps each
    ([(0, 1428, 0, 3445)], 32, 8, 128),                                     # by the estimates
    ([(0, 2668, 0, 2668)], 8, 8, 128),
    ([(0, 4335, 0, 4335)], 8, 2, 64),                                       # few blocks with long walks, which the other kernels cut
    ([(0, 899, 0, 899)], 64, 8, 64),
    ([(64 * i, 64, 64 * i, 64) for i in range(64)], 8, 8, 64),              # half of every block of 128 keys would be empty
])
def test_blocks_of_head_dim_256(segs, hq, hk, keys):
    tq, tkv = sum(s[1] for s in segs), segs[-1][2] + segs[-1][3]
    desc = ca.make_desc(segs, hq, hk, 256, tq, tkv, 0.0625)
    assert ca.chunk_attn_test_dkv_keys(desc) == keys
    assert bool(ca.chunk_attn_test_routes(desc) & ca.ROUTE_DKV_PIPELINED) == (keys == 128)


@pytest.mark.parametrize("segs,hq,hk,keys", [
    ([(0, 8192, 0, 16384)], 32, 8, 256), ([(0, 2048, 0, 16384)], 64, 8, 256),
    ([(0, 10790, 0, 10833)], 8, 2, 128),                                    # one of the kinds is not pipelined
    ([(0, 129, 0, 4351), (129, 1, 4360, 3900)], 512, 256, 128),             # short dK/dV walks
])
def test_blocks_of_head_dim_64(segs, hq, hk, keys):
    tq, tkv = sum(s[1] for s in segs), segs[-1][2] + segs[-1][3]
    desc = ca.make_desc(segs, hq, hk, 64, tq, tkv, 0.125)
    assert ca.chunk_attn_test_dkv_keys(desc) == keys


@pytest.mark.parametrize("segs,hq,hk,rows", [
    ([(0, 4096, 0, 4096)], 32, 8, 64), ([(0, 2048, 0, 32768)], 32, 8, 64), ([(300 * i, 300, 300 * i, 300) for i in range(64)], 32, 8, 64),
    ([(0, 640, 0, 640)], 256, 64, 64),
    ([(0, 1024, 0, 1024)], 32, 8, 32),                                      # no more blocks of 32 rows per wave than compute units
    ([(0, 2668, 0, 2668)], 8, 8, 32),                                       # the first, long blocks of 64 rows end last
    ([(128 * i, 128, 128 * i, 128) for i in range(64)], 16, 16, 32),        # half of every block of 256 rows would be empty
])
def test_forward_of_head_dim_256(segs, hq, hk, rows):
    tq, tkv = sum(s[1] for s in segs), segs[-1][2] + segs[-1][3]
    desc = ca.make_desc(segs, hq, hk, 256, tq, tkv, 0.0625)
    assert ca.chunk_attn_test_fwd_rows(desc) == rows and not ca.chunk_attn_test_routes(desc) & ca.ROUTE_FWD_PIPELINED


HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_steps_of_full_registers_touch_no_scratch(tmp_path):
    """The steps of kernels whose accumulators fill the accumulation registers spill nothing: a reload in a step waits for all copies in flight
    (two of them made the dK/dV blocks of head dimension 128 a fifth slower)."""
    for src, names in (("bwd_kernel.hip", ["bwd_pipe_kernelILi%dELb0ELb1" % d for d in (64, 96, 128, 256)]), ("fwd_kernel.hip", ["fwd_tall_kernel"])):
        out = str(tmp_path / "kernels.s")
        r = subprocess.run([HIPCC, *FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, src), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        text = open(out).read()
        for name in names:
            at = re.search(r"^\S*%s\S*:" % name, text, re.M).end()
            blocks = re.split(r"^\.LBB\S+:", text[at:text.index(".Lfunc_end", at)], flags=re.M)
            steps = [b for b in blocks if b.count("v_mfma") >= 4]
            assert steps and not any("scratch_" in b for b in steps), name

"""CPU-only tests of the C ABI: the library loads, exports every symbol the header declares, and rejects bad
descriptors on the host with the documented codes (no GPU is touched)."""
import ctypes
import os
import re

import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ca():
    import paper_2509_21275_amd as ca
    if not os.path.exists(ca.LIB_PATH):
        from paper_2509_21275_amd.build import build_library
        build_library()
    return ca


def test_library_exports_every_declared_symbol(ca):
    names = set()
    for h in sorted(os.listdir(os.path.join(ROOT, "include"))):
        header = open(os.path.join(ROOT, "include", h)).read()
        header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
        names |= set(re.findall(r"\b((?:chunk_attn|chunk_plan|chunk_sched|fused_ce)_[a-z0-9_]+)\s*\(", header))
    assert {"chunk_attn_fwd", "chunk_attn_bwd", "chunk_attn_bwd_f32kv", "chunk_attn_workspace_bytes", "chunk_attn_validate",
            "chunk_attn_pair_count", "chunk_attn_strerror", "chunk_attn_profile_events", "chunk_attn_shutdown",
            "chunk_attn_test_set_fwd_rescale_limit",
            "chunk_plan_time", "chunk_plan_mesh", "chunk_plan_build", "chunk_plan_segments", "fused_ce_inplace",
            "chunk_sched_act_bytes", "chunk_sched_f2b", "chunk_sched_windows", "chunk_sched_solve_ckpt", "chunk_sched_group",
            "chunk_sched_simulate", "chunk_sched_plan_batch"} <= names
    lib = ctypes.CDLL(ca.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), f"{n} declared in the header but not exported"


def desc(ca, segs, Hq=8, Hkv=2, d=128, tq=None, tkv=None, scale=0.1):
    tq = tq if tq is not None else max(s[0] + s[1] for s in segs)
    tkv = tkv if tkv is not None else max(s[2] + s[3] for s in segs)
    return ca.make_desc(segs, Hq, Hkv, d, tq, tkv, scale)


def test_valid_descriptors(ca):
    for idx in range(1, 6):
        c = synth.case_by_index(idx)
        d = ca.make_desc(c.segs, c.num_q_heads, c.num_kv_heads, c.head_dim, c.total_q, c.total_kv, c.scale)
        assert ca.chunk_attn_validate(d) == ca.OK
        assert ca.chunk_attn_pair_count(d) == c.pairs
        f, b = ca.chunk_attn_workspace_bytes(d)
        assert f > 0 and b > 0 and f % 256 == 0 and b % 256 == 0
    # key ranges may leave gaps; a hybrid chunk is legal; so are several segments with context
    assert ca.chunk_attn_validate(desc(ca, [(0, 4, 3, 10), (4, 6, 20, 9)], tkv=40)) == ca.OK


def test_head_dimensions(ca):
    """64, 96, 128 and 256 are accepted; a workspace for 96 has the size of one for 128 plus zero-padded copies
    of the tensors, which the one-pass backward runs on (Q, K, V, O for the forward; Q, K, V, O, dO, dQ and float32-sized dK, dV for the
    backward)."""
    segs = [(0, 300, 0, 500), (300, 212, 500, 212)]
    sizes = {}
    for d in (64, 96, 128, 256):
        dd = desc(ca, segs, Hq=8, Hkv=2, d=d)
        assert ca.chunk_attn_validate(dd) == ca.OK
        assert ca.chunk_attn_pair_count(dd) == 300 * 200 + 300 * 301 // 2 + 212 * 213 // 2
        sizes[d] = ca.chunk_attn_workspace_bytes(dd)
    up = lambda x: (x + 255) // 256 * 256
    qb, kb, gb = up(512 * 8 * 128 * 2), up(712 * 2 * 128 * 2), up(712 * 2 * 128 * 4)
    assert sizes[96][0] == sizes[128][0] + 2 * qb + 2 * kb
    assert sizes[96][1] == sizes[128][1] + 4 * qb + 2 * kb + 2 * gb
    for d in (32, 80, 192, 512):
        assert ca.chunk_attn_validate(desc(ca, segs, d=d)) == ca.UNSUPPORTED
    assert "64, 96, 128 or 256" in ca.chunk_attn_strerror(ca.UNSUPPORTED)


@pytest.mark.parametrize("segs,Hq,Hkv,dim", [
    ([(0, 1024, 0, 32768)], 32, 8, 128), ([(0, 1024, 0, 32768)], 32, 8, 96),   # dQ walks are cut
    ([(0, 4999, 0, 4999)], 32, 8, 128), ([(0, 1100, 5, 1400), (1100, 77, 1410, 77)], 6, 2, 96),  # dK/dV walks are cut
    ([(0, 300, 0, 300)], 32, 8, 128), ([(0, 300, 0, 700)], 8, 2, 64),
])
def test_workspace_size_does_not_depend_on_the_backward_mode(ca, segs, Hq, Hkv, dim):
    """The mode may change between the size query and the call (include/chunk_attn.h)."""
    d, lib = desc(ca, segs, Hq=Hq, Hkv=Hkv, d=dim), ctypes.CDLL(ca.LIB_PATH)
    try:
        sizes = []
        for mode in (0, 1, 2):
            assert lib.chunk_attn_test_set_bwd_mode(mode) == ca.OK
            sizes.append(ca.chunk_attn_workspace_bytes(d))
    finally:
        lib.chunk_attn_test_set_bwd_mode(0)
    assert sizes[0] == sizes[1] == sizes[2]


def packed(*lens):
    segs, at = [], 0
    for n in lens:
        segs.append((at, n, at, n))
        at += n
    return segs


@pytest.mark.parametrize("segs,Hq,Hkv,dim,fwd,dq,dkv", [
    # "": the plain kernel, "p": pipelined, "pc": pipelined with cut walks
    ([(0, 8192, 0, 32768)], 32, 8, 128, "p", "p", "p"),           # enough blocks: nothing is cut
    ([(0, 1024, 0, 32768)], 32, 8, 128, "pc", "p", "p"),           # (of the backward's walks those of one kind fill the gaps of the other's)
    ([(0, 4999, 0, 4999)], 32, 8, 128, "p", "p", "p"),
    ([(0, 1024, 0, 32768)], 32, 8, 96, "pc", "p", "p"),
    ([(0, 300, 0, 4000)], 8, 2, 128, "pc", "pc", "p"), ([(0, 1300, 0, 1300)], 8, 2, 96, "pc", "p", "pc"),
    ([(0, 3823, 0, 9114)], 8, 2, 128, "p", "pc", "pc"),
    (packed(*[4096] * 4), 32, 8, 64, "p", "p", "p"),
    (packed(256, 512, 128, 128), 8, 8, 64, "", "", ""),
    (packed(*[4096] * 4), 32, 8, 256, "", "", "p"),
    (packed(256, 512, 128, 128), 8, 8, 256, "", "", ""),
    # head dimension 64: blocks enough for the pipelined forward and dQ, but too few for their longest walk or their mean one
    (packed(*[6000] * 3), 8, 8, 64, "", "", "p"), ([(0, 5000, 0, 6000)], 32, 8, 64, "", "", ""),
    ([(0, 2048, 0, 16384)], 64, 8, 64, "p", "p", "p"), (packed(*[3000] * 10), 32, 8, 64, "p", "p", "p"),
    (packed(*[2048] * 8), 32, 8, 64, "", "", "p"),
    # (no walk of head dimension 64 is cut)
    ([(0, 3032, 0, 51484)], 64, 64, 64, "p", "p", "p"),
    # one or two long causal sequences that barely fill the chip
    (packed(4096, 4096), 32, 8, 64, "p", "p", ""), (packed(8192), 8, 8, 64, "", "", ""), (packed(16384, 16384), 8, 2, 64, "p", "p", ""),
    (packed(*[2048] * 4), 32, 8, 64, "", "", "p"), (packed(*[4096] * 3), 32, 8, 64, "p", "p", "p"), ([(0, 1024, 0, 8192)], 32, 8, 64, "", "", "p"),
    # many key blocks, but too little to walk for the pipelined dK/dV kernels
    (packed(*[70] * 64), 8, 8, 64, "", "", ""), (packed(*[128] * 64), 32, 8, 64, "", "", ""),
    (packed(*[256] * 64), 32, 8, 64, "", "", "p"), ([(0, 512, 0, 16896)], 8, 8, 64, "", "", "p"),
    (packed(*[70] * 64), 8, 8, 256, "", "", ""), ([(0, 64, 0, 4160)], 32, 8, 256, "", "", ""),
    (packed(*[200] * 32), 32, 8, 256, "", "", "p"),
])
def test_routes(ca, segs, Hq, Hkv, dim, fwd, dq, dkv):
    """Which kernels a chunk runs; the tests on the GPU assert with the same hook that they reach the path they are named for.  The table is that of mode 1:
    by default some of the small chunks run the kernels made for them, and the hook then says so and nothing of the kernels that do not run."""
    bits = {"": 0, "p": 1, "pc": 3}
    d = desc(ca, segs, Hq=Hq, Hkv=Hkv, d=dim)
    forward, backward = bits[fwd], bits[dq] << 2 | bits[dkv] << 4
    ca.chunk_attn_test_set_bwd_mode(1)
    try:
        assert ca.chunk_attn_test_routes(d) == forward | backward
        assert ca.chunk_attn_test_shared_heads(d) == ca.chunk_attn_test_shared_waves(d) == 0
    finally:
        ca.chunk_attn_test_set_bwd_mode(0)
    if ca.chunk_attn_test_shared_heads(d):
        forward = ca.ROUTE_FWD_SHARED
    if ca.chunk_attn_test_shared_waves(d):
        backward = ca.ROUTE_BWD_SHARED
    assert ca.chunk_attn_test_routes(d) == forward | backward
    assert (ca.ROUTE_FWD_CUT, ca.ROUTE_DQ_PIPELINED, ca.ROUTE_DKV_PIPELINED, ca.ROUTE_ONE_PASS) == (2, 4, 16, 64)
    assert (ca.ROUTE_FWD_SHARED, ca.ROUTE_BWD_SHARED) == (128, 256)


@pytest.mark.parametrize("dim,Hq,Hkv,segs,heads,waves", [
    # few queries on thousands of keys: the other kernels cut these walks over the whole chip, and were up to 1.7 times as fast
    (96, 64, 64, [(0, 13, 0, 14478)], 0, 0), (128, 32, 32, [(0, 33, 0, 7207), (33, 13, 7207, 17827)], 0, 0), (128, 128, 16, [(0, 4, 0, 7246)], 0, 0),
    (128, 1, 1, [(0, 4, 0, 3733)], 0, 0), (128, 64, 8, [(0, 7, 0, 2747)], None, 0), (96, 64, 8, [(0, 15, 0, 2381)], None, 0),
    (96, 32, 8, [(0, 38, 0, 2460)], None, 0), (128, 128, 16, [(0, 2, 0, 1125), (2, 15, 1125, 426)], None, 0), (128, 8, 8, [(0, 499, 0, 2440)], None, 0),
    # many short walks of many key/value heads
    (128, 64, 64, packed(51, 26, *[89] * 25), None, 0), (128, 64, 64, [(0, 189, 0, 264)], None, 0),
    # and what they are for
    (64, 8, 8, packed(256, 512, 128, 128), 1, 4), (64, 32, 8, [(0, 100, 0, 10100)], 1, 4), (96, 8, 8, packed(500), 1, 4), (128, 8, 8, packed(500), 1, 4),
    (128, 32, 8, [(0, 203, 0, 1704), (203, 246, 1704, 246), (449, 145, 1950, 145), (594, 220, 2095, 220)], 2, 0), (128, 32, 8, packed(*[128] * 8), 4, None),
])
def test_small_chunks_run_the_shared_kernels_where_those_are_faster(ca, dim, Hq, Hkv, segs, heads, waves):
    d = desc(ca, segs, Hq=Hq, Hkv=Hkv, d=dim)
    if heads is not None:
        assert ca.chunk_attn_test_shared_heads(d) == heads
    if waves is not None:
        assert ca.chunk_attn_test_shared_waves(d) == waves
    assert bool(ca.chunk_attn_test_routes(d) & ca.ROUTE_FWD_SHARED) == bool(ca.chunk_attn_test_shared_heads(d))
    assert bool(ca.chunk_attn_test_routes(d) & ca.ROUTE_BWD_SHARED) == bool(ca.chunk_attn_test_shared_waves(d))


def contexts(n, last=288):
    """n segments of 32 queries on 288 keys (10 tiles of 32 rows each), the last one on `last` keys."""
    return [(32 * i, 32, 288 * i, last if i == n - 1 else 288) for i in range(n)]


@pytest.mark.parametrize("dim", [64, 96, 128])
def test_bounds_of_the_small_chunks_kernels(ca, dim):
    """What their kernel arguments have room for (104 tiles of 32 query rows in the forward; 64 segments, 640 tiles of queries and keys in the
    backward), and the number of heads up to which their offsets stay in 32 bits: taken at the bound, left to the other kernels one past it."""
    heads = lambda segs, Hq=1, Hkv=1: ca.chunk_attn_test_shared_heads(desc(ca, segs, Hq, Hkv, dim))
    waves = lambda segs, Hq=1, Hkv=1: ca.chunk_attn_test_shared_waves(desc(ca, segs, Hq, Hkv, dim))
    assert heads(packed(*[20] * 104)) == 1 and heads(packed(*[20] * 105)) == 0
    assert heads(packed(*[20] * 103, 33)) == 0
    assert waves(packed(*[20] * 64)) == 4 and waves(packed(*[20] * 65)) == 0
    assert waves(contexts(64)) == 4 and waves(contexts(64, last=289)) == 0
    one = [(0, 1, 0, 1)]
    assert waves(one, 4096, 8) > 0 and waves(one, 8192, 8) == 0
    assert heads(one, 8192, 8) == 0 and (dim == 64 or heads(one, 4096, 8) == 4)


@pytest.mark.parametrize("segs,kw,code", [
    ([(0, 0, 0, 4)], {"tq": 4}, "BAD_SEGMENT"),                        # empty query range
    ([(0, 8, 0, 4)], {}, "BAD_SEGMENT"),                          # fewer keys than queries
    ([(1, 4, 0, 4)], {"tq": 5}, "BAD_SEGMENT"),                   # queries must start at row 0
    ([(0, 4, 0, 4), (5, 4, 4, 4)], {}, "BAD_SEGMENT"),            # hole in the query rows
    ([(0, 4, 0, 4), (4, 4, 2, 4)], {}, "BAD_SEGMENT"),            # overlapping key ranges
    ([(0, 4, 0, 4)], {"tq": 6}, "BAD_SEGMENT"),                   # queries do not cover total_q
    ([(0, 4, 0, 8)], {"tkv": 6}, "BAD_SEGMENT"),                  # key range past total_kv
    ([(0, 4, 0, 4)], {"d": 80}, "UNSUPPORTED"),
    ([(0, 4, 0, 4)], {"Hq": 6, "Hkv": 4}, "UNSUPPORTED"),
    ([(0, 4, 0, 4)], {"scale": 0.0}, "INVALID_ARG"),
    ([(0, 4, 0, 4)], {"scale": float("nan")}, "INVALID_ARG"),
    ([(0, 4, 0, 4)], {"Hq": 0}, "INVALID_ARG"),
])
def test_bad_descriptors(ca, segs, kw, code):
    d = desc(ca, segs, **kw)
    rc = ca.chunk_attn_validate(d)
    assert rc == getattr(ca, code), ca.chunk_attn_strerror(rc)
    with pytest.raises(ca.ChunkAttnError):
        ca.chunk_attn_workspace_bytes(d)
    with pytest.raises(ca.ChunkAttnError):
        ca.chunk_attn_pair_count(d)


def test_null_descriptor_and_messages(ca):
    lib = ctypes.CDLL(ca.LIB_PATH)
    lib.chunk_attn_validate.restype = ctypes.c_int
    assert lib.chunk_attn_validate(None) == ca.INVALID_ARG
    for code in (0, -1, -2, -3, -4, -5, -99):
        assert isinstance(ca.chunk_attn_strerror(code), str) and ca.chunk_attn_strerror(code)


def test_clock_log_hook_checks_its_buffer(ca):
    """The hook only stores the pointer: size and alignment are checked on the host, null switches it off."""
    import ctypes
    lib = ctypes.CDLL(ca.LIB_PATH)
    lib.chunk_attn_measure_set_clock_log.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    lib.chunk_attn_measure_set_clock_log.restype = ctypes.c_int
    assert ca.CLOCK_LOG_BYTES == 3 * 4096 * 8
    assert lib.chunk_attn_measure_set_clock_log(None, 0) == ca.OK
    assert lib.chunk_attn_measure_set_clock_log(ctypes.c_void_p(4096), ca.CLOCK_LOG_BYTES - 1) == ca.WORKSPACE_TOO_SMALL
    assert lib.chunk_attn_measure_set_clock_log(ctypes.c_void_p(4100), ca.CLOCK_LOG_BYTES) == ca.INVALID_ARG
    assert lib.chunk_attn_measure_set_clock_log(None, 0) == ca.OK


def test_shutdown_without_any_upload_is_a_no_op(ca):
    # nothing has been uploaded in this process: there is nothing to release, and no GPU call is made
    lib = ctypes.CDLL(ca.LIB_PATH)
    assert lib.chunk_attn_shutdown() == ca.OK
    assert lib.chunk_attn_shutdown() == ca.OK
    ca.chunk_attn_shutdown()


def test_synthetic_workloads_have_the_documented_shapes():
    c3 = synth.case_by_index(3); c4 = synth.case_by_index(4)
    assert c3.segs[0] == synth.Seg(0, 8192, 0, 65536) and c3.total_q == 16384 and c3.total_kv == 73728
    assert all(s.kv_len == s.q_len and 1 <= s.q_len <= 4096 for s in c3.segs[1:])
    assert sum(s.q_len for s in c4.segs) == 65536 and all(s.q_len <= 16384 for s in c4.segs)
    assert all(s.q_len >= 128 for s in c4.segs[:-1])
    for i in range(8):
        c5 = synth.case_by_index(5, i)
        assert c5.segs == [synth.Seg(0, 16384, 0, 16384 * (i + 1))]
    # determinism of the tensor generator: same (seed, id, index) -> same value, independent of blocking
    import torch
    a = synth.normal_bf16(7, 3, (5000,)); b = synth.normal_bf16(7, 3, (5000,), block=777)
    assert torch.equal(a, b)

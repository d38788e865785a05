"""Which blocks the estimates choose for chunks whose other blocks were measured to be faster, and what the choice costs the host."""
import os
import shutil
import subprocess
import time

import pytest

import paper_2509_21275_amd as ca


def _desc(segs, hq, hk, d):
    return ca.make_desc(segs, hq, hk, d, sum(s[1] for s in segs), segs[-1][2] + segs[-1][3], d ** -0.5)


def _packed(count, length):
    return [(length * i, length, length * i, length) for i in range(count)]


@pytest.mark.parametrize("count,length,hq,hk", [(350, 146, 28, 4), (145, 150, 28, 4), (348, 148, 8, 2)])
def test_blocks_are_numbered_as_they_start(count, length, hq, hk):
    """Two key blocks to a sequence, a long one and a short one, two or four key/value heads: every eighth block of a launch is as often one as the other."""
    assert ca.chunk_attn_test_dkv_keys(_desc(_packed(count, length), hq, hk, 128)) == 128


@pytest.mark.parametrize("count,length,hq,hk,d", [
    (94, 178, 32, 8, 128), (129, 222, 40, 8, 128), (126, 213, 32, 8, 128),    # 256 keys end as late as 128 by the estimate
    (10, 560, 32, 8, 128), (125, 255, 40, 8, 96)])
def test_equal_estimates_keep_the_smaller_blocks(count, length, hq, hk, d):
    assert ca.chunk_attn_test_dkv_keys(_desc(_packed(count, length), hq, hk, d)) == 128


@pytest.mark.parametrize("count,length,heads,d", [(8, 300, 64, 128), (8, 300, 64, 96), (32, 300, 16, 128), (8, 360, 64, 128), (40, 300, 64, 128)])
def test_a_query_head_to_a_key_value_head(count, length, heads, d):
    """Chunks that blocks of 256 keys make faster by 4 to 8 %."""
    assert ca.chunk_attn_test_dkv_keys(_desc(_packed(count, length), heads, heads, d)) == 256


@pytest.mark.parametrize("count,length,hq,hk", [
    (62, 241, 28, 4), (228, 256, 28, 4), (250, 235, 8, 8), (161, 101, 32, 8), (75, 124, 64, 8),  # short walks
    (8, 1520, 8, 8), (9, 1428, 8, 2), (11, 701, 8, 8)])                                                            # the last sequences' long blocks start late
def test_forward_of_256_keeps_32_rows(count, length, hq, hk):
    assert ca.chunk_attn_test_fwd_rows(_desc(_packed(count, length), hq, hk, 256)) == 32


@pytest.mark.parametrize("segs,hq,hk", [(_packed(8, 255), 28, 4), (_packed(9, 369), 16, 8), ([(0, 2214, 0, 7168)], 16, 16)])
def test_forward_of_256_whose_blocks_all_start_at_once(segs, hq, hk):
    """No more blocks of 64 rows per wave than compute units: faster by 14 to 17 %."""
    assert ca.chunk_attn_test_fwd_rows(_desc(segs, hq, hk, 256)) == 64


@pytest.mark.parametrize("segs,hq,hk,keys", [
    (_packed(166, 57), 28, 4, 64), (_packed(331, 51), 28, 4, 64), (_packed(278, 70), 28, 4, 128),   # a block of 128 keys would be half empty, or not
    (_packed(10, 200), 4, 4, 64), (_packed(11, 200), 4, 4, 64), (_packed(15, 352), 8, 8, 64), (_packed(15, 370), 8, 8, 128),   # dQ walks of 5.5, of 7.7 and of 8 stages
    ([(0, 371, 0, 2337)] + [(371 + 172 * i, 172, 2337 + 172 * i, 172) for i in range(19)], 8, 2, 64)])  # ahead by less than the estimates are off by
def test_blocks_of_256_that_stay(segs, hq, hk, keys):
    assert ca.chunk_attn_test_dkv_keys(_desc(segs, hq, hk, 256)) == keys


@pytest.mark.parametrize("d,keys,in_step", [(128, 256, True), (96, 256, True), (64, 256, False)])
def test_long_walks_that_start_in_groups(d, keys, in_step):
    desc = _desc([(0, 8192, 0, 16384)], 64, 8, d)
    assert ca.chunk_attn_test_dkv_keys(desc) == keys and ca.chunk_attn_test_dkv_in_step(desc) == in_step


@pytest.mark.parametrize("segs,hq,hk,keys", [
    ([(0, 16317, 0, 16594)], 16, 16, 128), ([(0, 12000, 0, 12000)], 32, 32, 128),                       # a query head to a key/value head: two launches
    ([(0, 12000, 0, 12000)], 32, 16, 256), ([(0, 223, 0, 5186)], 512, 256, 256), ([(0, 451, 0, 9405)], 512, 128, 256)])  # several: one, walks of few steps, too
def test_one_launch_of_64(segs, hq, hk, keys):
    assert ca.chunk_attn_test_dkv_keys(_desc(segs, hq, hk, 64)) == keys


def test_walks_are_counted_by_segment(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    root, exe = os.path.dirname(os.path.dirname(os.path.abspath(__file__))), str(tmp_path / "walk_counts")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(root, "include"), os.path.join(root, "tests", "native", "walk_counts.cpp"),
                        os.path.join(root, "paper_2509_21275_amd", "csrc", "plan.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:]


@pytest.mark.parametrize("d", [96, 128, 256])
def test_large_chunks_cost_the_choice_no_list(d):
    """2^27 query rows (a list of their blocks took seconds and gigabytes) in less than 20 ms, most of it the tiles' parities at 256."""
    desc = _desc([(0, 1 << 27, 0, 1 << 27)], 64, 64, d)
    best = 1.0
    for _ in range(5):
        begin = time.perf_counter()
        ca.chunk_attn_workspace_bytes(desc)
        best = min(best, time.perf_counter() - begin)
    assert best < 0.02


@pytest.mark.parametrize("segs,heads", [
    ([(0, 11481, 0, 11581)] + [(11481 + 292 * i, 292, 11581 + 292 * i, 292) for i in range(22)], 8),   # faster by 8 %
    ([(0, 5863, 0, 10447)] + [(5863 + 190 * i, 190, 10447 + 190 * i, 190) for i in range(3)], 8)])
def test_dq_blocks_that_start_first(segs, heads):
    assert ca.chunk_attn_test_dkv_keys(_desc(segs, heads, heads, 128)) == 256

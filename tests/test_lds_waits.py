"""LDS reads written as instructions (lds_asm_read*) are invisible to the compiler: a register they fill may be used only after
an s_waitcnt that covers the read, and only naming the register in that statement (or in an empty one behind it) keeps the
compiler from moving the use in front of it.  This looks at the source of every pipelined step, and of the small chunks' kernels: each
array that a read fills is an operand of a wait in the same step or kernel."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_21275_amd.build import FLAGS

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_21275_amd", "csrc")


def bodies(text, head):
    """Bodies of the lambdas or functions that start with `head` (a pattern up to the parameters)."""
    for m in re.finditer(head, text):
        at = text.index("{", m.end())
        depth, i = 0, at
        while True:
            depth += {"{": 1, "}": -1}.get(text[i], 0)
            i += 1
            if depth == 0:
                break
        yield text[at:i], text.count("\n", 0, at) + 1


def statements(body):
    """Operand texts of the asm statements that wait for LDS reads or stand for one that did (empty, tying registers)."""
    for m in re.finditer(r'asm volatile\("((?:[^"\\]|\\.)*)"', body):
        end, depth = m.start() + len("asm volatile"), 0
        while True:
            depth += {"(": 1, ")": -1}.get(body[end], 0)
            end += 1
            if depth == 0:
                break
        if "lgkmcnt" in m.group(1) or m.group(1) == "":
            yield body[m.end():end]


@pytest.mark.parametrize("source", ["fwd_kernel.hip", "bwd_kernel.hip", "bwd_fused_kernel.hip"])
def test_every_array_read_in_a_step_is_tied_to_a_wait(source):
    text = open(os.path.join(CSRC, source)).read()
    steps = list(bodies(text, r"auto step = \[&\]"))
    found = 0
    for body, line in steps:
        filled = set(re.findall(r"\b(\w+)(?:\[[^=;]*\])? = (?:lds_asm_read\w*|load_\w+)\b", body))
        found += len(filled)
        tied = set(re.findall(r'"\+v"\((\w+)', " ".join(statements(body))))
        assert filled <= tied, f"{source}:{line}: {sorted(filled - tied)} read from LDS, but no wait names them"
    assert found >= 1


@pytest.mark.parametrize("source,kernel,arrays", [("fwd_kernel.hip", "fwd_share_kernel", 4), ("bwd_share_kernel.hip", "share_dq_block", 8),
                                                 ("bwd_share_kernel.hip", "share_dkv_block", 11)])
def test_every_array_read_in_a_small_chunks_kernel_is_tied_to_a_wait(source, kernel, arrays):
    text = open(os.path.join(CSRC, source)).read()
    (body, line), = bodies(text, r"void %s\(" % kernel)
    filled = set(re.findall(r"\b(\w+)(?:\[[^=;]*\])? = lds_asm_read\w*\b", body)) | set(re.findall(r'asm volatile\("ds_read[^"]*" : "=v"\((\w+)', body))
    tied = set(re.findall(r'"\+v"\((\w+)', " ".join(statements(body))))
    assert len(filled) == arrays, sorted(filled)
    assert filled <= tied, f"{source}:{line}: {sorted(filled - tied)} read from LDS, but no wait names them"


HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_unpipelined_dkv_steps_wait_for_their_reads_one_by_one(tmp_path):
    """Each of bwd_dkv_kernel's four unrolled steps starts its vector work on the first of its reads while five later ones are still
    out.  (The compiler places these waits; it waits for all reads at once where it has lost count of them.)"""
    out = str(tmp_path / "bwd.s")
    r = subprocess.run([HIPCC, *FLAGS, "-x", "hip", "--cuda-device-only", "-S", os.path.join(CSRC, "bwd_kernel.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = open(out).read()
    for name in ("bwd_dkv_kernelILi64ELi4ELb0", "bwd_dkv_kernelILi64ELi4ELb1", "bwd_short_kernelILi64ELi4ELb0", "bwd_short_kernelILi64ELi4ELb1"):
        at = re.search(r"^\S*%s\S*:" % name, text, re.M).end()
        body = text[at:text.index(".Lfunc_end", at)]
        assert body.count("lgkmcnt(5)") >= 4, name

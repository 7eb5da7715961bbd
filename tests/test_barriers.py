"""The kernels wait for what a wavefront has written to LDS before it reaches a barrier, in the code that the compiler emits.

A barrier does not wait for a wavefront's own LDS writes; the wait is an instruction in front of it, which the compiler places and once
left out where the barrier is reached over a loop's back edge.  The test compiles every source to assembly and follows every path.
"""
import functools
import os
import re
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2604_11288_amd import build


def _lines(text):
    """A kernel's instructions and labels, and where each label stands."""
    lines = [re.sub(r"\s+", " ", line.split(";")[0]).strip() for line in text.split("\n")]
    lines = [line for line in lines if line and (not line.startswith(".") or line.startswith(".LBB"))]
    return lines, {line[:-1]: i for i, line in enumerate(lines) if line.endswith(":")}


def _passable(text):
    """Lines of the barriers that a path reaches with an LDS write outstanding."""
    lines, label = _lines(text)
    seen, todo, found = {}, [(0, False)], set()
    while todo:
        i, pending = todo.pop()
        while i < len(lines) and not (i in seen and (seen[i] or not pending)):
            seen[i] = pending or seen.get(i, False)
            op, _, rest = lines[i].partition(" ")
            if op.startswith("ds_") and not op.startswith(("ds_read", "ds_bpermute", "ds_permute", "ds_swizzle")):
                pending = True
            elif op == "s_waitcnt" and "lgkmcnt(0)" in rest:
                pending = False
            elif op == "s_barrier" and pending:
                found.add(i)
            elif op == "s_endpgm":
                break
            elif op == "s_branch":
                i = label[rest]
                continue
            elif op.startswith("s_cbranch"):
                todo.append((label[rest], pending))
            i += 1
    return sorted(found)


def _polls(text):
    """Lines by which a workgroup may wait for another one: a sleep, or a read past the caches that workgroups do not share from
    which a path leads back to it."""
    lines, label = _lines(text)
    found = [i for i, line in enumerate(lines) if line.startswith("s_sleep")]
    for read in (i for i, line in enumerate(lines) if re.match(r"(global|flat|buffer)_load.*\bsc1\b", line)):
        seen, todo = set(), [read + 1]
        while todo:
            i = todo.pop()
            while i < len(lines) and i not in seen:
                seen.add(i)
                op, _, rest = lines[i].partition(" ")
                if op == "s_endpgm":
                    break
                if op == "s_branch":
                    i = label[rest]
                    continue
                if op.startswith("s_cbranch"):
                    todo.append(label[rest])
                i += 1
        if read in seen:
            found.append(read)
    return found


def test_the_check_finds_a_missing_wait():
    body = "k:\n.LBB0_1:\n%ss_barrier\nds_write_b32 v0, v1\ns_cbranch_scc0 .LBB0_1\ns_endpgm\n"
    assert _passable(body % "") and not _passable(body % "s_waitcnt lgkmcnt(0)\n")


def test_the_check_finds_a_wait_for_another_workgroup():
    body = "k:\n.LBB0_1:\nglobal_load_dword v0, v1, s[0:1]%s\ns_cbranch_vccz .LBB0_%d\ns_nop 0\n.LBB0_2:\ns_endpgm\n"
    assert _polls(body % (" sc1", 1)) and not _polls(body % (" sc1", 2)) and not _polls(body % ("", 1))


@functools.lru_cache(maxsize=None)
def _emitted():
    """The text that the compiler emits for every source, by source."""
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as tmp:
        def emit(source):
            out = os.path.join(tmp, source + ".s")
            subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", out],
                           check=True, stderr=subprocess.DEVNULL)
            with open(out) as f:
                return f.read()
        with ThreadPoolExecutor(max_workers=len(build.SOURCES)) as pool:
            return dict(zip(build.SOURCES, pool.map(emit, build.SOURCES)))


def _kernels(source):
    """(name, emitted text) of a source's kernels."""
    text = _emitted()[source]
    return [(m.group(1), text[m.start():text.index(".Lfunc_end", m.start())]) for m in re.finditer(r"^(_Z\S+):\s*; @", text, re.M)]


needs_hipcc = pytest.mark.skipif(shutil.which(build.HIPCC) is None and not os.path.exists(build.HIPCC), reason="no hipcc")
AT_LEAST = {"ta_api.hip": 0, "ta_score.hip": 20, "ta_select.hip": 30, "ta_decode.hip": 50}       # kernels of a source; of the others one


@needs_hipcc
@pytest.mark.parametrize("source", build.SOURCES)
def test_kernels_wait_for_lds_writes(source):
    kernels = _kernels(source)
    assert len(kernels) >= AT_LEAST.get(source, 1)
    assert not [name for name, body in kernels if _passable(body)]


@needs_hipcc
def test_no_workgroup_of_a_generation_step_waits_for_another():
    """Steps of different states may overlap on one GPU: a workgroup that waited could hold the place of the one it waits for."""
    kernels = _kernels("ta_decode.hip")
    assert len(kernels) > 50
    assert not [name for name, body in kernels if _polls(body)]

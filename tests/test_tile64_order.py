"""The order of the 64-row kernel's requests to raise a maximum, on the CPU.

Two waves run the accesses that one step of the kernel makes to the requests
(a barrier, the read of those of stage i, the write of its own for stage i + 1)
in every order that the barriers allow.  A wave must always read the request
that the other one wrote for the stage of its step, wherever it is held back.
The places come from the kernel's own header, compiled here, and the kernel's
source names a place only through it.
"""
import os
import re
import subprocess

import pytest

from paper_2606_01502_amd import build as B

N_STAGES = 5


def _places(tmp_path):
    src = tmp_path / "places.cc"
    src.write_text('#include "mla_kernels.h"\n#include <cstdio>\n'
                   "int main() { for (int i = 0; i < 16; ++i) "
                   'std::printf("%d %d\\n", mla::ask_place(i), mla::kAskBytes); }\n')
    exe = tmp_path / "places"
    rocm = os.path.dirname(os.path.dirname(B.HIPCC))
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", B.CSRC, "-o", str(exe), str(src)], check=True)
    rows = [tuple(map(int, ln.split()))
            for ln in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()]
    return [r[0] for r in rows], rows[0][1]


def _wrong_reads(place):
    """Reads of another stage's request over every interleaving of two waves."""
    # step i: meet the other wave, read the requests of stage i, write for i + 1
    prog = [("write", 0)]
    for i in range(N_STAGES):
        prog += [("meet", i), ("read", i)] + ([("write", i + 1)] if i + 1 < N_STAGES else [])
    wrong, seen = set(), set()
    # state: program counters, and each wave's bytes (place -> stage written)
    todo = [((0, 0), ((), ()))]
    while todo:
        state = todo.pop()
        if state in seen:
            continue
        seen.add(state)
        pcs, mem = state
        at = [prog[pc] if pc < len(prog) else ("end", -1) for pc in pcs]
        if at[0][0] == at[1][0] == "meet":
            todo.append(((pcs[0] + 1, pcs[1] + 1), mem))
            continue
        for w in (0, 1):
            op, stage = at[w]
            if op in ("meet", "end"):
                continue
            new = list(mem)
            if op == "write":
                d = dict(mem[w])
                d[place(stage)] = stage
                new[w] = tuple(sorted(d.items()))
            elif dict(mem[1 - w]).get(place(stage)) != stage:
                wrong.add((w, stage))
            todo.append((tuple(pc + (k == w) for k, pc in enumerate(pcs)), tuple(new)))
    return wrong


def test_requests_are_read_before_they_are_written_again(tmp_path):
    places, size = _places(tmp_path)
    assert size == 64 * 8  # a byte per lane and wave
    # stages that share a place share all of it, others nothing
    assert all(a == b or abs(a - b) >= size for a in places for b in places)
    assert max(places) + size == 2 * size
    assert _wrong_reads(lambda i: places[i]) == set()


def test_one_place_for_all_stages_is_found_out():
    assert _wrong_reads(lambda i: 0)


def test_kernel_names_the_place_by_the_stage():
    with open(os.path.join(B.CSRC, "mla_partial.hip")) as f:
        src = re.sub(r"//[^\n]*", "", f.read())
    # one way to the requests' bytes, and the stage of every use
    assert src.count("L::kAsk") == 1 and "smem + L::kAsk + ask_place(stage)" in src
    uses = re.findall(r"\basks\(([^)]*)\)", src)
    assert sorted(uses) == ["i", "i", "stage", "stage"]
    # written in the softmax of the stage after the step's, read in the step's own
    assert "soft(f, i + 1)" in src

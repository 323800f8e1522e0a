"""The PQ decode scorer and the residual scorer keep tiles in LDS rings that
direct-to-LDS loads refill. Those loads are inline assembly, so the compiler
orders nothing between them and the LDS reads of a slot: the sources have to
state the wait. Build both files to gfx950 assembly on the CPU and follow every
path from each LDS read to the loads after it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# LDS-DMA loads that may follow a read before the wait: a step of the PQ ring
# reads slot k + 1, refills slot k with one load and waits before the next
# step's load refills slot k + 1; a residual slot is read and refilled in one
# step.
RUNS = {"pq_mfma": 1, "residual": 0}
clobbers, scratch = {}, {}


@pytest.fixture(scope="module", params=sorted(RUNS))
def program(request, tmp_path_factory):
    """(file, instructions as (text, whether from inline assembly), labels)."""
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    src = os.path.join(ROOT, "paper_2606_26439_amd", "csrc", request.param + ".hip")
    out = tmp_path_factory.mktemp("asm") / (request.param + ".s")
    cmd = [HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
           "-Xclang", "-packed-fp32-ops", "-fno-honor-nans", "-I", os.path.join(ROOT, "include"),
           "-x", "hip", "--cuda-device-only", "-S", src, "-o", str(out)]
    r = subprocess.run(cmd, check=True, capture_output=True, text=True)
    clobbers[request.param] = [ln for ln in r.stderr.splitlines() if "clobber" in ln]
    ins, labels, inline = [], {}, False
    scratch[request.param] = [int(n) for n in re.findall(r"^; ScratchSize: (\d+)", out.read_text(),
                                                         re.M)]
    for ln in out.read_text().splitlines():
        if "#ASMSTART" in ln or "#ASMEND" in ln:
            inline = "#ASMSTART" in ln
            continue
        ln = ln.split(";")[0].strip()
        if ln.endswith(":"):
            labels[ln[:-1]] = len(ins)
        elif ln and not ln.startswith("."):
            ins.append((ln, inline))
    return request.param, ins, labels


def _unwaited_loads(ins, labels, start):
    """The most LDS-DMA loads that a path from `start` meets before the wait
    that the source states (two or more count as two)."""
    todo, seen, most = [(start, 0)], set(), 0
    while todo:
        pos, n = todo.pop()
        while pos < len(ins) and (pos, n) not in seen:
            seen.add((pos, n))
            ln, inline = ins[pos]
            if inline and ln == "s_waitcnt lgkmcnt(0)":
                break
            if ln.startswith("global_load_lds"):
                n = min(n + 1, 2)
                most = max(most, n)
            m = re.match(r"s_(c?branch)\w*\s+(\S+)", ln)
            if m and m.group(2) in labels:
                if m.group(1) == "branch":
                    pos = labels[m.group(2)]
                    continue
                todo.append((labels[m.group(2)], n))
            elif ln.startswith(("s_endpgm", "s_setpc")):
                break
            pos += 1
    return most


def test_a_slot_is_refilled_only_after_the_wait_for_its_reads(program):
    name, ins, labels = program
    loads = [i for i, (ln, _) in enumerate(ins) if ln.startswith("global_load_lds")]
    assert len(loads) >= 16
    # the reads of a step: those that the ring's counted wait precedes
    starts = [i for i, (ln, inline) in enumerate(ins)
              if inline and re.match(r"s_waitcnt vmcnt\(\d+\)", ln)]
    assert len(starts) >= 4
    for i in starts:
        assert _unwaited_loads(ins, labels, i) <= RUNS[name], (name, i)


def test_m0_belongs_to_the_inline_loads(program):
    # they set it without saying so to the compiler, which may keep nothing
    # of its own there
    name, ins, _ = program
    assert not clobbers[name]
    assert not [ln for ln, inline in ins if not inline and re.search(r"\bm0\b", ln)]



def test_few_registers_spill(program):
    # a spilled operand of the inner loop comes back from memory for every tile
    # (residual, d = 256, 64 tokens: 2.5 to 6 times the time with 172 to 324 bytes)
    sizes = scratch[program[0]]
    assert len(sizes) >= 16 and max(sizes) <= 128

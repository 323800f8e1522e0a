"""The queries whose top-k parts a workgroup of the fused scorer writes, for
candidate offsets that keep the contract and for ones that break it: the
wave loop (which positions belong to which query) is followed here on the CPU,
its owner words go through the kernel's own scored_queries, and the result
has to stay inside [0, n_queries) and cover every query that was scored."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    out = tmp_path_factory.mktemp("owners") / "scored_queries"
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-w",
                    os.path.join(ROOT, "tests", "scored_queries_host.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    return str(out)


def _owner(off, n_q, p):
    """The last query starting at or before p by the search the kernel uses
    (-1: none)."""
    past = np.nonzero(np.asarray(off[:n_q + 1]) > p)[0]
    return int(past[0]) - 1 if past.size else n_q - 1


def _wave(off, n_q, lo, hi):
    """Pieces (query, first, end) of a wave's range, and its owner words."""
    pieces, first, last, p = [], -1, -1, lo
    while p < hi:
        a = _owner(off, n_q, p)
        end = off[a + 1]
        if a < 0:
            p = end
            continue
        if end <= p:
            break
        e = min(end, hi)
        pieces.append((a, p, e))
        if first < 0:
            first = a
        last = a
        p = e
    return pieces, first, last


@pytest.mark.parametrize("nw", [4, 8])
@pytest.mark.parametrize("off,n_total", [
    ([0, 10, 10, 60, 100], 100),     # the contract
    ([0, 100], 100),
    ([0, 0, 0, 100, 100], 100),
    ([0, 10, 20], 100),              # ends before the candidates do
    ([0, 0, 0], 100),                # no position owned at all
    ([40, 60, 100], 100),            # starts after the first candidate
    ([90, 95, 99], 100),
    ([0, 50, 400], 100),             # ends after the candidates do
    ([0, 80, 20, 60], 100),          # not ascending
])
def test_stays_inside_the_queries(program, nw, off, n_total):
    n_q = len(off) - 1
    lines, want = [], []
    for grid in (1, 2, 5):
        share = [n_total * w // (grid * nw) for w in range(grid * nw + 1)]
        for wg in range(grid):
            waves = [_wave(off, n_q, share[wg * nw + w], share[wg * nw + w + 1])
                     for w in range(nw)]
            lines.append(" ".join(map(str, [nw, n_q] + [w[1] for w in waves]
                                      + [w[2] for w in waves])))
            want.append({a for w in waves for a, _, _ in w[0]})
    out = subprocess.run([program], input="\n".join(lines) + "\n", text=True, check=True,
                         capture_output=True, timeout=60).stdout.split("\n")
    for got, scored in zip(out, want):
        any_, a0, a1 = map(int, got.split())
        assert any_ == (1 if scored else 0)
        if scored:
            assert 0 <= a0 and a1 < n_q
            if off == sorted(off):
                assert a0 == min(scored) and a1 == max(scored)


def test_words_past_the_last_query_are_cut(program):
    out = subprocess.run([program], input="4 3 -1 1 2 -1 -1 2 9 -1\n4 3 -1 -1 -1 -1 5 5 5 5\n",
                         text=True, check=True, capture_output=True, timeout=60).stdout.split("\n")
    assert out[0].split() == ["1", "1", "2"]
    assert out[1].split()[0] == "0"

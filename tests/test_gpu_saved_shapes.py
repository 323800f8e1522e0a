"""Launch shapes of the fused scorer that come from a tuning cache: which calls
a saved shape holds for, and that every call it holds for can run it."""
import json

import numpy as np
import pytest
import torch

import paper_2606_26439_amd as M
import workloads as W
from tests._gpu import dev, device_tokens

pytestmark = pytest.mark.gpu

_CODE = {"f32": 0, "bf16": 1, "f16": 2, "fp8": 3}


def _problem(dtype, dim, lens, n_docs=200):
    g = W.rng(dim + len(lens))
    d_off = W.offsets_from_lengths(g.integers(0, 40, size=n_docs))
    d = W.unit_tokens(int(d_off[-1]), dim, g)
    q = W.unit_tokens(sum(lens), dim, g)
    return (device_tokens(q, W.offsets_from_lengths(lens), dtype),
            device_tokens(d, d_off, dtype))


def _load(path, entries):
    path.write_text(json.dumps({"version": 1, "entries": entries}))
    M.load_tune_cache(str(path))


@pytest.mark.parametrize("lens", [[64], [32, 32], [32, 7, 20, 32]])
@pytest.mark.parametrize("dtype,dim,nw", [("f16", 768, 8), ("bf16", 768, 8), ("f32", 384, 4)])
def test_a_shape_that_fills_the_lds_serves_top_k_too(dtype, dim, nw, lens, tmp_path):
    # four query blocks and the ring take all 160 KB: the scores alone run
    # staged, with the top-k the same waves have to fit as well
    Q, D = _problem(dtype, dim, lens)
    want = M.score(Q, D)
    shape = {"pf": 2, "nw": nw, "wg_per_cu": 0, "stage": 1}
    _load(tmp_path / "t.json", [{"dtype": _CODE[dtype], "dim": dim, "nqb": 4, "units": u, **shape}
                                for u in (0, 1, 2)])
    assert torch.equal(M.score(Q, D), want)
    n = len(lens)
    off = dev(W.offsets_from_lengths([200] * n))
    ids = dev(np.tile(np.arange(200, dtype=np.int32), n))
    rs, ri = M.topk(want, off, 10)
    for cand in (None, M.Candidates(off, ids)):
        ts, ti = M.score_topk(Q, D, 10, cand)
        assert torch.equal(ts, rs) and torch.equal(ti, ri)


def _entries(path, dtype, dim):
    return [e for e in json.loads(path.read_text())["entries"]
            if e.get("dtype") == _CODE[dtype] and e.get("dim") == dim]


def test_the_cache_survives_its_round_trip(tmp_path):
    # a shape tuned for one query holds for that alone, in the process that
    # tuned it, in the file, and in a process that reads the file
    Q, D = _problem("f16", 80, [32])
    first, second = tmp_path / "a.json", tmp_path / "b.json"
    M.autotune(Q, D, reps=1, cache_path=str(first))
    tuned = _entries(first, "f16", 80)
    assert [e["units"] for e in tuned] == [0]
    entry = {**tuned[0], "dim": 112}  # as a process that has tuned nothing reads it
    _load(tmp_path / "c.json", [entry])
    M.autotune(*_problem("f16", 80, [32]), reps=1, cache_path=str(second))
    assert _entries(second, "f16", 112) == [entry]


@pytest.mark.parametrize("generic_last", [False, True])
def test_entries_for_a_form_stay_beside_those_for_all(tmp_path, generic_last):
    dim = 208 + 16 * generic_last
    base = {"dtype": 2, "dim": dim, "nqb": 2, "pf": 3, "wg_per_cu": 0, "stage": 0, "rows": 16}
    files = [[{**base, "units": 2, "nw": 8}], [{**base, "nw": 4}]]
    for i, entries in enumerate(files if generic_last else files[::-1]):
        _load(tmp_path / f"{i}.json", entries)
    out = tmp_path / "all.json"
    M.autotune(*_problem("f16", 80, [32]), reps=1, cache_path=str(out))
    assert {e.get("units"): e["nw"] for e in _entries(out, "f16", dim)} == {None: 4, 2: 8}

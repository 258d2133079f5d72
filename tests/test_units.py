"""The pair tables as matrix operands: the operand words and their products on
the CPU (plain integers as the reference), and the matrix sweep on the GPU at
the sizes where its layouts and tiles change, against the oracle."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2603_29942_amd", "csrc")


def test_operand_words(tmp_path):
    exe = os.path.join(str(tmp_path), "unit_checks")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-DBZ_HD=inline", "-I", CSRC, "-I",
                    os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "unit_checks.cpp"), "-o", exe],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.splitlines() == ["OK weights", "OK order", "OK triples", "OK reports"]


# (p, columns processed, k): the first and last column count of every layout
# (F_7: 21 | 32 | 42 | 64 | 128, F_3: 64 | 128), and k around the tiles of 32
# units (F_3: 2 units a pair, 17 pairs end in a second tile; F_7: 6 a pair)
SHAPES = [(3, 1, 5), (3, 31, 6), (3, 32, 7), (3, 33, 8), (3, 64, 9), (3, 65, 7), (3, 96, 6), (3, 97, 6),
          (7, 1, 5), (7, 20, 5), (7, 21, 6), (7, 22, 5), (7, 32, 6), (7, 33, 5), (7, 42, 6), (7, 43, 5), (7, 64, 5),
          (7, 65, 5), (7, 96, 5), (7, 97, 5), (7, 122, 6)]


@pytest.mark.gpu
@pytest.mark.parametrize("p,nsym,k", SHAPES)
def test_sweep_at_layout_edges(p, nsym, k):
    """Every stage of a code (no early end) on the plain path with tables, with
    and without histograms, and batched: the oracle's trace, the histograms'
    lowest weight and their sum being the stage's minimum and count."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from oracle import bzref
    from paper_2603_29942_amd import bz
    rng = np.random.default_rng([31, p, nsym, k])
    G = rng.integers(0, p, size=(k, nsym + k), dtype=np.uint8)
    G[:, :k] = np.eye(k, dtype=np.uint8)  # full rank
    if nsym > 3:
        G[:, k + 1] = 0  # a column that no sum fills
    ref = bzref.min_distance(p, G, no_termination=True)
    got = [bz.min_distance(p, G, no_termination=True, pair_tables=1),
           bz.min_distance(p, G, no_termination=True, pair_tables=1, histograms=True)]
    got += bz.min_distance_batch([(p, G)], no_termination=True, device="cuda:0")
    for r in got:
        for key in ("status", "d", "m", "ranks", "stages", "codewords_total"):
            assert r[key] == ref[key], (key, r[key], ref[key])
    for stage, h in zip(got[1]["stages"], got[1]["hist"]):
        assert int(h.sum()) == stage[2] and int(np.nonzero(h)[0][0]) == stage[3]


@pytest.mark.gpu
@pytest.mark.parametrize("p,n,k,hist,tables", [(3, 30, 13, False, False), (3, 30, 14, False, True),
                                               (3, 30, 14, True, False), (7, 16, 5, False, True),
                                               (7, 20, 7, True, False), (7, 20, 8, True, True)])
def test_default_tables(p, n, k, hist, tables):
    """Which plain calls take tables by default, and that both ways agree."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    G = np.random.default_rng([32, p, n, k]).integers(0, p, size=(k, n), dtype=np.uint8)
    G[:, :k] = np.eye(k, dtype=np.uint8)
    r = bz.min_distance(p, G, histograms=hist)
    assert bool(r["info"] & bz.INFO_PAIRS) == tables
    for pt in (-1, 1):
        o = bz.min_distance(p, G, histograms=hist, pair_tables=pt)
        for key in ("status", "d", "m", "ranks", "stages", "codewords_total"):
            assert o[key] == r[key], (key, o[key], r[key])


@pytest.mark.gpu
@pytest.mark.parametrize("p,n,k", [(7, 48, 20), (7, 56, 24), (7, 63, 21), (3, 80, 28), (3, 89, 29), (3, 100, 50)])
def test_rounds_of_triples(p, n, k):
    """Rounds far enough up to take triples, in runs and not: batched (a few
    codes, so that some rounds have too few tasks for runs) and plain with
    tables, against the kernel without tables."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    G = np.random.default_rng([33, p, n, k]).integers(0, p, size=(k, n), dtype=np.uint8)
    limit = 1 << 34
    ref = bz.min_distance(p, G, no_termination=True, max_codewords=limit, pair_tables=-1)
    assert max(st[0] for st in ref["stages"]) >= 6
    got = [bz.min_distance(p, G, no_termination=True, max_codewords=limit, pair_tables=1)]
    got += bz.min_distance_batch([(p, G)] * 2, no_termination=True, max_codewords=limit, device="cuda:0")
    for r in got:
        for key in ("status", "d", "m", "ranks", "stages", "codewords_total"):
            assert r[key] == ref[key], (key, r[key], ref[key])


# every layout with a table of triples, at the first or last column counts of
# the layout where a code that takes them has one: (p, n, k, identity skip)
TRIPLE_SHAPES = [(7, 43, 22, True), (7, 54, 22, True), (7, 55, 22, True), (7, 63, 21, True), (7, 59, 15, True),
                 (7, 78, 13, True), (7, 109, 12, True), (7, 59, 15, False), (7, 78, 13, False),
                 (3, 67, 35, True), (3, 80, 28, True), (3, 100, 30, True), (3, 116, 19, True), (3, 116, 19, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("p,n,k,skip", TRIPLE_SHAPES)
def test_triples_on_every_layout(p, n, k, skip):
    """Rounds of triples ran (they are in the schedule, and without the bound
    test every stage of it runs), plain and batched: the kernel without tables
    gives the same stages."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    G = np.random.default_rng([34, p, n, k]).integers(0, p, size=(k, n), dtype=np.uint8)
    kw = {"no_termination": True, "identity_skip": skip, "max_codewords": 1 << 31}
    ref = bz.min_distance(p, G, pair_tables=-1, **kw)
    assert not ref["info"] & bz.INFO_TRIPLES
    got = [bz.min_distance(p, G, pair_tables=1, **kw)]
    got += bz.min_distance_batch([(p, G)] * 2, device="cuda:0", **kw)
    for r in got:
        assert r["info"] & bz.INFO_TRIPLES
        for key in ("status", "d", "m", "ranks", "stages", "codewords_total"):
            assert r[key] == ref[key], (key, r[key], ref[key])


@pytest.mark.gpu
@pytest.mark.parametrize("p,n,k,skip", [(7, 43, 22, True), (7, 59, 15, True), (7, 78, 13, True), (7, 78, 13, False),
                                        (3, 67, 35, True), (3, 116, 19, True)])
def test_histograms_of_triples(p, n, k, skip):
    """A spectrum whose rounds take triples (units outside a task's range are
    masked there too) equals the kernel without tables', bin for bin."""
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    G = np.random.default_rng([35, p, n, k]).integers(0, p, size=(k, n), dtype=np.uint8)
    kw = {"no_termination": True, "identity_skip": skip, "max_codewords": 1 << 31, "histograms": True}
    ref = bz.min_distance(p, G, pair_tables=-1, **kw)
    got = bz.min_distance(p, G, pair_tables=1, **kw)
    assert got["info"] & bz.INFO_TRIPLES
    assert got["stages"] == ref["stages"] and np.array_equal(got["hist"], ref["hist"])


@pytest.mark.gpu
@pytest.mark.parametrize("p,k", [(7, 6), (7, 12), (7, 23), (3, 20), (3, 64)])
@pytest.mark.parametrize("tables", [-1, 0, 1])
@pytest.mark.parametrize("skip", [True, False])
def test_whole_space(p, k, tables, skip):
    import torch
    assert torch.cuda.is_available(), "no GPU visible"
    from paper_2603_29942_amd import bz
    # n = k, no column left to process: a codeword of g rows has weight g
    G = np.eye(k, dtype=np.uint8)
    r = bz.min_distance(p, G, no_termination=True, max_codewords=10**8, pair_tables=tables, identity_skip=skip)
    assert r["d"] == 1
    assert [s[3] for s in r["stages"]] == [s[0] for s in r["stages"]]
    assert [s[4] for s in r["stages"]] == [1] * len(r["stages"])

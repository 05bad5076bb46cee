"""The guess of the single pass is made on the device (clique search, choice of
the reduction and the key tiles, selection, row table of a worker-major
upload): every outcome against the oracle, and the guess right where the
probe covers the vector."""
import random

import numpy as np
import pytest

import oracle
import synth
from paper_2108_02416_amd import aspis

from test_gpu_steady import _compare, _oracle, _run

pytestmark = pytest.mark.gpu


def _honest(K, r, d):
    wl = synth.Workload(0, K, r, 0, d, synth.DIST_NORMAL, "weak", "reversed", "fixed")
    s = oracle.assign(K, r)
    g, _ = synth.generate(wl, s, d=d)
    return g, s


@pytest.mark.parametrize("K,r,q,pairs", [
    (7, 3, 3, []),                                  # complete graph
    (9, 3, 2, [(0, 8)]),                            # two maximum cliques
    (10, 3, 4, [(0, 1), (0, 2), (0, 3)]),           # one maximum clique
    (10, 3, 1, [(0, 1), (2, 3)]),                   # none large enough
    (12, 5, 3, [(0, 11), (1, 11), (2, 11)]),
    (24, 3, 11, [(2 * j, 2 * j + 1) for j in range(12)]),   # the even workers: one too few
])
@pytest.mark.parametrize("mode", ["median", "paper"])
def test_guess_of_planted_graphs(K, r, q, pairs, mode):
    """Worker v's replica differs from every other one of each file that it
    shares with worker u."""
    d = 40
    g, s = _honest(K, r, d)
    for u, v in pairs:
        for i in np.flatnonzero((s == u).any(axis=1) & (s == v).any(axis=1)):
            g[i, int(np.flatnonzero(s[i] == v)[0]), (u * K + v) % d] += np.float32(1.0)
    ref = _oracle(g, K, r, q, mode)
    for layout in ("file", "worker"):
        got = _run(g, K, r, q, mode, 0, layout)
        _compare(got, ref, K, mode)
        assert got["stats"]["fused"] == 1 and got["stats"]["speculation_hit"] == 1


@pytest.mark.parametrize("K,q,deg,seed", [
    (30, 14, 3, 6), (30, 14, 3, 5), (30, 14, 3, 0), (27, 13, 3, 8), (30, 14, 2, 3), (25, 12, 3, 5),
])
@pytest.mark.parametrize("mode,layout", [("median", "file"), ("paper", "file"), ("paper", "worker"),
                                         ("median", "worker")])
def test_guess_of_sparse_disagreement(K, q, deg, seed, mode, layout):
    """Every adversary disagrees with `deg` honest workers only, so the graph
    has up to thousands of maximal cliques (1,935, 1,770, 690, 1,145, 2,576
    and 561 here): the guess has to decide it all the same, both where one
    clique is the largest and where several are."""
    r, d = 3, 64
    g, s = _honest(K, r, d)
    rng = random.Random(seed)
    against = [rng.sample(range(q, K), deg) for _ in range(q)]
    for i, (a, u, v) in enumerate(s):
        if a < q <= u and u in against[a] and v in against[a]:
            g[i, 0, (int(a) * 7) % d] += np.float32(1.0)
    ref = _oracle(g, K, r, q, mode)
    assert ref["clique"]["success"] == ((deg, seed) not in ((3, 0), (2, 3)))
    got = _run(g, K, r, q, mode, 0, layout)
    _compare(got, ref, K, mode)
    assert got["stats"]["fused"] == 1 and got["stats"]["speculation_hit"] == 1


@pytest.mark.parametrize("K,r", [(41, 3), (64, 3), (14, 7), (19, 5)])
def test_row_table_of_many_workers(K, r):
    g, _ = _honest(K, r, 4)
    got = _run(g, K, r, 2, "mean", 0, "worker")
    _compare(got, _oracle(g, K, r, 2, "mean"), K, "mean")


@pytest.mark.parametrize("d", [128 * 256, 128 * 256 + 4, 128 * 256 + 133])
@pytest.mark.parametrize("K,layout", [(K, lay) for K in (7, 9, 10) for lay in ("file", "worker")])
def test_few_files_either_side_of_the_half_key_line(K, layout, d):
    """35, 84 and 120 files take half-key tiles from 32,769 coordinates on."""
    r, q = 3, 2
    wl = synth.Workload(0, K, r, q, d, synth.DIST_NORMAL, "weak", "reversed", "fixed")
    g, _ = synth.generate(wl, oracle.assign(K, r), d=d)
    got = _run(g, K, r, q, layout=layout)
    _compare(got, _oracle(g, K, r, q, "median"), K, "median")
    assert (got["stats"]["tile_cols"], got["stats"]["half_keys"]) == \
        ((128, 1) if d > 128 * 256 else (64, 0))
    full = _run(g, K, r, q, flags=aspis.FLAG_FULL_KEYS, layout=layout)
    assert full["stats"]["half_keys"] == 0
    assert (full["out"] == got["out"]).all()

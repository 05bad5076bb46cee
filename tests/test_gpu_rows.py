"""Rows of any length: the kernels read 16-byte chunks at 4-byte boundaries,
and the chunk holding a row's end is read four coordinates before it.  Every
remainder of the row length by four and by the tile, in the persistent grid's
steady state, against the oracle.  Row lengths that keep rows on 128-byte
lines and others take different kernels (the tile order and the loads)."""
import numpy as np
import pytest

import oracle
import synth
from paper_2108_02416_amd import aspis

from test_gpu_repair import _attack_only_at, _late_workload, _repaired
from test_gpu_steady import CUS, _compare, _oracle, _run

pytestmark = pytest.mark.gpu


# d = 128 * 256 * k + extra: a last tile of one chunk short of, at and past
# its end, and a last tile that is one coordinate
@pytest.mark.parametrize("K,r,q,layout,flags,tiles,extra", [
    (15, 3, 4, "file", 0, 3 * CUS, 1),
    (15, 3, 4, "file", 0, CUS + 3, 127),
    (15, 3, 4, "worker", 0, CUS + 3, 2),
    (15, 3, 4, "file", aspis.FLAG_TWO_PASS, CUS + 3, 3),
    (15, 3, 4, "file", aspis.FLAG_FULL_KEYS, CUS + 3, 5),
    (15, 3, 4, "worker", aspis.FLAG_FULL_KEYS, CUS + 3, 6),
    (11, 5, 3, "file", 0, CUS + 1, 1),
    (21, 3, 5, "file", 0, 70, 33),
    (25, 3, 6, "worker", 0, 40, 3),
    (24, 3, 5, "worker", 0, 130, 3),
    (7, 3, 2, "file", 0, 3 * CUS, 3),
    (10, 7, 2, "file", 0, 20, 1),
    (15, 3, 4, "file", 0, 0, 5),
    (15, 3, 4, "file", 0, 0, 7),
    # r = 5 and 7: full keys, half keys, the row table
    (9, 5, 2, "file", 0, CUS + 1, 4),
    (9, 5, 2, "worker", 0, CUS + 1, 1),
    (11, 5, 3, "worker", 0, CUS + 1, 36),
    (9, 7, 2, "worker", 0, CUS + 1, 32),
    (11, 7, 2, "file", 0, CUS // 2 + 1, 32),
    (11, 7, 2, "worker", 0, CUS // 2 + 1, 3),
    (12, 7, 2, "file", 0, 10, 7),
    # rows on 128-byte lines, the last tile ragged
    (15, 3, 4, "file", 0, 2 * CUS + 3, 32),
    (15, 3, 4, "worker", 0, CUS + 3, 96),
    (21, 3, 5, "file", 0, 2 * CUS // 4 + 1, 32),
    (25, 3, 6, "file", 0, CUS // 4 + 1, 64),
    (11, 5, 3, "file", 0, CUS + 1, 64),
])
def test_any_row_length(K, r, q, layout, flags, tiles, extra):
    d = 128 * tiles + extra
    print(f"K={K} r={r} d={d} layout={layout} flags={flags}", flush=True)
    wl = synth.Workload(0, K, r, q, d, synth.DIST_NORMAL, "weak", "alie", "fixed")
    g, _ = synth.generate(wl, oracle.assign(K, r), d=d)
    got = _run(g, K, r, q, "median", flags, layout)
    _compare(got, _oracle(g, K, r, q, "median"), K, "median")


@pytest.mark.parametrize("mode,K,r,q,d", [
    ("mean", 10, 3, 2, 4 * 256 * 11 + 3),
    ("paper", 10, 3, 2, 4 * 256 * 11 + 3),
    ("mean", 5, 3, 1, 1024 * (5 * CUS - 1)),    # either side of the line to bursts
    ("mean", 5, 3, 1, 1024 * (5 * CUS - 1) + 1),
    ("mean", 5, 3, 1, 1024 * 8 * CUS + 5),      # and back, two rounds of the grid
    ("mean", 8, 5, 2, 1024 * 3 + 2),
    ("mean", 8, 7, 2, 1024 * 3 + 1),
    ("mean", 7, 3, 2, 3),                       # rows shorter than a chunk
    ("mean", 7, 5, 2, 2),
    ("mean", 8, 7, 2, 1),
    ("mean", 7, 3, 2, 4),
])
def test_any_row_length_mean(mode, K, r, q, d):
    wl = synth.Workload(0, K, r, q, d, synth.DIST_NORMAL, "weak", "reversed", "fixed")
    g, _ = synth.generate(wl, oracle.assign(K, r), d=d)
    for layout in ("file", "worker"):
        _compare(_run(g, K, r, q, mode, 0, layout), _oracle(g, K, r, q, mode), K, mode)


def test_repair_of_a_chunk_shared_by_two_tiles():
    """d = 128 n + 1: the last tile's one chunk starts three coordinates
    before it, in the tile before.  A deviation at the last coordinate alone
    and one in that other tile alone each repair one tile."""
    wl, kw = _late_workload(15, 3, 4)
    d = 128 * (CUS + 40) + 1
    s = oracle.assign(wl.K, wl.r)
    for coord in (d - 1, d - 2):
        g = _attack_only_at(wl, s, d, np.array([coord]), **kw)
        _, _, groups = _repaired(g, wl.K, wl.r, wl.q)
        assert groups == 1

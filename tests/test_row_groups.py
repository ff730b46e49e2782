"""The workgroups of the forward and dQ kernels: units of 32 rows of one query head, four to a workgroup, numbered heads
first.  For group sizes that divide four, are divided by it and do neither, every (head, row) must be owned by exactly one
wave, and the walk of its workgroup must visit every visible pair of it once and skip no visible one (checked against the
oracle's mask, pair by pair)."""
import numpy as np
import pytest

import oracle
import paper_2509_15763_amd as u
from test_walk_plan import FULL, SKIP, compact_positions

SHAPES = [
    # L, r, W, sinks, units
    (1, 4, 4, 0, False),
    (33, 1, 3, 0, False),
    (1000, 4, 129, 0, False),
    (777, 3, 40, 70, False),
    (1283, 2, 1, 5, True),
    (1500, 4, 20, 64, True),
    (640, 1000, 2000, 0, False),
]


@pytest.mark.parametrize("kernel", [u.UNIGIST_WALK_FWD, u.UNIGIST_WALK_DQ])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 7, 8])
@pytest.mark.parametrize("L,r,W,sinks,units", SHAPES)
def test_every_pair_once(L, r, W, sinks, units, G, kernel):
    M = oracle.mask_rows(np.arange(L), L, r, W, sinks=sinks, units=units)
    owned = np.zeros((G, L), dtype=np.int8)
    n_groups = u.unigist_plan_row_group(L, r, W, sinks, int(units), G, kernel, 0)["n_groups"]
    assert n_groups == -(-(-(-L // 32) * G) // 4)
    for group in range(n_groups):
        p = u.unigist_plan_row_group(L, r, W, sinks, int(units), G, kernel, group)
        Bn, ngt, nfar, kind = p["Bn"], p["n_gist_steps"], p["nfar"], p["kind"]
        assert Bn == (32 if kernel == u.UNIGIST_WALK_FWD else 64) and ngt == -(-nfar // Bn)
        pos = compact_positions(nfar, r, sinks)
        assert nfar == 0 or pos.max() < p["wstart"]
        live = [w for w in range(4) if p["head"][w] >= 0]
        assert live == list(range(len(live))) and (len(live) == 4 or group == n_groups - 1)
        assert p["i0"] == min(p["row0"][w] for w in live)
        assert p["i1"] == min(L, max(p["row0"][w] for w in live) + 32) - 1
        for w in live:
            r0, r1 = p["row0"][w], min(L, p["row0"][w] + 32)
            assert p["head"][w] < G and r0 % 32 == 0 and r0 < L
            owned[p["head"][w], r0:r1] += 1
            rows = M[r0:r1]
            cover = np.zeros(rows.shape, dtype=np.int8)
            assert rows[:, pos].all()
            cover[:, pos] += 1
            for it in range(ngt):
                assert kind[w, it] == (FULL if (it + 1) * Bn <= nfar else 2)
            for n in range(p["n_window_steps"]):
                j0 = p["wstart"] + n * Bn
                part = rows[:, j0:j0 + Bn]
                if kind[w, ngt + n] == SKIP:
                    assert not part.any()
                    continue
                assert kind[w, ngt + n] != FULL or (part.all() and part.shape[1] == Bn)
                cover[:, j0:j0 + Bn] += 1
            assert cover.max() <= 1 and (cover[rows] == 1).all()
    assert (owned == 1).all()


def test_group_of_one_is_the_row_tile():
    L, r, W, sinks = 1000, 4, 100, 7
    for kernel in (u.UNIGIST_WALK_FWD, u.UNIGIST_WALK_DQ):
        for t in range(-(-L // 128)):
            a, b = u.unigist_plan_row_tile(L, r, W, sinks, 0, kernel, t), u.unigist_plan_row_group(L, r, W, sinks, 0, 1, kernel, t)
            assert all(a[n] == b[n] for n in ("Bn", "wstart", "nfar", "n_gist_steps", "n_window_steps"))
            live = [w for w in range(4) if b["head"][w] == 0]
            assert [b["row0"][w] for w in live] == list(range(128 * t, min(L, 128 * t + 128), 32))
            assert (a["kind"][live] == b["kind"][live]).all()


@pytest.mark.parametrize("L", [1, 100, 128, 300, 777])
@pytest.mark.parametrize("B,Hq,Hkv", [(1, 1, 1), (1, 32, 8), (3, 28, 4), (32, 32, 8), (2, 16, 16), (5, 12, 3), (40, 8, 8), (65, 28, 7),
                                      (191, 4, 1), (193, 4, 1), (9, 24, 8)])
def test_launch_order(B, Hq, Hkv, L):
    G, NP = Hq // Hkv, B * Hkv
    per = -(-(-(-L // 32) * G) // 4)
    order = [u.unigist_plan_row_slot(B, Hq, Hkv, L, n) for n in range(NP * per)]
    assert len(set(order)) == NP * per
    assert all(0 <= pair < NP and 0 <= group < per for pair, group in order)
    if NP % 8 == 0:  # a pair stays on one XCD
        assert all(pair % 8 == n % 8 for n, (pair, _) in enumerate(order))
    # one after the other on the XCD (or in the launch): the groups of a bunch, longest walk first, then the next pair
    lanes = [order[x::8] for x in range(8)] if NP % 8 == 0 else [order]
    w = G if NP % 8 == 0 or NP >= 192 else 1
    for lane in lanes:
        pairs = sorted({pair for pair, _ in lane})
        want = [(pair, group) for top in range(per, 0, -w) for pair in pairs for group in range(top - 1, max(top - w, 0) - 1, -1)]
        assert lane == want


def test_arguments():
    for bad in [(0, 4, 1, 10, 0), (1, 4, 3, 10, 0), (1, 4, 1, 0, 0), (1, 4, 1, 100, 4), (1, 4, 1, 100, -1)]:
        with pytest.raises(u.UnigistError):
            u.unigist_plan_row_slot(*bad)
    assert u.load().unigist_plan_row_group(100, 4, 8, 0, 0, 4, 0, 0, None, 0, None) == 1
    for bad in [(0, 4, 8, 0, 0, 4, 0, 0), (100, 4, 8, 0, 0, 0, 0, 0), (100, 4, 8, 0, 0, 4, 2, 0), (100, 4, 8, 0, 0, 4, 0, 4),
                (100, 4, 8, 0, 0, 4, 0, -1), (100, 4, 8, 0, 2, 4, 0, 0)]:
        with pytest.raises(u.UnigistError):
            u.unigist_plan_row_group(*bad)

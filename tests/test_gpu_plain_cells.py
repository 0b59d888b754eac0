"""The plain 16-bit cells, which serve what offset cells cannot hold: gaps that open for less than they extend by, or
with Go past 255 or Ge past 32.  Every kernel of theirs at its edges, against the oracle (tolerance 0)."""
import numpy as np
import pytest

import oracle
from inputs import synth

pytestmark = pytest.mark.gpu

GAPS = [(1, 11), (33, 33), (300, 2)]


def _db(seed, lens):
    rng = np.random.default_rng(seed)
    subs = [synth.background_residues(rng, int(L)) for L in lens]
    offs = np.concatenate([[0], np.cumsum([s.size for s in subs])]).astype(np.int64)
    return synth.Database(np.concatenate(subs), offs)


def _query(db, m):
    """Half of it a stretch of the first subject, so that some scores are high."""
    q = synth.small_query(seed=m, m=m)
    k = min(m // 2, int(db.offsets[1]))
    q[m - k:] = db.residues[:k]
    return q


def _check(got, q, db, blosum, go, ge, what, mode="local"):
    want = oracle.scores(q, db.residues, db.offsets, blosum, go, ge, mode=mode)
    assert (got == want).all(), f"{what} {go}/{ge}: {np.nonzero(got != want)[0][:5]}"


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("lanes", [1, 2, 16, 32, 64])
def test_rows_and_lanes(gpu, blosum, rows, lanes):
    db = _db(8000, [900, 700, 0, 1, 2, 3, 4, 5] + list(range(20, 140)))
    D = gpu.Database(db.residues, db.offsets, rows_per_lane=rows, force_lanes=lanes)
    for m in (1, rows - 1, rows, rows + 1, rows * lanes, rows * lanes + 1, 333):
        q = _query(db, m)
        for go, ge in GAPS:
            _check(D.search(q, blosum, go, ge).cpu().numpy(), q, db, blosum, go, ge, f"m={m}")
            assert D.stats()["rows_per_lane"] == rows
    D.close()


@pytest.mark.parametrize("rows", [0, 8, 16])
@pytest.mark.parametrize("lanes", [0, 1, 8, 32])
def test_query_pairs(gpu, blosum, rows, lanes):
    """Two queries per lane, of like length and not, and one that is left over."""
    db = _db(8100, [900, 500, 0, 1] + list(range(20, 200)))
    D = gpu.Database(db.residues, db.offsets, rows_per_lane=rows, force_lanes=lanes, lane_pack=2)
    qs = [_query(db, m) for m in (1, 40, 333, 330, 700)]
    for go, ge in GAPS:
        got = D.search_batch(qs, blosum, go, ge, k=0)[0].cpu().numpy()
        for i, q in enumerate(qs):
            _check(got[i], q, db, blosum, go, ge, f"query {i}")
    D.close()


def test_long_pairs_among_the_others(gpu, blosum):
    db = _db(8200, [9000, 5000, 4999] + list(np.random.default_rng(1).integers(0, 300, 700)))
    D, D2 = gpu.Database(db.residues, db.offsets), gpu.Database(db.residues, db.offsets, lane_pack=2)
    qs = [_query(db, m) for m in (1, 30, 255, 257, 400, 1025)]
    for go, ge in GAPS:
        for q in qs:
            _check(D.search(q, blosum, go, ge).cpu().numpy(), q, db, blosum, go, ge, f"m={q.size}")
        for d in (D, D2):
            got = d.search_batch(qs, blosum, go, ge, k=0)[0].cpu().numpy()
            for i, q in enumerate(qs):
                _check(got[i], q, db, blosum, go, ge, f"batch, m={q.size}")
    D.close()
    D2.close()


@pytest.mark.parametrize("mode", ["global", "semiglobal"])
def test_end_to_end_long_pairs_beside_the_launch(gpu, blosum, mode):
    """Short queries: the long pairs run beside the 16-row launch at the rows per lane that take the least, 4 up to 256
    residues and 8 up to 512."""
    db = _db(8300, [6000, 5000, 4000, 3500] + list(np.random.default_rng(2).integers(1, 400, 600)))
    D = gpu.Database(db.residues, db.offsets)
    rows = {}
    for m in (1, 30, 256, 257, 500):
        q = _query(db, m)
        for go, ge in ((7, 9), (33, 33)):
            _check(D.search(q, blosum, go, ge, mode=mode).cpu().numpy(), q, db, blosum, go, ge, f"{mode} m={m}", mode)
            st = D.stats()
            if (go, ge) == (33, 33):
                assert st["side_items"] > 0, st
                rows[m] = st["side_rows_per_lane"]
    assert rows == {1: 4, 30: 4, 256: 4, 257: 8, 500: 8}, rows
    D.close()


def test_scores_past_the_range(gpu, blosum):
    """High scorers are flagged and recomputed; their 16-bit result is poisoned, so a missed one would show."""
    W = 17
    q = np.full(3000, W, np.int8)
    rng = np.random.default_rng(3)
    subs = [np.concatenate([synth.background_residues(rng, 500), q]), np.full(2900, W, np.int8), np.full(2500, W, np.int8)]
    subs += [synth.background_residues(rng, int(L)) for L in rng.integers(1, 300, 200)]
    offs = np.concatenate([[0], np.cumsum([s.size for s in subs])]).astype(np.int64)
    db = synth.Database(np.concatenate(subs), offs)
    for pack in (1, 2):
        D = gpu.Database(db.residues, db.offsets, poison=1, lane_pack=pack)
        for go, ge in GAPS:
            got = D.search_batch([q, q[:2000]], blosum, go, ge, k=0)[0].cpu().numpy()
            assert D.stats()["rerun_pairs"] >= 1
            for i, x in enumerate((q, q[:2000])):
                _check(got[i], x, db, blosum, go, ge, f"pack {pack} query {i}")
        D.close()

"""Long subjects on a workgroup each (chained waves, windows of the subject) and
end-to-end modes on offset cells, at the edges of waves (256 rows), passes (1,024
rows) and windows, against the oracle (tolerance 0)."""
import numpy as np
import pytest

import oracle
from inputs import synth

pytestmark = pytest.mark.gpu


def _db(seed, long_ones):
    rng = np.random.default_rng(seed)
    lens = list(long_ones) + [0, 1, 2, 3] + list(rng.integers(1, 260, 60))
    subs = [synth.background_residues(rng, int(L)) for L in lens]
    offs = np.zeros(len(subs) + 1, np.int64)
    offs[1:] = np.cumsum(lens)
    return synth.Database(np.concatenate(subs), offs)


def _query(db, m):
    """Half of it a stretch from the end of the longest subject, so that some scores are high."""
    q = synth.small_query(seed=m, m=m)
    k = min(m // 2, 400)
    if k:
        at = int(db.offsets[1]) - 37 - k
        q[m - k:] = db.residues[at:at + k]
    return q


@pytest.mark.parametrize("mode", ["local", "global", "semiglobal"])
@pytest.mark.parametrize("m", [1, 4, 5, 64, 255, 256, 257, 511, 512, 513, 769, 1024, 1025, 2049])
def test_edges_of_waves_and_passes(gpu, blosum, mode, m):
    db = _db(51, (9001, 6000, 5997, 4100))
    D = gpu.Database(db.residues, db.offsets)
    q = _query(db, m)
    for go, ge in ((10, 2), (11, 1)):
        got = D.search(q, blosum, go, ge, mode=mode).cpu().numpy()
        want = oracle.scores(q, db.residues, db.offsets, blosum, go, ge, mode=mode)
        assert (got == want).all(), f"{mode} m={m} {go}/{ge}: {np.nonzero(got != want)[0][:5]}"
    D.close()


@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("lanes", [1, 2, 16, 32, 64])
def test_end_to_end_rows_and_lanes(gpu, blosum, rows, lanes):
    db = _db(52, (1200, 700))
    D = gpu.Database(db.residues, db.offsets, rows_per_lane=rows, force_lanes=lanes)
    for m in (1, rows - 1, rows, rows + 1, rows * lanes, rows * lanes + 1, 333):
        q = _query(db, m)
        for mode in ("global", "semiglobal"):
            for go, ge in ((10, 2), (7, 7), (12, 0)):
                got = D.search(q, blosum, go, ge, mode=mode).cpu().numpy()
                want = oracle.scores(q, db.residues, db.offsets, blosum, go, ge, mode=mode)
                assert (got == want).all(), f"{mode} m={m} {go}/{ge}: {np.nonzero(got != want)[0][:5]}"
    D.close()


@pytest.mark.parametrize("mode", ["local", "global", "semiglobal"])
def test_scores_past_the_range_on_a_workgroup(gpu, blosum, mode):
    """A repeat that scores beyond 16 bits in a chained pair is found and recomputed; the 16-bit result is poisoned,
    so a missed recompute would show."""
    rng = np.random.default_rng(53)
    W = 17
    q = np.full(3000, W, np.int8)
    first = np.concatenate([synth.background_residues(rng, 5000), q, synth.background_residues(rng, 4000)])
    subs = [first, synth.background_residues(rng, 11000)] + [synth.background_residues(rng, int(L)) for L in rng.integers(1, 300, 40)]
    offs = np.zeros(len(subs) + 1, np.int64)
    offs[1:] = np.cumsum([s.size for s in subs])
    db = synth.Database(np.concatenate(subs), offs)
    D = gpu.Database(db.residues, db.offsets, poison=1)
    got = D.search(q, blosum, 10, 2, mode=mode).cpu().numpy()
    want = oracle.scores(q, db.residues, db.offsets, blosum, 10, 2, mode=mode)
    assert (got == want).all(), np.nonzero(got != want)[0][:5]
    D.close()


@pytest.mark.parametrize("m", [(100, 60), (257, 256), (700, 30, 1025)])
def test_query_pairs_chain(gpu, blosum, m):
    db = _db(54, (9001, 6000))
    D = gpu.Database(db.residues, db.offsets, lane_pack=2)
    qs = [_query(db, x) for x in m]
    got = D.search_batch(qs, blosum, 10, 2)[0].cpu().numpy()
    for i, q in enumerate(qs):
        want = oracle.scores(q, db.residues, db.offsets, blosum, 10, 2)
        assert (got[i] == want).all(), f"query {i}: {np.nonzero(got[i] != want)[0][:5]}"
    D.close()


@pytest.mark.parametrize("lens", [(769, 800, 1024), (944, 1100, 1563, 1888), (1537, 1549, 2048, 2305)])
@pytest.mark.parametrize("subjects", [1343, 6000])
def test_rows_past_the_query_in_passes_of_768(gpu, blosum, lens, subjects):
    """A pass of 64 lanes x 12 rows reads the profile in steps of 768 rows, past a multiple of 1,024."""
    rng = np.random.default_rng(55)
    n = np.clip(np.exp(rng.normal(5.7, 0.6, subjects)), 20, 2400).astype(np.int64)
    offs = np.concatenate([[0], np.cumsum(n)])
    res = synth.background_residues(rng, int(offs[-1]))
    qs = [synth.background_residues(rng, m) for m in lens]
    D = gpu.Database(res, offs)
    got = D.search_batch(qs + qs + qs, blosum, 11, 1)[0].cpu().numpy()
    for i, q in enumerate(qs):
        want = oracle.scores(q, res, offs, blosum, 11, 1)
        one = D.search(q, blosum, 11, 1).cpu().numpy()
        assert (one == want).all(), f"alone m={q.size}: {np.nonzero(one != want)[0][:5]}"
        for k in (i, i + len(qs), i + 2 * len(qs)):
            assert (got[k] == want).all(), f"batched m={q.size}: {np.nonzero(got[k] != want)[0][:5]}"
    D.close()

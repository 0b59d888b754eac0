"""What the planner makes of a search, read from the launch's statistics, with scores against the oracle (tolerance 0)."""
import numpy as np
import pytest

import oracle
from inputs import synth

pytestmark = pytest.mark.gpu


def _db(lens, seed=7000):
    rng = np.random.default_rng(seed)
    subs = [synth.background_residues(rng, int(L)) for L in lens]
    offs = np.concatenate([[0], np.cumsum([s.size for s in subs])]).astype(np.int64)
    return synth.Database(np.concatenate(subs), offs)


def _query(m):
    return synth.background_residues(np.random.default_rng(7100 + m), m)


@pytest.mark.parametrize("lens", [(1211, 1217), (68, 115)])
def test_query_pairs_fill_their_workgroups(gpu, blosum, lens):
    """A small database, whose units all exceed a wave's share at the most lanes: two queries of any lengths go as one
    pair, 64 units a group, four to an item."""
    db = _db([300] * 2500)
    D = gpu.Database(db.residues, db.offsets, lane_pack=2)
    qs = [_query(m) for m in lens]
    got = D.search_batch(qs, blosum, 10, 2, k=0)[0].cpu().numpy()
    groups = -(-db.n // 128)
    assert D.stats()["items"] <= groups * 64 // 4 + 1, D.stats()
    for i, q in enumerate(qs):
        assert (got[i] == oracle.scores(q, db.residues, db.offsets, blosum, 10, 2)).all()
    D.close()


def test_long_pair_on_plain_cells_takes_the_rows_that_fit(gpu, blosum):
    """Gaps that offset cells cannot hold (Ge > Go): a long subject against 400 residues is one pass of 64 lanes at 8
    rows, not two at 4 or a half-empty one at 16."""
    db = _db([6000, 50])
    D = gpu.Database(db.residues, db.offsets)
    q = _query(400)
    got = D.search(q, blosum, 3, 5).cpu().numpy()
    st = D.stats()
    assert st["rows_per_lane"] == 8 and st["side_items"] == 0, st
    assert (got == oracle.scores(q, db.residues, db.offsets, blosum, 3, 5)).all()
    D.close()


@pytest.mark.parametrize("lens", [(400,), (150, 7, 3111, 20, 480, 99, 12, 1500)])
@pytest.mark.parametrize("lane_pack", [1, 2])
def test_plain_cells_in_a_callers_workspace(gpu, blosum, lens, lane_pack):
    """sw_batch_workspace_bytes does not know the gaps: a workspace of exactly its size serves every scoring, whichever
    plan fits it."""
    rng = np.random.default_rng(7200)
    db = _db(rng.integers(0, 60, 20000), seed=7201)
    D = gpu.Database(db.residues, db.offsets, lane_pack=lane_pack, memory="torch")
    qs = [_query(m) for m in lens]
    for go, ge in ((3, 5), (10, 2), (3, 5)):
        D.ws = None
        got = D.search_batch(qs, blosum, go, ge, k=0)[0].cpu().numpy() if len(qs) > 1 else \
            D.search(qs[0], blosum, go, ge).cpu().numpy()[None]
        for i, q in enumerate(qs):
            assert (got[i] == oracle.scores(q, db.residues, db.offsets, blosum, go, ge)).all(), (q.size, go, ge)
    D.close()


@pytest.mark.parametrize("mode", ["local", "semiglobal"])
def test_a_long_pair_in_parts(gpu, blosum, mode):
    """One long subject on several workgroups, beside 16 items of the group's other pairs, at 10/2 and 11/1, where an
    alignment covers a bounded stretch of it; on one at Ge = 0, where it may cover all."""
    db = _db([20000])
    D = gpu.Database(db.residues, db.offsets)
    for m in (100, 300, 1025):
        q = _query(m)
        for go, ge in ((10, 2), (11, 1), (12, 0)):
            got = D.search(q, blosum, go, ge, mode=mode).cpu().numpy()
            items = D.stats()["items"] + D.stats()["side_items"]
            assert items == 17 if ge == 0 else items > 17, (m, go, ge, items)
            assert (got == oracle.scores(q, db.residues, db.offsets, blosum, go, ge, mode=mode)).all(), (m, go, ge)
    D.close()


@pytest.mark.parametrize("mode", ["local", "semiglobal"])
@pytest.mark.parametrize("m", [60, 257, 513, 1100])
def test_parts_and_spans(gpu, blosum, mode, m):
    """From a span of the query's own length (no gap pays) to one past the subject, on a caller's workspace too."""
    db = _db([20011, 16000, 9001, 50, 40])
    q = _query(m)
    q[m // 2:] = db.residues[19500:19500 + m - m // 2]
    for memory in ("library", "torch"):
        D = gpu.Database(db.residues, db.offsets, memory=memory)
        for go, ge in ((127, 32), (40, 20), (10, 5), (10, 2), (11, 1), (4, 1), (12, 0)):
            got = D.search(q, blosum, go, ge, mode=mode).cpu().numpy()
            want = oracle.scores(q, db.residues, db.offsets, blosum, go, ge, mode=mode)
            assert (got == want).all(), (memory, go, ge, got, want)
        D.close()


@pytest.mark.parametrize("mode", ["local", "global", "semiglobal"])
@pytest.mark.parametrize("subjects,length,m", [(300, 300, 700), (300, 300, 760), (300, 300, 1100), (300, 300, 1500),
                                               (300, 300, 2300), (250_000, 20, 144), (250_000, 20, 300)])
def test_twelve_rows_per_lane(gpu, blosum, mode, subjects, length, m):
    """Passes of 64 and of 16 lanes x 12 rows, which no option asks for, where the planner takes them."""
    rng = np.random.default_rng(7400 + m)
    lens = np.full(subjects, length)
    lens[subjects // 2:] -= rng.integers(0, 4, subjects - subjects // 2)
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    res = synth.background_residues(rng, int(offs[-1]))
    q = _query(m)
    D = gpu.Database(res, offs)
    got = D.search(q, blosum, 10, 2, mode=mode).cpu().numpy()
    assert D.stats()["rows_per_lane"] == 12, D.stats()
    want = oracle.scores(q, res, offs, blosum, 10, 2, mode=mode)
    assert (got == want).all(), np.nonzero(got != want)[0][:5]
    D.close()

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

"""Local scores on offset cells (16-bit cells whose offset grows by Ge per row
and per column step, lowered every K steps) against the oracle.

The CPU part follows the kernel's per-cell order, cooperating lanes, boundary
words between passes and the lowering included, on plain integers, and checks
that no stored value ever leaves 0..0x7BFF (so that packed integer additions
carry nothing between halves and half-float maxima order every value).  The GPU
part runs the kernels at the edges of what the host's rule sends to them.
Integer arithmetic: tolerance 0.
"""
import numpy as np
import pytest

import oracle
from inputs import synth

SAT = 0x7C00


def period(ge):
    return min(64, 4 * (32 // ge)) if ge > 0 else 64


def offset_score(q, d, sm, go, ge, R, B):
    """S of one pair on offset cells: passes of B lanes x R rows, lane b one step behind lane b - 1."""
    m, n = len(q), len(d)
    K, goe, cr = period(ge), go - ge, ge * (R - 1)
    prof = lambda i, x: int(sm[q[i]][x]) + go + ge if i < m and x >= 0 else 0  # noqa: E731
    ok = lambda v: (v if 0 <= v < SAT else pytest.fail(f"stored value {v} outside the exact range"))  # noqa: E731
    bnd = {}
    best = 0
    passes = -(-m // (R * B))
    for p in range(passes):
        P = [[ge * r for r in range(R + 1)] for _ in range(B)]
        E = [[go + ge * (r + 1) for r in range(R)] for _ in range(B)]
        S = [[ge * (2 * i + 1) for i in range(R // 2)] for _ in range(B)]
        F = [ge * R] * B
        tau, out = 1, {}
        for t in range(4 * (-(-(n + B - 1) // 4))):
            hand = [(P[b][R], F[b]) for b in range(B)]
            for b in range(B):
                j = t - b
                x = d[j] if 0 <= j < n else -1
                if b == 0:
                    g, f = bnd.get(j, (0, 0)) if p else (0, 0)
                    top, f = ok(g + ge * tau), ok(f + ge * tau)
                else:
                    top, f = ok(hand[b - 1][0] - cr), ok(hand[b - 1][1] - cr)
                hd = [ok(P[b][r] + prof((p * B + b) * R + r, x)) for r in range(R)]
                S[b] = [ok(s + ge) for s in S[b]]
                P[b][0] = top
                old = list(P[b])
                for r in range(R):
                    h = max(hd[r], E[b][r], f)
                    g = ok(h - goe)
                    P[b][r + 1] = g
                    E[b][r] = max(E[b][r], g, go + ge * (r + tau + 1))
                    f = max(f, g)
                for i in range(R // 2):
                    S[b][i] = max(S[b][i], P[b][2 * i + 1], old[2 * i + 2])
                F[b] = f
            j = t - (B - 1)
            if 0 <= j < n:
                off = ge * (R + tau)
                out[j] = (ok(P[B - 1][R] - off), ok(F[B - 1] - off))
            tau += 1
            if tau > K:
                down = ge * K
                P = [[ok(v - down) for v in row] for row in P]
                E = [[ok(v - down) for v in row] for row in E]
                S = [[ok(v - down) for v in row] for row in S]
                F = [ok(v - down) for v in F]
                tau -= K
        bnd = out
        last = ge * (tau - 1)
        for b in range(B):
            for i in range(R // 2):
                best = max(best, S[b][i] - last - ge * (2 * i + 1), P[b][2 * i + 2] - last - ge * (2 * i + 2))
    return best


# gap pairs at the edges of the rule (Ge <= Go, SM + Go + Ge in 0..255, Ge <= 32), with BLOSUM62 (-4..11)
GAPS = [(10, 2), (11, 1), (4, 0), (2, 2), (5, 5), (32, 32), (31, 30), (232, 12), (244, 0), (60, 17)]


@pytest.mark.parametrize("gaps", GAPS)
@pytest.mark.parametrize("R,B", [(4, 1), (4, 2), (8, 1), (8, 4), (16, 2)])
def test_emulated_offset_cells_equal_the_oracle(blosum, gaps, R, B):
    rng = np.random.default_rng(R * 100 + B * 10 + gaps[0])
    for m, n in [(1, 1), (R, 3), (R * B + 1, 70), (2 * R * B, 150), (37, 66)]:
        q, d = rng.integers(0, 20, m).astype(np.int8), rng.integers(0, 20, n).astype(np.int8)
        k = min(m, n) * 3 // 4
        d[:k] = q[:k]
        want = oracle.scores(q, d, np.array([0, n], np.int64), blosum, *gaps)[0]
        assert offset_score(q.tolist(), d.tolist(), blosum, *gaps, R, B) == want, (m, n)


def _db(seed):
    db = synth.small_db(seed=seed, n=391, lo=0, hi=420)
    rng = np.random.default_rng(seed)
    subs = [db.subject(k).copy() for k in range(db.n)]
    subs[7] = rng.integers(0, 20, 2311).astype(np.int8)
    offs = np.zeros(len(subs) + 1, np.int64)
    offs[1:] = np.cumsum([s.size for s in subs])
    return synth.Database(np.concatenate(subs), offs, name="offset")


@pytest.mark.gpu
@pytest.mark.parametrize("gaps", GAPS + [(233, 12), (33, 33), (10, 11), (1, 1)])      # the last four: plain cells
def test_gaps_at_the_edges_of_the_rule(gpu, blosum, gaps):
    import torch
    db = _db(61)
    queries = [synth.small_query(seed=m, m=m) for m in (1, 15, 16, 17, 129, 300, 1025)]
    for q in queries[3:]:
        db.residues[db.offsets[7]: db.offsets[7] + q.size] = q
    want = [oracle.scores(q, db.residues, db.offsets, blosum, *gaps) for q in queries]
    for pack in (1, 2):
        D = gpu.Database(db.residues, db.offsets, lane_pack=pack)
        got, _, _ = D.search_batch(queries, blosum, *gaps, k=0)
        alone = [D.search(q, blosum, *gaps).cpu().numpy() for q in queries] if pack == 1 else []
        torch.cuda.synchronize()
        for i, w in enumerate(want):
            assert (got[i].cpu().numpy() == w).all(), (pack, queries[i].size)
            assert not alone or (alone[i] == w).all(), queries[i].size
        D.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [4, 8, 16])
@pytest.mark.parametrize("lanes", [1, 2, 8, 16, 32, 64])
def test_lanes_and_rows(gpu, blosum, lanes, rows):
    import torch
    db = _db(62)
    for m in (rows * lanes - 1, rows * lanes, rows * lanes + 1, 2 * rows * lanes + 3):
        q = synth.small_query(seed=m, m=m)
        D = gpu.Database(db.residues, db.offsets, force_lanes=lanes, rows_per_lane=rows)
        got = D.search(q, blosum, 10, 2)
        torch.cuda.synchronize()
        assert (got.cpu().numpy() == oracle.scores(q, db.residues, db.offsets, blosum, 10, 2)).all(), m
        D.close()


@pytest.mark.gpu
@pytest.mark.parametrize("pack", [1, 2])
def test_scores_at_the_end_of_the_offset_range(gpu, blosum, pack):
    """Self scores around 0x7C00 - Go - Ge (K + 17) = 31,572 at 10/2 (W scores 11, A 4, N 6).  A query that can
    score there but not beyond 31,739 keeps plain cells and needs no recompute; one that can reach the plain
    limit runs on offset cells, whose recompute starts at 31,572."""
    import torch
    W, A, N = 17, 0, 2
    top = [np.full(2870, W), np.concatenate([np.full(2869, W), [A, A, A]]), np.concatenate([np.full(2885, W), [A]])]
    longer = np.concatenate([np.full(2870, W), np.full(30, N)])        # can score 31,750
    subs = [np.asarray(x, np.int8) for x in top] + [np.full(60, W, np.int8), longer.astype(np.int8)]
    offs = np.zeros(len(subs) + 1, np.int64)
    offs[1:] = np.cumsum([s.size for s in subs])
    res = np.concatenate(subs)
    D = gpu.Database(res, offs, lane_pack=pack, poison=1)
    for q, flagged in ((top[0], False), (top[1], False), (top[2], False), (longer, True)):
        batch = [np.asarray(q, np.int8)] * pack
        got, _, _ = D.search_batch(batch, blosum, 10, 2, k=0)
        torch.cuda.synchronize()
        want = oracle.scores(batch[0], res, offs, blosum, 10, 2)
        assert all((g.cpu().numpy() == want).all() for g in got)
        assert (D.stats()["rerun_pairs"] > 0) == flagged, q.size
    D.close()

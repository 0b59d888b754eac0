"""A CPU model of how a chained pair is cut into windows and parts of the subject (run_chain in sw_kernels.hip,
alignment_span and semiglobal_span in sw_api.cpp): the largest score of the windows, each starting `span` columns
before its own ones, is the pair's."""
import numpy as np
import pytest

import oracle
from inputs import blosum62, synth

WHOLE = 1 << 28


def span_of(q, sm, go, ge, mode):
    m, top = q.size, int(np.maximum(sm[q].max(axis=1), 0).sum())
    if mode == "local":
        if top <= go:
            return min(m + 1, WHOLE)
        return WHOLE if ge <= 0 or ge > go else min(m + (top - go) // ge + 1, WHOLE)
    return WHOLE if ge <= 0 or ge > go else min(m + (top + (m - 1) * ge) // ge + 1, WHOLE)


def windows(cols, count, span):
    """Column ranges [start, end) of `count` windows over all parts."""
    core = ((cols // 4 + count - 1) // count) * 4
    for at in range(count):
        if at * core < cols:
            yield max(0, at * core - span) & ~3, min(cols, (at + 1) * core)


def subject_with(rng, q, n):
    """Mutated stretches of the query with long gaps in them, spread over the subject."""
    s = synth.background_residues(rng, n)
    for _ in range(6):
        a, b = sorted(rng.integers(0, q.size + 1, 2))
        gap = int(rng.integers(0, 3 * q.size))
        piece = np.concatenate([q[a:(a + b) // 2], synth.background_residues(rng, gap), q[(a + b) // 2:b]])[:n]
        at = int(rng.integers(0, n - piece.size + 1))
        s[at:at + piece.size] = piece
    return s


@pytest.mark.parametrize("mode", ["local", "semiglobal"])
@pytest.mark.parametrize("go,ge", [(10, 2), (11, 1), (3, 1), (1, 1), (0, 0), (12, 0), (30, 5), (400, 1)])
def test_the_windows_hold_the_pairs_score(mode, go, ge):
    sm = blosum62()
    rng = np.random.default_rng(9000 + 10 * go + ge)
    cut = 0
    for m in (1, 2, 7, 30, 61):
        q = synth.background_residues(rng, m)
        span = span_of(q, sm, go, ge, mode)
        for n in (1, 5, 64, 333, 1200):
            s = subject_with(rng, q, n)
            want = oracle.pair_mode(q, s, sm, go, ge, mode)
            for count in (1, 2, 3, 4, 8, 32):
                got = [oracle.pair_mode(q, s[a:b], sm, go, ge, mode) for a, b in windows(-(-n // 4) * 4, count, span) if a < n]
                assert max(got) == want, (m, n, count, span, got, want)
                cut += len(got) > 1
    assert cut > 20


def test_a_shorter_span_loses_scores():
    """The span is not far from the least: at half of it, some pair's best alignment lies in no window."""
    sm = blosum62()
    rng = np.random.default_rng(9100)
    W, lost = 17, 0
    for m in (8, 20, 40):
        q = np.full(m, W, np.int8)
        for gap in range(m, 5 * m, 3):
            # the two halves of the query, as far apart as a gap still pays for
            s = np.concatenate([np.full(40, 2, np.int8), q[:m // 2], np.full(gap, 2, np.int8), q[m // 2:],
                                np.full(40, 2, np.int8)])
            want = oracle.pair(q, s, sm, 10, 2)
            for span, must in ((span_of(q, sm, 10, 2, "local"), True), (m // 2, False)):
                got = max(oracle.pair(q, s[a:b], sm, 10, 2) for a, b in windows(-(-s.size // 4) * 4, 8, span) if a < s.size)
                assert got == want or not must
                lost += got != want
    assert lost > 0

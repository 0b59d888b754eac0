"""Bands of rows behind one another (sw_pair and the traceback fill) at the edges
of a band, of a read of 32 columns and of the waves' 64 steps of skew, and with
more bands than waves, against the oracle (tolerance 0)."""
import numpy as np
import pytest

import oracle
from inputs import synth

pytestmark = pytest.mark.gpu


def _related(rng, q, n):
    """n residues, two thirds of them a stretch of q with an insertion halfway."""
    s = synth.background_residues(rng, n)
    k = min(q.size, 2 * n // 3) - 3
    if k >= 8:
        a = int(rng.integers(0, q.size - k + 1))
        s[: k // 2] = q[a:a + k // 2]
        s[k // 2 + 3:k + 3] = q[a + k // 2:a + k]
    return s


@pytest.mark.parametrize("m", [31, 127, 128, 129, 255, 256, 257, 512, 513, 900])
def test_pair_and_alignment_at_band_edges(gpu, blosum, m):
    rng = np.random.default_rng(6100 + m)
    q = synth.background_residues(rng, m)
    lens = [1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 700]
    subs = [_related(rng, q, n) for n in lens]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    D = gpu.Database(np.concatenate(subs), offs)
    for go, ge in ((10, 2), (0, 1), (3, 5), (2**31 - 1, 2**31 - 1)):
        got = D.align(q, list(range(len(lens))), blosum, go, ge)
        for a, s in zip(got, subs):
            want = oracle.align(q, s, blosum, min(go, 1 << 28), min(ge, 1 << 28))
            for key in ("score", "q_begin", "q_end", "s_begin", "s_end", "ops"):
                assert a[key] == want[key], f"m={m} n={s.size} {go}/{ge} {key}: got {a[key]!r} want {want[key]!r}"
            assert int(gpu.sw_pair(q, s, blosum, go, ge).item()) == want["score"], (m, s.size, go, ge)
    D.close()


def test_more_bands_than_waves(gpu, blosum):
    rng = np.random.default_rng(6200)
    q = synth.background_residues(rng, 270_000)            # 1,055 bands of 256 rows, 2,110 of 128
    s = np.concatenate([q[200_000:200_030], synth.background_residues(rng, 9)])
    want = oracle.align(q, s, blosum, 10, 2)
    assert int(gpu.sw_pair(q, s, blosum, 10, 2).item()) == want["score"]
    assert int(gpu.sw_pair(s, q, blosum, 10, 2).item()) == want["score"]
    D = gpu.Database(s, np.array([0, s.size], np.int64))
    a = D.align(q, [0], blosum, 10, 2)[0]
    assert all(a[k] == want[k] for k in ("score", "q_begin", "q_end", "s_begin", "s_end", "ops"))
    D.close()


def test_pair_matrix_that_is_not_symmetric(gpu):
    rng = np.random.default_rng(6300)
    sm = rng.integers(-9, 10, (20, 20)).astype(np.int8)
    for m, n in ((300, 90), (90, 300)):
        q, s = synth.background_residues(rng, m), synth.background_residues(rng, n)
        assert int(gpu.sw_pair(q, s, sm, 7, 1).item()) == oracle.pair(q, s, sm, 7, 1)


@pytest.mark.parametrize("longest,count", [(35_000, 150), (2_200_000, 3)])
def test_alignments_that_come_back_in_pieces(gpu, blosum, longest, count):
    """More operations than the handle's pinned buffer (2 MiB) holds, of all pairs together or of one."""
    rng = np.random.default_rng(6400)
    q = synth.background_residues(rng, 60)
    lens = [longest] + [int(x) for x in rng.integers(1, 200, count - 1)]
    subs = [_related(rng, q, n) for n in lens]
    offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    D = gpu.Database(np.concatenate(subs), offs)
    order = [int(x) for x in rng.permutation(count)]
    for _ in range(2):
        for a, k in zip(D.align(q, order, blosum, 10, 2), order):
            want = oracle.align(q, subs[k], blosum, 10, 2)
            assert a["subject"] == k
            for key in ("score", "q_begin", "q_end", "s_begin", "s_end", "ops"):
                assert a[key] == want[key], f"n={subs[k].size} {key}: got {a[key]!r} want {want[key]!r}"
    D.close()

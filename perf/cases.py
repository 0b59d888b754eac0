"""Timed cases of the protein search library: what its users call, over the sizes they call it with.

A case is a dict of plain values.  ``kind`` names the entry point:

* ``search``   ``Database.search``: one query against a packed database, local, global or semi-global;
* ``batch``    ``Database.search_batch``: several queries at once, scores and top hits or the top hits alone;
* ``align``    ``Database.align_batch``: the alignments of each query's top hits;
* ``pair``     ``sw_pair``: one long query against one long subject over the whole GPU;
* ``topk``     ``topk``: the best subjects of one score vector.

The databases follow the repository's workloads: log-normal subject lengths (median 300, clipped to
20..35,000), i.i.d. residues with protein background frequencies, mutated copies of every query planted
among the subjects and, from 10,000 subjects on, a tail of 16 subjects of 5,000..35,000 residues.  The
packed handle is what a program keeps between calls, so it belongs to the state; the query arrives in
host memory with every call, as in a search service.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2309_09609_amd as sw

SIGMA = 0.61          # shape of the log-normal subject lengths
LONGEST = 35_000      # residues of the longest protein

LETTERS = "ARNDCQEGHILKMFPSTWYVBZX*"
FREQUENCIES = (0.07805, 0.05129, 0.04487, 0.05364, 0.01925, 0.04264, 0.06295, 0.07377, 0.02199, 0.05142,
               0.09019, 0.05744, 0.02243, 0.03856, 0.05203, 0.07120, 0.05841, 0.01330, 0.03216, 0.06441)
# BLOSUM62 (Henikoff & Henikoff 1992), lower triangle in the order of LETTERS
BLOSUM62 = """
4
-1 5
-2 0 6
-2 -2 1 6
0 -3 -3 -3 9
-1 1 0 0 -3 5
-1 0 0 2 -4 2 5
0 -2 0 -1 -3 -2 -2 6
-2 0 1 -1 -3 0 0 -2 8
-1 -3 -3 -3 -1 -3 -3 -4 -3 4
-1 -2 -3 -4 -1 -2 -3 -4 -3 2 4
-1 2 0 -1 -3 1 1 -2 -1 -3 -2 5
-1 -1 -2 -3 -1 0 -2 -3 -2 1 2 -1 5
-2 -3 -3 -3 -2 -3 -3 -3 -1 0 0 -3 0 6
-1 -2 -2 -1 -3 -1 -1 -2 -2 -3 -3 -1 -2 -4 7
1 -1 1 0 -1 0 0 0 -1 -2 -2 0 -1 -2 -1 4
0 -1 0 -1 -1 -1 -1 -2 -2 -1 -1 -1 -1 -2 -1 1 5
-3 -3 -4 -4 -2 -2 -3 -2 -2 -3 -2 -3 -1 1 -4 -3 -2 11
-2 -2 -2 -3 -2 -1 -2 -3 2 -1 -1 -2 -1 3 -3 -2 -2 2 7
0 -3 -3 -3 -1 -2 -2 -3 -3 3 1 -2 1 -1 -2 -2 0 -3 -1 4
-2 -1 3 4 -3 0 1 -1 0 -3 -4 0 -3 -3 -2 0 -1 -4 -3 -3 4
-1 0 0 1 -3 3 4 -2 0 -3 -3 1 -1 -3 -1 0 -1 -3 -2 -2 1 4
0 -1 -1 -1 -2 -1 -1 -1 -1 -1 -1 -1 -1 -1 -2 0 0 -2 -1 -1 -1 -1 -1
-4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 -4 1
"""


def matrix(letters: int) -> np.ndarray:
    m = np.zeros((24, 24), np.int8)
    for i, line in enumerate(BLOSUM62.split("\n")[1:25]):
        for j, v in enumerate(line.split()):
            m[i, j] = m[j, i] = int(v)
    return np.ascontiguousarray(m[:letters, :letters])


# ------------------------------------------------------------------ the cases
def _search(name, subjects, qlen, mode="local", clip=LONGEST, go=10, ge=2, letters=20):
    return {"name": name, "kind": "search", "subjects": subjects, "clip": clip, "qlen": qlen, "mode": mode,
            "go": go, "ge": ge, "letters": letters}


def _batch(name, subjects, queries, lo, hi, lane_pack, k, scores, memory="library", shortest=20):
    return {"name": name, "kind": "batch", "subjects": subjects, "queries": queries, "qmin": lo, "qmax": hi,
            "lane_pack": lane_pack, "k": k, "scores": scores, "memory": memory, "shortest": shortest,
            "go": 10, "ge": 2, "letters": 20}


def listed():
    return [
        # a query against one organism's or family's small database: latency and launches count
        _search("search_144_2k", 2_000, 144, clip=1_000),
        # the shortest query of the paper-scale workload against the whole 570,000-subject database
        _search("search_144_570k", 570_000, 144),
        # an ordinary query of odd length against it
        _search("search_1003_570k", 570_000, 1_003),
        # the longest query of the workload: the largest single search
        _search("search_5478_570k", 570_000, 5_478),
        # the end-to-end modes (the whole query against whole subjects, or against any stretch of them)
        _search("global_405_570k", 570_000, 405, mode="global"),
        _search("semiglobal_331_100k", 100_000, 331, mode="semiglobal"),
        # many queries against a mid-sized database in one call, two queries per lane, scores and top hits
        _batch("batch_16_40k", 40_000, 16, 50, 5_000, lane_pack=2, k=10, scores=True),
        # a few queries with the handle's defaults against a small database
        _batch("batch_6_5k", 5_000, 6, 144, 1_100, lane_pack=1, k=10, scores=True),
        # two length-matched requests of a search service: the caller's workspace, the top hits alone
        _batch("served_2_200k", 200_000, 2, 330, 361, lane_pack=2, k=10, scores=False, memory="torch"),
        # the alignments behind ten top hits of each of eight queries
        {"name": "align_8x10", "kind": "align", "subjects": 20_000, "queries": 8, "hits": 10, "qmin": 144, "qmax": 2_600,
         "go": 10, "ge": 2, "letters": 20},
        # one long pair over the whole GPU
        {"name": "pair_20k", "kind": "pair", "qlen": 20_001, "slen": 19_500, "go": 10, "ge": 2, "letters": 20},
        # the top ten of one search's scores
        {"name": "topk_10_570k", "kind": "topk", "subjects": 570_000, "k": 10},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any entry point, sizes spread over their logarithm, the options
    that are used in earnest (11/1 gaps, the 24-letter alphabet, either lane packing, either memory)."""
    kind = rng.choice(("search", "search", "search", "mode", "batch", "batch", "align", "pair", "topk"))
    go, ge = rng.choice(((10, 2), (10, 2), (11, 1)))
    letters = rng.choice((20, 20, 24))
    if kind in ("search", "mode"):
        mode = "local" if kind == "search" else rng.choice(("global", "semiglobal"))
        qlen = _log(rng, 30, 5_478 if mode == "local" else 3_000)
        c = _search("", _log(rng, 200, 570_000), qlen, mode=mode, go=go, ge=ge, letters=letters)
    elif kind == "batch":
        queries = rng.randint(2, 24)
        hi = _log(rng, 100, 5_000)
        lane_pack = rng.choice((1, 2))
        subjects = _log(rng, 500, max(600, min(200_000, int(1.2e9 / (queries * hi)))))
        shortest = 20
        if rng.random() < 0.25:        # a database of long subjects
            subjects, shortest = max(64, subjects // 40), 3_000
        c = _batch("", subjects, queries, max(30, hi // rng.choice((2, 10))), hi, lane_pack=lane_pack,
                   k=rng.choice((1, 10, 100)), scores=rng.random() < 0.5, memory=rng.choice(("library", "torch")),
                   shortest=shortest)
        c.update(go=go, ge=ge, letters=letters)
    elif kind == "align":
        qmax = _log(rng, 150, 5_478)
        c = {"kind": "align", "subjects": _log(rng, 1_000, 20_000), "queries": rng.randint(1, 12),
             "hits": rng.choice((1, 5, 10)), "qmin": max(50, qmax // 8), "qmax": qmax, "go": go, "ge": ge,
             "letters": letters}
    elif kind == "pair":
        c = {"kind": "pair", "qlen": _log(rng, 500, 40_000), "slen": _log(rng, 500, 40_000), "go": go, "ge": ge,
             "letters": letters}
    else:
        c = {"kind": "topk", "subjects": _log(rng, 1_000, 10_000_000), "k": rng.choice((1, 10, 100, 1_000))}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs
def _rng(seed, stream):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence(seed, spawn_key=(stream,))))


def _frequencies(letters):
    f = np.array(FREQUENCIES, np.float64)
    if letters > 20:                   # the ambiguity codes are rare, but they occur
        f = np.concatenate([f / f.sum(), np.full(letters - 20, 1e-4)])
    return f / f.sum()


def _protein(rng, length, letters):
    return rng.choice(letters, size=int(length), p=_frequencies(letters)).astype(np.int8)


def _homolog(rng, seq, letters):
    """A mutated copy: 10-60 % substitutions and a few short gaps."""
    s = seq.copy()
    hit = rng.random(s.size) < rng.uniform(0.1, 0.6)
    s[hit] = _protein(rng, int(hit.sum()), letters)
    for _ in range(int(rng.integers(0, 2 + s.size // 200))):
        at, gap = int(rng.integers(0, s.size)), int(rng.geometric(0.4))
        s = np.concatenate([s[:at], s[at + gap:] if rng.random() < 0.5 else np.concatenate([_protein(rng, gap, letters), s[at:]])])
    return s if s.size else seq.copy()


def _lengths(c, seed):
    """Subject lengths, the same for a case whatever the seed's residues (work() needs their sum)."""
    n, shortest = c["subjects"], c.get("shortest", 20)
    rng = _rng(c["subjects"], 0)
    if shortest > 20:
        return rng.integers(shortest, LONGEST + 1, size=n).astype(np.int64)
    lens = np.clip(np.rint(np.exp(rng.normal(math.log(300), SIGMA, size=n))), shortest, c.get("clip", LONGEST))
    lens = lens.astype(np.int64)
    if n >= 10_000 and c.get("clip", LONGEST) == LONGEST:
        lens[-16:] = np.rint(np.exp(rng.uniform(math.log(5_000), math.log(LONGEST), size=16)))
        lens[-1] = LONGEST
    return lens


def _qlens(c):
    if "qlen" in c:
        return [c["qlen"]]
    rng = _rng(c["queries"], 1)
    return [int(x) for x in np.rint(np.exp(rng.uniform(math.log(c["qmin"]), math.log(c["qmax"]), size=c["queries"])))]


def _device_residues(seed, count, letters):
    cum = torch.from_numpy(np.cumsum(_frequencies(letters))[:-1] * 65536).round().to(torch.int32).cuda()
    lut = torch.bucketize(torch.arange(65536, dtype=torch.int32, device="cuda"), cum, right=True).to(torch.int8)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = torch.empty(count, dtype=torch.int8, device="cuda")
    for a in range(0, count, 1 << 26):
        b = min(count, a + (1 << 26))
        out[a:b] = lut[torch.randint(0, 65536, (b - a,), generator=g, device="cuda", dtype=torch.int32)]
    return out


def _database(c, seed):
    """(queries, residues on the GPU, offsets, planted subjects of each query)"""
    rng = _rng(seed, 2)
    letters = c["letters"]
    queries = [_protein(rng, m, letters) for m in _qlens(c)]
    lens = _lengths(c, seed)
    n = lens.size
    planted, inserts = [], {}
    per = min(c.get("hits", 5), max(1, n // (4 * len(queries))))
    place = _rng(c["subjects"], 3).permutation(max(1, n - 16))
    for qi, q in enumerate(queries):
        mine = [int(x) for x in place[qi * per:(qi + 1) * per]]
        planted.append(mine)
        for k in mine:
            h = _homolog(rng, q, letters)[: lens[k]]       # homologous along the subject's whole length
            inserts[k] = h
    offsets = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offsets[1:])
    res = _device_residues(seed, int(offsets[-1]), letters)
    for k, h in inserts.items():
        res[offsets[k]: offsets[k] + h.size] = torch.from_numpy(h).cuda()
    return queries, res, offsets, planted


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "topk":
        # scores as a search leaves them: an extreme-value background, a few homologs, many ties
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        u = torch.rand(c["subjects"], generator=g, device="cuda").clamp_(1e-7, 1 - 1e-7)
        s = (38.0 - 4.2 * torch.log(-torch.log(u))).to(torch.int32)
        at = torch.randint(0, c["subjects"], (20,), generator=g, device="cuda")
        s[at] = torch.randint(150, 3_000, (20,), generator=g, device="cuda", dtype=torch.int32)
        return {"case": c, "scores": s}
    if kind == "pair":
        rng = _rng(seed, 2)
        q = _protein(rng, c["qlen"], c["letters"])
        s = _protein(rng, c["slen"], c["letters"])
        seg = _homolog(rng, q[: min(q.size, s.size) // 3], c["letters"])[: s.size]
        at = int(rng.integers(0, s.size - seg.size + 1))
        s[at: at + seg.size] = seg
        return {"case": c, "query": q, "subject": s, "subst": matrix(c["letters"])}
    queries, res, offsets, planted = _database(c, seed)
    db = sw.Database(res, offsets, alphabet=c["letters"], lane_pack=c.get("lane_pack", 0),
                     memory=c.get("memory", "library"))
    state = {"case": c, "db": db, "queries": queries, "subst": matrix(c["letters"])}
    if kind == "align":
        rng = _rng(seed, 4)
        state["subjects"] = [np.array(p + [int(x) for x in rng.integers(0, db.n, size=c["hits"] - len(p))], np.int64)
                             for p in planted]
        lens = np.diff(offsets)
        state["room"] = sum(_qlens(c)) * c["hits"] + c["queries"] * c["hits"] * int(lens.max())
    return state


# ------------------------------------------------------------------ one pass
def _paths(alignments, room):
    """Every operation of every alignment, one after the other, in an array whose size the case alone decides."""
    ops = "".join(a["ops"] for a in alignments).encode()
    out = np.zeros(room, np.uint8)
    out[: len(ops)] = np.frombuffer(ops, np.uint8)
    return out


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "search":
        return state["db"].search(state["queries"][0], state["subst"], c["go"], c["ge"], mode=c["mode"])
    if kind == "batch":
        scores, top, index = state["db"].search_batch(state["queries"], state["subst"], c["go"], c["ge"], k=c["k"],
                                                      keep_scores=c["scores"])
        return {"scores": scores, "top": top, "index": index} if c["scores"] else {"top": top, "index": index}
    if kind == "align":
        rows = state["db"].align_batch(state["queries"], state["subjects"], state["subst"], c["go"], c["ge"])
        flat = [a for row in rows for a in row]
        return {"ends": np.array([[a["score"], a["q_begin"], a["q_end"], a["subject"], a["s_begin"], a["s_end"],
                                   len(a["ops"])] for a in flat], np.int64),
                "ops": _paths(flat, state["room"])}
    if kind == "pair":
        return sw.sw_pair(state["query"], state["subject"], state["subst"], c["go"], c["ge"], alphabet=c["letters"])
    top, index = sw.topk(state["scores"], c["k"])
    return {"top": top, "index": index}


def work(case):
    """Residues (or scores) read once, results written once; 10 elementary integer operations per cell
    (Eq. 1-3 with H - Go shared, and the running maximum)."""
    kind = case["kind"]
    if kind == "topk":
        return {"bytes": 4 * case["subjects"] + 12 * case["k"], "flops": case["subjects"]}
    if kind == "pair":
        return {"bytes": case["qlen"] + case["slen"], "flops": 10 * case["qlen"] * case["slen"]}
    qlens = _qlens(case)
    if kind == "align":
        # each hit: its matrix once, the residues and the path
        mean = 300 * math.exp(SIGMA * SIGMA / 2)
        return {"bytes": int(sum(qlens) * 2 + case["queries"] * case["hits"] * mean * 2),
                "flops": int(10 * sum(qlens) * case["hits"] * mean)}
    lens = _lengths(case, 0)
    out = 4 * lens.size * len(qlens)
    return {"bytes": int(lens.sum()) + out, "flops": 10 * sum(qlens) * int(lens.sum())}


# ------------------------------------------------------------------ plain 64-bit values
EXACT_CELLS = 3_000_000_000        # padded cells that plain torch sweeps in a few seconds
NEG = -(1 << 40)


def _scores64(q, res, offsets, sm, go, ge, mode):
    """Scores of one query against every subject, all subjects' anti-diagonals at once, int64."""
    dev = res.device
    n, m = offsets.size - 1, int(q.size)
    lens = torch.from_numpy(np.diff(offsets)).to(dev)
    width = int(lens.max())
    A = sm.shape[0]
    cols = torch.arange(width, device=dev)
    pad = torch.full((n, width + 2 * m), A, dtype=torch.int64, device=dev)
    at = torch.from_numpy(offsets[:-1]).to(dev)[:, None] + cols[None]
    inside = cols[None] < lens[:, None]
    pad[:, m: m + width] = torch.where(inside, res[at.clamp_(max=res.numel() - 1)].long(), torch.tensor(A, device=dev))
    table = torch.zeros((A, A + 1), dtype=torch.int64, device=dev)
    table[:, :A] = torch.from_numpy(sm.astype(np.int64)).to(dev)
    base = torch.from_numpy(q.astype(np.int64)).to(dev) * (A + 1)
    rows = torch.arange(m + 1, device=dev)
    gap = lambda k: torch.where(k > 0, -(go + (k - 1) * min(go, ge)), torch.zeros_like(k))  # noqa: E731
    local = mode == "local"
    border = torch.zeros(m + 1, dtype=torch.int64, device=dev) if local else gap(rows)
    H2 = torch.full((n, m + 1), 0 if local else NEG, dtype=torch.int64, device=dev)
    H1 = H2.clone()
    H1[:, 0] = 0
    E = torch.full((n, m + 1), NEG, dtype=torch.int64, device=dev)
    F = E.clone()
    best = torch.full((n,), 0 if local else NEG, dtype=torch.int64, device=dev)
    if mode == "semiglobal":
        best[:] = border[m]
    for d in range(1, m + width + 1):
        E = torch.maximum(H1 - go, E - ge)
        F = torch.roll(torch.maximum(H1 - go, F - ge), 1, 1)
        hd = torch.full_like(H1, NEG)
        if d >= 2:
            code = pad[:, d - 1: d - 1 + m].flip(1)
            hd[:, 1:] = H2[:, :-1] + table.view(-1)[base[None] + code]
        H = torch.maximum(hd, torch.maximum(E, F))
        if local:
            H.clamp_(min=0)
        j = d - rows
        H[:, 0] = 0 if (local or mode == "semiglobal") else gap(torch.tensor(d)).item()
        if d <= m:
            H[:, d] = border[d]
            E[:, d] = NEG
        F[:, 0] = NEG
        if local:
            ok = (j[None] >= 1) & (j[None] <= lens[:, None])
            ok[:, 0] = False
            best = torch.maximum(best, torch.where(ok, H, torch.zeros_like(H)).amax(1))
        else:
            jm = d - m
            if jm >= 1:
                best = torch.where(lens == jm, H[:, m], best) if mode == "global" else \
                    torch.where(lens >= jm, torch.maximum(best, H[:, m]), best)
        H2, H1 = H1, H
    return best


def _top64(scores, k):
    s = scores.cpu().numpy()
    order = np.lexsort((np.arange(s.size), -s))[:k]
    top = np.full(k, -1, np.int64)
    index = np.full(k, -1, np.int64)
    top[: order.size] = s[order]
    index[: order.size] = order
    return torch.from_numpy(top), torch.from_numpy(index)


def exact(case, seed):
    kind = case["kind"]
    if kind == "topk":
        top, index = _top64(prepare(case, seed)["scores"], case["k"])
        return {"top": top, "index": index}
    if kind == "align":
        return None                    # paths: whole values
    if kind == "pair":
        s = prepare(case, seed)
        res = torch.from_numpy(s["subject"]).cuda()
        if case["qlen"] + case["slen"] > 45_000:
            return None
        return _scores64(s["query"], res, np.array([0, res.numel()], np.int64), s["subst"], case["go"], case["ge"],
                         "local")
    lens = _lengths(case, seed)
    qlens = _qlens(case)
    if lens.size * int(lens.max()) * sum(qlens) > EXACT_CELLS or len(qlens) > 8:
        return None
    queries, res, offsets, _ = _database(dict(case), seed)
    sm = matrix(case["letters"])
    rows = [_scores64(q, res, offsets, sm, case["go"], case["ge"], case.get("mode", "local")) for q in queries]
    if kind == "search":
        return rows[0]
    tops = [_top64(r, case["k"]) for r in rows]
    out = {"top": torch.stack([t for t, _ in tops]), "index": torch.stack([i for _, i in tops])}
    if case["scores"]:
        out["scores"] = torch.stack(rows)
    return out

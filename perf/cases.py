"""Timed cases of the word counter: the calls its users make, over the sizes they make them at.

A case is a dict of plain values; `listed()` names twelve, `draw()` gives more of the same
ranges. `prepare()` makes on the GPU what a program holds before the call (text, offsets, a kept
workspace, a batch plan, a running server), `run()` makes one pass through the public entry
points of `paper_2206_05269_amd.wc`, `work()` states the bytes such a pass cannot do without.

Text. Words of a seeded vocabulary drawn with a finite Zipf law, one separator after each, one
word in twenty capitalised: the recipe of the package's synthetic corpora, written here without
its bookkeeping so that inputs take little time to make. With "long" set, one vocabulary word in
500 has 17 to 40 bytes (compounds, links, file names); with kind "utf8", a third of the words are
made of two- and three-byte letters. Documents end right after a delimiter and have lognormal
sizes.

Order. The library leaves the order of a table's entries open (it depends on which lane claims a
slot first), so two right answers differ as arrays. What `run()` returns is a `Read`: a dict that
holds the pass's tables as the call left them and puts them in canonical order (by document, then
by word) when its values are read, followed by zeros up to a length that the case alone gives (the
number of distinct words differs a little from seed to seed). The order is for comparing; a
program that uses a table does not need it, and a pass does not make it.
"""
import functools
import math
import statistics

import numpy as np
import torch

from paper_2206_05269_amd import wc

KiB, MiB, GiB = 1 << 10, 1 << 20, 1 << 30
DEV = "cuda:0"
_SEP = b"        \n,"  # space 0.8, newline 0.1, punctuation 0.1


# ------------------------------------------------------------------------------------------
# the cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # one small request counted by itself: the median-and-below request of a serving mix
        _count("request-24k", 24 * KiB + 77, vocab=500_000, zipf=1.05, shift=5, count_bytes=8),
        # the smallest corpus of the benchmark: four documents, one megabyte, a kept workspace
        _count("plain-1mb", 1_000_000, docs=4, vocab=5000, zipf=1.1, keep=True),
        # one corpus of the per-corpus comparison: 2,000 documents, 20 MB, one table
        _count("corpus-20mb", 20_000_000, docs=2000, vocab=50_000, zipf=1.05),
        # the largest request of a serving mix: one text of 64 MB with long words, odd in
        # size and placed at an odd address
        _count("text-64mb", 64 * MiB - 4099, vocab=500_000, zipf=1.05, shift=11, count_bytes=8,
               long=True),
        # the single-stream benchmark: 8 GiB, a million words, 2^22 slots, 64-bit counts
        _count("stream-8gib", 8 * GiB, vocab=1_000_000, max_len=16, zipf=1.0, keep=True,
               count_bytes=8, slots=1 << 22),
        # one table per document of the same 20 MB corpus (the map of a per-corpus comparison)
        _docs("perdoc-2000", 2000, median=8 * KiB, lo=2 * KiB, hi=20 * KiB, vocab=50_000,
              zipf=1.05),
        # the batch benchmark: 100,000 documents of 200 B to 1 MiB through a captured graph
        _docs("batch-100k", 100_000, median=16 * KiB, lo=200, hi=MiB, vocab=200_000, zipf=1.1,
              batch=True),
        # the reduce: per-document tables of 2,000 documents summed into one table
        _merge("merge-2000", 2000, vocab=50_000, zipf=1.05),
        # the per-corpus comparison itself: the top 50 words of four corpora
        _topk("topk-4x20mb", 4, 20_000_000, k=50, vocab=50_000, zipf=1.05),
        # text in other languages, under the UTF-8 reading
        _utf8("utf8-16mb", 16 * MiB + 1021, docs=200, vocab=100_000, zipf=1.05),
        # a burst of requests to the server, then a merge query over their tables
        _serve("serve-96", 96, vocab=500_000, zipf=1.05),
        # a text in pinned host memory, copied and counted
        _host("host-192mb", 192 * MiB + 333, vocab=500_000, zipf=1.05),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def size(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | (rng.random() < 0.5)

    text = dict(vocab=size(5000, 1_000_000), zipf=round(rng.uniform(1.0, 1.15), 3))
    kind = rng.choice(["count"] * 5 + ["docs"] * 2 + ["batch", "merge", "topk", "utf8", "serve", "host"])
    if kind == "count":
        return _count(None, size(KiB, 3 * GiB), docs=rng.choice([1, 1, 1, size(2, 3000)]),
                      max_len=rng.choice([12, 12, 16]), shift=rng.randrange(16),
                      count_bytes=rng.choice([4, 8]), long=rng.random() < 0.4,
                      keep=rng.random() < 0.3, **text)
    if kind == "docs":
        m = size(2 * KiB, 24 * KiB)
        return _docs(None, size(20, 4000), median=m, lo=m // 8 + 16, hi=m * 8,
                     count_bytes=rng.choice([4, 8]), long=rng.random() < 0.4, **text)
    if kind == "batch":
        return _docs(None, size(1000, 30_000), median=size(4 * KiB, 24 * KiB), lo=200, hi=MiB,
                     batch=True, **text)
    if kind == "merge":
        return _merge(None, size(20, 4000), **text)
    if kind == "topk":
        return _topk(None, rng.randint(2, 8), size(MiB, 24 * MiB), k=rng.choice([10, 50, 200]),
                     **text)
    if kind == "utf8":
        return _utf8(None, size(32 * KiB, 48 * MiB), docs=size(1, 500), **text)
    if kind == "serve":
        return _serve(None, rng.randint(16, 128), **text)
    return _host(None, size(2 * MiB, 384 * MiB), **text)


def _case(name, **kw):
    return {"name": name, **kw} if name else kw


def _count(name, nbytes, docs=1, vocab=50_000, max_len=12, zipf=1.05, shift=0, count_bytes=4,
           long=False, keep=False, slots=0):
    """wc.count into one table. shift: address of the text mod 16; keep: the program keeps the
    call's workspace (else each call takes one from the caching allocator)."""
    return _case(name, kind="count", bytes=nbytes, docs=min(docs, nbytes // 64 + 1), vocab=vocab,
                 max_len=max_len, zipf=zipf, shift=shift, count_bytes=count_bytes, long=long,
                 keep=keep, slots=slots)


def _docs(name, docs, median, lo, hi, vocab, zipf, count_bytes=4, long=False, batch=False):
    """One table per document: wc.count(per_doc=True), or wc.Batch with its captured graph."""
    return _case(name, kind="docs", docs=docs, median=median, lo=lo, hi=hi, vocab=vocab,
                 max_len=12, zipf=zipf, count_bytes=count_bytes, long=long, batch=batch)


def _merge(name, docs, vocab, zipf):
    return _case(name, kind="merge", docs=docs, median=8 * KiB, lo=2 * KiB, hi=20 * KiB,
                 vocab=vocab, max_len=12, zipf=zipf, long=False)


def _topk(name, corpora, nbytes, k, vocab, zipf):
    return _case(name, kind="topk", corpora=corpora, bytes=nbytes, k=k, vocab=vocab, max_len=12,
                 zipf=zipf)


def _utf8(name, nbytes, docs, vocab, zipf):
    return _case(name, kind="utf8", bytes=nbytes, docs=min(docs, nbytes // 64 + 1), vocab=vocab,
                 max_len=12, zipf=zipf, count_bytes=8)


def _serve(name, requests, vocab, zipf):
    """A burst of requests of 1 KiB to 4 MiB (lognormal, median 64 KiB) in device memory."""
    return _case(name, kind="serve", docs=requests, median=64 * KiB, lo=KiB, hi=4 * MiB,
                 vocab=vocab, max_len=12, zipf=zipf)


def _host(name, nbytes, vocab, zipf):
    return _case(name, kind="host", bytes=nbytes, vocab=vocab, max_len=12, zipf=zipf)


# ------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------
def _zipf(n, s, factor=None):
    w = np.arange(1, n + 1, dtype=np.float64) ** (-s)
    if factor is not None:
        w *= factor
    return w / w.sum()


def _vocabulary(case, seed):
    """(words uint8[n, L] zero padded, lengths int64[n]) on the GPU."""
    rng = np.random.default_rng(seed)
    n, top = case["vocab"], case["max_len"]
    lens = rng.integers(1, top + 1, size=n)
    if case.get("long"):
        pick = rng.random(n) < 0.002
        lens[pick] = rng.integers(17, 41, size=int(pick.sum()))
    L = int(lens.max())
    w = rng.integers(ord("a"), ord("z") + 1, size=(n, L), dtype=np.uint8)
    w[np.arange(L)[None, :] >= lens[:, None]] = 0
    if case["kind"] == "utf8":
        # a third of the words: letters of two bytes (U+0430..U+044F) or of three (U+4E00..)
        other = np.flatnonzero(rng.random(n) < 1 / 3)
        letters = np.maximum(1, lens[other] // 2)
        wide = rng.random(len(other)) < 0.5
        wide3 = np.zeros((n, 3 * max(1, top // 2)), dtype=np.uint8)
        cp = rng.integers(0, 32, size=(len(other), max(1, top // 2)))
        for j in range(max(1, top // 2)):
            m2, m3 = ~wide & (letters > j), wide & (letters > j)
            c2, c3 = 0x430 + cp[m2, j], 0x4E00 + 7 * cp[m3, j]
            wide3[other[m2], 2 * j] = 0xC0 | (c2 >> 6)
            wide3[other[m2], 2 * j + 1] = 0x80 | (c2 & 63)
            wide3[other[m3], 3 * j] = 0xE0 | (c3 >> 12)
            wide3[other[m3], 3 * j + 1] = 0x80 | ((c3 >> 6) & 63)
            wide3[other[m3], 3 * j + 2] = 0x80 | (c3 & 63)
        lens[other] = letters * np.where(wide, 3, 2)
        full = np.zeros((n, max(L, wide3.shape[1])), dtype=np.uint8)
        full[:, :L] = w
        full[other] = 0
        full[other, :wide3.shape[1]] = wide3[other]
        w = full
    return torch.from_numpy(w).to(DEV), torch.from_numpy(lens.astype(np.int64)).to(DEV)


def _text(case, nbytes, seed, words=None, probs=None):
    """uint8[nbytes] on the GPU: drawn words with their separators, spaces after the last."""
    words, lens = words if words is not None else _vocabulary(case, seed)
    p = probs if probs is not None else _zipf(case["vocab"], case["zipf"])
    mean = float((p * (lens.cpu().numpy() + 1)).sum())
    cdf = torch.from_numpy(np.cumsum(p)).to(DEV)
    sep = torch.tensor(list(_SEP), dtype=torch.uint8, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    out = torch.full((nbytes,), 0x20, dtype=torch.uint8, device=DEV)
    at, done = 0, False
    while not done:
        want = min(1 << 26, int((nbytes - at) / mean * 1.1) + 4096)
        u = torch.rand(want, generator=gen, device=DEV, dtype=torch.float64)
        r = torch.searchsorted(cdf, u, right=True).clamp_(max=case["vocab"] - 1)
        z = lens[r] + 1
        end = torch.cumsum(z, 0) + at
        keep = int((end <= nbytes).sum())
        done = keep < want
        r, z, end = r[:keep], z[:keep], end[:keep]
        pos, n = end - z, z - 1
        up = torch.rand(keep, generator=gen, device=DEV) < 0.05
        s = torch.randint(0, len(_SEP), (keep,), generator=gen, device=DEV)
        for i in range(words.shape[1]):
            m = torch.nonzero(n > i)[:, 0]
            if not m.numel():
                break
            b = words[r[m], i]
            if i == 0:
                b = torch.where(up[m] & (b < 0x80), b - 32, b)
            out[pos[m] + i] = b
        out[end - 1] = sep[s]
        at = int(end[-1]) if keep else at
    return out


@functools.lru_cache(maxsize=64)
def _quantiles(n, sigma):
    normal = statistics.NormalDist()
    return np.exp(sigma * np.array([normal.inv_cdf((i + 0.5) / n) for i in range(n)]))


def _sizes(case, seed):
    """Lognormal document sizes: its quantiles (so that a case's total does not depend on the
    seed), clipped, in a random order."""
    n = case["docs"]
    if "median" in case:
        x = np.clip(_quantiles(n, 1.0) * case["median"], case["lo"], case["hi"]).astype(np.int64)
    else:
        x = _quantiles(n, 0.7)
        x = np.maximum(1, x * (case["bytes"] / x.sum())).astype(np.int64)
    return np.random.default_rng(seed).permutation(x)


def _ends(text, sizes):
    """int64 offsets [0, ..., len] near the given sizes, each right after a delimiter."""
    n = text.numel()
    t = torch.from_numpy(np.minimum(np.cumsum(sizes), n)).to(DEV)
    idx = (t[:, None] + torch.arange(48, device=DEV) - 1).clamp(0, n - 1)
    b = text[idx]
    delim = (b < 0x30) & (b != 0x27)
    first = torch.where(delim.any(1), delim.to(torch.int8).argmax(1), torch.zeros_like(t))
    ends = torch.cummax((t + first).clamp(max=n), 0).values
    ends[-1] = n
    return torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), ends])


def _at(text, shift):
    """The text at an address of `shift` mod 16."""
    if not shift:
        return text
    buf = torch.empty(text.numel() + 16, dtype=torch.uint8, device=DEV)
    buf[shift:shift + text.numel()] = text
    return buf[shift:shift + text.numel()]


def _corpus(case, seed):
    """(text, offsets) of a case with documents."""
    sizes = _sizes(case, seed + 2)
    text = _text(case, int(sizes.sum()) if "median" in case else case["bytes"], seed)
    return text, _ends(text, sizes)


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "count":
        if case["docs"] > 1:
            text, off = _corpus(case, seed)
        else:
            text = _text(case, case["bytes"], seed)
            off = torch.tensor([0, text.numel()], dtype=torch.int64, device=DEV)
        s["text"], s["offsets"], s["workspace"] = _at(text, case["shift"]), off, None
        if case["keep"]:
            plan = wc.count_plan(text.numel(), off.numel() - 1, count_bytes=case["count_bytes"],
                                 table_slots=case["slots"])
            s["workspace"] = torch.empty(plan.workspace_bytes, dtype=torch.uint8, device=DEV)
    elif kind in ("docs", "merge", "utf8"):
        s["text"], s["offsets"] = _corpus(case, seed)
        if kind == "merge":
            s["per"] = wc.count(s["text"], s["offsets"], per_doc=True, count_bytes=4)
        elif case.get("batch"):
            n = s["text"].numel()
            # a quarter more room than text of this kind fills, as a program plans it
            s["batch"] = wc.Batch(max_docs=case["docs"], max_bytes=n,
                                  **wc.output_sizes(s["text"], s["offsets"], count_bytes=4))
    elif kind == "topk":
        words = _vocabulary(case, seed)
        rng = np.random.default_rng(seed + 3)
        s["tables"] = []
        for c in range(case["corpora"]):
            # each corpus uses 200 words of the shared vocabulary five times as often
            f = np.ones(case["vocab"])
            f[rng.choice(case["vocab"], size=200, replace=False)] = 5.0
            text = _text(case, case["bytes"], seed + 10 * (c + 1), words,
                         _zipf(case["vocab"], case["zipf"], f))
            s["tables"].append(wc.count(text, count_bytes=4))
    elif kind == "serve":
        text, off = _corpus(case, seed)
        o = off.cpu().numpy()
        s["texts"] = [text[o[i]:o[i + 1]] for i in range(len(o) - 1)]
        s["server"], s["ids"] = wc.Server(mem_budget=GiB, max_streams=8), []
    else:
        text = _text(case, case["bytes"], seed)
        s["text"] = torch.empty(text.numel(), dtype=torch.uint8, pin_memory=True)
        s["text"].copy_(text)
        s["device"] = torch.empty_like(text)
    return s


# ------------------------------------------------------------------------------------------
# a pass
# ------------------------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "count":
        t = wc.count(s["text"], s["offsets"], count_bytes=case["count_bytes"],
                     table_slots=case["slots"], workspace=s["workspace"])
    elif kind == "docs" and case["batch"]:
        t = s["batch"].run(s["text"], s["offsets"])
    elif kind == "docs":
        t = wc.count(s["text"], s["offsets"], per_doc=True, count_bytes=case["count_bytes"])
    elif kind == "merge":
        t = wc.merge([s["per"]], count_bytes=8)
    elif kind == "utf8":
        t = wc.count(s["text"], s["offsets"], count_bytes=8, utf8=True)
    elif kind == "host":
        t = wc.count_host(s["text"], count_bytes=8, d_text=s["device"])
    elif kind == "topk":
        k = wc.topk_ratio(s["tables"], case["k"])
        return Read(("words", "n_c", "n_rest", "score", "vocab"), lambda: _topk_arrays(k, case))
    else:
        return _serve_pass(s)
    return Read(("counts", "words", "lengths", "tokens") + (("docs",) if t.docs() is not None else ()),
                lambda: _arrays(t, *_room(case)))


def _serve_pass(s):
    """Submit the burst and a merge query over it, wait for all; the tables stay with the server
    until the next burst."""
    srv = s["server"]
    for i in s["ids"]:
        srv.release(i)
    ids = [srv.submit(t, count_bytes=8) for t in s["texts"]]
    merged = srv.merge(ids)
    s["ids"] = ids + [merged]
    res = [srv.wait(i) for i in ids]
    total = srv.wait(merged)

    def read(held=s):  # the tables are in the server's memory
        out = {}
        for name, tabs in (("requests", res), ("merged", [total])):
            d = [sorted(wc.result_to_dict(r).items()) for r in tabs]
            room, cols = _room(held["case"], merged=name == "merged")
            words = np.array([w for t in d for w, _ in t], dtype="S%d" % (8 * cols))
            words = words.view(np.uint8).reshape(-1, 8 * cols)
            out[name + "_counts"] = _padded(np.array([c for t in d for _, c in t], np.int64), room)
            out[name + "_words"] = _padded(words, room)
            out[name + "_entries"] = np.array([len(t) for t in d], dtype=np.int64)
            out[name + "_tokens"] = np.array([r.total_tokens for r in tabs], dtype=np.int64)
        return out

    return Read(tuple(a + b for a in ("requests", "merged")
                      for b in ("_counts", "_words", "_entries", "_tokens")), read)


class Read(dict):
    """The outputs of a pass under their names, in canonical order once they are read."""

    def __init__(self, names, read):
        super().__init__(dict.fromkeys(names))
        self._read, self._got = read, None

    def __getitem__(self, name):
        if self._got is None:
            self._got = self._read()
        return self._got[name]


def _pack(words, off, col):
    """Bytes 8 col .. 8 col + 7 of every entry's word as one int64, zero padded, the first byte
    highest."""
    n, step = off.numel() - 1, 1 << 23
    out = torch.zeros(n, dtype=torch.int64, device=off.device)
    at = 8 * col + torch.arange(8, device=off.device)
    for a in range(0, n, step):
        o = off[a:min(a + step, n) + 1]
        i = (o[:-1, None] + at).clamp_(max=words.numel() - 1)
        v = torch.where(at < (o[1:] - o[:-1])[:, None], words[i], 0).to(torch.int64)
        out[a:a + step] = (v << (56 - 8 * (at & 7))).sum(1)
    return out


def _room(case, merged=False):
    """(rows, int64 values a word) that a case's tables are padded to: a text with a word table
    has at most the vocabulary's words; per-document tables have about the expected pairs."""
    cols = 5 if case.get("long") else 3 if case["kind"] == "utf8" else 2
    if case["kind"] == "docs" or (case["kind"] == "serve" and not merged):
        return int(1.5 * _pairs(case)) + 4096, cols
    return case["vocab"] + 64, cols


def _padded(x, rows):
    """x followed by zeros up to `rows` rows (as it is when it has more)."""
    if len(x) >= rows:
        return x
    if isinstance(x, np.ndarray):
        return np.concatenate([x, np.zeros((rows - len(x),) + x.shape[1:], x.dtype)])
    return torch.cat([x, x.new_zeros((rows - len(x),) + tuple(x.shape[1:]))])


def _arrays(t, rows, cols):
    """A device table in canonical order, padded to rows and columns."""
    n, words, off, counts = t.n_entries, t.words(), t.word_offsets(), t.counts()
    lens = off[1:] - off[:-1]
    cols = max(cols, (int(lens.max()) + 7) // 8) if n else cols
    key = [_pack(words, off, c) for c in range(cols)]
    perm = _order(key, t.docs())
    out = {"counts": _padded(counts[perm], rows), "lengths": _padded(lens[perm], rows),
           "words": [_padded(x[perm], rows) for x in key], "tokens": t.total_tokens}
    if t.docs() is not None:
        out["docs"] = _padded(t.docs()[perm], rows)
    return out


def _order(cols, docs=None):
    perm = None
    for col in list(reversed(cols)) + ([docs] if docs is not None else []):
        x = col if perm is None else col[perm]
        i = torch.sort(x, stable=True).indices
        perm = i if perm is None else perm[i]
    return perm


def _topk_arrays(k, case):
    rows = case["corpora"] * case["k"]
    words = np.array([w for c in k.words for w in c], dtype="S16").view(np.uint8).reshape(-1, 16)
    return {"words": _padded(words, rows), "n_c": _padded(np.concatenate(k.n_c), rows),
            "n_rest": _padded(np.concatenate(k.n_rest), rows),
            "score": _padded(np.concatenate(k.score), rows), "vocab": k.vocab_size}


# ------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------
@functools.lru_cache(maxsize=256)
def _distinct(vocab, zipf, tokens):
    """Expected distinct words among so many drawn tokens."""
    return float(-np.expm1(tokens * np.log1p(-np.minimum(_zipf(vocab, zipf), 1 - 1e-12))).sum())


def _expected(case, nbytes):
    """Expected distinct words of a text of so many bytes."""
    return _distinct(case["vocab"], case["zipf"], round(nbytes / ((case["max_len"] + 1) / 2 + 1)))


def _pairs(case):
    """Expected (document, word) pairs: documents of 64 sizes stand for all."""
    n = min(case["docs"], 4096)
    q = np.sort(_sizes(dict(case, docs=n), 1))
    q = q[np.linspace(0, n - 1, min(n, 64)).astype(int)] if n < 128 else q[n // 128::n // 64]
    return float(np.mean([_expected(case, float(x)) for x in q])) * case["docs"]


def work(case):
    """Each input byte read once, each output byte written once: text and offsets in; words,
    offsets and counts of the expected distinct words out."""
    kind = case["kind"]
    mean_word = (case["max_len"] + 1) / 2
    cb = case.get("count_bytes", 8)
    if kind in ("count", "utf8", "host"):
        e = _expected(case, case["bytes"])
        return {"bytes": case["bytes"] + 8 * case.get("docs", 1) + e * (mean_word + 8 + cb),
                "flops": 0}
    if kind == "topk":
        e = _expected(case, case["bytes"]) * case["corpora"]
        return {"bytes": e * (mean_word + 8 + 4) + case["corpora"] * case["k"] * (mean_word + 32),
                "flops": 0}
    text, per = float(_sizes(case, 1).sum()), _pairs(case)
    if kind == "docs":
        return {"bytes": text + 8 * case["docs"] + per * (mean_word + 8 + cb + 8)
                + 16 * case["docs"], "flops": 0}
    out = _expected(case, text) * (mean_word + 16)
    if kind == "merge":
        return {"bytes": per * (mean_word + 8 + 4) + out, "flops": 0}
    # serve: each request's table written, and read again by the merge
    return {"bytes": text + 2 * per * (mean_word + 16) + out, "flops": 0}


def tolerance(case):
    """Counts, lengths, documents and words are whole numbers and the same in every right answer;
    a score is three divisions of exactly held numbers in double precision, each correctly
    rounded, so it is the same too."""
    return "exact"


def exact(case, seed):
    """The scores of the distinctive words (the only computed floating numbers), from a count of
    the same texts in plain torch; None elsewhere."""
    if case["kind"] != "topk":
        return None
    words = _vocabulary(case, seed)
    rng = np.random.default_rng(seed + 3)
    keys, which = [], []
    for c in range(case["corpora"]):
        f = np.ones(case["vocab"])
        f[rng.choice(case["vocab"], size=200, replace=False)] = 5.0
        text = _text(case, case["bytes"], seed + 10 * (c + 1), words,
                     _zipf(case["vocab"], case["zipf"], f))
        low = torch.where((text >= 65) & (text <= 90), text + 32, text)
        word = ((low >= 97) & (low <= 122)) | ((low >= 48) & (low <= 57)) | (low == 39)
        pad = torch.zeros(1, dtype=torch.bool, device=DEV)
        start = torch.nonzero(word & ~torch.cat([pad, word[:-1]]))[:, 0]
        end = torch.nonzero(word & ~torch.cat([word[1:], pad]))[:, 0] + 1
        key = torch.zeros((start.numel(), 2), dtype=torch.int64, device=DEV)
        for j in range(case["max_len"]):
            b = torch.where(start + j < end, low[(start + j).clamp(max=low.numel() - 1)], 0)
            key[:, j // 8] |= b.to(torch.int64) << (56 - 8 * (j % 8))
        keys.append(key)
        which.append(torch.full((start.numel(),), c, dtype=torch.int64, device=DEV))
    key, which = torch.cat(keys), torch.cat(which)
    perm = _order([key[:, 0], key[:, 1]])
    key, which = key[perm], which[perm]
    new = torch.ones(key.shape[0], dtype=torch.bool, device=DEV)
    new[1:] = (key[1:] != key[:-1]).any(1)
    e = torch.cumsum(new, 0) - 1
    key, C = key[new].cpu().numpy(), case["corpora"]
    V = len(key)
    joint = torch.bincount(e * C + which, minlength=V * C).reshape(V, C).cpu().numpy()
    total, col = joint.sum(1), joint.sum(0)
    score = []
    for c in range(C):
        nc, nr = joint[:, c], total - joint[:, c]
        at = np.flatnonzero(nc >= 1)
        # enough of the best by the ratio in double precision to hold every tie with the last
        # row, then those in the exact order
        ratio = (nc[at] + 1.0) / (nr[at] + 1.0)
        cut = np.partition(ratio, -min(case["k"], len(at)))[-min(case["k"], len(at))]
        at = at[ratio >= cut * (1 - 1e-12)]
        best = sorted(at, key=functools.cmp_to_key(
            lambda a, b: _before(a, b, nc, nr, key)))[:case["k"]]
        a, b = nc[best].astype(np.float64), nr[best].astype(np.float64)
        score.append(((a + 1) / (col[c] + V)) / ((b + 1) / (col.sum() - col[c] + V)))
    return {"words": None, "n_c": None, "n_rest": None, "score": _padded(np.concatenate(score), C * case["k"]),
            "vocab": None}


def _before(a, b, nc, nr, key):
    """-1 when word a ranks before word b: the larger ratio, the larger count, the smaller word."""
    x, y = (int(nc[a]) + 1) * (int(nr[b]) + 1), (int(nc[b]) + 1) * (int(nr[a]) + 1)
    if x != y:
        return -1 if x > y else 1
    if nc[a] != nc[b]:
        return -1 if nc[a] > nc[b] else 1
    return -1 if tuple(key[a]) < tuple(key[b]) else 1

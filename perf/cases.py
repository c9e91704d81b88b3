"""Workloads of the KmerCo library, each one pass through its public entry points.

The sizes are those of the repository's own workloads (``synth/reads.py``,
``synth/serving.py``, ``bench.py``): from a read set of 1 Mbase to 2 Gbases
into a 2 GB countBF, plain, batched and served, plus the two lookups of a
finished countBF.  Reads are simulated on the GPU from the seed alone: a
uniform genome, reads at uniform positions of either strand, substitutions,
and 'N' calls.
"""
import math

import torch

import paper_2305_07545_amd as P
from paper_2305_07545_amd import kmerco

DEV = "cuda"


def _insert(reads, lo, hi, genome, err, k, tau, **more):
    """A plain insertion + classification of `reads` reads of lo..hi bases.  size: the countBF is
    dimensioned (Eq. 1) for this multiple of twice the expected distinct k-mers."""
    return dict(dict(kind="insert", reads=reads, lo=lo, hi=hi, genome=genome, err=err, n_rate=0.0, k=k, tau=tau,
                     alpha=8, k_h=1, size=1.0, two_calls=False), **more)


def listed():
    return [
        # the smallest call: 10,000 reads of a 100 kbp genome; latency and launches count
        _insert(10_000, 100, 100, 100_000, 0.01, 21, 2, name="tiny_k21"),
        # one ordinary read set of ragged reads (the median set of the 256-set workload)
        _insert(20_000, 50, 300, 175_000, 0.01, 25, 2, name="one_set_k25"),
        # a bacterial sequencing run, the size of the paper's own files (41-164 M k-mers)
        _insert(1_000_000, 150, 150, 5_000_000, 0.0055, 31, 3, name="bacterial_k31", n_rate=0.001),
        # the same reads at the paper's longer k-mer length: two-word keys
        _insert(1_000_000, 150, 150, 5_000_000, 0.0055, 55, 3, name="bacterial_k55", n_rate=0.001),
        # several hash functions and a counter length that is no power of two (the paper's sweeps),
        # inserted and classified by separate calls
        _insert(150_000, 100, 250, 1_000_000, 0.005, 28, 3, name="multi_hash", alpha=5, k_h=2, two_calls=True),
        # the bacterial run into a countBF sixteen times as large (fewest collisions): beyond the caches
        _insert(1_000_000, 150, 150, 5_000_000, 0.0055, 31, 3, name="roomy_k31", n_rate=0.001, size=16.0),
        # the largest: a quarter of the 8 Gbase workload, 2 Gbases into a 2 GB countBF
        _insert(8_000_000, 250, 250, 50_000_000, 0.003, 31, 5, name="large_k31", size=4.71),
        # many read sets of mixed sizes, each with its own countBF, one batched call
        dict(name="sets_mixed", kind="sets", sets=64, median=20_000, spread=1.0, err=0.01),
        # many small read sets in one call
        dict(name="sets_small", kind="sets", sets=256, median=1_500, spread=0.4, err=0.01),
        # sessions filled by requests from host memory, then classified
        dict(name="serving", kind="serving", sessions=3, requests=12, reads=60_000, lo=100, hi=250, genome=1_500_000,
             err=0.005, k=21, tau=3),
        # frequencies of a key list: stored k-mers and absent ones
        dict(name="query_20m", kind="query", keys=20_000_000, reads=600_000, genome=5_000_000, err=0.0055, k=31, alpha=8,
             k_h=1),
        # the distinct list of a finished countBF split at a threshold, as when a run is classified again
        dict(name="classify", kind="classify", reads=1_000_000, genome=5_000_000, err=0.0055, k=31, tau=4, alpha=8,
             k_h=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["insert"] * 11 + ["sets"] * 4 + ["query", "query", "classify"] + ["serving"] * 2)
    k = rng.choice([21, 25, 28, 31, 31, 55])
    if kind == "insert":
        lo = rng.randint(50, 250)
        hi = rng.choice([lo, rng.randint(lo, 300)])
        k_h = rng.choice([1, 1, 1, 1, 2, 3])
        bases = _log(rng, 500_000, 300_000_000 // k_h)
        genome, err = max(20_000, bases // rng.randint(10, 40)), rng.uniform(0.001, 0.02)
        # countBFs of up to the 2 GB of the largest listed case
        size = min(2.0 ** rng.uniform(-2, 4), 0.9e9 / _expected(genome, bases, err, k))
        return _insert(max(100, 2 * bases // (lo + hi)), lo, hi, genome, err, k, rng.randint(2, 5),
                       alpha=rng.choice([8, 8, 8, 8, 4, 5, 12, 16]), k_h=k_h, n_rate=rng.choice([0.0, 0.001]),
                       size=round(size, 2), two_calls=rng.random() < 0.25)
    if kind == "sets":
        sets = _log(rng, 8, 256)
        return dict(kind="sets", sets=sets, median=_log(rng, 1_000, min(20_000, 1_500_000 // sets)),
                    spread=round(rng.uniform(0.0, 1.0), 2), err=rng.uniform(0.001, 0.02))
    if kind == "serving":
        return dict(kind="serving", sessions=rng.randint(1, 4), requests=rng.randint(2, 14), reads=_log(rng, 5_000, 80_000),
                    lo=100, hi=rng.randint(100, 250), genome=_log(rng, 500_000, 2_000_000), err=0.005,
                    k=rng.choice([21, 31]), tau=rng.randint(2, 5))
    reads = _log(rng, 20_000, 1_000_000)
    c = dict(kind=kind, reads=reads, genome=max(20_000, reads * 5), err=rng.uniform(0.001, 0.02), k=k,
             alpha=rng.choice([8, 8, 5, 16]), k_h=rng.choice([1, 1, 2]))
    if kind == "query":
        c["keys"] = _log(rng, 1_000, 20_000_000)
    else:
        c["tau"] = rng.randint(2, 5)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _expected(genome, bases, err, k):
    """Expected distinct canonical k-mers: the genome's own and up to k novel ones per error."""
    return genome + bases * err * k


def _simulate(g, genome_len, lengths, err, n_rate=0.0):
    """Reads of the given lengths from a uniform genome; (uint8 ASCII, int64 offsets) on the GPU."""
    n = lengths.numel()
    offsets = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(lengths, 0, out=offsets[1:])
    total = int(offsets[-1])
    genome = torch.randint(0, 4, (genome_len,), generator=g, device=DEV, dtype=torch.uint8)
    span = genome_len - int(lengths.max()) + 1
    starts = (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * span).long()
    reverse = torch.rand(n, generator=g, device=DEV) < 0.5
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=DEV)
    reads = torch.empty(total, dtype=torch.uint8, device=DEV)
    step = max(1, 40_000_000 * n // max(total, 1))
    for a in range(0, n, step):  # some 40 M bases at a time
        b = min(n, a + step)
        p0, p1 = int(offsets[a]), int(offsets[b])
        at = torch.repeat_interleave(torch.arange(a, b, device=DEV), lengths[a:b])
        i = torch.arange(p0, p1, device=DEV) - offsets[at]
        rev = reverse[at]
        codes = genome[starts[at] + torch.where(rev, lengths[at] - 1 - i, i)]
        codes = torch.where(rev, 3 - codes, codes)
        wrong = torch.rand(p1 - p0, generator=g, device=DEV) < err
        other = torch.randint(1, 4, (p1 - p0,), generator=g, device=DEV, dtype=torch.uint8)
        codes = torch.where(wrong, (codes + other) & 3, codes)
        out = letters[codes.long()]
        if n_rate:
            out[torch.rand(p1 - p0, generator=g, device=DEV) < n_rate] = ord("N")
        reads[p0:p1] = out
    return reads, offsets


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _sizes():
    """Sizes (read lengths, reads of a set) are the case's own, whatever the seed of the reads' content."""
    return _generator(2305)


def _lengths(sizes, n, lo, hi):
    return torch.randint(lo, hi + 1, (n,), generator=sizes, device=DEV, dtype=torch.int64)


def _zeros(n):
    return torch.zeros(max(1, int(n)), dtype=torch.int64, device=DEV)


def _filled(case, g):
    """A countBF holding a read set and its distinct list (the state of the lookups)."""
    lengths = _lengths(_sizes(), case["reads"], 150, 150)
    reads, offsets = _simulate(g, case["genome"], lengths, case["err"])
    k, bases = case["k"], reads.numel()
    items = 2.0 * _expected(case["genome"], bases, case["err"], k)
    bf = P.CountBF(*P.dims(items), case["alpha"], case["k_h"])
    distinct = bf.insert(reads, offsets, k, distinct=_zeros(min(bases, 0.6 * items) * kmerco.key_words(k)))
    bf.sync()
    return bf, distinct


def _prepare_insert(case, g):
    lengths = _lengths(_sizes(), case["reads"], case["lo"], case["hi"])
    reads, offsets = _simulate(g, case["genome"], lengths, case["err"], case["n_rate"])
    k, bases = case["k"], reads.numel()
    expected = _expected(case["genome"], bases, case["err"] + case["n_rate"], k)
    bf = P.CountBF(*P.dims(2.0 * expected * case["size"]), case["alpha"], case["k_h"])
    bf.reserve(bases)
    room = int(min(bases, 1.2 * expected + 1000)) * kmerco.key_words(k)
    counts = _zeros(4)
    return dict(case=case, reads=reads, offsets=offsets, bf=bf, counts=counts,
                n_distinct=counts[0:1], n_windows=counts[1:2], n_trust=counts[2:3], n_err=counts[3:4],
                distinct=_zeros(room), trust=_zeros(room), err=_zeros(room))


def _run_insert(s):
    c, bf = s["case"], s["bf"]
    bf.reset()
    s["counts"].zero_()
    if c["two_calls"]:
        bf.insert(s["reads"], s["offsets"], c["k"], distinct=s["distinct"], n_distinct=s["n_distinct"],
                  n_windows=s["n_windows"])
        bf.classify(s["distinct"], s["n_distinct"], c["tau"], trust=s["trust"], err=s["err"], n_trust=s["n_trust"],
                    n_err=s["n_err"])
    else:
        bf.insert_classify(s["reads"], s["offsets"], c["k"], c["tau"], distinct=s["distinct"], trust=s["trust"],
                           err=s["err"], n_distinct=s["n_distinct"], n_windows=s["n_windows"], n_trust=s["n_trust"],
                           n_err=s["n_err"])
    return {n: s[n] for n in ("counts", "distinct", "trust", "err")} | {"words": bf.words}


def _prepare_sets(case, g):
    n_sets, sizes = case["sets"], _sizes()
    z = torch.randn(n_sets, generator=sizes, device=DEV)
    reads_of = (case["median"] * torch.exp(case["spread"] * z)).long().clamp(1_000, 100_000).tolist()
    picks = torch.randint(0, 3, (n_sets,), generator=sizes, device=DEV).tolist()
    parts, offs, sets, pos = [], [_zeros(1)], [], 0
    for n, pick in zip(reads_of, picks):
        lengths = _lengths(sizes, n, 50, 300)
        bases = int(lengths.sum())
        pad = -pos % kmerco.SET_ALIGN
        if pad:  # every set starts at a multiple of SET_ALIGN, the gap is a read of 'N'
            parts.append(torch.full((pad,), ord("N"), dtype=torch.uint8, device=DEV))
            pos += pad
            offs.append(torch.tensor([pos], device=DEV))
        genome = max(2_000, bases // 20)
        reads, o = _simulate(g, genome, lengths, case["err"])
        parts.append(reads)
        offs.append(o[1:] + pos)
        k = (21, 25, 31)[pick]
        expected = _expected(genome, bases, case["err"], k)
        X, Y = P.dims(2.0 * expected)
        sets.append(dict(first_base=pos, n_bases=bases, k=k, X=X, Y=Y, room=int(min(bases, 1.2 * expected + 1000))))
        pos += bases
    words = torch.empty(sum(q["X"] * q["Y"] for q in sets), dtype=torch.int64, device=DEV)
    lists = {n: _zeros(sum(q["room"] for q in sets)) for n in ("distinct", "trust", "err")}
    counts = _zeros(4 * n_sets)
    entries, w, r = [], 0, 0
    for i, q in enumerate(sets):
        f = P.CountBF(q["X"], q["Y"], words=words[w:w + q["X"] * q["Y"]])
        w += q["X"] * q["Y"]
        e = dict(filter=f, first_base=q["first_base"], n_bases=q["n_bases"], k=q["k"], tau=2)
        for n in lists:
            e[n] = lists[n][r:r + q["room"]]
        r += q["room"]
        for j, n in enumerate(("n_distinct", "n_windows", "n_trust", "n_err")):
            e[n] = counts[4 * i + j:4 * i + j + 1]
        entries.append(e)
    return dict(case=case, batch=P.Batch(), entries=entries, reads=torch.cat(parts), offsets=torch.cat(offs),
                counts=counts, words=words, stream=torch.cuda.Stream(), **lists)


def _run_sets(s):
    s["batch"].insert(s["entries"], s["reads"], s["offsets"], reset=True, graph=True, stream=s["stream"])
    return {n: s[n] for n in ("counts", "distinct", "trust", "err", "words")}


def _prepare_serving(case, g):
    k, n_sessions, n = case["k"], case["sessions"], case["requests"]
    requests, bases_of, sizes = [], [0] * n_sessions, _sizes()
    for i, z in enumerate(torch.randn(n, generator=sizes, device=DEV).tolist()):
        lengths = _lengths(sizes, max(1000, int(case["reads"] * math.exp(0.5 * z))), case["lo"], case["hi"])
        reads, offsets = _simulate(g, case["genome"], lengths, case["err"])
        bases_of[i % n_sessions] += reads.numel()
        requests.append((reads.cpu().pin_memory(), offsets.cpu().pin_memory()))
    sessions = []
    for bases in bases_of:
        # every request of a session has a genome of its own size
        expected = _expected(case["genome"] * -(-n // n_sessions), bases, case["err"], k)
        sessions.append(dict(dims=P.dims(2.0 * expected), room=int(min(max(bases, 1000), 1.2 * expected + 1000))))
    lists = [(_zeros(q["room"]), _zeros(q["room"])) for q in sessions]
    server = P.Server(memory_budget=16 << 30, lane_bases=2 * max(r.numel() for r, _ in requests) + (1 << 20),
                      lane_reads=2 * max(o.numel() for _, o in requests) + 1024)
    return dict(case=case, server=server, requests=requests, sessions=sessions, lists=lists)


def _run_serving(s):
    c, server = s["case"], s["server"]
    ids = [server.open(*q["dims"], c["k"], q["room"]) for q in s["sessions"]]
    tickets = [server.submit(ids[i % len(ids)], reads=r, offsets=o) for i, (r, o) in enumerate(s["requests"])]
    tickets += [server.submit(sid, classify=True, insert=False, tau=c["tau"], trust=t, err=e)
                for sid, (t, e) in zip(ids, s["lists"])]
    server.wait()
    results = [server.result(t) for t in tickets]
    for t in tickets:
        server.release(t)
    for sid in ids:
        server.close(sid)
    counts = [[int(r[n]) for n in ("status", "n_windows", "distinct_first", "n_new", "n_trust", "n_err")] for r in results]
    return dict(counts=torch.tensor(counts), trust=[t for t, _ in s["lists"]], err=[e for _, e in s["lists"]])


def _prepare_lookup(case, g):
    bf, distinct = _filled(case, g)
    w = kmerco.key_words(case["k"])
    s = dict(case=case, bf=bf, distinct=distinct)
    if case["kind"] == "classify":
        n = distinct.numel()
        return dict(s, trust=_zeros(n), err=_zeros(n), n_trust=_zeros(1), n_err=_zeros(1))
    # three stored keys to one absent key, in random order
    n = case["keys"]
    stored = distinct.view(-1, w)[:int(bf.n_distinct)]
    keys = stored[(torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * stored.shape[0]).long()]
    absent = torch.rand(n, generator=g, device=DEV) < 0.25
    bits = 2 * case["k"]
    top = min(bits, 62)
    random = torch.randint(0, 1 << top, (n, w), generator=g, device=DEV)
    if w == 2:
        random[:, 1] &= (1 << (bits - 64)) - 1
    keys = torch.where(absent[:, None], random, keys).reshape(-1).contiguous()
    return dict(s, keys=keys, freq=torch.empty(n, dtype=torch.int32, device=DEV))


def _run_query(s):
    return s["bf"].query(s["keys"], freq=s["freq"])


def _run_classify(s):
    s["bf"].classify(s["distinct"], s["bf"].n_distinct, s["case"]["tau"], trust=s["trust"], err=s["err"],
                     n_trust=s["n_trust"], n_err=s["n_err"])
    return {n: s[n] for n in ("trust", "err", "n_trust", "n_err")}


_PREPARE = {"insert": _prepare_insert, "sets": _prepare_sets, "serving": _prepare_serving, "query": _prepare_lookup,
            "classify": _prepare_lookup}
_RUN = {"insert": _run_insert, "sets": _run_sets, "serving": _run_serving, "query": _run_query,
        "classify": _run_classify}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _generator(seed))


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---------------------------------------------------------------------------
# what a pass cannot do without: every input read once, every output written
# once; operations are the 32-bit integer ones of hashing each k-mer (117 at
# one hash function, 74 for each further one, 181 + 102 for two-word keys)
# ---------------------------------------------------------------------------

def _insert_work(bases, reads, genome, err, k, items, k_h=1):
    windows = max(0, bases - reads * (k - 1))
    distinct = min(windows, genome * (1 - math.exp(-bases / genome)) + 0.7 * bases * err * k)
    X, Y = P.dims(items)
    key = 8 * kmerco.key_words(k)
    ops = 117 + 74 * (k_h - 1) if k <= 32 else 181 + 102 * (k_h - 1)
    return {"bytes": bases + 8 * reads + 8 * X * Y + 2 * key * distinct, "flops": ops * windows}


def work(case):
    c = case
    if c["kind"] == "insert":
        bases = c["reads"] * (c["lo"] + c["hi"]) // 2
        items = 2 * c["size"] * _expected(c["genome"], bases, c["err"] + c["n_rate"], c["k"])
        return _insert_work(bases, c["reads"], c["genome"], c["err"], c["k"], items, c["k_h"])
    if c["kind"] == "sets":
        reads = max(1_000, int(c["median"] * math.exp(c["spread"] ** 2 / 2)))
        w = _insert_work(175 * reads, reads, max(2_000, 175 * reads // 20), c["err"], 25,
                         2 * _expected(175 * reads // 20, 175 * reads, c["err"], 25))
        return {n: c["sets"] * v for n, v in w.items()}
    if c["kind"] == "serving":
        bases = c["reads"] * (c["lo"] + c["hi"]) // 2
        w = _insert_work(bases, c["reads"], c["genome"], c["err"], c["k"],
                         2 * _expected(c["genome"], bases, c["err"], c["k"]))
        return {n: c["requests"] * v for n, v in w.items()}
    key = 8 * kmerco.key_words(c["k"])
    bases = 150 * c["reads"]
    distinct = c["genome"] * (1 - math.exp(-bases / c["genome"])) + 0.7 * bases * c["err"] * c["k"]
    n = c["keys"] if c["kind"] == "query" else distinct
    return {"bytes": n * (key + 8 * c["k_h"] + (4 if c["kind"] == "query" else key)), "flops": 74 * n * c["k_h"]}


# ---------------------------------------------------------------------------
# the same results from the definitions, in 64-bit torch arithmetic
# ---------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _rotl(x, r):
    return ((x << r) | (x >> (32 - r))) & _M32


def _murmur(words, seed):
    """MurmurHash3_x86_32 of keys given as 32-bit words, first word first."""
    h = torch.full_like(words[0], seed)
    for w in words:
        w = (_rotl((w * 0xCC9E2D51) & _M32, 15) * 0x1B873593) & _M32
        h = (_rotl(h ^ w, 13) * 5 + 0xE6546B64) & _M32
    h = h ^ (4 * len(words))
    h = ((h ^ (h >> 16)) * 0x85EBCA6B) & _M32
    h = ((h ^ (h >> 13)) * 0xC2B2AE35) & _M32
    return h ^ (h >> 16)


def _halves(keys):
    """32-bit words of keys given as a list of 64-bit words, low first."""
    return [v for k in keys for v in (k & _M32, (k >> 32) & _M32)]


def _mod(hi, lo, d):
    return (hi * ((1 << 32) % d) + lo) % d


def _slots(keys, X, Y, alpha, k_h):
    eta = 64 // alpha
    w = _halves(keys)
    for a in range(k_h):
        hi, lo = _murmur(w, 2 * a), _murmur(w, 2 * a + 1)
        yield (_mod(hi, lo, X) * Y + _mod(hi, lo, Y)) * eta + _mod(hi, lo, eta)


def _strand(codes, k, p, reverse):
    """The k-base keys starting at p as 64-bit words, low first."""
    words = [torch.zeros_like(p) for _ in range(kmerco.key_words(k))]
    for i in range(k):
        c = codes[p + i] if not reverse else 3 - codes[p + k - 1 - i]
        if len(words) == 2:
            words[1] = (words[1] << 2) | ((words[0] >> 62) & 3)
        words[0] = (words[0] << 2) | c
    return words


def exact(case, seed):
    if case["kind"] != "insert" or case["reads"] * case["hi"] > 60_000_000:
        return None
    s = _prepare_insert(case, _generator(seed))
    k, alpha, k_h = case["k"], case["alpha"], case["k_h"]
    X, Y = int(s["bf"].layout.X), int(s["bf"].layout.Y)
    reads, offsets = s["reads"], s["offsets"]
    table = torch.full((256,), 4, dtype=torch.int64, device=DEV)
    table[torch.tensor(list(b"ACGT"), device=DEV)] = torch.arange(4, device=DEV)
    codes = table[reads.long()]
    bad = torch.zeros(reads.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum((codes == 4).long(), 0, out=bad[1:])
    owner = torch.repeat_interleave(torch.arange(offsets.numel() - 1, device=DEV), offsets[1:] - offsets[:-1])
    p = torch.arange(reads.numel(), device=DEV)
    p = p[p + k <= offsets[owner + 1]]
    p = p[bad[p + k] == bad[p]]
    fwd, rev = _strand(codes, k, p, False), _strand(codes, k, p, True)
    hf, hr = _murmur(_halves(fwd), 0), _murmur(_halves(rev), 0)
    lf, lr = _murmur(_halves(fwd), 1), _murmur(_halves(rev), 1)
    take = (hf < hr) | ((hf == hr) & (lf < lr))
    keys = [torch.where(take, f, r) for f, r in zip(fwd, rev)]
    eta, top = 64 // alpha, (1 << alpha) - 1
    count = torch.zeros(X * Y * eta, dtype=torch.int64, device=DEV)
    first = torch.full((X * Y * eta,), 1 << 62, dtype=torch.int64, device=DEV)
    slots = list(_slots(keys, X, Y, alpha, k_h))
    for at in slots:
        count.index_add_(0, at, torch.ones_like(at))
        first.scatter_reduce_(0, at, p, "amin")
    new = torch.zeros_like(p, dtype=torch.bool)
    freq = torch.full_like(p, top)
    for at in slots:
        new |= first[at] == p
        freq = torch.minimum(freq, count[at])
    count = count.clamp(max=top).view(X * Y, eta)
    words = torch.zeros(X * Y, dtype=torch.int64, device=DEV)
    for i in range(eta):
        words |= count[:, i] << (alpha * i)
    keys, above = torch.stack(keys, 1)[new], (freq > case["tau"])[new]

    def laid_out(name, rows):
        out = torch.zeros_like(s[name])
        out[:rows.numel()] = rows.reshape(-1)
        return out

    n = [keys.shape[0], p.numel(), int(above.sum()), int((~above).sum())]
    return dict(counts=torch.tensor(n, device=DEV), distinct=laid_out("distinct", keys),
                trust=laid_out("trust", keys[above]), err=laid_out("err", keys[~above]), words=words)

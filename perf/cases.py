"""Performance cases: the work that users of this framework have it do, through
its public entry points.

A case is a dict of plain values. Two kinds of reference sets are used, shaped
as this repository's generators make them: clusters of ten mutated copies of a
random root genome (``set = "clusters"``), and identical copies of one genome
(``set = "copies"``, redundant strain collections). Read records are sampled
from the set with substitutions, from a random strand, 5% of them foreign:
``reads`` is ``"short"`` (one length), ``"uneven"`` (half single-end of 50 to
250 bp, half pairs 2 x 150 bp of one fragment, one paired-layout offsets array)
or ``"long"`` (lengths log-uniform between len_lo and len_hi).

Inputs are made on the GPU from the seed alone (torch generators).
"""
import math

import numpy as np
import torch

import paper_2106_08150_amd as mc

K, WINDOW, SKETCH = 16, 128, 16
STRIDE = WINDOW - K + 1
REUSE_BYTES = 64 << 30      # blocks kept by a process that rebuilds databases

_ACGT = (65, 67, 71, 84)


def listed():
    return [
        # --- query: bucket table ------------------------------------------
        # one interactive request: a few hundred reads, answered at once
        # (launches and host time count, not the kernels)
        dict(name="query_few", op="classify", set="clusters", genomes=50, total_bp=200_000_000,
             reads="short", records=200, len_lo=150, len_hi=150, top=False, shape=512),
        # the small reference set of the tests: 8 genomes of 100 kbp, 10,000
        # reads of 100 bp, with the top-hit lists
        dict(name="query_small_set", op="classify", set="clusters", genomes=8, total_bp=800_000,
             reads="short", records=10_000, len_lo=100, len_hi=100, top=True, shape=512),
        # the benchmark's classification: 10M reads of 150 bp against 1,000
        # genomes / 4 Gbp, in the launch shape the benchmark uses
        dict(name="query_scale", op="classify", set="clusters", genomes=1000,
             total_bp=4_000_000_000, reads="short", records=10_000_000, len_lo=150, len_hi=150,
             top=False, shape=256),
        # an uneven batch (mixed single-end and paired records), top hits kept
        dict(name="query_uneven", op="classify", set="clusters", genomes=250,
             total_bp=1_000_000_000, reads="uneven", records=2_000_001, len_lo=50, len_hi=250,
             top=True, shape=512),
        # long reads (kilobases, as the tests' 1,000 to 5,000 bp records and
        # longer): candidate lists of hundreds to thousands of locations
        dict(name="query_long", op="classify", set="clusters", genomes=250,
             total_bp=1_000_000_000, reads="long", records=20_000, len_lo=800, len_hi=10_000,
             top=True, shape=512),
        # reads of a redundant collection: hundreds of identical genomes, so
        # every feature is at the per-feature location cap
        dict(name="query_redundant", op="classify", set="copies", genomes=300,
             total_bp=300 * 20_000, reads="uneven", records=4_000, len_lo=50, len_hi=250,
             top=True, shape=512),
        # --- query: other forms --------------------------------------------
        # the query-only form of a database: condensed layout, table released
        dict(name="query_condensed", op="condensed", set="clusters", genomes=500,
             total_bp=2_000_000_000, reads="short", records=2_000_000, len_lo=150, len_hi=150,
             top=False, shape=512),
        # a captured classification of a small fixed-size batch, replayed
        dict(name="query_graph", op="graph", set="clusters", genomes=50, total_bp=200_000_000,
             reads="uneven", records=3_001, len_lo=50, len_hi=250, top=True, shape=512),
        # a burst of host batches through the served loop (sizes log-uniform),
        # from submission to the labels in host memory
        dict(name="served_burst", op="served", set="clusters", genomes=250,
             total_bp=1_000_000_000, reads="long", records=400_000, len_lo=100, len_hi=250,
             top=False, shape=512, batches=12),
        # --- build ----------------------------------------------------------
        # the benchmark's build: 4 Gbp of genomes already in device memory,
        # into a fresh database, then a first batch of reads
        dict(name="build_scale", op="build", set="clusters", genomes=1000,
             total_bp=4_000_000_000, reads="short", records=20_000, len_lo=150, len_hi=150,
             top=True, shape=512),
        # a small collection of ragged contigs from host memory, added in two
        # calls (the second one is an on-demand addition to a live database)
        dict(name="build_contigs", op="build_host", set="clusters", genomes=400,
             total_bp=20_000_000, reads="short", records=20_000, len_lo=150, len_hi=150,
             top=True, shape=512),
        # conversion of a built table to the condensed query layout, then a
        # first batch of reads
        dict(name="condense", op="condense", set="clusters", genomes=250,
             total_bp=1_000_000_000, reads="short", records=20_000, len_lo=150, len_hi=150,
             top=True, shape=512),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges. Sizes are odd as they fall."""
    op = rng.choice(["classify", "classify", "classify", "condensed", "graph", "noalloc", "served",
                     "build", "build_host", "condense"])
    c = dict(op=op, set="clusters", reads="short", top=rng.random() < 0.5,
             shape=rng.choice([256, 512]), len_lo=150, len_hi=150)
    if op == "build":
        c["total_bp"] = _log_uniform(rng, 5_000_000, 4_000_000_000)
    elif op == "build_host":
        c["total_bp"] = _log_uniform(rng, 500_000, 80_000_000)
    else:
        c["total_bp"] = _log_uniform(rng, 2_000_000, 1_000_000_000)
    # genomes of 40 kbp to 4 Mbp (contigs on the host path), at least 2
    size = _log_uniform(rng, 5_000, 200_000) if op == "build_host" else _log_uniform(rng, 40_000,
                                                                                    4_000_000)
    c["genomes"] = max(2, min(2_000, c["total_bp"] // size))
    if op in ("build", "build_host", "condense"):
        c["len_lo"] = c["len_hi"] = rng.randint(80, 260)
        c["records"] = _log_uniform(rng, 100, 20_000)
        return c
    kind = rng.choice(["short", "uneven", "long", "copies"])
    if kind == "copies" and op in ("classify", "condensed"):
        c.update(set="copies", genomes=rng.randint(20, 300), reads=rng.choice(["short", "uneven"]),
                 records=_log_uniform(rng, 50, 4_000))
        c["total_bp"] = c["genomes"] * rng.randint(8_000, 40_000)
        if c["reads"] == "short":
            c["len_lo"] = c["len_hi"] = rng.randint(80, 260)
        else:
            c.update(len_lo=50, len_hi=250)
        return c
    c["reads"] = "short" if kind == "copies" else kind
    if c["reads"] == "long" and op in ("classify", "condensed"):
        c.update(len_lo=rng.randint(300, 1_000), len_hi=rng.randint(1_500, 12_000),
                 records=_log_uniform(rng, 50, 16_000))
        return c
    if c["reads"] == "long":
        c["reads"] = "short"
    if c["reads"] == "short":
        c["len_lo"] = c["len_hi"] = rng.randint(60, 300)
    else:
        c.update(len_lo=50, len_hi=250)
    c["records"] = {"classify": lambda: _log_uniform(rng, 50, 4_000_000),
                    "condensed": lambda: _log_uniform(rng, 1_000, 2_000_000),
                    "graph": lambda: _log_uniform(rng, 50, 30_000),
                    "noalloc": lambda: _log_uniform(rng, 50, 300_000),
                    "served": lambda: _log_uniform(rng, 20_000, 400_000)}[op]()
    if op == "served":
        c["top"] = False
        c["batches"] = rng.randint(2, 16)
    return c


# ------------------------------------------------------------------ inputs --
def _letters(dev):
    return torch.tensor(_ACGT, dtype=torch.uint8, device=dev)


def _complement(dev):
    t = torch.arange(256, dtype=torch.uint8, device=dev)
    for a, b in ((65, 84), (84, 65), (67, 71), (71, 67)):
        t[a] = b
    return t


def _substitute(codes, rate, gen):
    """2-bit codes with each one replaced by another one at `rate`."""
    hit = torch.rand(codes.shape, device=codes.device, generator=gen) < rate
    step = torch.randint(1, 4, codes.shape, dtype=torch.uint8, device=codes.device, generator=gen)
    return (codes + step * hit) & 3


def _genomes(case, seed):
    """Reference text (device), lengths, taxa and parents of the set."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    rng = np.random.default_rng(seed)
    n, total = int(case["genomes"]), int(case["total_bp"])
    lut = _letters(dev)
    if case["set"] == "copies":
        L = total // n
        root = torch.randint(0, 4, (L,), dtype=torch.uint8, device=dev, generator=gen)
        text = lut[root.long()].repeat(n)
        return (text, np.full(n, L, np.uint64), np.arange(1, n + 1, dtype=np.uint32),
                np.zeros(n + 1, np.uint32))
    lens = np.clip(rng.lognormal(0.0, 0.4, n), 0.25, 2.5)
    lens = np.maximum((lens * (total / lens.sum())).astype(np.int64), 300)
    text = torch.empty(int(lens.sum()), dtype=torch.uint8, device=dev)
    per, at = 10, 0
    for c0 in range(0, n, per):
        members = lens[c0:c0 + per]
        root = torch.randint(0, 4, (int(members.max()),), dtype=torch.uint8, device=dev,
                             generator=gen)
        for L in members:
            d = float(rng.uniform(0.02, 0.15))
            text[at:at + int(L)] = lut[_substitute(root[:int(L)], d, gen).int()]
            at += int(L)
    # some genomes hold a run of unknown bases
    ends = np.cumsum(lens)
    for g in np.nonzero(rng.random(n) < 0.05)[0]:
        run = int(rng.integers(20, 200))
        s = int(ends[g] - lens[g] + rng.integers(0, lens[g] - run))
        text[s:s + run] = ord("N")
    # taxonomy: root, one node per cluster, one leaf per genome
    clusters = (n + per - 1) // per
    parents = np.zeros(1 + clusters + n, np.uint32)
    parents[1 + clusters:] = 1 + np.arange(n) // per
    taxa = (1 + clusters + np.arange(n)).astype(np.uint32)
    return text, lens.astype(np.uint64), taxa, parents


def _records(case, text, lengths, seed):
    """Read bytes and offsets (device) sampled from the set."""
    dev = text.device
    gen = torch.Generator(device=dev).manual_seed(seed * 7 + 1)
    rng = np.random.default_rng(seed * 7 + 2)
    n, lo, hi = int(case["records"]), int(case["len_lo"]), int(case["len_hi"])
    g_len = lengths.astype(np.int64)
    g_off = np.concatenate([[0], np.cumsum(g_len)[:-1]])
    gi = rng.integers(0, g_len.size, n)
    rev = rng.random(n) < 0.5
    if case["reads"] == "uneven":
        pair = rng.random(n) < 0.5
        span = np.where(pair, np.clip(rng.normal(400, 50, n), 150, 700).astype(np.int64),
                        rng.integers(lo, hi + 1, n))
        span = np.minimum(span, g_len[gi])
        start = g_off[gi] + (rng.random(n) * (g_len[gi] - span + 1)).astype(np.int64)
        m1 = np.where(pair, np.minimum(150, span), span)
        m2 = np.where(pair, np.minimum(150, span), 0)
        mates = np.empty((n, 2, 2), np.int64)       # start, length of each mate
        mates[:, 0, 0] = np.where(pair & rev, start + span - m1, start)
        mates[:, 1, 0] = np.where(rev, start, start + span - m2)
        mates[:, 0, 1], mates[:, 1, 1] = m1, m2
        mrev = np.stack([rev, ~rev], 1).reshape(-1)
        mstart, mlen = mates[:, :, 0].reshape(-1), mates[:, :, 1].reshape(-1)
    else:
        if case["reads"] == "long":
            mlen = np.exp(rng.uniform(math.log(lo), math.log(hi + 1), n)).astype(np.int64)
        else:
            mlen = np.full(n, lo, np.int64)
        mlen = np.minimum(mlen, g_len[gi])
        mstart = g_off[gi] + (rng.random(n) * (g_len[gi] - mlen + 1)).astype(np.int64)
        mrev = rev
    foreign = rng.random(n) < 0.05
    if case["reads"] == "uneven":
        foreign = np.repeat(foreign, 2)
    off = np.zeros(mlen.size + 1, np.int64)
    np.cumsum(mlen, out=off[1:])
    out = torch.empty(int(off[-1]), dtype=torch.uint8, device=dev)
    d_off = torch.from_numpy(off).to(dev)
    lut, comp = _letters(dev), _complement(dev)
    block = max(1, int(60_000_000 / max(1.0, float(mlen.mean()))))
    for a in range(0, mlen.size, block):
        b = min(mlen.size, a + block)
        L = torch.from_numpy(mlen[a:b]).to(dev)
        base, size = int(off[a]), int(off[b] - off[a])
        if size == 0:
            continue
        row = torch.repeat_interleave(torch.arange(b - a, device=dev), L, output_size=size)
        pos = torch.arange(size, device=dev) - (d_off[a:b] - base)[row]
        r = torch.from_numpy(mrev[a:b]).to(dev)[row]
        src = torch.from_numpy(mstart[a:b]).to(dev)[row] + torch.where(r, L[row] - 1 - pos, pos)
        t = text[src]
        t = torch.where(r, comp[t.int()], t)
        # substitutions (1%), a rare unknown base, and foreign records
        u = torch.rand(size, device=dev, generator=gen)
        rnd = lut[torch.randint(0, 4, (size,), dtype=torch.int32, device=dev, generator=gen)]
        f = torch.from_numpy(foreign[a:b]).to(dev)[row]
        t = torch.where(f | (u < 0.0133), rnd, t)
        out[base:base + size] = torch.where(u > 0.99995, torch.full_like(t, ord("N")), t)
    return out, d_off


def _database(case, text, lengths, taxa, parents):
    db = mc.Database(K, WINDOW, SKETCH, 254)
    db.add_targets(text, lengths, taxa)
    db.set_taxonomy(parents)
    mc.mc_db_set_launch_config(db.h, int(case["shape"]), 4, 16384)
    return db


def _opts(case):
    """Query options: the defaults; records with pairs give their insert size."""
    uneven = case["reads"] == "uneven"
    return dict(top_m=4, min_hits=4, hit_diff=0, insert_size=400 if uneven else 0, paired=uneven)


def prepare(case, seed):
    op = case["op"]
    text, lengths, taxa, parents = _genomes(case, seed)
    reads, off = _records(case, text, lengths, seed)
    st = dict(op=op, reads=reads, off=off, n=int(case["records"]), top=bool(case["top"]),
              opts=_opts(case))
    if op in ("build", "build_host"):
        mc.mc_set_cached_memory_limit(REUSE_BYTES)
        half = lengths.size // 2
        cut = int(lengths[:half].sum())
        st.update(text=text, lengths=lengths, taxa=taxa, parents=parents, half=half, cut=cut)
        if op == "build_host":
            st["text"] = text.cpu().numpy()
        return st
    db = _database(case, text, lengths, taxa, parents)
    del text
    if op == "condensed":
        db.condense(release_table=True)
    elif op in ("graph", "noalloc"):
        n, top_m = st["n"], st["opts"]["top_m"]
        st["labels"] = torch.empty(n, dtype=torch.int32, device="cuda")
        st["tops"] = (torch.empty((n, top_m, 3), dtype=torch.int32, device="cuda")
                      if st["top"] else None)
        o = st["opts"]
        st["q"] = mc.QueryOpts(o["top_m"], o["min_hits"], o["hit_diff"], o["insert_size"],
                               int(o["paired"]))
        if op == "graph":
            st["graph"] = mc.ClassifyGraph(db.h, reads, off, n, st["q"], st["labels"], st["tops"])
    elif op == "served":
        # host batches with log-uniform sizes (the same for every seed), every
        # other one in pinned memory
        rng = np.random.default_rng(st["n"] + int(case["batches"]))
        per = 2 if st["opts"]["paired"] else 1
        w = np.exp(rng.uniform(0.0, math.log(100.0), int(case["batches"])))
        cuts = np.concatenate([[0], np.round(np.cumsum(w) / w.sum() * st["n"])]).astype(np.int64)
        h_reads, h_off = reads.cpu(), off.cpu().numpy()
        batches = []
        for i, (a, b) in enumerate(zip(cuts[:-1], cuts[1:])):
            if b == a:
                continue
            o = h_off[per * a:per * b + 1]
            t = h_reads[int(o[0]):int(o[-1])].clone()
            batches.append((t.pin_memory() if i % 2 else t.numpy(),
                            (o - o[0]).astype(np.uint64)))
        st["batches"] = batches
        st["srv"] = mc.Server(db, slots=4)
        del st["reads"], st["off"]
    st["db"] = db
    return st


def _classify(db, st):
    labels, top = db.classify(st["reads"], st["off"], st["n"], with_top=st["top"], **st["opts"])
    return [labels, top] if st["top"] else [labels]


def run(st):
    op = st["op"]
    if op in ("classify", "condensed"):
        return _classify(st["db"], st)
    if op == "graph":
        st["graph"].launch()
        return [st["labels"], st["tops"]]
    if op == "noalloc":
        mc.mc_classify_noalloc(st["db"].h, st["reads"], st["off"], st["n"], st["q"], st["labels"],
                               st["tops"])
        return [st["labels"], st["tops"]]
    if op == "served":
        o = st["opts"]
        tickets = [st["srv"].submit(t, off, **o) for t, off in st["batches"]]
        return [st["srv"].wait(t)[0] for t in tickets]
    if op == "condense":
        st["db"].condense()
        return _classify(st["db"], st)
    # a fresh database: one addition of device text, or two of host text
    db = mc.Database(K, WINDOW, SKETCH, 254)
    if op == "build":
        db.add_targets(st["text"], st["lengths"], st["taxa"])
    else:
        h, c = st["half"], st["cut"]
        db.add_targets(st["text"][:c], st["lengths"][:h], st["taxa"][:h])
        db.add_targets(st["text"][c:], st["lengths"][h:], st["taxa"][h:])
    db.set_taxonomy(st["parents"])
    return _classify(db, st)


def exact(case, seed):
    """Every output is a whole number (taxon ids, target ids, scores, windows)
    and has to stay equal: there is nothing that rounds."""
    return None


# -------------------------------------------------------------------- work --
def _mean_len(case):
    lo, hi = case["len_lo"], case["len_hi"]
    if case["reads"] == "short" or lo == hi:
        return float(lo)
    return (hi - lo) / math.log(hi / lo)


def work(case):
    """Bytes one pass cannot do without: the reads, their offsets and results
    once, and per sketch element looked up one 64-byte piece of the index; a
    build reads the text once and writes its table once (a sketch element is an
    8-byte entry, the table is half full), a conversion reads that table once
    and writes the layout of about the same size."""
    n = int(case["records"])
    if case["reads"] == "uneven":
        mates, bases, windows = 2 * n, n * (0.5 * 300 + 0.5 * 150), n * (0.5 * 4 + 0.5 * 1.7)
    else:
        m = _mean_len(case)
        mates, bases, windows = n, n * m, n * max(1.0, math.ceil((m - K + 1) / STRIDE))
    out = 4 * n + (48 * n if case["top"] else 0)
    query = bases + 8 * (mates + 1) + out + windows * SKETCH * 64
    table = case["total_bp"] / STRIDE * SKETCH * 8 * 2
    if case["op"] in ("build", "build_host"):
        return {"bytes": query + case["total_bp"] + table, "flops": 0}
    if case["op"] == "condense":
        return {"bytes": query + 2 * table, "flops": 0}
    return {"bytes": query, "flops": 0}

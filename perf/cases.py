"""The calls a read mapper makes of this library, at the sizes it makes them.

A case names one step of the filter's path (or the whole of it), a synthetic
reference and a read set. The references follow the repository's workloads:
1 Mbp, 100 Mbp with 1.5% repeats, and 3.1 Gbp with 45% repeats (64 families of
300 bp and 64 of 6 kbp at 5-25% divergence); reads are 100, 150 or 250 bp, or
the 30/40/30 mix of the three, with 2-5% edits in the proportion 8:1:1. All
random numbers come from the seed, on the GPU.

Fields of a case:
  kind      scan | candidates | verify | seeds | sweep | pipeline
  genome    reference length; bin, overlap, q: the index
  reads     number of reads; length: their length (0: the mix)
  edits     one explicit budget E for every read (0: each read's own error rate)
  counts    scan: bytes of the per-bin counts asked for (0: pass masks only)
  summary   scan: the masks' per-read pass counts and digests are taken too
  cap       candidate bins kept per read
  bounded   verify: distances above E_r reported as E_r + 1
  non_acgt  reads and reference hold runs and single bytes that are no base
"""

from __future__ import annotations

import math

import torch

from paper_1708_04329_amd import grim

HUMAN = 3_100_000_000
LENGTHS, SHARES, RATES = (100, 150, 250), (30, 40, 30), (20, 30, 40, 50)  # read mix; error rates per mille
SEED_K = 12

_BASE = dict(genome=HUMAN, bin=2048, overlap=263, q=5, reads=1, length=0, edits=0, counts=0, summary=False, cap=0,
             bounded=False, non_acgt=False)


def _case(kind, name="", **kw):
    c = dict(_BASE, kind=kind, **kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the plain small batch: 2000 reads against one bacterial-size reference, counts wanted beside the masks
        _case("scan", "scan_1Mbp_2000x100_counts", genome=1_000_000, overlap=105, reads=2000, length=100, edits=5,
              counts=1),
        # a light request of the serving stream (sizes are log-uniform in 1..20000): latency
        _case("scan", "scan_human_17_mixed", reads=17, summary=True),
        # a request of about the stream's mean size
        _case("scan", "scan_human_1201_mixed", reads=1201, summary=True, non_acgt=True),
        # the human-scale batch: every bin of 3.1 Gbp, 150 bp reads with E = 7
        _case("scan", "scan_human_49999x150", reads=49_999, length=150, edits=7),
        # a handful of reads with their seed-hit lists: a mapper's interactive call
        _case("candidates", "cand_100Mbp_67x100", genome=100_000_000, overlap=105, reads=67, length=100, edits=5,
              cap=256),
        # short lists, cache-resident index: the 100 Mbp candidate batch
        _case("candidates", "cand_100Mbp_1000003x100", genome=100_000_000, overlap=105, reads=1_000_003, length=100,
              edits=5, cap=256),
        # long lists over an index larger than the caches, uneven reads
        _case("candidates", "cand_human_q6_40001_mixed", q=6, reads=40_001, cap=1024),
        # alignment of the pairs that passed, as a mapper asks for it: only up to each read's budget
        _case("verify", "verify_bounded_human_100003", q=6, reads=100_003, cap=1024, bounded=True),
        # exact distances of every passing pair (false-negative study, no bound)
        _case("verify", "verify_exact_100Mbp_20011", genome=100_000_000, overlap=105, reads=20_011, length=100,
              edits=5, cap=256),
        # seed lookup and ranking: the step that makes the candidate lists
        _case("seeds", "seeds_human_20011_mixed", reads=20_011, cap=1024),
        # one point of the read-existence study: index build, all-bins scan, pass counts
        _case("sweep", "sweep_human_158bp_2000x100", bin=158, overlap=105, reads=2000, length=100),
        # one point of the false-negative study: seed table, index, lists, filter, verification of every candidate
        _case("pipeline", "pipeline_100Mbp_2000x100", genome=100_000_000, overlap=105, reads=2000, length=100,
              edits=5, cap=2048, bounded=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "scan", "candidates", "candidates", "verify", "verify", "seeds", "sweep",
                       "pipeline"])
    length = rng.choice([0, 0, 100, 150, 250])
    kw = dict(length=length, overlap=105 if length == 100 else 263, non_acgt=rng.random() < 0.3)
    if length:
        kw["edits"] = rng.choice([0, length // 20])
    big = HUMAN if rng.random() < 0.4 else _log_int(rng, 1_000_000, HUMAN)
    if kind == "scan":
        q = rng.choice([4, 5, 5, 5, 6])
        B = rng.choice([2048, 2048, 2048, 474, 237, 158])
        bins = -(-big // B)
        # at most the largest listed case's additions, and 8 GB of masks
        most = 49_999 * 146 * -(-HUMAN // 2048) / (bins * (length or 250))
        n = _log_int(rng, 1, max(1, min(60_000, most, 6.4e10 / bins)))
        counts = rng.choice([0, 0, 0, 1, 2]) if n * bins < 4e8 and length in (100, 150, 250) else 0
        return _case(kind, genome=big, bin=B, q=q, reads=n, counts=counts, summary=rng.random() < 0.3, **kw)
    if kind == "sweep":
        G = _log_int(rng, 1_000_000, HUMAN)
        kw.update(length=100, overlap=105, edits=0)
        return _case(kind, genome=G, bin=rng.choice([474, 237, 158]), q=rng.choice([4, 5, 6]),
                     reads=_log_int(rng, 50, 2000), **kw)
    if kind == "pipeline":
        G = _log_int(rng, 1_000_000, 100_000_000)
        return _case(kind, genome=G, q=rng.choice([5, 6]), bin=rng.choice([2048, 474]),
                     reads=_log_int(rng, 50, 2000), cap=rng.choice([256, 2048]), bounded=rng.random() < 0.7, **kw)
    if kind == "seeds":
        return _case(kind, genome=big, bin=rng.choice([2048, 2048, 474]), reads=_log_int(rng, 10, 20_000),
                     cap=rng.choice([256, 1024, 2048]), **kw)
    if rng.random() < 0.5:
        G, q, cap, most = HUMAN, 6, 1024, 40_000 if kind == "candidates" else 100_000
    else:
        G, q, cap, most = _log_int(rng, 10_000_000, 100_000_000), 5, 256, 1_000_000 if kind == "candidates" else 20_000
    return _case(kind, genome=G, q=q, reads=_log_int(rng, 20, most), cap=cap,
                 bounded=kind == "verify" and rng.random() < 0.6, **kw)


# ---------------------------------------------------------------------------
# Inputs, made on the GPU from the seed.
# ---------------------------------------------------------------------------
_PER_PAIR = (("count", torch.int16), ("pass", torch.uint8), ("dist", torch.int16), ("match", torch.uint8))
_SLOT = 6000  # the reference is made in slots: uniform bases, a long repeat copy, or short repeat copies


def _rand(gen, *shape):
    return torch.rand(*shape, generator=gen, device="cuda")


def _randint(gen, lo, hi, shape, dtype=torch.int64):
    return torch.randint(lo, hi, shape, generator=gen, device="cuda", dtype=dtype)


def _ascii(codes):
    lut = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device="cuda")  # A C G T
    return lut.index_select(0, codes.reshape(-1).int()).reshape(codes.shape)


def _codes(ascii_):
    return ((ascii_ >> 1) ^ (ascii_ >> 2)) & 3


def _diverge(codes, rate, gen):
    """Substitutions at the given per-row rates."""
    other = (codes + _randint(gen, 1, 4, codes.shape, torch.uint8)) & 3
    return torch.where(_rand(gen, *codes.shape) < rate, other, codes)


def _reference(case, gen):
    G = case["genome"]
    repeats = 0.45 if G > 1_000_000_000 else (0.015 if G > 10_000_000 else 0.0)
    ref = torch.empty(G, dtype=torch.uint8, device="cuda")
    long_fam = _randint(gen, 0, 4, (64, _SLOT), torch.uint8)
    short_fam = _randint(gen, 0, 4, (64, 300), torch.uint8)
    step = 16384 * _SLOT
    for lo in range(0, G, step):
        n = min(step, G - lo)
        slots = -(-n // _SLOT)
        base = _randint(gen, 0, 4, (slots, _SLOT), torch.uint8)
        u = _rand(gen, slots)
        rows = (u < repeats / 2).nonzero().flatten()
        if len(rows):
            fam = long_fam[_randint(gen, 0, 64, (len(rows),))]
            base[rows] = _diverge(fam, 0.05 + 0.2 * _rand(gen, len(rows), 1), gen)
        rows = ((u >= repeats / 2) & (u < repeats)).nonzero().flatten()
        if len(rows):
            per = _SLOT // 300
            fam = short_fam[_randint(gen, 0, 64, (len(rows) * per,))]
            base[rows] = _diverge(fam, 0.05 + 0.2 * _rand(gen, len(rows) * per, 1), gen).reshape(-1, _SLOT)
        text = _ascii(base)
        if case["non_acgt"]:
            text[_rand(gen, slots) < 0.002] = 78  # assembly gaps: N runs
        ref[lo:lo + n] = text.reshape(-1)[:n]
    return ref


def _read_set(case, ref, gen):
    """(bases, offsets, max_edits or None, err_permille or None)."""
    n, G = case["reads"], case["genome"]
    if case["length"]:
        lens = torch.full((n,), case["length"], dtype=torch.int64, device="cuda")
    else:
        w = torch.tensor(SHARES, dtype=torch.float32, device="cuda")
        kind = torch.multinomial(w, n, replacement=True, generator=gen)
        lens = torch.tensor(LENGTHS, dtype=torch.int64, device="cuda")[kind]
    rate = torch.tensor(RATES, dtype=torch.int64, device="cuda")[_randint(gen, 0, len(RATES), (n,))]
    if case["edits"]:
        edits = torch.full((n,), case["edits"], dtype=torch.int64, device="cuda")
    else:
        edits = lens * rate // 1000
    offsets = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = lens.cumsum(0)
    Lm = int(lens.max())
    Em = max(1, int(edits.max()))
    parts = []
    for lo in range(0, n, 1 << 17):
        ln, ed = lens[lo:lo + (1 << 17), None], edits[lo:lo + (1 << 17), None]
        m = len(ln)
        at = torch.arange(Lm, device="cuda")[None, :]
        live = at < ln
        key = torch.where(live, _rand(gen, m, Lm), 2.0)
        spots = key.topk(Em, dim=1, largest=False).indices
        edit = torch.zeros(m, Lm, dtype=torch.bool, device="cuda")
        edit.scatter_(1, spots, torch.arange(Em, device="cuda")[None, :] < ed)
        u = _rand(gen, m, Lm)
        ins, dele = edit & (u < 0.1), edit & (u >= 0.1) & (u < 0.2)
        pos = (_rand(gen, m, 1).double() * (G - Lm - Em - 2)).long()
        src = pos + (1 + dele.long() - ins.long()).cumsum(1) - 1
        codes = _codes(ref[src.clamp_(0, G - 1)])
        codes = torch.where(edit & (u >= 0.2), (codes + _randint(gen, 1, 4, (m, Lm), torch.uint8)) & 3, codes)
        codes = torch.where(ins, _randint(gen, 0, 4, (m, Lm), torch.uint8), codes)
        text = _ascii(codes)
        if case["non_acgt"]:
            text = torch.where(_rand(gen, m, Lm) < 0.001, 78, text)  # uncalled bases
        parts.append(text[live])
    bases = torch.cat(parts)
    if case["edits"]:
        return bases, offsets, edits.to(torch.int16).view(torch.uint16), None
    return bases, offsets, None, rate.to(torch.int16).view(torch.uint16)


def _zeros(n, dtype):
    return torch.zeros(max(1, n), dtype=dtype, device="cuda")


def _lists(case, ref, reads):
    """Seed-hit candidate lists (cand_off, cand_bin) from the library's own seeding."""
    co, cb = _zeros(case["reads"] + 1, torch.int64), _zeros(case["reads"] * case["cap"], torch.int32)
    seeds = grim.grim_seeds_build(ref, SEED_K)
    total = grim.grim_seed_candidates(seeds, reads, case["bin"], case["cap"], co, cb)
    seeds.free()
    return co, cb[:max(1, total)].clone()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ref = _reference(case, gen)
    reads = grim.ReadSet(*_read_set(case, ref, gen))
    s = {"case": case, "reads": reads}
    kind, B, O, q, n = case["kind"], case["bin"], case["overlap"], case["q"], case["reads"]
    # outputs of one list entry each have room for the longest lists, as the lists' own buffer has
    room = n * case["cap"]
    if kind == "scan":
        s["index"] = grim.grim_build_index(ref, B, O, q, grim.LAYOUT_TM)
        info = s["index"].info()
        s["mask"] = torch.empty((n, info["mask_words"]), dtype=torch.int32, device="cuda")
        if case["counts"]:
            s["counts"] = torch.empty((n, info["n_bins"]), device="cuda",
                                      dtype=torch.uint8 if case["counts"] == 1 else torch.int16)
    elif kind == "candidates":
        s["off"], s["bin"] = _lists(case, ref, reads)
        s["index"] = grim.grim_build_index(ref, B, O, q, grim.LAYOUT_BM)
        s["count"], s["pass"] = _zeros(room, torch.int16), _zeros(room, torch.uint8)
    elif kind == "verify":
        s["off"], s["bin"] = _lists(case, ref, reads)
        s["index"] = grim.grim_build_index(ref, B, O, q, grim.LAYOUT_BM | grim.LAYOUT_REF)
        s["pass"] = _zeros(room, torch.uint8)
        grim.grim_filter_candidates(s["index"], reads, s["off"], s["bin"], None, s["pass"])
        s["dist"], s["match"] = _zeros(room, torch.int16), _zeros(room, torch.uint8)
    elif kind == "seeds":
        s["seeds"] = grim.grim_seeds_build(ref, SEED_K)
        s["off"], s["bin"] = _zeros(n + 1, torch.int64), _zeros(room, torch.int32)
    else:  # sweep, pipeline: the reference itself is what the call starts from
        s["ref"] = ref
    if kind == "pipeline":
        s["off"], s["bin"] = _zeros(n + 1, torch.int64), _zeros(room, torch.int32)
        for name, dtype in _PER_PAIR:
            s[name] = _zeros(room, dtype)
    if kind in ("scan", "sweep"):
        s["passed"], s["digest"] = _zeros(n, torch.int32), _zeros(n, torch.int64)
    return s


# ---------------------------------------------------------------------------
# One pass.
# ---------------------------------------------------------------------------
def _run_sweep(s):
    """One point of sweep.existence_study: build, scan, pass counts."""
    c = s["case"]
    idx = grim.grim_build_index(s["ref"], c["bin"], c["overlap"], c["q"], grim.LAYOUT_TM)
    mask = torch.empty((c["reads"], idx.info()["mask_words"]), dtype=torch.int32, device="cuda")
    grim.grim_filter_scan(idx, s["reads"], mask.view(torch.uint32))
    grim.grim_mask_summary(mask.view(torch.uint32), pass_count=s["passed"].view(torch.uint32))
    idx.free()
    return {"mask": mask, "passed": s["passed"]}


def _run_pipeline(s):
    """One point of sweep.fn_study: seed table, index, lists, filter, verification of every candidate."""
    c = s["case"]
    seeds = grim.grim_seeds_build(s["ref"], SEED_K)
    idx = grim.grim_build_index(s["ref"], c["bin"], c["overlap"], c["q"], grim.LAYOUT_BM | grim.LAYOUT_REF)
    P = grim.grim_seed_candidates(seeds, s["reads"], c["bin"], c["cap"], s["off"], s["bin"])
    if P:
        bins = s["bin"][:P]
        grim.grim_filter_candidates(idx, s["reads"], s["off"], bins, s["count"].view(torch.uint16), s["pass"])
        verify = grim.grim_verify_candidates_bounded if c["bounded"] else grim.grim_verify_candidates
        verify(idx, s["reads"], s["off"], bins, None, s["dist"].view(torch.uint16), s["match"])
    idx.free()
    seeds.free()
    return {name: s[name] for name in ("off", "bin") + tuple(name for name, _ in _PER_PAIR)}


def run(s):
    c, kind = s["case"], s["case"]["kind"]
    if kind == "scan":
        mask, counts = s["mask"].view(torch.uint32), s.get("counts")
        if c["counts"] == 2:
            counts = counts.view(torch.uint16)
        grim.grim_filter_scan(s["index"], s["reads"], mask, counts)
        out = {"mask": s["mask"]}
        if c["counts"]:
            out["counts"] = s["counts"]
        if c["summary"]:
            grim.grim_mask_summary(mask, s["passed"].view(torch.uint32), s["digest"].view(torch.uint64))
            out.update(passed=s["passed"], digest=s["digest"])
        return out
    if kind == "candidates":
        grim.grim_filter_candidates(s["index"], s["reads"], s["off"], s["bin"], s["count"].view(torch.uint16),
                                    s["pass"])
        return {"count": s["count"], "pass": s["pass"]}
    if kind == "verify":
        verify = grim.grim_verify_candidates_bounded if c["bounded"] else grim.grim_verify_candidates
        verify(s["index"], s["reads"], s["off"], s["bin"], s["pass"], s["dist"].view(torch.uint16), s["match"])
        return {"dist": s["dist"], "match": s["match"]}
    if kind == "seeds":
        grim.grim_seed_candidates(s["seeds"], s["reads"], c["bin"], c["cap"], s["off"], s["bin"])
        return {"off": s["off"], "bin": s["bin"]}
    return _run_sweep(s) if kind == "sweep" else _run_pipeline(s)


# ---------------------------------------------------------------------------
# What one pass cannot do without.
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: each input read once and each output written once. Flops: one addition per token of a read and
    bin it is checked against. List lengths are the expected ones."""
    G, n, q, B = case["genome"], case["reads"], case["q"], case["bin"]
    L = case["length"] or sum(l * s for l, s in zip(LENGTHS, SHARES)) / 100
    bins, tokens = -(-G // B), L - q + 1
    reads = n * (L + 10)
    bits = bins * 4 ** q / 8
    hits = math.floor(L / SEED_K) * G / 4 ** SEED_K
    pairs = n * max(1.0, min(case["cap"], hits)) if case["cap"] else 0
    mask = n * bins / 8
    kind = case["kind"]
    if kind == "scan":
        return {"bytes": bits + reads + mask + n * bins * case["counts"] + (12 * n if case["summary"] else 0),
                "flops": n * bins * tokens}
    if kind == "sweep":
        return {"bytes": G + bits + reads + mask + 4 * n, "flops": n * bins * tokens}
    if kind == "candidates":
        return {"bytes": min(bits, pairs * 4 ** q / 8) + reads + 8 * n + 7 * pairs, "flops": pairs * tokens}
    if kind == "verify":
        return {"bytes": min(G, pairs * B) + reads + 8 * n + 8 * pairs, "flops": 0}
    if kind == "seeds":
        return {"bytes": reads + 8 * n + 4 * n * hits + 4 * pairs, "flops": 0}
    return {"bytes": G + bits + reads + 8 * n + 10 * pairs, "flops": pairs * tokens}


# ---------------------------------------------------------------------------
# The same outputs from plain torch, for the sizes where that is quick. Every
# output is a whole number.
# ---------------------------------------------------------------------------
def _tokens(text, q):
    """Code of the q bases at every position and whether they are all bases."""
    codes = _codes(text).long()
    base = (text == 65) | (text == 67) | (text == 71) | (text == 84)
    m = len(text) - q + 1
    code = torch.zeros(m, dtype=torch.int64, device=text.device)
    ok = torch.ones(m, dtype=torch.bool, device=text.device)
    for i in range(q):
        code = code * 4 + codes[i:i + m]
        ok &= base[i:i + m]
    return code, ok


def _bits(ref, case):
    B, O, q, G = case["bin"], case["overlap"], case["q"], case["genome"]
    code, ok = _tokens(ref, q)
    at = ok.nonzero().flatten()
    code = code[at]
    bits = torch.zeros(-(-G // B), 4 ** q, dtype=torch.bool, device=ref.device)
    for back in range(-(-O // B) + 1):
        x = at // B - back
        live = (x >= 0) & (at - x * B < B + O)
        bits[x[live], code[live]] = True
    return bits


def _histograms(case, reads):
    """Token counts [n, 4^q] in 64 bits and thresholds [n]."""
    q, off = case["q"], reads.offsets
    lens = off[1:] - off[:-1]
    code, ok = _tokens(reads.bases, q)
    at = torch.arange(len(code), device=code.device)
    r = torch.searchsorted(off, at, right=True) - 1
    live = ok & (at + q <= off[r + 1])
    h = torch.zeros(len(lens), 4 ** q, dtype=torch.float64, device=code.device)
    h.index_put_((r[live], code[live]), torch.ones((), dtype=torch.float64, device=code.device), accumulate=True)
    if reads.max_edits is not None:
        E = reads.max_edits.view(torch.int16).long()
    else:
        E = (lens * reads.err_permille.view(torch.int16).long() + 999) // 1000
    return h, lens - q + 1 - q * E, E


def _exact_scan(case, ref, reads):
    bits = _bits(ref, case)
    h, T, _ = _histograms(case, reads)
    cnt = (h @ bits.T.double()).long()
    nb = bits.shape[0]
    ok = torch.zeros(len(T), -(-nb // 32) * 32, dtype=torch.int64, device=ref.device)
    ok[:, :nb] = cnt >= T[:, None]
    word = (ok.reshape(len(T), -1, 32) << torch.arange(32, device=ref.device)).sum(2)
    return cnt, torch.where(word >= 1 << 31, word - (1 << 32), word).to(torch.int32), ok.sum(1)


def _exact_pairs(case, ref, reads, off, bins):
    bits = _bits(ref, case)
    h, T, _ = _histograms(case, reads)
    r = torch.repeat_interleave(torch.arange(len(T), device=ref.device), off[1:] - off[:-1])
    cnt = torch.cat([(h[r[i:i + 65536]] * bits[bins[i:i + 65536].long()]).sum(1).long()
                     for i in range(0, len(r), 65536)])
    return cnt, cnt >= T[r]


def _exact_distances(case, ref, reads, off, bins, mask):
    """Smallest edit distance of each masked pair's read to any part of its bin, column by column."""
    B, O, q, G = case["bin"], case["overlap"], case["q"], case["genome"]
    lens = reads.offsets[1:] - reads.offsets[:-1]
    _, _, E = _histograms(case, reads)
    pair_r = torch.repeat_interleave(torch.arange(len(lens), device=ref.device), off[1:] - off[:-1])
    dist = torch.full((len(bins),), 0xFFFF, dtype=torch.int64, device=ref.device)
    todo = mask.nonzero().flatten()
    Lm = int(lens.max())
    row = torch.arange(Lm + 1, device=ref.device)[None, :]
    for i in range(0, len(todo), 1 << 17):
        p = todo[i:i + (1 << 17)]
        r, x = pair_r[p], bins[p].long()
        at = (reads.offsets[r][:, None] + row[:, :Lm]).clamp_(max=len(reads.bases) - 1)
        text = reads.bases[at]
        lo = x * B
        hi = torch.minimum(lo + B + O + q - 1, torch.full_like(lo, G))
        col = row.repeat(len(p), 1)
        best = col.gather(1, lens[r][:, None])[:, 0]
        for j in range(int((hi - lo).max())):
            t = ref[(lo + j).clamp_(max=G - 1)]
            sub = ((text != t[:, None]) | (t == 78)[:, None]).long()
            nxt = torch.cat([torch.zeros_like(col[:, :1]), torch.minimum(col[:, :-1] + sub, col[:, 1:] + 1)], 1)
            nxt = (nxt - row).cummin(1).values + row
            col = torch.where((lo + j < hi)[:, None], nxt, col)
            best = torch.minimum(best, col.gather(1, lens[r][:, None])[:, 0])
        dist[p] = torch.minimum(best, E[r] + 1) if case["bounded"] else best
    return dist, (dist <= E[pair_r]) & mask.bool()


def _exact_lists(case, ref, reads):
    n, B, cap, dev = case["reads"], case["bin"], case["cap"], ref.device
    nb = case["genome"] // B + 1
    code, ok = _tokens(ref, SEED_K)
    at = ok.nonzero().flatten()
    key, order = code[at].sort()
    pos = at[order]
    rcode, rok = _tokens(reads.bases, SEED_K)
    lens = reads.offsets[1:] - reads.offsets[:-1]
    r = torch.repeat_interleave(torch.arange(n, device=dev), lens // SEED_K)
    o = torch.cat([torch.arange(int(k), device=dev) for k in lens // SEED_K]) * SEED_K
    s = reads.offsets[r] + o
    r, o, s = r[rok[s]], o[rok[s]], s[rok[s]]
    lo, hi = torch.searchsorted(key, rcode[s]), torch.searchsorted(key, rcode[s], right=True)
    rep = torch.repeat_interleave(torch.arange(len(s), device=dev), hi - lo)
    first = (hi - lo).cumsum(0) - (hi - lo)
    hit = lo[rep] + torch.arange(len(rep), device=dev) - first[rep]
    bins = (pos[hit] - o[rep]).clamp_(min=0) // B
    cell, votes = torch.unique(r[rep] * nb + bins, return_counts=True)
    rank = torch.argsort((cell // nb) * (1 << 20) - votes, stable=True)  # by read, votes (more first), bin
    read = (cell // nb)[rank]
    start = torch.searchsorted(read, torch.arange(n + 1, device=dev))
    keep = rank[torch.arange(len(rank), device=dev) - start[read] < cap].sort().values
    off = torch.searchsorted(cell[keep] // nb, torch.arange(n + 1, device=dev))
    return off, (cell[keep] % nb).int()


def exact(case, seed):
    G, n, kind = case["genome"], case["reads"], case["kind"]
    bins = -(-G // case["bin"])
    L = case["length"] or 250
    if G > 200_000_000 or bins * 4 ** case["q"] > 1 << 31 or (kind in ("scan", "sweep") and n * bins > 1 << 30):
        return None
    w = n * max(1, min(case["cap"] or 1, L // SEED_K * (G >> (2 * SEED_K)) + 16))  # pairs listed, about
    if w > 4_000_000 or (kind in ("verify", "pipeline") and w * L * (case["bin"] + case["overlap"]) > 1 << 37):
        return None
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    ref = _reference(case, gen)
    reads = grim.ReadSet(*_read_set(case, ref, gen))
    if kind in ("scan", "sweep"):
        cnt, mask, passed = _exact_scan(case, ref, reads)
        out = {"mask": mask}
        if case["counts"]:
            out["counts"] = cnt
        if case["summary"] or kind == "sweep":
            out["passed"] = passed
        if case["summary"]:
            out["digest"] = None
        return out
    off, lists = _exact_lists(case, ref, reads)
    out = {"off": off, "bin": lists}
    if kind != "seeds":
        out["count"], out["pass"] = _exact_pairs(case, ref, reads, off, lists)
    if kind in ("verify", "pipeline"):
        every = torch.ones_like(out["pass"]) if kind == "pipeline" else out["pass"]
        dist, out["match"] = _exact_distances(case, ref, reads, off, lists, every)
        out["dist"] = torch.where(dist > 0x7FFF, dist - 0x10000, dist)  # outputs are read as int16
    room = n * case["cap"]
    given = {"seeds": ("off", "bin"), "candidates": ("count", "pass"), "verify": ("dist", "match")}
    return {name: v if name == "off" else torch.cat([v, v.new_zeros(max(1, room) - len(v))])
            for name, v in out.items() if name in given.get(kind, out)}

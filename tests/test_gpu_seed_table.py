"""The seed table's build by partitions: seed lengths on both sides of every
change of its partition bits (codes that are partitions themselves up to k = 6,
low bits left above, more partition bits from k = 13), references of one tile
(32768 positions), its edges and several, skewed ones, byte-wise ones; and the
counter build that takes over without memory for the partitions. The candidate
lists do not depend on the order within a bucket: equal to the oracle's."""

from __future__ import annotations

import random

import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu


def lists(ref_dev, rd, k, B, cap):
    import torch
    seeds = grim.grim_seeds_build(ref_dev, k)
    info = seeds.info()
    co = empty((rd.n + 1,), torch.int64)
    cb = empty((max(1, rd.n * cap),), torch.int32)
    P = grim.grim_seed_candidates(seeds, grim.ReadSet(dev(rd.bases), dev(rd.offsets)), B, cap, co, cb)
    return host(co), host(cb)[:P], info


@pytest.mark.parametrize("counters", [False, True])
@pytest.mark.parametrize("k,G", [(1, 3000), (2, 32768), (5, 65540), (6, 32769), (6, 131073), (7, 70001), (8, 65535), (11, 200003),
                                 (12, 32768 + 11), (12, 600011), (13, 140000), (14, 131072 + 13), (14, 14)])
def test_table_matches_oracle(oracle, monkeypatch, k, G, counters):
    if counters:
        monkeypatch.setenv("GRIM_SEED_BUILD_COUNTERS", "1")
    rng = random.Random(100 * k + G)
    ref = bytearray(rng.choices(b"ACGTacgt", weights=[6, 2, 2, 3, .1, .1, .1, .1], k=G))
    if G > 2000:
        for p, n, b in ((G // 3, 700, b"A"), (G // 2, 300, b"N"), (G - 60, 60, b"T"), (64, 1, b"N")):
            ref[p:p + n] = b * len(ref[p:p + n])
        unit = bytes(ref[1000:1200])
        for _ in range(40):
            p = rng.randrange(0, G - 200)
            ref[p:p + 200] = unit
    ref = np.frombuffer(bytes(ref), np.uint8).copy()
    n = 6 if k < 4 else 60
    seqs = []
    for _ in range(n):
        L = min(rng.choice([k, 30, 100, 151]), G)
        p = rng.randrange(0, G - L + 1)
        s = bytearray(ref[p:p + L].tobytes())
        if L > 20:
            s[rng.randrange(L)] = rng.choice(b"ACGTN")
        seqs.append(bytes(s))
    rd = synth.reads_from_strings(seqs)
    want_o, want_b = oracle.seed_candidates(ref, rd.bases, rd.offsets, k, 500, 64)
    want_n = 0
    ok = np.isin(ref, np.frombuffer(b"ACGTacgt", np.uint8))
    run = np.convolve(ok, np.ones(k, np.int64), "valid") if G >= k else np.zeros(0)
    want_n = int((run == k).sum())
    got_o, got_b, info = lists(dev(ref), rd, k, 500, 64)
    assert info["n_positions"] == want_n
    assert np.array_equal(got_o, want_o) and np.array_equal(got_b, want_b)
    # the same bytes at an odd address (no 16-byte loads), and from the host
    odd = dev(np.concatenate([np.zeros(1, np.uint8), ref]))[1:]
    for other in (odd, ref):
        got_o, got_b, info = lists(other, rd, k, 500, 64)
        assert info["n_positions"] == want_n
        assert np.array_equal(got_o, want_o) and np.array_equal(got_b, want_b)

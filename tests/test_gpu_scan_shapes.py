"""The all-bins scan at the edges of its launch shapes: read counts around a
wavefront's group, around the chunk counts that change the workgroup order and
around the one-workgroup length order; indexes of one tile, of a few, and of
more than one round over the XCDs. Bit-exact against the CPU oracle."""

from __future__ import annotations

import random

import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host, unpack_mask
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu


def mixed_reads(rng, ref, n, lens, with_n=True):
    seqs = []
    for _ in range(n):
        L = rng.choice(lens)
        p = rng.randrange(0, len(ref) - L)
        s = bytearray(ref[p:p + L].tobytes())
        for _ in range(rng.randrange(0, 6)):
            s[rng.randrange(L)] = rng.choice(b"ACGTN" if with_n else b"ACGT")
        seqs.append(bytes(s))
    return synth.reads_from_strings(seqs)


def check(oracle, ref, B, O, q, rd, counts=None):
    import torch
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_TM)
    info = idx.info()
    nb, W = info["n_bins"], info["mask_words"]
    mask = empty((rd.n, W), torch.uint32)
    mask.view(torch.int32).fill_(-1)
    cnt = None if counts is None else empty((rd.n, nb), counts)
    grim.grim_filter_scan(idx, grim.ReadSet(dev(rd.bases), dev(rd.offsets), err_permille_all=40,
                                            allow_short_overlap=True), mask, cnt)
    torch.cuda.synchronize()
    bits = oracle.bits(ref, B, O, q)
    want_c, want_p = oracle.scan_all(bits, q, rd.bases, rd.offsets, err_permille=40)
    m = host(mask)
    assert np.array_equal(unpack_mask(m, nb), want_p)
    if nb % 32:
        assert not np.any(m[:, -1] >> np.uint32(nb % 32))
    if cnt is not None:
        assert np.array_equal(host(cnt), want_c)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 31, 33, 127, 130, 515])
@pytest.mark.parametrize("q,bins", [(5, 37), (5, 1024), (5, 1025), (4, 3000), (6, 3000), (7, 700), (3, 9000), (5, 70000)])
def test_read_counts(oracle, n, q, bins):
    rng = random.Random(n * 1000 + q + bins)
    B = 16
    if bins * n > 4_000_000:
        n = max(1, 4_000_000 // bins)
    ref = np.frombuffer(bytes(rng.choices(b"ACGT", k=bins * B - 5)), np.uint8).copy()
    check(oracle, ref, B, 40, q, mixed_reads(rng, ref, n, (q, 33, 100, 150, 255 + q, 300)))


@pytest.mark.parametrize("chunk", [64, 256, 4096])
@pytest.mark.parametrize("n", [449, 512, 513, 1031])
def test_chunk_counts(oracle, monkeypatch, chunk, n):
    # 64 reads a chunk: 7, 8 and more chunks (the order of workgroups changes at 8)
    monkeypatch.setenv("GRIM_SCAN_CHUNK", str(chunk))
    rng = random.Random(n + chunk)
    ref = np.frombuffer(bytes(rng.choices(b"ACGTN", weights=[9, 9, 9, 9, 0.1], k=40_000)), np.uint8).copy()
    check(oracle, ref, 16, 40, 5, mixed_reads(rng, ref, n, (20, 64, 100, 250)))


@pytest.mark.parametrize("n", [16384, 16385])
def test_length_order(oracle, n):
    rng = random.Random(n)
    ref = np.frombuffer(bytes(rng.choices(b"ACGT", k=3000)), np.uint8).copy()
    check(oracle, ref, 64, 40, 5, mixed_reads(rng, ref, n, (20, 40, 80, 150), with_n=False))

"""Calls that run out of memory after their first launch: they return only when
that work is done (their workspace may go to another handle next), and the
handle then works as before."""

from __future__ import annotations

import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu
B, O, q, E = 256, 160, 5, 5


@pytest.fixture(scope="module")
def world(oracle):
    ref = synth.genome(synth.GenomeSpec(length=60_000, seed=21))
    rd = synth.reads(synth.ReadSpec(n_reads=200, seed=22, lens=(100, 150), len_w=(1, 1), edit_mode=0, edits=4), ref)
    budget = np.full(rd.n, E, np.uint16)
    return ref, rd, budget, oracle


def busy(stream):
    """Some tens of milliseconds of work ahead of the call on its stream."""
    import torch
    with torch.cuda.stream(stream):
        torch.cuda._sleep(100_000_000)
    assert not stream.query()


def fails_when_done(monkeypatch, stream, call):
    busy(stream)
    monkeypatch.setenv("GRIM_POOL_TEST_FAIL", "1")
    with pytest.raises(grim.GrimError) as e:
        call()
    left = not stream.query()
    monkeypatch.delenv("GRIM_POOL_TEST_FAIL")
    assert e.value.code == grim.GRIM_ENOMEM
    assert not left, "the call returned with its work still on the stream"


def test_scan(world, monkeypatch):
    import torch
    ref, rd, budget, oracle = world
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_TM)
    reads = grim.ReadSet(dev(rd.bases), dev(rd.offsets), max_edits=dev(budget))
    mask = empty((rd.n, idx.info()["mask_words"]), torch.uint32)
    counts = empty((rd.n, idx.info()["n_bins"]), torch.uint16)
    monkeypatch.setenv("GRIM_SCAN_SORT", "0")  # tokens and thresholds get their memory, the order does not
    grim.grim_filter_scan(idx, reads, mask, counts)
    monkeypatch.delenv("GRIM_SCAN_SORT")
    stream = torch.cuda.Stream()
    fails_when_done(monkeypatch, stream, lambda: grim.grim_filter_scan(idx, reads, mask, counts, stream=stream))
    counts.view(torch.int16).zero_()
    torch.cuda.synchronize()
    grim.grim_filter_scan(idx, reads, mask, counts, stream=stream)
    want, _ = oracle.scan_all(oracle.bits(ref, B, O, q), q, rd.bases, rd.offsets, max_edits=budget)
    assert np.array_equal(host(counts), want)


def test_verify(world, monkeypatch):
    import torch
    ref, rd, budget, oracle = world
    idx = grim.grim_build_index(dev(ref), B, O, q, grim.LAYOUT_TM | grim.LAYOUT_REF)
    nb = idx.info()["n_bins"]
    reads = grim.ReadSet(dev(rd.bases), dev(rd.offsets), max_edits=dev(budget))
    grim.grim_filter_scan(idx, reads, empty((rd.n, idx.info()["mask_words"]), torch.uint32))  # thresholds
    co = np.arange(rd.n + 1, dtype=np.int64) * 3
    cb = np.sort(np.random.default_rng(3).integers(0, nb, (rd.n, 3)), axis=1).reshape(-1).astype(np.int32)
    off, bins = dev(co), dev(cb)
    dist, match = empty((len(cb),), torch.uint16), empty((len(cb),), torch.uint8)
    stream = torch.cuda.Stream()
    fails_when_done(monkeypatch, stream, lambda: grim.grim_verify_candidates_bounded(idx, reads, off, bins, None, dist,
                                                                                    match, stream=stream))
    torch.cuda.synchronize()
    grim.grim_verify_candidates_bounded(idx, reads, off, bins, None, dist, match, stream=stream)
    want_d, want_m = oracle.verify_bounded(ref, B, O, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
    assert np.array_equal(host(dist.view(torch.int16)).view(np.uint16), want_d) and np.array_equal(host(match), want_m)

"""Seed candidates of more reads than one launch of 16 threads a read can hold
(2^28): one-base reads with one-base seeds on a reference of one A and fifty C,
so that a read's best bin is known from its base alone."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_util import dev, host, log
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu


def test_more_reads_than_a_launch_holds(monkeypatch):
    import torch
    monkeypatch.setenv("GRIM_SEED_BATCH_KEYS", str(1 << 24))
    n = (1 << 28) + 77
    seeds = grim.grim_seeds_build(dev(np.frombuffer(b"A" + b"C" * 50, np.uint8).copy()), 1)
    g = torch.Generator(device="cuda")
    g.manual_seed(28)
    bases = torch.tensor([65, 67, 71], dtype=torch.uint8, device="cuda")[
        torch.randint(0, 3, (n,), generator=g, device="cuda", dtype=torch.int32)]
    reads = grim.ReadSet(bases, torch.arange(n + 1, dtype=torch.int64, device="cuda"))
    off = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
    bins = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    log("inputs made")
    total = grim.grim_seed_candidates(seeds, reads, 10, 1, off, bins)
    log("candidates", total)
    # A: its one hit is in bin 0; C: bins 1..4 hold ten hits each, the smallest wins; G: none
    hit = bases != 71
    assert total == int(hit.sum())
    assert int(off[0]) == 0 and bool((off[1:] - off[:-1] == hit).all())
    assert torch.equal(bins[:total], (bases[hit] == 67).int())
    assert host(bins[total:total + 1]).tolist() == [-1]

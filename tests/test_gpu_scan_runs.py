"""The all-bins scan on either side of the chunk count and chunk size from which a
chunk takes a run of the reads in length order. Bit-exact against the CPU oracle."""

from __future__ import annotations

import random

import numpy as np
import pytest

from test_gpu_scan_shapes import check, mixed_reads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,chunk", [(60_000, 640), (51_201, 540), (49_000, 520), (60_000, 4096), (50_001, 530)])
def test_runs_of_reads(oracle, monkeypatch, n, chunk):
    """96 chunks and more of 512 reads and more, a few less, and far fewer."""
    monkeypatch.setenv("GRIM_SCAN_CHUNK", str(chunk))
    rng = random.Random(n + chunk)
    ref = np.frombuffer(bytes(rng.choices(b"ACGTN", weights=[9, 9, 9, 9, 0.1], k=1500)), np.uint8).copy()
    check(oracle, ref, 64, 40, 5, mixed_reads(rng, ref, n, (20, 64, 100, 250)))

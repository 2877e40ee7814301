"""Bounded verification of a bin whose text is nearly 2^32 bases: pieces of the
read at both ends, so that the stretch to align is as long as the text. The
reference is one base repeated, the read does not hold it, and two copies with
one substitution are planted: the distance is 1 by construction."""

from __future__ import annotations

import numpy as np
import pytest

from gpu_util import empty, host, log
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("short_by", [100])
def test_text_of_nearly_all_offsets(short_by):
    import torch
    G = (1 << 32) - short_by
    read = np.frombuffer(b"ACGGCAACGCAGCGAACGGACACGCA", np.uint8)  # 26 bases: two pieces of 13, one edit
    ref = torch.full((G,), ord("T"), dtype=torch.uint8, device="cuda")
    for at, edit in ((40, 20), (G - 60, 3)):
        copy = torch.from_numpy(read.copy()).cuda()
        copy[edit] = ord("T")
        ref[at:at + len(read)] = copy
    idx = grim.grim_build_index(ref, (1 << 32) - 1, 0, 5, grim.LAYOUT_REF)
    assert idx.info()["n_bins"] == 1
    del ref
    log("index built")
    reads = grim.ReadSet(torch.from_numpy(read.copy()).cuda(), torch.tensor([0, len(read)], device="cuda"),
                         max_edits=torch.ones(1, dtype=torch.int16, device="cuda").view(torch.uint16),
                         allow_short_overlap=True)
    dist, match = empty((1,), torch.int16), empty((1,), torch.uint8)
    dist.fill_(77)
    match.fill_(77)
    grim.grim_verify_candidates_bounded(idx, reads, torch.tensor([0, 1], device="cuda"),
                                        torch.zeros(1, dtype=torch.int32, device="cuda"), None,
                                        dist.view(torch.uint16), match)
    log("verified")
    assert host(dist).tolist() == [1] and host(match).tolist() == [1]
    idx.free()

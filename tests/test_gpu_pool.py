"""Device memory kept between handles: it comes back by itself without another
call of the library, at once when asked for, and at the process's end; blocks that
go from handle to handle between threads and streams give the oracle's results."""

from __future__ import annotations

import os
import subprocess
import sys
import threading
import time

import numpy as np
import pytest

import synth
from gpu_util import dev, empty, host, log
from paper_1708_04329_amd import grim

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GB = 1 << 30


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def back_within(seconds, level):
    end = time.monotonic() + seconds
    while free_bytes() < level:
        if time.monotonic() > end:
            return False
        time.sleep(0.02)
    return True


@pytest.fixture()
def reference():
    import torch
    ref = torch.full((GB,), ord("A"), dtype=torch.uint8, device="cuda")
    grim.grim_build_index(ref, 4096, 0, 5, grim.LAYOUT_REF).free()  # whatever a first call sets up
    grim.grim_trim_memory()
    time.sleep(0.2)
    return ref


def test_idle_memory_comes_back_without_a_call(reference):
    before = free_bytes()
    grim.grim_build_index(reference, 4096, 0, 5, grim.LAYOUT_REF).free()
    log("kept", before - free_bytes())
    assert back_within(6.0, before)


def test_memory_comes_back_when_asked_for(reference):
    before = free_bytes()
    grim.grim_build_index(reference, 4096, 0, 5, grim.LAYOUT_REF).free()
    assert free_bytes() <= before - GB // 2  # kept for the next handle
    grim.grim_trim_memory()
    assert back_within(1.0, before)  # well before idle blocks go by themselves


def test_long_lived_memory_is_not_kept(reference):
    before = free_bytes()
    idx = grim.grim_build_index(reference, 4096, 0, 5, grim.LAYOUT_REF)
    time.sleep(2.1)
    idx.free()
    assert back_within(1.0, before - (64 << 20))


@pytest.mark.parametrize("last", ["idx.free()", "pass", "idx.free(); time.sleep(1.99)",
                                  "idx.free(); seeds.free(); grim.grim_trim_memory()"])
def test_process_ends_with_blocks_idle(last):
    code = ("import time, torch\nfrom paper_1708_04329_amd import grim\n"
            "ref = torch.full((1 << 22,), 65, dtype=torch.uint8, device='cuda')\n"
            "seeds = grim.grim_seeds_build(ref, 6)\n"
            "idx = grim.grim_build_index(ref, 4096, 0, 5, grim.LAYOUT_REF | grim.LAYOUT_BM)\n" + last + "\nprint('done')\n")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.strip().endswith("done"), (out.returncode, out.stderr[-500:])


def test_threads_and_streams_exchange_blocks(oracle):
    import torch
    B, O, q, k, cap = 256, 160, 5, 8, 16
    jobs = []
    for t in range(2):
        ref = synth.genome(synth.GenomeSpec(length=150_000 + 1000 * t, seed=50 + t))
        rd = synth.reads(synth.ReadSpec(n_reads=300, seed=60 + t, lens=(100, 150), len_w=(1, 1), edit_mode=0, edits=4), ref)
        budget = np.full(rd.n, 5, np.uint16)
        co, cb = oracle.seed_candidates(ref, rd.bases, rd.offsets, k, B, cap)
        bits = oracle.bits(ref, B, O, q)
        cnt, _ = oracle.scan_candidates(bits, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
        dist, _ = oracle.verify_bounded(ref, B, O, q, rd.bases, rd.offsets, co, cb, max_edits=budget)
        jobs.append((ref, rd, budget, co, cb, cnt, dist))
    wrong = []

    def work(t):
        ref, rd, budget, co, cb, want_c, want_d = jobs[t]
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            dref, reads = dev(ref), grim.ReadSet(dev(rd.bases), dev(rd.offsets), max_edits=dev(budget))
            off, bins = empty((rd.n + 1,), torch.int64), empty((rd.n * cap,), torch.int32)
            cnt, dist = empty((len(cb),), torch.uint16), empty((len(cb),), torch.uint16)
            match = empty((len(cb),), torch.uint8)
            for i in range(40):
                for out in (off, bins, cnt.view(torch.int16), dist.view(torch.int16)):
                    out.zero_()
                seeds = grim.grim_seeds_build(dref, k, stream=stream)
                idx = grim.grim_build_index(dref, B, O, q, grim.LAYOUT_BM | grim.LAYOUT_REF, stream=stream)
                n = grim.grim_seed_candidates(seeds, reads, B, cap, off, bins, stream=stream)
                grim.grim_filter_candidates(idx, reads, off, bins[:n], cnt, match, stream=stream)
                grim.grim_verify_candidates_bounded(idx, reads, off, bins[:n], None, dist, match, stream=stream)
                ok = (n == len(cb) and np.array_equal(host(off), co) and np.array_equal(host(bins)[:n], cb)
                      and np.array_equal(host(cnt), want_c)
                      and np.array_equal(host(dist.view(torch.int16)).view(np.uint16), want_d))
                idx.free()
                seeds.free()
                if not ok:
                    wrong.append((t, i))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong

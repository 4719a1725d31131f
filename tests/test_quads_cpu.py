"""Host self-check of the row-quad packings (sdnn_plan_check_host re-walks every program of a
default plan: each entry once, in its row, in ascending column order, with its weight bits and
inside the chunks its descriptor states)."""
import os
import re

import numpy as np
import pytest

import paper_2101_07948_amd as sd
from conftest import ROOT, random_csr


def check(row_ptr, col_idx, values, M, K, **kw):
    info = sd.plan_check_host(row_ptr, col_idx, values, M, K, **kw)
    assert info["nnz"] == len(col_idx) and info["packings"] == 5


@pytest.mark.parametrize("M,K,density", [(1, 1, 1.0), (7, 64, 0.5), (33, 65, 0.3), (100, 513, 0.02),
                                         (257, 700, 0.9), (40, 9000, 0.01)])
def test_random_patterns(M, K, density):
    rp, ci, v, _ = random_csr(np.random.default_rng([M, K]), M, K, density)
    check(rp, ci, v, M, K)
    check(rp, ci, v, M, K, out_permuted=True)
    check(rp, ci, v, M, K, split_chunks=2)


def test_info_reports_the_packings_and_their_memory():
    """quad_packings and quad_kib: at least 8 bytes per entry and packing for a default plan, none
    for a plan that fixes a panel height, a grouping or a tile width: these are the
    panel kernel's, and its calls stay there."""
    rp, ci, v, _ = random_csr(np.random.default_rng(3), 256, 512, 0.1)
    info = sd.plan_check_host(rp, ci, v, 256, 512)
    assert info["quad_packings"] == 4
    assert 4 * 8 * len(ci) <= 1024 * info["quad_kib"] <= 4 * 16 * len(ci)
    for kw in ({"panel_rows": 8}, {"tile_cols": 128}, {"tile_cols": 256}, {"grouping": "order"},
               {"grouping": "balanced"}):
        info = sd.plan_check_host(rp, ci, v, 256, 512, **kw)
        assert info["quad_packings"] == 0 and info["quad_kib"] == 0


def scattered_runs(M, K, n, seed):
    """M rows of n neighbouring entries each, at random places."""
    start = np.random.default_rng(seed).integers(0, K - n + 1, M)
    cols = (start[:, None] + np.arange(n)).astype(np.int32).ravel()
    return np.arange(0, M * n + 1, n, dtype=np.int32), cols, np.ones(M * n, np.float32)


@pytest.mark.parametrize("M,K,rows", [(4096, 8000, "runs"), (4096, 60000, "runs"),
                                      (2048, 262144, "uniform"), (20000, 50000, "uniform")])
def test_memory_stays_within_the_panel_packings(M, K, rows):
    """Rows whose entries a block cannot put together (16 neighbours scattered over K; 26 or 2
    entries spread over all of K): the row-quad packings together take at most twice what the panel
    packings take, a packing that would take more than its share is left out."""
    if rows == "runs":
        rp, ci, v = scattered_runs(M, K, 16, M + K)
    else:
        n = 26 if K > 100000 else 2
        ci = np.sort(np.random.default_rng(M).integers(0, K // n, (M, n)) + np.arange(n) * (K // n), 1)
        rp, ci, v = np.arange(0, M * n + 1, n, dtype=np.int32), ci.astype(np.int32).ravel(), np.ones(M * n, np.float32)
    info = sd.plan_check_host(rp, ci, v, M, K, permute="identity")
    assert 1024 * info["quad_kib"] <= 2 * info["packed_bytes"]
    assert (info["quad_packings"] < 4) == (rows == "runs")


def test_empty_and_extreme_rows():
    """No entries at all, one full row among empty ones, and rows at opposite ends of K (fillers
    everywhere, more than 64 descriptors in a program)."""
    check(np.zeros(6, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32), 5, 100)
    K = 20000
    rp = np.array([0, 0, K, K, K, K, K, K, K], np.int32)
    check(rp, np.arange(K, dtype=np.int32), np.ones(K, np.float32), 8, K)
    lo, hi = np.arange(0, 300), np.arange(K - 300, K)
    cols = np.concatenate([lo, hi, lo, hi, np.arange(0, K, 70)]).astype(np.int32)
    rp = np.cumsum([0, 300, 300, 300, 300, len(range(0, K, 70))]).astype(np.int32)
    check(rp, cols, np.ones(len(cols), np.float32), 5, K)


def test_no_wait_on_a_counter_at_its_end():
    """The LDS counter has 4 bits: at 15 it may stand for more, and a wait for "at most 15 in flight"
    waits for nothing.  Every wait of the generated loops is on 14 or fewer (the loads' counter,
    of 6 bits, on 62 or fewer)."""
    text = open(os.path.join(ROOT, "paper_2101_07948_amd", "csrc", "quad_asm_gen.h")).read()
    lds = [int(n) for n in re.findall(r"lgkmcnt\((\d+)\)", text)]
    loads = [int(n) for n in re.findall(r"vmcnt\((\d+)\)", text)]
    assert lds and max(lds) <= 14 and loads and max(loads) <= 62


@pytest.mark.parametrize("header", ["quad_asm_gen.h", "spmm_asm_gen.h"])
def test_consumer_loops_hand_back_their_poll_budget(header):
    """A wave runs its loop once per item: the loop starts from what the items before have left of
    the budget (handed on in a register, or in the wave's word of LDS), so that the bound on a wave's
    waiting does not grow with its items."""
    text = open(os.path.join(ROOT, "paper_2101_07948_amd", "csrc", header)).read()
    loops = len(re.findall(r"__device__ __forceinline__ void consume_", text))
    count = lambda pattern: len(re.findall(pattern, text))
    assert loops > 0
    if header == "quad_asm_gen.h":
        assert count(r'\[budget\] "\+[sv]"\(budget\)') == count(r"a\.poll_budget = budget;") == loops
        assert count(r"[sv]_mov_b32 %\[budget\], s\d+") == loops
    else:
        assert count(r"ds_read_b32 v30, %\[pa\] offset:128") == count(r"ds_write_b32 %\[pa\], v30 offset:128") == loops

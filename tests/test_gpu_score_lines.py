"""Batched scoring at the lines between its two kernels: rows on either side of
each line, against the oracle bit for bit, and the time of calls that the
wrong kernel makes much slower."""
import numpy as np
import pytest

import workloads as W
from test_gpu_score import DEV, P, check, rows_of  # noqa: F401  (P: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F,T,depth,offset,leaves", [
    # with leaf indices: either side of each line
    (24577, 176, 30, 4, 0, True), (24576, 176, 30, 4, 0, True), (24577, 192, 15, 6, 1, True),
    (32769, 110, 9, 7, 0, True), (32768, 110, 9, 7, 3, True), (32769, 176, 9, 8, 0, True),
    (45057, 176, 65, 8, 0, True), (45056, 192, 65, 8, 0, True), (65537, 176, 24, 9, 0, True),
    (81921, 192, 25, 9, 0, True), (131072, 176, 25, 9, 0, True), (131073, 176, 25, 9, 0, True),
    # scores alone
    (32769, 176, 25, 8, 0, False), (32768, 176, 25, 8, 0, False), (32769, 110, 1600, 1, 2, False),
    (49153, 192, 80, 7, 0, False), (49152, 176, 80, 7, 1, False), (65537, 176, 24, 9, 0, False),
    (98305, 176, 112, 6, 0, False), (98304, 192, 112, 6, 0, False), (98305, 110, 60, 8, 0, False),
    (98305, 176, 49, 9, 0, False), (114689, 176, 170, 7, 0, False), (114688, 192, 156, 8, 0, False),
    (114689, 192, 156, 8, 0, False), (131072, 176, 157, 8, 0, False), (131071, 110, 157, 8, 1, False)])
def test_scores_at_the_lines(P, n, F, T, depth, offset, leaves):
    print(f"[gpu-score] lines: n {n} F {F} T {T} depth {depth} offset {offset} leaves {leaves}", flush=True)
    check(P, W.make_ensemble(T, depth, F, 29), rows_of(n, F, n + F), leaves, offset)


def call_us(P, tables, n, F, leaves):
    """Time of one scoring call among others: the best of nine runs of ten."""
    import torch
    ens = P.at_ensemble_create(*tables, F)
    feats = torch.from_numpy(rows_of(1 << 12, F, 3)).to(DEV).repeat((n + (1 << 12) - 1) >> 12, 1)[:n].contiguous()
    sc = torch.empty(n, dtype=torch.float32, device=DEV)
    lv = torch.empty((n, tables[0].shape[0]), dtype=torch.int16, device=DEV) if leaves else None
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = np.inf
    for _ in range(9):
        a.record()
        for _ in range(10):
            P.at_gbt_predict(ens, feats, sc, lv)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 100)
    return best


@pytest.mark.parametrize("n,T,depth", [(131072, 100, 4), (131072, 250, 6)])
def test_leaf_indices_of_many_rows_cost_no_second_walk(P, n, T, depth):
    """The kernel that walks a row on one lane takes 1.4 to 1.6 times its own
    time with the indices (their stores), the other one 2.4 to 2.8 times."""
    tables = W.make_ensemble(T, depth, 176, 5)
    scores, leaves = call_us(P, tables, n, 176, False), call_us(P, tables, n, 176, True)
    print(f"[gpu-score] n {n} T {T} depth {depth}: {scores:.1f} us, with leaf indices {leaves:.1f} us", flush=True)
    assert leaves < 2.0 * scores


@pytest.mark.parametrize("F", [109, 110, 111, 112, 173, 174, 175, 176, 189, 190, 191, 192])
@pytest.mark.parametrize("n", [131072, 131329])
def test_rows_that_end_within_their_last_quad(P, F, n):
    """Every row length of the one-lane-a-row kernel: its last load takes the
    row's last four features and moves them to their places."""
    fid, thr, leaf = W.make_ensemble(12, 4, F, 5)
    fid[:, 0] = F - 1 - np.arange(12) % 5                # every tree looks at the row's end first
    print(f"[gpu-score] row ends: F {F} n {n}", flush=True)
    check(P, (fid, thr, leaf), rows_of(n, F, F), False, F % 4)
    check(P, (fid, thr, leaf), rows_of(n, F, F), True, 0)


@pytest.mark.parametrize("T,depth", [(40, 3), (100, 4)])
def test_one_row_fewer_costs_no_more(P, T, depth):
    """131071 rows against 131072, where one row decided the kernel: 26 us
    against 21 for 40 trees of depth 3."""
    tables = W.make_ensemble(T, depth, 176, 5)
    below, at = call_us(P, tables, 131071, 176, False), call_us(P, tables, 131072, 176, False)
    print(f"[gpu-score] T {T} depth {depth}: 131071 rows {below:.1f} us, 131072 {at:.1f}", flush=True)
    assert below < 1.1 * at

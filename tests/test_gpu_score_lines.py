"""Batched scoring at the lines between its two kernels: rows on either side of
each line, against the oracle bit for bit, and the time of calls that the
wrong kernel makes much slower."""
import numpy as np
import pytest

import workloads as W
from test_gpu_score import DEV, P, check, rows_of  # noqa: F401  (P: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,F,T,depth,offset", [
    (24577, 176, 30, 4, 0), (24576, 176, 30, 4, 0), (28673, 192, 15, 6, 0), (28672, 110, 15, 6, 0), (36865, 110, 9, 7, 0),
    (36865, 176, 9, 8, 0), (49153, 176, 65, 8, 0), (49152, 192, 65, 8, 0), (98305, 176, 7, 9, 0), (28673, 192, 9, 5, 1),
    (28673, 110, 9, 5, 3)])
def test_leaves_at_the_lines(P, n, F, T, depth, offset):
    print(f"[gpu-score] leaf lines: n {n} F {F} T {T} depth {depth} offset {offset}", flush=True)
    check(P, W.make_ensemble(T, depth, F, 29), rows_of(n, F, n + F), True, offset)


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

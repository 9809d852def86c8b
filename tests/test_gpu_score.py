"""GPU parity of batched scoring at the edges of its kernels' plans: rows a
workgroup (8 .. 64), partial workgroups, chunks and tree groups, both tree
forms, unaligned rows, and the three kinds of ensembles (thresholds within
six bits; above them only in splits that decide nothing; above them).
Scores are fp32 left folds in tree order, so they are compared bit for bit
with the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def P():
    import torch
    torch.cuda.set_device(0)
    import paper_1805_08166_amd
    return paper_1805_08166_amd


def check(P, tables, feats, leaves, offset=0):
    """Scores (and leaf indices) of feats against the oracle; offset: ints
    the feature rows start past a 16-byte boundary."""
    import torch
    n, F = feats.shape
    ens = P.at_ensemble_create(*tables, F)
    buf = torch.zeros(n * F + 4, dtype=torch.int32, device=DEV)
    d = buf[offset: offset + n * F].view(n, F)
    d.copy_(torch.from_numpy(feats))
    guard = 64
    sc = torch.full((n + guard,), 7.0, dtype=torch.float32, device=DEV)
    T = tables[0].shape[0]
    lv = torch.full((n + guard, T), -1, dtype=torch.int16, device=DEV) if leaves else None
    P.at_gbt_predict(ens, d, sc[:n], lv[:n] if leaves else None)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(min(n, 300)), n - 1 - np.arange(min(n, 300))]))
    # the library reads features as bytes: values are clamped to [0, 255]
    want, wl = oracle.predict(*tables, np.clip(feats[rows], 0, 255), True)
    got = sc.cpu().numpy()
    assert np.array_equal(got[rows].view(np.uint32), want.view(np.uint32))
    assert (got[n:] == 7.0).all()
    if leaves:
        g = lv.cpu().numpy()
        assert np.array_equal(g[rows].view(np.uint16), wl)
        assert (g[n:] == -1).all()


def rows_of(n, F, seed, hi=40):
    f = np.random.default_rng(seed).integers(-3, hi, size=(n, F), dtype=np.int64)
    return f.astype(np.int32)


@pytest.mark.parametrize("n,F,T,depth", [
    (1, 1, 1, 1), (7, 110, 3, 2), (9, 5, 101, 4), (63, 176, 4, 5), (2048, 176, 257, 8), (2049, 110, 130, 6),
    (4097, 192, 61, 9), (8193, 208, 97, 7), (12289, 176, 45, 10), (24577, 130, 90, 4), (24577, 176, 50, 8),
    (98305, 110, 30, 6), (131072, 110, 9, 8), (131073, 176, 9, 8), (131072, 192, 9, 7), (131072, 256, 5, 9),
    (300, 256, 33, 11), (300, 255, 21, 12), (2050, 240, 17, 3)])
@pytest.mark.parametrize("leaves", [False, True])
def test_scores_at_plan_edges(P, n, F, T, depth, leaves):
    print(f"[gpu-score] n {n} F {F} T {T} depth {depth} leaves {leaves}", flush=True)
    check(P, W.make_ensemble(T, depth, F, 17 + depth), rows_of(n, F, n + F), leaves)


@pytest.mark.parametrize("F,n", [(176, 500), (176, 131072), (110, 500), (110, 131072)])
@pytest.mark.parametrize("offset", [1, 2, 3])
def test_scores_of_unaligned_rows(P, F, n, offset):
    print(f"[gpu-score] unaligned: F {F} n {n} offset {offset}", flush=True)
    check(P, W.make_ensemble(11, 6, F, 5), rows_of(n, F, 3), True, offset)
    check(P, W.make_ensemble(11, 6, F, 5), rows_of(n, F, 3), False, offset)


@pytest.mark.parametrize("F", [110, 176, 192, 130])
@pytest.mark.parametrize("n", [70, 5000])
def test_scores_with_thresholds_above_six_bits(P, F, n):
    """Thresholds up to 255 with features up to 300 (clamped to 255): a
    six-bit threshold would decide differently."""
    print(f"[gpu-score] wide thresholds: F {F} n {n}", flush=True)
    fid, thr, leaf = W.make_ensemble(13, 6, F, 9)
    thr = np.random.default_rng(4).integers(0, 256, size=thr.shape).astype(np.uint8)
    check(P, (fid, thr, leaf), rows_of(n, F, 8, hi=300), False)
    check(P, (fid, thr, leaf), rows_of(n, F, 8, hi=300), True)


@pytest.mark.parametrize("hi", [40, 300])
def test_scores_of_padded_trees(P, hi):
    """Splits with threshold 255 over copies of one leaf (trained trees
    padded to full ones), features on both sides of 63 and 255."""
    print(f"[gpu-score] padded trees: features below {hi}", flush=True)
    trees = W.make_node_trees(40, 6, 176, 3)
    fid, thr, leaf = P.at_trees_pad(trees, 176, 7)
    thr = np.where(thr == 255, 255, np.minimum(thr, 63)).astype(np.uint8)
    check(P, (fid, thr, leaf), rows_of(777, 176, 5, hi=hi), False)
    check(P, (fid, thr, leaf), rows_of(777, 176, 5, hi=hi), True)


def test_scores_at_the_six_bit_edge(P):
    """Thresholds and features around 62 .. 64, where the clamp begins."""
    print("[gpu-score] six-bit edge", flush=True)
    fid, thr, leaf = W.make_ensemble(9, 5, 176, 2)
    r = np.random.default_rng(1)
    f = r.integers(60, 67, size=(400, 176)).astype(np.int32)
    for top in (63, 64):
        thr = r.integers(60, top + 1, size=thr.shape).astype(np.uint8)
        check(P, (fid, thr, leaf), f, True)
        check(P, (fid, thr, leaf), f, False)


def test_scores_of_more_rows_than_one_launch_takes(P):
    """2^29 rows and some: eight threads a row would be more than the 2^32
    threads of one launch.  One feature, so the oracle's scores of its 64
    values give every row's."""
    import torch
    n, part = (1 << 29) + 77, 1 << 26
    print(f"[gpu-score] n {n}", flush=True)
    tables = W.make_ensemble(28, 2, 1, 6)
    want = oracle.predict(*tables, np.arange(64, dtype=np.int32)[:, None], False)
    want = torch.from_numpy(np.asarray(want[0] if isinstance(want, tuple) else want, np.float32)).to(DEV)
    assert want.unique().numel() > 1
    ens = P.at_ensemble_create(*tables, 1)
    f = torch.randint(0, 64, (n, 1), dtype=torch.int32, device=DEV)
    sc = torch.full((n,), 7.0, dtype=torch.float32, device=DEV)
    P.at_gbt_predict(ens, f, sc, None)
    for lo in range(0, n, part):
        assert torch.equal(sc[lo: lo + part], want[f[lo: lo + part, 0].long()])

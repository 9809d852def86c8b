"""GPU parity of the tree-partitioned path on both sides of its chain kernel's
width rule: four or eight waves by trees, chains and whether a block of 16
chains has its space's tables in LDS; compact tiles (a space with constant
features) and whole ones; traced, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SMALL = (3, (1, 4, 8, 8, 6, 3, 3, 1, 1))                  # conv2d with the vectorize and vthread knobs
C2 = (1, (1, 64, 56, 56, 64, 3, 3, 1, 1))                 # ResNet-18 C2: compact tiles
PLAIN = (1, SMALL[1])
ONE = (0, (32, 1, 8))                                     # GEMM with a unit axis: compact tiles


@pytest.fixture(scope="module")
def P():
    import torch
    torch.cuda.set_device(0)
    import paper_1805_08166_amd
    return paper_1805_08166_amd


@pytest.mark.parametrize("members,n,trees,depth,waves", [
    ([SMALL], 37, 700, 4, 8), ([SMALL], 37, 701, 4, 4), ([C2], 4096, 90, 3, 8), ([C2], 4097, 90, 3, 4),
    ([C2], 37, 1, 1, 8), ([C2], 33, 720, 3, 4), ([ONE], 33, 40, 3, 8), ([ONE], 33, 720, 3, 4),
    ([PLAIN, C2, PLAIN], 50, 720, 3, 8),                  # blocks over two spaces
    ([PLAIN, C2], 48, 720, 3, 4), ([PLAIN, C2, C2], 21, 30, 4, 8)])
def test_runs_on_both_widths(P, members, n, trees, depth, waves):
    """n chains a space; `waves` is what the rule gives (a compute unit a
    workgroup at most, and at most 700 trees or a block over two spaces)."""
    import torch
    print(f"[gpu-chain] spaces {members} chains {n} trees {trees} depth {depth} waves {waves}", flush=True)
    spaces = [P.at_space_create(*m) for m in members]
    offs = np.arange(len(members) + 1) * n
    sp = spaces[0] if len(members) == 1 else P.at_spaceset_create(spaces, offs)
    total = n * len(members)
    blocks_apart = len(members) == 1 or n % 16 == 0
    assert waves == (8 if (total + 15) // 16 <= 256 and (trees <= 700 or not blocks_apart) else 4)
    tables = W.make_ensemble(trees, depth, sp.n_features, 11)
    ens = P.at_ensemble_create(*tables, sp.n_features)
    seed, k, base = 17, 6, 0
    ch = P.at_chains_create(sp, 0, total, k, seed)
    P.at_chains_set_path(ch, P.AT_SA_PATH_TREES)
    m = min(n, 20)                                        # the last chains of every space
    och = [oracle.Chains([oracle.Space(*members[i])], [0, m], seed=seed, chain0=int(offs[i + 1]) - m, topk=k)
           for i in range(len(members))]
    for steps in (6, 3):
        thr = P.at_sa_thresholds(seed, 0, total, base, steps)
        best = torch.zeros((total, k, 4), dtype=torch.int32, device=DEV)
        trace = torch.zeros((total, steps, 4), dtype=torch.int32, device=DEV)
        P.at_sa_run_traced(sp, ens, ch, steps, torch.from_numpy(thr).to(DEV), best, trace)
        torch.cuda.synchronize()
        tr, top = P.entries(trace), P.entries(best)
        for i, oc in enumerate(och):
            lo, hi = int(offs[i + 1]) - m, int(offs[i + 1])
            otr = oc.run(tables, steps, oracle.thresholds(seed, lo, m, base, steps), trace=True)
            assert np.array_equal(tr["cfg"][lo:hi], otr["cfg"])
            assert np.array_equal(tr["score"][lo:hi].view(np.uint32), otr["score"].view(np.uint32))
            assert np.array_equal(tr["flag"][lo:hi], otr["valid"])
            assert np.array_equal(top["cfg"][lo:hi], oc.top["cfg"])
            assert np.array_equal(top["score"][lo:hi].view(np.uint32), oc.top["score"].view(np.uint32))
        base += steps
    assert P.at_chains_last_path(ch) == P.AT_SA_PATH_TREES

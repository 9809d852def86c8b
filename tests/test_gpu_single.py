"""GPU parity of the chain-local kernels at the edges of their plans: one, two
and four chains a workgroup, one, two, four and more trees a lane, whole
trees and tails, 512 and 1024 threads, waves that do not walk, and streamed
tree tops; a run that draws its chains and one that continues them, traced,
against the oracle."""
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


# n, trees, depth, then what the plan is to be: chains and threads a workgroup,
# and whole trees resident, tree tops resident ("tail") or streamed ("stream")
@pytest.mark.parametrize("n,trees,depth,cpb,threads,form", [
    (5, 1, 1, 1, 512, "whole"), (40, 7, 3, 1, 512, "whole"), (40, 300, 8, 1, 512, "tail"),
    (256, 447, 6, 1, 512, "tail"), (256, 449, 6, 1, 512, "tail"), (130, 1000, 6, 1, 512, "tail"),
    (300, 223, 6, 2, 512, "whole"), (300, 225, 4, 2, 512, "whole"), (300, 600, 7, 2, 1024, "tail"),
    (511, 520, 5, 2, 1024, "whole"),
    (1021, 96, 8, 4, 512, "whole"), (1000, 112, 8, 4, 512, "tail"), (1000, 113, 6, 4, 512, "whole"),
    (1000, 255, 5, 4, 512, "whole"), (1000, 257, 8, 4, 1024, "tail"), (1000, 520, 8, 4, 1024, "tail"),
    (520, 1000, 4, 4, 1024, "whole"),
    (1000, 257, 6, 4, 1024, "whole"), (1000, 257, 7, 4, 1024, "tail"), (1000, 257, 9, 4, 1024, "tail"),
    (1000, 257, 10, 4, 512, "stream"),                   # the deepest of either form at 1024 threads, and past them
    (40, 700, 9, 1, 512, "stream"), (1000, 200, 10, 4, 512, "stream"), (2000, 600, 8, 8, 512, "stream")])
@pytest.mark.parametrize("tmpl,shape", [(0, (24, 36, 30)), (3, (1, 4, 8, 8, 6, 3, 3, 1, 1))])
def test_runs_at_plan_edges(P, tmpl, shape, n, trees, depth, cpb, threads, form):
    import torch
    print(f"[gpu-single] template {tmpl} chains {n} trees {trees} depth {depth}", flush=True)
    sp, osp = P.at_space_create(tmpl, shape), oracle.Space(tmpl, shape)
    tables = W.make_ensemble(trees, depth, sp.n_features, 7)
    ens = P.at_ensemble_create(*tables, sp.n_features)
    seed, k = 61, 5
    ch = P.at_chains_create(sp, 3, n, k, seed)
    P.at_chains_set_path(ch, P.AT_SA_PATH_LOCAL)
    m = min(n, 24)
    lo = n - m                                    # the last workgroup may be short
    och = oracle.Chains([osp], [0, m], seed=seed, chain0=3 + lo, topk=k)
    base = 0
    for steps in (7, 1, 4):
        thr = P.at_sa_thresholds(seed, 3, n, base, steps)
        best = torch.zeros((n, k, 4), dtype=torch.int32, device=DEV)
        trace = torch.zeros((n, steps, 4), dtype=torch.int32, device=DEV)
        P.at_sa_run_traced(sp, ens, ch, steps, torch.from_numpy(thr).to(DEV), best, trace)
        torch.cuda.synchronize()
        tr, top = P.entries(trace)[lo:], P.entries(best)[lo:]
        otr = och.run(tables, steps, oracle.thresholds(seed, 3 + lo, m, base, steps), trace=True)
        assert np.array_equal(tr["cfg"], otr["cfg"])
        assert np.array_equal(tr["score"].view(np.uint32), otr["score"].view(np.uint32))
        assert np.array_equal(tr["flag"], otr["valid"])
        assert np.array_equal(top["cfg"], och.top["cfg"]) and np.array_equal(top["flag"], och.top["valid"])
        assert np.array_equal(top["score"].view(np.uint32), och.top["score"].view(np.uint32))
        base += steps
    plan = P.at_chains_last_plan(ch)
    assert plan["path"] == P.AT_SA_PATH_LOCAL
    assert (plan["chains_per_wg"], plan["threads"]) == (cpb, threads)
    assert (plan["chunks"] > 1, plan["gather"]) == {"whole": (False, 0), "tail": (False, 2), "stream": (True, 1)}[form]

"""GPU parity of the chain-local runs of eight and more chains a workgroup:
every form of their plan (whole trees resident in one pass and in chunks, tree
tops resident, whole trees and tree tops streamed) on one space, on a set
whose boundaries fall inside workgroups and on a space with more split choices
than the LDS takes, with full and short last workgroups; traced, against the
oracle."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CONV = [(1, (1, 2, 4, 4, 2, 3, 3, 1, 1)), (1, (1, 2, 6, 6, 2, 1, 1, 0, 2)), (1, (1, 1, 8, 8, 2, 7, 7, 3, 2))]
BIG = (0, (720, 720, 64))                                 # 2807 split choices

# form -> (whether the trees stream, what at_chains_last_plan calls gather)
FORMS = {"resident": (False, 0), "resident chunks": (False, 0), "tail": (False, 2), "streamed": (True, 0),
         "gathered": (True, 1)}


@pytest.fixture(scope="module")
def P():
    import torch
    torch.cuda.set_device(0)
    import paper_1805_08166_amd
    return paper_1805_08166_amd


@pytest.mark.parametrize("form,trees,depth,n", [
    ("resident", 120, 6, 1500), ("resident", 81, 5, 2500), ("resident", 37, 4, 4500),
    ("resident chunks", 300, 5, 2000), ("resident chunks", 300, 5, 1500), ("resident chunks", 400, 4, 2500),
    ("tail", 250, 8, 1500), ("tail", 251, 7, 2500), ("tail", 130, 8, 4500), ("tail", 250, 8, 1536),
    ("streamed", 1300, 4, 1500), ("streamed", 1201, 4, 2500), ("streamed", 1202, 4, 4500),
    ("gathered", 400, 9, 1500), ("gathered", 350, 9, 2500), ("gathered", 350, 9, 2560), ("gathered", 302, 9, 4500)])
@pytest.mark.parametrize("where", ["one space", "three spaces", "big space"])
def test_plans_of_many_chains(P, where, form, trees, depth, n):
    import torch
    print(f"[gpu-local] {where}, {form}: {n} chains, {trees} trees of depth {depth}", flush=True)
    members = {"one space": CONV[:1], "three spaces": CONV, "big space": [BIG]}[where]
    # the inner boundaries are not multiples of 8 (nor of 16 or 32)
    offs = np.array([0, 5, 701, n] if len(members) == 3 else [0, n], np.int64)
    spaces, ospaces = [P.at_space_create(*m) for m in members], [oracle.Space(*m) for m in members]
    sp = spaces[0] if len(members) == 1 else P.at_spaceset_create(spaces, offs)
    if where == "big space":
        assert sum(int(x) for x in ospaces[0].knob_sizes[:3]) > 1024
    tables = W.make_ensemble(trees, depth, ospaces[0].n_features, 23)
    ens = P.at_ensemble_create(*tables, ospaces[0].n_features)
    seed, k, base = 29, 4, 0
    ch = P.at_chains_create(sp, 11, n, k, seed)
    P.at_chains_set_path(ch, P.AT_SA_PATH_LOCAL)
    # the first chains (the inner boundaries among them) and the last
    cuts = [(0, min(n, 760 if len(members) == 3 else 40)), (n - 40, n)]
    och = []
    for lo, hi in cuts:
        o = np.clip(offs, lo, hi) - lo
        keep = [i for i in range(len(members)) if o[i + 1] > o[i]]
        och.append(oracle.Chains([ospaces[i] for i in keep], np.array([0] + [o[i + 1] for i in keep], np.int64),
                                 seed=seed, chain0=11 + lo, topk=k))
    for steps in (5, 1, 3):
        thr = P.at_sa_thresholds(seed, 11, n, base, steps)
        best = torch.zeros((n, k, 4), dtype=torch.int32, device=DEV)
        trace = torch.zeros((n, steps, 4), dtype=torch.int32, device=DEV)
        P.at_sa_run_traced(sp, ens, ch, steps, torch.from_numpy(thr).to(DEV), best, trace)
        torch.cuda.synchronize()
        tr, top = P.entries(trace), P.entries(best)
        for (lo, hi), oc in zip(cuts, och):
            otr = oc.run(tables, steps, oracle.thresholds(seed, 11 + lo, hi - lo, base, steps), trace=True)
            assert np.array_equal(tr["cfg"][lo:hi], otr["cfg"])
            assert np.array_equal(tr["score"][lo:hi].view(np.uint32), otr["score"].view(np.uint32))
            assert np.array_equal(tr["flag"][lo:hi], otr["valid"])
            assert np.array_equal(top["cfg"][lo:hi], oc.top["cfg"])
            assert np.array_equal(top["flag"][lo:hi], oc.top["valid"])
            assert np.array_equal(top["score"][lo:hi].view(np.uint32), oc.top["score"].view(np.uint32))
        base += steps
    plan = P.at_chains_last_plan(ch)
    streams, gather = FORMS[form]
    assert plan["path"] == P.AT_SA_PATH_LOCAL
    assert plan["chains_per_wg"] == (8 if n <= 2048 else 16 if n <= 4096 else 32)
    assert (plan["chunks"] > 1) == streams and plan["gather"] == gather
    if not streams:
        assert (plan["trees_per_chunk"] < trees) == (form == "resident chunks")

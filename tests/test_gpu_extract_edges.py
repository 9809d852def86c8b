"""GPU parity of the feature rows at the edges of the extraction kernels'
64-row workgroups: partial workgroups, out-of-range indices in them, rows
whose length is no multiple of four, unaligned outputs, every row form and
template."""
import numpy as np
import pytest

import oracle
import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CONV = (1, 6, 9, 7, 12, 3, 5, 1, 2)
GEMM = (48, 30, 14)


@pytest.fixture(scope="module")
def P():
    import torch
    torch.cuda.set_device(0)
    import paper_1805_08166_amd
    return paper_1805_08166_amd


@pytest.mark.parametrize("tmpl,shape", [(0, GEMM), (1, CONV), (2, GEMM), (3, CONV)])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 130])
def test_rows_at_workgroup_edges(P, tmpl, shape, n):
    import torch
    print(f"[gpu-extract] template {tmpl} n {n}", flush=True)
    sp, osp = P.at_space_create(tmpl, shape), oracle.Space(tmpl, shape)
    cfgs = W.make_configs(n, osp.n_configs, 40 + n)
    bad = np.zeros(n, bool)
    bad[[0, n // 2, n - 1]] = n > 1
    cfgs[bad] = [osp.n_configs, np.uint64(2 ** 40), np.uint64(2 ** 63)][: int(bad.sum())]
    good = cfgs.copy()
    good[bad] = 0
    d = torch.from_numpy(cfgs.view(np.int64)).to(DEV)
    forms = [(P.at_extract_features, osp.features, sp.n_features),
             (P.at_extract_features_full, osp.features_full, 13 * sp.n_loops),
             (P.at_extract_features_onehot, osp.features_onehot, 24 * sp.n_loops),
             (P.at_extract_relation_features, osp.relation_features, 192)]
    for f, ref, width in forms:
        want = ref(good).astype(np.int64)
        want[bad] = -1
        for offset in ((0,) if width == 192 else (0, 1)):   # relation rows must be 16-byte aligned
            buf = torch.full((n * width + 8,), -7, dtype=torch.int32, device=DEV)
            f(sp, d, buf[offset: offset + n * width].view(n, width))
            got = buf.cpu().numpy()
            assert np.array_equal(got[offset: offset + n * width].reshape(n, width), want)
            assert (got[:offset] == -7).all() and (got[offset + n * width:] == -7).all()
            assert P.at_space_errors(sp) == int(bad.sum())


@pytest.mark.parametrize("tmpl,shape,form,width", [(1, CONV, "full", 208), (1, CONV, "relation", 192), (0, GEMM, "onehot", 240)])
def test_rows_past_the_caches(P, tmpl, shape, form, width):
    """Outputs above 320 MB, whose blocks an XCD takes 16 at a time, the last
    blocks of the grid in order: every row is written, and by its own block
    (the rows of the same indices in calls below that size)."""
    import torch
    n = (320 << 20) // (4 * width) // 64 * 64 + 64 * 37 + 5
    print(f"[gpu-extract] template {tmpl} {form} n {n}", flush=True)
    sp = P.at_space_create(tmpl, shape)
    f = {"full": P.at_extract_features_full, "onehot": P.at_extract_features_onehot,
         "relation": P.at_extract_relation_features}[form]
    cfgs = torch.randint(0, sp.n_configs, (n,), dtype=torch.int64, device=DEV)
    out = torch.full((n, width), -7, dtype=torch.int32, device=DEV)
    f(sp, cfgs, out)
    part = 100003
    for lo in range(0, n, part):
        c = cfgs[lo: lo + part].clone()
        want = torch.full((len(c), width), -9, dtype=torch.int32, device=DEV)
        f(sp, c, want)
        assert torch.equal(out[lo: lo + part], want)

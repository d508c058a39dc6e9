"""Thin-film queries in batches by kind: the same bits whatever the order of
the queries, at the edges of batches (64), of a workgroup's chunk (2048) and
beyond one chunk per workgroup, with invalid queries among them, and for a
stack that leaves no room for the chunk's list."""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu

CASES = [(n, 31, p) for p in (0, 1, 2) for n in (1, 63, 65, 257, 2049, 70001)] + [(1300, 3440, 0), (1300, 3440, 1)]


@pytest.mark.parametrize("n,L,precision", CASES)
def test_tmm_independent_of_query_order(gctx, n, L, precision):
    rng = np.random.default_rng(n + L)
    lam = np.array([450.0, 633.0])
    # glass, silica, silver: the long stack of one lossless material
    n_re = np.array([[1.9, 1.46, 0.05], [1.9, 1.46, 0.06]])
    n_im = np.array([[0.0, 0.0, 2.4], [0.0, 0.0, 4.2]])
    mat = np.ones(L, np.uint8)
    if L < 1000:
        mat[1::2] = 0
        mat[L // 2] = 2
    thk = torch.tensor(rng.uniform(0.05, 120.0 if L < 1000 else 1.0, L), device="cuda:0")
    th = rng.uniform(0.0, 1.5, n)
    th[rng.random(n) < 0.1] = np.arcsin(1.46 / 1.9)          # near critical
    th[rng.random(n) < 0.02] = 1.7                           # no such angle
    li = rng.integers(0, 2, n).astype(np.int32)
    li[rng.random(n) < 0.02] = 5                             # no such wavelength
    print(f"tmm order n={n} L={L} precision={precision}", flush=True)

    def run(idx):
        return gctx.tmm_rt(thk, mat, 0, 0, lam, n_re, n_im, torch.tensor(li[idx]), torch.tensor(th[idx]),
                           precision).cpu().numpy()

    a = run(np.arange(n))
    bad = (li > 1) | (th > np.pi / 2)
    assert np.all(np.isnan(a[bad])) and not np.any(np.isnan(a[~bad]))
    for perm in (rng.permutation(n), np.argsort(th, kind="stable")):
        assert np.array_equal(run(perm).view(np.uint64), a[perm].view(np.uint64))

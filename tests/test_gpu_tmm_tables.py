"""Thin-film queries over many wavelengths: the call enqueues and returns
(header: asynchronous), its results are those of one call per wavelength bit
for bit, whether the tables travel with the launch (up to 31 wavelengths of
long stacks) or are copied, and whether queries are solved in order or by kind
(mixed precision; lossless stacks in double precision where the launch has
more queries than run at once: 131072 lanes of 256 CUs)."""
import time

import numpy as np
import pytest
import torch

import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu


def _queries(n, n_lam, L, ag, seed):
    rng = np.random.default_rng(seed)
    lam = 400.0 + 300.0 * np.arange(n_lam) / max(n_lam - 1, 1)
    # glass, silica (crosses the critical angle), titania, alumina, silver
    n_re = np.tile([1.52, 1.46, 2.35, 1.63, 0.12], (n_lam, 1)) + 0.01 * (550.0 / lam[:, None] - 1.0)
    n_im = np.tile([0.0, 0.0, 0.0, 0.0, 3.3], (n_lam, 1))
    mat = (1 + np.arange(L) % 3).astype(np.uint8)
    if ag:
        mat[L // 2] = 4
    thk = torch.tensor(rng.uniform(1.0, 200.0, L), device="cuda:0")
    li = torch.tensor(rng.integers(0, n_lam, n).astype(np.int32), device="cuda:0")
    th = torch.tensor(rng.uniform(0.0, 1.5, n), device="cuda:0")
    return thk, mat, lam, n_re, n_im, li, th


@pytest.mark.parametrize("n_lam,L,ag,precision", [(9, 8, False, 0), (9, 40, True, 1), (31, 400, True, 1), (31, 250, False, 2)])
def test_calls_of_many_wavelengths_do_not_wait(gctx, n_lam, L, ag, precision):
    thk, mat, lam, n_re, n_im, li, th = _queries(64, n_lam, L, ag, 1)
    call = lambda: gctx.tmm_rt(thk, mat, 0, 0, lam, n_re, n_im, li, th, precision)   # noqa: E731
    want = call()
    torch.cuda.synchronize()
    took = []
    for f in (torch.cuda.synchronize, call):                 # waiting for the stream; the call
        torch.cuda._sleep(40_000_000)
        t = time.perf_counter()
        got = f()
        took.append(time.perf_counter() - t)
        torch.cuda.synchronize()
    print(f"stream busy for {took[0]:.4f} s, call {took[1]:.4f} s", flush=True)
    assert took[0] > 2e-3, "the stream was not kept busy"
    assert took[1] < 0.5 * took[0], "the call waited for the stream"
    assert torch.equal(torch.view_as_real(got), torch.view_as_real(want))


@pytest.mark.parametrize("n,n_lam,L,ag,precision", [
    (3000, 1, 8, True, 1), (3000, 9, 40, True, 1), (3000, 31, 400, True, 1), (3000, 300, 5, False, 1), (3000, 300, 5, True, 0),
    (131072, 3, 33, False, 0), (131073, 3, 32, False, 0), (140001, 9, 31, False, 0), (150000, 9, 12, True, 1),
    (150000, 9, 12, False, 2), (140001, 3, 40, True, 0)])
def test_wavelengths_together_equal_one_by_one(gctx, n, n_lam, L, ag, precision):
    thk, mat, lam, n_re, n_im, li, th = _queries(n, n_lam, L, ag, n + n_lam)
    print(f"tmm tables n={n} wavelengths={n_lam} L={L} ag={ag} precision={precision}", flush=True)
    got = gctx.tmm_rt(thk, mat, 0, 0, lam, n_re, n_im, li, th, precision)
    assert not torch.isnan(torch.view_as_real(got)).any()
    for k in range(0, n_lam, 1 + n_lam // 40):
        sel = (li == k).nonzero().flatten()
        # descending angles: other waves, other batches
        sel = sel[torch.argsort(th[sel], descending=True)]
        one = gctx.tmm_rt(thk, mat, 0, 0, lam[k:k + 1], n_re[k:k + 1], n_im[k:k + 1], torch.zeros_like(li[sel]), th[sel],
                          precision)
        assert torch.equal(torch.view_as_real(one), torch.view_as_real(got[sel]))

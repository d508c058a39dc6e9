"""A layer material that absorbs at some wavelengths of the table and not at
others: coefficients, traces and gradients at every wavelength against the
oracle.  Tolerances are those of the tests of absorbing stacks: 1e-11 for
coefficients and weights, 1e-9 of the largest gradient."""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg
from inputs import MAT_AG, MAT_GLASS

pytestmark = pytest.mark.gpu

LAMS = (430.0, 530.0, 640.0)


def _indices(inp, above):
    """MAT_AG's place: absorbing at the first wavelength only; its index at the
    others above or below the glass's (evanescent layers among the hits)."""
    inp["n_re"][:, MAT_AG] = (0.8, 1.9, 2.1) if above else (0.8, 1.4, 1.3)
    inp["n_im"][:, MAT_AG] = (1.7, 0.0, 0.0)


@pytest.mark.parametrize("above", [True, False])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_coefficients(gctx, orc, above, precision):
    w = inputs.small_variant("diff_1200", n_layers=21, lambdas_nm=LAMS)
    inp = inputs.make_inputs(w)
    _indices(inp, above)
    mat, thk = inp["mat"][0, 0].copy(), inp["thk"][0, 0].copy()
    mat[7] = mat[15] = MAT_AG
    thk[7], thk[15] = 35.0, 60.0
    rng = np.random.default_rng(2)
    n = 600
    li = rng.integers(0, 3, n).astype(np.int32)
    th = rng.uniform(0.0, 1.45, n)
    nre, nim, lam = inp["n_re"], inp["n_im"], inp["lambda_nm"]
    got = gctx.tmm_rt(torch.tensor(thk), mat, MAT_GLASS, MAT_GLASS, lam, nre, nim, torch.tensor(li), torch.tensor(th),
                      precision).cpu().numpy()
    err = np.zeros(n)
    for q in range(n):
        l = li[q]
        ref = orc.tmm_rt(thk, nre[l, mat] + 1j * nim[l, mat], nre[l, MAT_GLASS], nre[l, MAT_GLASS] + 0j, lam[l], theta=th[q])
        err[q] = np.max(np.abs(got[q] - ref)) / max(1.0, np.max(np.abs(ref)))
    print(f"above={above} precision={precision}: max error {err.max():.1e}, median {np.median(err):.1e}", flush=True)
    if precision == 0:
        assert err.max() <= 1e-11
    else:                                                    # single precision: the bulk (as for silver stacks)
        assert np.median(err) <= 1e-4


@pytest.mark.parametrize("above", [True, False])
def test_trace_and_gradient(gctx, orc, above):
    w = inputs.small_variant("diff_1200", n_layers=9, lambdas_nm=LAMS, fov_n=2, rays_per_point=150)
    inp = inputs.make_inputs(w)
    _indices(inp, above)
    inp["mat"][:, 1::2, 4] = MAT_AG
    inp["thk"][:, 1::2, 4] = 25.0
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    dLdI = np.random.default_rng(4).standard_normal(scene.shape)
    print(f"partial absorption above={above}", flush=True)
    osc = orc.OracleScene(w, inp, step=1)
    orec = osc.trace_rays(np.arange(w.n_rays))
    ow = np.array([r.w for r in orec])
    og = osc.backward(dLdI, 1)
    scale = np.max(np.abs(og))
    assert scale > 0
    for mode in ("hit", "memo", "regenerated"):
        _, _, _, rec, _ = gctx.trace_forward(scene, thk, w.seed, 1, 0, record_stride=1, grad=mode != "regenerated",
                                             memo=mode == "memo")
        rec = gwg.records_view(rec)
        g = gctx.trace_backward(torch.tensor(dLdI), scene).cpu().numpy()
        assert np.array_equal(rec["bin"], [r.bin for r in orec])
        assert np.max(np.abs(rec["w"] - ow)) <= 1e-11 * max(1.0, ow.max()), mode
        assert np.max(np.abs(g - og)) <= 1e-9 * scale, mode

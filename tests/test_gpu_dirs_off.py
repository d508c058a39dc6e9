"""Rays that leave the direction table (test_dir_tree_cpu.py shows that the scenes
have them).

- Beams that meet the first mirror within 1e-4 of normal incidence (|d x n|
  from 0 to 1e-4: the general walk takes over at the hit) and just above it;
- beams with more directions than the table keeps (64): the deepest reflections
  walk in general.

Against the oracle: paths, bins and categories equal, weights to 1e-11 (the
mirror basis is undetermined at normal incidence, but the coefficients of s and
p then agree to |d x n|^2, so its rounding, 2^-53 / |d x n|, drops out), the
gradient to 1e-9 of its largest component, the reflection-probability gradient
to 1e-11."""
import functools

import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg
from tests.dir_tree import off_table_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["normal_incidence", "many_directions"])
def test_rays_off_the_table_match_oracle(gctx, orc, name):
    w, inp, ng, fov = off_table_case(name)
    print(f"off the table: {name}", flush=True)
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    dLdI = np.random.default_rng(8).standard_normal(scene.shape)
    osc = orc.OracleScene(w, inp, step=1)
    n = len(fov) * w.rays_per_point
    osc.events = functools.partial(osc.events, cap=w.max_events)     # the score estimator asks for 64
    orec = osc.trace_rays(np.arange(n))
    ow = np.array([r.w for r in orec])
    og = osc.backward(dLdI, 1)
    scale = np.max(np.abs(og))
    hit = np.array([r.n_prma > 0 and r.bin >= 0 for r in orec]).reshape(len(fov), -1)
    assert np.all(hit.sum(1) > 10) and scale > 0             # mirrors met on the way to a bin, from every point
    for mode in ("hit", "memo", "regenerated"):
        _, c, _, rec, _ = gctx.trace_forward(scene, thk, w.seed, 1, 0, record_stride=1, grad=mode != "regenerated",
                                             memo=mode == "memo")
        rec = gwg.records_view(rec)
        W = np.random.default_rng(3).uniform(-1.0, 2.0, scene.shape)
        om = gctx.omega_gradient(torch.tensor(W), c, scene).cpu().numpy()
        g = gctx.trace_backward(torch.tensor(dLdI), scene).cpu().numpy()
        assert np.array_equal(rec["bin"], [r.bin for r in orec]), mode
        assert np.array_equal(rec["category"], [r.category for r in orec]), mode
        assert np.array_equal(rec["n_events"], [r.n_events for r in orec]), mode
        assert np.max(np.abs(rec["w"] - ow)) <= 1e-11 * max(1.0, ow.max()), mode
        assert np.max(np.abs(g - og)) <= 1e-9 * scale, mode
        oom, _ = orc.omega_score_gradient(osc, W, c.cpu().numpy())
        print(f"  {mode}: reflection-probability gradient {om}, largest difference {np.max(np.abs(om - oom)):.1e}", flush=True)
        assert np.allclose(om, oom, rtol=1e-11, atol=1e-13 * np.abs(oom).max()), mode
    gctx.set_tuning(table_nodes=128)
    try:
        _, _, _, rec, _ = gctx.trace_forward(scene, thk, w.seed, 1, 0, record_stride=1, table=True, grad=True)
        g = gctx.trace_backward(torch.tensor(dLdI), scene).cpu().numpy()
    finally:
        gctx.set_tuning()
    tsc = orc.OracleScene(w, inp, table_nodes=128, step=1)
    tw = np.array([r.w for r in tsc.trace_rays(np.arange(n))])
    assert np.max(np.abs(gwg.records_view(rec)["w"] - tw)) <= 1e-10 * max(1.0, np.max(np.abs(tw)))
    tg = tsc.backward(dLdI, 1)
    assert np.max(np.abs(g - tg)) <= 1e-9 * np.max(np.abs(tg))

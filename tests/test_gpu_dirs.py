"""Direction states of collimated beams: scenes at the edges of what the
per-point direction table holds, against the oracle's general walk.

- many mirrors close together: long paths and more directions than the table
  keeps (rays that leave it walk in general);
- tilts at which beams meet the mirrors near normal incidence, run nearly
  parallel to the faces, or leave along the face normal (basis fallbacks);
- one field point, one ray per point, one event, the largest event count;
- more eyebox bins than a workgroup keeps in LDS.

Paths, bins and categories are equal; weights agree to the rounding of two
double-precision formulations (as in the full-size comparisons: 1e-11).
"""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu

SCENES = {
    "many_mirrors": dict(n_mirrors=16, pitch_mm=1.3, n_layers=3, max_events=256, fov_n=3, rays_per_point=300),
    "normal_incidence": dict(tilt_deg=12.5, n_layers=5, fov_n=3, rays_per_point=200),
    "along_the_slab": dict(tilt_deg=45.0, n_layers=5, fov_n=3, rays_per_point=150),
    "steep": dict(tilt_deg=38.0, n_layers=4, fov_n=2, rays_per_point=150),
    "one_field_point": dict(fov_n=1, n_layers=7, rays_per_point=700),
    "one_ray": dict(fov_n=2, n_layers=2, rays_per_point=1),
    "one_event": dict(fov_n=2, n_layers=2, rays_per_point=65, max_events=1),
    "many_bins": dict(fov_n=2, n_layers=3, rays_per_point=257, bins=(64, 40)),
}


def _trace(gctx, w, inp, **kw):
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    q, c, irr, rec, st = gctx.trace_forward(scene, thk, w.seed, 1, 0, record_stride=1, stats=True, **kw)
    return scene, thk, q.cpu().numpy(), c.cpu().numpy(), gwg.records_view(rec), st


@pytest.mark.parametrize("name", list(SCENES))
def test_direction_table_edges_match_oracle(gctx, orc, name):
    w = inputs.small_variant("diff_1200", lambdas_nm=(460.0, 620.0), **SCENES[name])
    inp = inputs.make_inputs(w)
    print(f"directions {name} {SCENES[name]}", flush=True)
    osc = orc.OracleScene(w, inp, step=1)
    scene, thk, q, c, rec, st = _trace(gctx, w, inp, grad=True)
    L, dLdI = gctx.loss(torch.tensor(q.astype(np.float64) * 2.0 ** -24 / w.rays_per_point), 0)
    g = gctx.trace_backward(dLdI, scene).cpu().numpy()
    orec = osc.trace_rays(np.arange(w.n_rays))
    ow = np.array([r.w for r in orec])
    assert np.array_equal(rec["bin"], [r.bin for r in orec])
    assert np.array_equal(rec["category"], [r.category for r in orec])
    assert np.array_equal(rec["n_events"], [r.n_events for r in orec])
    assert np.array_equal(rec["n_prma"], [r.n_prma for r in orec])
    assert np.max(np.abs(rec["w"] - ow)) <= 1e-11 * max(1.0, ow.max())
    assert st["interactions"] == sum(r.n_events for r in orec) and st["rays"] == w.n_rays
    og = osc.backward(dLdI.cpu().numpy(), 1)
    assert np.max(np.abs(g - og)) <= 1e-9 * max(np.max(np.abs(og)), 1e-300)
    # each key's coefficients solved once: the per-hit bits
    _, _, qm, cm, recm, _ = _trace(gctx, w, inp, memo=True)
    assert np.array_equal(qm, q) and np.array_equal(cm, c) and np.array_equal(recm["w"], rec["w"])
    # plain forward: the same as with the gradient flag
    _, _, qp, cp, _, _ = _trace(gctx, w, inp)
    assert np.array_equal(qp, q) and np.array_equal(cp, c)
    # angle table: keys against the oracle's per-hit interpolation
    gctx.set_tuning(table_nodes=128)
    try:
        _, _, _, ct, rect, _ = _trace(gctx, w, inp, table=True)
    finally:
        gctx.set_tuning()
    assert np.array_equal(ct, c) and np.array_equal(rect["bin"], rec["bin"])
    tsc = orc.OracleScene(w, inp, table_nodes=128, step=1)
    tw = np.array([r.w for r in tsc.trace_rays(np.arange(w.n_rays))])
    assert np.max(np.abs(rect["w"] - tw)) <= 1e-10 * max(1.0, np.max(np.abs(tw)))

"""Keyed gradients: entries that carry their key's slot, summed per item and
(memoized) per field point, at the edges of the key tables.

- items of one wave, many items to a point, a last item that is nearly empty;
- key tables so small that some or all items have no keys (they are searched),
  and entry regions so small that items are regenerated;
- more keys in a point than are gathered at a time, rays off the direction
  table.

The sums have n terms of one sign or the other in a different order than hit
by hit: n eps of the summed magnitudes, for n <= 2^16 below 1e-10 of the larger
of the value and 1e-3 of the largest gradient (the bound of the full-size
comparisons).  The angle table's sums are 64-bit fixed point: 1e-9 of the
largest gradient covers their last bits.
"""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu

CASES = {
    "many_items": (dict(rays_per_point=641, n_layers=9, fov_n=2), dict(rays_per_block=64)),
    "one_item": (dict(rays_per_point=300, n_layers=5, fov_n=3), dict(rays_per_block=4096)),
    "some_without_keys": (dict(rays_per_point=900, n_layers=6, fov_n=2), dict(rays_per_block=64, memo_keys=24)),
    "none_with_keys": (dict(rays_per_point=200, n_layers=4, fov_n=2), dict(rays_per_block=64, memo_keys=1)),
    "regions_overflow": (dict(rays_per_point=700, n_layers=4, fov_n=2), dict(rays_per_block=128, adj_entries_per_ray=3)),
    "many_keys": (dict(n_mirrors=16, pitch_mm=1.3, n_layers=3, max_events=256, fov_n=2, rays_per_point=700),
                  dict(rays_per_block=64)),
    "no_layers": (dict(rays_per_point=65, n_layers=1, fov_n=2), dict(rays_per_block=64)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_keyed_gradient_edges(gctx, name):
    kw, tune = CASES[name]
    w = inputs.small_variant("diff_1200", lambdas_nm=(460.0, 620.0), **kw)
    inp = inputs.make_inputs(w)
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    print(f"keyed {name} {kw} {tune}", flush=True)
    dLdI = torch.tensor(np.random.default_rng(3).standard_normal(scene.shape), device="cuda:0")
    dLdI[:, :, 0, ::3] = 0.0                               # bins without a gradient
    out = {}
    for mode in ("hit", "memo", "table", "table_regen"):
        extra = {k: v for k, v in tune.items() if mode != "table_regen" or k == "rays_per_block"}
        if mode == "table_regen":
            extra["adj_entries_per_ray"] = 1
        gctx.set_tuning(table_nodes=512, **extra)
        try:
            gctx.trace_forward(scene, thk, w.seed, 2, 0, grad=True, memo=mode == "memo", table=mode.startswith("table"))
            a, st = gctx.trace_backward(dLdI, scene, stats=True)
            b = gctx.trace_backward(dLdI, scene)
        finally:
            gctx.set_tuning()
        assert torch.equal(a, b)
        print(f"  {mode}: adjoints {st['adjoint_hits']}, regenerated rays {st['rays']}", flush=True)
        out[mode] = a.cpu().numpy()
    scale = np.max(np.abs(out["hit"]))
    assert scale > 0
    assert np.all(np.abs(out["memo"] - out["hit"]) <= 1e-10 * np.maximum(np.abs(out["hit"]), 1e-3 * scale))
    assert np.max(np.abs(out["table"] - out["table_regen"])) <= 1e-9 * np.max(np.abs(out["table"]))

"""Sorted adjoint of lossless stacks: layer counts at the ends of segments and
half segments (24 and 48 layers), of the eight staged layers and of the
pipelined reads, every mirror of the largest scene, batches of a few entries
and of many, groups of one and of several items.

Against the oracle's adjoint: both are double precision, and a gradient entry
sums up to 1e4 hits' terms; 1e-9 of the largest entry is far above their
rounding and far below a wrong layer or a lost batch.
"""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu

CASES = [(n, dict(fov_n=2, rays_per_point=130), {}) for n in (1, 2, 3, 7, 9, 24, 25, 47, 49, 73, 97, 145)] + [
    (5, dict(fov_n=3, rays_per_point=65, n_mirrors=16, pitch_mm=1.3), {}),
    (50, dict(fov_n=3, rays_per_point=1), {}),
    (26, dict(fov_n=2, rays_per_point=700), dict(rays_per_block=64)),
    (26, dict(fov_n=2, rays_per_point=700), dict(rays_per_block=64, ck_entries_per_ray=-1)),
    (26, dict(fov_n=2, rays_per_point=700), dict(rays_per_block=1024, adj_entries_per_ray=2)),
]


@pytest.mark.parametrize("n_layers,kw,tune", CASES)
def test_sorted_adjoint_matches_oracle(gctx, orc, n_layers, kw, tune):
    w = inputs.small_variant("diff_1200", n_layers=n_layers, lambdas_nm=(430.0, 640.0), **kw)
    inp = inputs.make_inputs(w)
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    print(f"sorted adjoint L={n_layers} {kw} {tune}", flush=True)
    dLdI = np.random.default_rng(7).standard_normal(scene.shape)
    gctx.set_tuning(**tune)
    try:
        gctx.trace_forward(scene, thk, w.seed, 1, 0, grad=True)
        g, st = gctx.trace_backward(torch.tensor(dLdI), scene, stats=True)
    finally:
        gctx.set_tuning()
    og = orc.OracleScene(w, inp, step=1).backward(dLdI, 1)
    scale = np.max(np.abs(og))
    err = np.max(np.abs(g.cpu().numpy() - og))
    print(f"  hits {st['adjoint_hits']}, max |g| {scale:.3e}, error {err / max(scale, 1e-300):.1e}", flush=True)
    assert err <= 1e-9 * scale


# stacks with absorbing layers: (layers, positions of silver)
SILVER = {
    "first_and_last": (27, (0, 26)),
    "neighbours": (30, (10, 11, 12)),
    "after_a_whole_run": (50, (24, 49)),
    "before_a_whole_run": (49, (0, 25)),
    "runs_of_one": (9, (1, 3, 5, 7)),
    "only": (1, (0,)),
    "all": (6, tuple(range(6))),
    "as_many_pieces_as_are_kept": (32, tuple(range(0, 32, 2))),
    "one_piece_more": (33, tuple(range(0, 33, 2))),
}


@pytest.mark.parametrize("name", list(SILVER))
def test_sorted_adjoint_with_absorbing_layers(gctx, orc, name):
    """Pieces of stacks with silver layers (up to 32 pieces; with one more the
    general adjoint).  Silver damps what passes it, so gradients of a
    formulation and of the oracle's agree to 1e-9 of the largest."""
    n_layers, silver = SILVER[name]
    w = inputs.small_variant("diff_1200", n_layers=n_layers, lambdas_nm=(430.0, 640.0), fov_n=2, rays_per_point=200)
    inp = inputs.make_inputs(w)
    for j in silver:
        inp["mat"][:, ::2, j] = inputs.MAT_AG               # every other mirror: the others stay lossless
        inp["thk"][:, ::2, j] = 4.0 + j % 3
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    print(f"silver {name} L={n_layers}", flush=True)
    dLdI = np.random.default_rng(9).standard_normal(scene.shape)
    gctx.trace_forward(scene, thk, w.seed, 1, 0, grad=True)
    g = gctx.trace_backward(torch.tensor(dLdI), scene).cpu().numpy()
    og = orc.OracleScene(w, inp, step=1).backward(dLdI, 1)
    scale = np.max(np.abs(og))
    assert scale > 0
    err = np.max(np.abs(g - og))
    print(f"  max |g| {scale:.3e}, error {err / scale:.1e}", flush=True)
    assert err <= 1e-9 * scale

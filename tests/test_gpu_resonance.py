"""Gradients of reflected hits near a resonance: mirrors coated with a half-wave
cavity between two quarter-wave stacks of 20 pairs, 1 to 10 pm off its
resonance at the mirrors' first incidence (kappa = n_glass sin 25 deg).  On its
way from the exit to the incident side the state grows to the cavity and shrinks
again; what a backward carries through the layers must not keep the rounding of
its largest value squared.

The backward over stored entries against the one that traces the paths again,
which forms every 16 layers anew from the state there.  Both solve the same hits
with the same kappa.  A hit's own conditioning is the rounding of a phase over
the distance from the resonance in relative wavelength, 2^-53 / (1e-3 nm / 530
nm) = 6e-11 of its largest gradient at 1 pm, and less further off; thirty times
that, 2e-9, leaves room for some hundred hits whose gradients cancel in part.
(The oracle's sums differ by more: its rays' fields, which weigh the hits, pass
the same resonances in another formulation.)"""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg
from inputs import MAT_GLASS, MAT_SIO2, MAT_TIO2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pm", [1.0, 3.0, 10.0])
@pytest.mark.parametrize("stored", [True, False])
def test_gradient_off_a_cavity_resonance(gctx, pm, stored):
    w = inputs.small_variant("diff_1200", lambdas_nm=(530.0 + 1e-3 * pm,), n_layers=81, fov_n=1, rays_per_point=400)
    inp = inputs.make_inputs(w)
    kap = inp["n_re"][0, MAT_GLASS] * np.sin(np.radians(w.tilt_deg))
    side = [MAT_TIO2, MAT_SIO2] * 20
    mats = np.array(side + [MAT_TIO2] + side[::-1], dtype=np.uint8)
    n = inp["n_re"][0, mats]
    thk_q = 530.0 / (4.0 * np.sqrt(n * n - kap * kap))
    thk_q[40] *= 2.0
    inp["mat"][0, :, :], inp["thk"][0, :, :] = mats, thk_q
    scene = gwg.SceneSpec.from_workload(w, inp)
    thk = torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")
    dLdI = torch.tensor(np.random.default_rng(6).standard_normal(scene.shape))
    gctx.set_tuning(ck_entries_per_ray=0 if stored else -1)
    try:
        gctx.trace_forward(scene, thk, w.seed, 1, 0, grad=True)
        g = gctx.trace_backward(dLdI, scene).cpu().numpy()
    finally:
        gctx.set_tuning()
    gctx.trace_forward(scene, thk, w.seed, 1, 0)
    ref = gctx.trace_backward(dLdI, scene).cpu().numpy()
    scale = np.max(np.abs(ref))
    assert scale > 0
    err = np.max(np.abs(g - ref)) / scale
    print(f"{pm} pm off, stored={stored}: largest gradient {scale:.3e}, difference {err:.1e}", flush=True)
    assert err <= 2e-9 / pm

"""The autotuner tries the configuration that an untuned forward takes, so it can
never choose a slower one: small launches, memoized ones, and large ones."""
import pytest

from tests.host_only import run

SCENES = {
    "one_small_point": dict(fov_n=1, rays_per_point=2048, n_layers=8),
    "some_small_points": dict(fov_n=3, rays_per_point=300, n_layers=40, lambdas_nm=tuple(400.0 + 30.0 * k for k in range(9))),
    "a_wave_per_simd": dict(fov_n=3, rays_per_point=2048, n_layers=40),
    "more": dict(fov_n=5, rays_per_point=8192, n_layers=40),
    "whole_points": dict(fov_n=21, rays_per_point=8192, n_layers=20, n_designs=8),
}


@pytest.mark.parametrize("name", list(SCENES))
@pytest.mark.parametrize("grad,memo", [(False, False), (True, False), (False, True), (True, True)])
def test_autotune_tries_the_automatic_configuration(name, grad, memo):
    out = run(f"""
sc = h.scene(**{SCENES[name]!r})
assert h.forward(sc, grad={grad}, memo={memo}) == 0, h.error()
k = h.kernels('k_trace_fwd')[-1]
out['auto'] = [k[2], int(k[3]['rays'])]
out['memo'] = int(k[3]['memo'])
rc, t = h.autotune(sc, grad={grad}, memo={memo})
out['rc'] = rc
out['tried'] = [[k[2], int(k[3]['rays'])] for k in h.kernels('k_trace_fwd')]
""")
    assert out["rc"] == 0 and (out["memo"] > 0) == memo
    assert out["auto"] in out["tried"]
    assert {b for b, _ in out["tried"]} == {128, 256}

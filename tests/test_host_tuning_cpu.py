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


# per-hit forwards: rounds of a tile by points and rays (512 workgroups run at
# once); the items of a launch that fits one pass are as small as they get
@pytest.mark.parametrize("fov_n,n_lam,rays,rounds", [
    (1, 1, 100000, 1), (1, 1, 131072, 1), (5, 3, 8192, 2), (1, 1, 1000000, 2), (1, 9, 116500, 2), (1, 3, 174700, 2),
    (1, 1, 4000000, 4), (11, 3, 250, 1)])
@pytest.mark.parametrize("grad", [False, True])
def test_rounds_of_forward_tiles(fov_n, n_lam, rays, rounds, grad):
    out = run(f"""
sc = h.scene(fov_n={fov_n}, rays_per_point={rays}, n_layers=8, lambdas_nm={tuple(400.0 + 10.0 * k for k in range(n_lam))!r})
assert h.forward(sc, grad={grad}) == 0, h.error()
k = h.kernels('k_trace_fwd')[-1]
out['k'] = [k[2], int(k[3]['rays'])]
""")
    threads, tile = out["k"]
    assert threads == 256 and tile == min(256 * rounds, rays)

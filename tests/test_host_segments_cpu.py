"""Which entries' segments the forward keeps in the memory it has: all, not the
evanescent hits', or those of the first items."""
import pytest

from tests.host_only import run


@pytest.mark.parametrize("earlier,n_layers,evan,part", [(80, 97, 0, 1.0), (30, 97, 0, 2 / 3), (5, 97, 0, 1 / 3), (80, 200, 0, 4 / 5),
                                                        (200, 97, 1, 1.0)])
def test_storage_while_capturing(earlier, n_layers, evan, part):
    """The scenes of test_gpu_segments.py."""
    out = run(f"""
kw = dict(lambdas_nm=(430.0, 640.0), fov_n=3, rays_per_point=200)
assert h.forward(h.scene(n_layers={earlier}, **kw), grad=True) == 0
sc = h.scene(n_layers={n_layers}, **kw)
h.tuning(ck_entries_per_ray=-1)
assert h.forward(sc, grad=True) == 0 and h.backward() == 0
assert h.kernels('k_trace_fwd')[-1][3]['ck_regions'] == '0'
h.tuning()
h.fake.fake_capture(1)
assert h.forward(sc, grad=True) == 0, h.error()
out.update({{k: int(v) for k, v in h.kernels('k_trace_fwd')[-1][3].items() if k in ('regions', 'ck_regions', 'ck_nb', 'ck_evan')}})
out['kept'] = h.kept()
assert h.backward() == 0, h.error()
out['sorted'] = len(h.kernels('k_adj_sorted'))
""")
    assert out["kept"] == 1 and out["sorted"] == 1
    assert out["ck_evan"] == evan
    assert out["ck_nb"] == (n_layers // 24 if evan else n_layers // 48) + 1
    assert 0 < out["ck_regions"] <= out["regions"]
    assert abs(out["ck_regions"] / out["regions"] - part) <= 2.0 / out["regions"]

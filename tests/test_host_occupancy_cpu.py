"""Persistent grids are sized by the occupancy of the kernel that is launched, not
of another instance of its template."""
import pytest

from tests.host_only import run

PERSISTENT = ("k_trace_fwd", "k_trace_bwd", "k_adj_sorted", "k_adj_entries", "k_adj_memo", "k_key_adj", "k_omega_grad")


@pytest.mark.parametrize("kw", [dict(), dict(ag_layer_at=4), dict(fov_mode=1, fov_n=1)])
@pytest.mark.parametrize("mode", ["hit", "memo", "table", "regenerated"])
@pytest.mark.parametrize("precision", [0, 1, 2])
def test_grids_are_sized_for_the_launched_kernels(kw, mode, precision):
    out = run(f"""
h.tuning(table_nodes=16)
sc = h.scene(**{dict(dict(fov_n=3, rays_per_point=500, n_layers=9), **kw)!r})
assert h.forward(sc, grad={mode != "regenerated"}, memo={mode == "memo"}, table={mode == "table"}, precision={precision}) == 0, h.error()
assert h.backward() == 0, h.error()
out['names'] = [x[0] for x in h.log()]
out['asked'] = h.asked()
""")
    launched = {n for n in out["names"] if any(k in n for k in PERSISTENT)}
    assert len(launched) >= 2
    assert launched <= set(out["asked"]), launched - set(out["asked"])

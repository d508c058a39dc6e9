"""Buffers that the sorted adjoint adds to the stored entries: where one of them
cannot be allocated the backward traces the paths again, as where the entries
themselves do not fit; no call fails for it."""
import pytest

from tests.host_only import run

STEP = """
sc = h.scene(fov_n=3, rays_per_point=500, n_layers=40)
def step(refuse=None):
    if refuse: h.fake.fake_refuse(refuse, refuse)
    rc = [h.forward(sc, grad=True)]
    kept, fwd = h.kept(), h.sizes()
    h.log()
    rc.append(h.backward())
    bwd = h.sizes()
    return rc, kept, fwd, bwd, [x[0] for x in h.log()]
"""


def _sizes(which):
    out = run(STEP + """
rc, kept, fwd, bwd, _ = step()
assert rc == [0, 0] and kept == 1
out['fwd'], out['bwd'] = fwd, bwd
""")
    if which == "order":                                     # 4 bytes an entry of 48
        return next(n for n in out["fwd"] if n * 12 in out["fwd"])
    rows = [n for n in out["bwd"] if n % (8 * 6 * 40) == 0]
    return max(rows) if which == "rows" else next(n for n in out["bwd"] if n % (4 * 129) == 0)


@pytest.mark.parametrize("which", ["order", "rows", "classes"])
def test_step_without_room_for(which):
    n = _sizes(which)
    out = run(STEP + f"""
rc, kept, _, _, names = step({n})
out['rc'], out['kept'], out['error'] = rc, kept, h.error()
out['sorted'] = sum('k_adj_sorted' in x for x in names)
out['regen'] = sum('k_trace_bwd' in x for x in names)
h.fake.fake_refuse(1, 0)                                     # room again: entries and their sort
rc, kept, _, _, names = step()
out['again'] = [rc, kept, sum('k_adj_sorted' in x for x in names)]
""")
    assert out["rc"] == [0, 0], out["error"]
    assert out["kept"] == (0 if which == "order" else 1) and out["sorted"] == 0 and out["regen"] == 1
    assert out["again"] == [[0, 0], 1, 1]


@pytest.mark.parametrize("mode", ["memo", "table", "hit"])
def test_forward_with_little_memory_for_hit_queues(mode):
    """Pools of several rounds take several times the memory of one: with less
    the forward takes smaller pools."""
    out = run(f"""
kw = dict(fov_n=21, rays_per_point=8192, n_layers=8)
flag = dict(memo={mode == "memo"}, table={mode == "table"})
h.tuning(table_nodes=64)
assert h.forward(h.scene(**kw), **flag) == 0, h.error()
k = h.kernels('k_trace_fwd', clear=False)[-1]
n = max(h.sizes())                                           # the queues
out['pool'] = int(k[3]['pool'])
h2 = type(h)()
h2.fake.fake_clear()
h2.tuning(table_nodes=64)
h2.fake.fake_refuse(n // out['pool'] + n // 16, 1 << 62)     # room for one round, not for two
out['rc'] = h2.forward(h2.scene(**kw), **flag)
out['error'] = h2.error()
out['small'] = [int(x[3]['pool']) for x in h2.kernels('k_trace_fwd')]
""")
    assert out["pool"] >= 4
    assert out["rc"] == 0, out["error"]
    assert out["small"] == [1]


@pytest.mark.parametrize("mode", ["memo", "table"])
def test_keyed_forwards_reserve_no_segment_matrices(mode):
    """Only the per-hit solves store them (25 GB for 1323 points x 8192 rays of 200 layers)."""
    out = run(f"""
sc = h.scene(fov_n=3, rays_per_point=512, n_layers=40)
h.tuning(table_nodes=16, rays_per_block=256)
assert h.forward(sc, grad=True) == 0
out['hit'] = h.sizes()
g = type(h)()
g.fake.fake_clear()
g.tuning(table_nodes=16, rays_per_block=256)
assert g.forward(sc, grad=True, memo={mode == "memo"}, table={mode == "table"}) == 0
out['keyed'] = g.sizes()
""")
    entries = 12 * next(n for n in out["hit"] if n * 12 in out["hit"])      # 8 a ray, 48 bytes
    matrices = entries * 4 * 2 * 64 // (8 * 48)                             # of 4 entries a ray, 2 blocks of 64 bytes
    assert matrices in out["hit"] and entries in out["keyed"]
    assert matrices not in out["keyed"]

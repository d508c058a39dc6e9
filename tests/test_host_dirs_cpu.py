"""Direction tables: one for all scenes with the same directions, within a bound,
and done without where there is no room."""
from tests.host_only import run


def test_scenes_with_the_same_directions_share_a_table():
    """An optimisation of the reflection probabilities and a batch in chunks of
    designs make a scene each iteration or chunk."""
    out = run("""
import numpy as np
used = []
for k in range(12):
    assert h.forward(h.scene(fov_n=21, rays_per_point=64, omega=np.full(6, 0.2 + 0.01 * k))) == 0, h.error()
    used.append(h.fake.fake_used())
for d in range(4):
    s = h.scene(fov_n=21, rays_per_point=64); s.first_design = d
    assert h.forward(s) == 0, h.error()
out['built'] = len(h.kernels('k_dir_states'))
out['grown'] = used[-1] - used[0]
assert h.forward(h.scene(fov_n=21, rays_per_point=64, tilt_deg=26.0)) == 0
out['other'] = len(h.kernels('k_dir_states'))
""")
    assert out["built"] == 1
    assert out["grown"] < 8 << 20                            # 16 MB a table, 1323 points
    assert out["other"] == 1


def test_no_room_for_a_table():
    """The call does without: rays walk in general, memoized solves go hit by hit."""
    out = run("""
n = 1323 * 64 * 24 * 8                                       # a table's bytes
h.fake.fake_refuse(n, n)
out['rc'] = h.forward(h.scene(fov_n=21, rays_per_point=64), memo=True)
k = h.kernels('k_trace_fwd')
out['dirs'], out['memo'] = k[-1][3]['dirs'], int(k[-1][3]['memo'])
h.fake.fake_refuse(1, 0)
s = h.scene(fov_n=21, rays_per_point=65)
out['rc2'] = h.forward(s, memo=True)
out['memo2'] = int(h.kernels('k_trace_fwd')[-1][3]['memo'])
""")
    assert out["rc"] == 0 and out["dirs"] in ("(nil)", "0x0") and out["memo"] == 0
    assert out["rc2"] == 0 and out["memo2"] > 0


def test_tables_are_bounded():
    """288 GiB of memory, scenes of 30000 points (1.1 GB a table): the tables of
    all cached scenes together stay within 32 GiB; a small card keeps most of
    its memory for the rest."""
    out = run("""
import numpy as np
g = np.linspace(-10.0, 10.0, 30000)
fov = np.stack([g, g], 1)
for k in range(40):
    sc = h.scene(fov=fov + 0.01 * k, rays_per_point=1, n_layers=2, bins=(4, 4), lambdas_nm=(450.0, 530.0, 620.0))
    assert h.forward(sc) == 0, h.error()
out['used'] = h.fake.fake_used()
out['memo'] = 0
h.forward(h.scene(fov=fov, rays_per_point=1, n_layers=2, bins=(4, 4), lambdas_nm=(450.0, 530.0, 620.0)), memo=True)
out['memo'] = int(h.kernels('k_trace_fwd')[-1][3]['memo'])
""")
    assert out["used"] < 40 << 30
    assert out["memo"] > 0                                   # 90000 points are memoized
    out = run("""
import numpy as np
h.fake.fake_memory(4 << 30)
g = np.linspace(-10.0, 10.0, 30000)
out['rc'] = h.forward(h.scene(fov=np.stack([g, g], 1), rays_per_point=1, n_layers=2, bins=(4, 4)))
out['dirs'] = h.kernels('k_trace_fwd')[-1][3]['dirs']
""")
    assert out["rc"] == 0 and out["dirs"] in ("(nil)", "0x0")

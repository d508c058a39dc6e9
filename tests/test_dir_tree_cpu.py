"""The scenes of test_gpu_dirs_off.py hold rays that leave the direction table."""
import math

import pytest

from tests.dir_tree import guided, off_table_case, tree

MIRROR = 5


def test_beams_meet_the_first_mirror_near_normal_incidence():
    """|d x n| at the first hit: 0, between 1e-6 and 1e-4 (the general walk's), just above, far above."""
    w, inp, ng, fov = off_table_case("normal_incidence")
    beta = math.radians(w.tilt_deg)
    nx, nz = -math.sin(beta), math.cos(beta)
    first = []
    for x, y in fov:
        d = guided(x, y, ng, nx, nz)
        first.append(math.sqrt((d[1] * nz) ** 2 + (d[2] * nx - d[0] * nz) ** 2 + (d[1] * nx) ** 2))
    assert first[0] < 1e-15 and 1e-6 < first[1] < 1e-4 and 1e-6 < first[2] < 1e-4 and 1e-4 < first[3] < 1e-3
    assert 1e-6 < first[4] < 1e-4 and first[5] > 0.1


@pytest.mark.parametrize("point", [0, 1])
def test_rays_take_directions_beyond_the_kept_ones(orc, point):
    w, inp, ng, fov = off_table_case("many_directions")
    states, _, full = tree(*fov[point], ng, 1.0, w.tilt_deg)
    osc = orc.OracleScene(w, inp, step=1)
    off = 0
    for i in range(w.rays_per_point):
        ev = osc.events(point * w.rays_per_point + i, cap=256)
        off += any((e[5], abs(e[7])) not in states for e in ev if e[0] == MIRROR)
    print(f"point {point}: {len(states)} states, full {full}, {off} of {w.rays_per_point} rays leave")
    assert len(states) == 64 and full
    assert 3 <= off < w.rays_per_point

"""The direction tree of a collimated beam, as the library's per-point table holds
it: replayed on the host (same operations in the same order as k_dir_states)."""
import math

import numpy as np

import inputs
from inputs import MAT_GLASS

KEPT = 64


def guided(thx, thy, ng, nx, nz):
    tx, ty = math.tan(thx * (math.pi / 180.0)), math.tan(thy * (math.pi / 180.0))
    inv = 1.0 / math.sqrt(tx * tx + ty * ty + 1.0)
    ax, ay = tx * inv, ty * inv
    gx, gy, gz = ax / ng, ay / ng, math.sqrt(1.0 - (ax * ax + ay * ay) / (ng * ng))
    t2 = 2.0 * (nx * gx + nz * gz)
    return gx - t2 * nx, gy, gz - t2 * nz


def tree(thx, thy, ng, na, tilt_deg):
    """(states [(dx, |dz|)], smallest |d x n| over the reached (state, sign) pairs, whether the table overflowed)."""
    beta = tilt_deg * (math.pi / 180.0)
    nx, nz = -math.sin(beta), math.cos(beta)
    d = guided(thx, thy, ng, nx, nz)
    dy = d[1]
    states, queue, seen, full = [], [], set(), False

    def state(dx, adz):
        nonlocal full
        if (dx, adz) in states:
            return states.index((dx, adz))
        if len(states) == KEPT:
            full = True
            return -1
        states.append((dx, adz))
        return len(states) - 1

    def push(e, neg):
        if (e, neg) not in seen:
            seen.add((e, neg))
            queue.append((e, neg))

    def reach(e, neg):
        dx = states[e][0]
        push(e, neg)
        if (ng * ng) * (dx * dx + dy * dy) > na * na:
            push(e, 1 - neg)

    low = 1.0
    if d[2] != 0.0:
        reach(state(d[0], abs(d[2])), 1 if d[2] < 0.0 else 0)
    q = 0
    while q < len(queue):
        e, neg = queue[q]
        q += 1
        dx, dz = states[e][0], -states[e][1] if neg else states[e][1]
        low = min(low, math.sqrt((dy * nz) ** 2 + (dz * nx - dx * nz) ** 2 + (dy * nx) ** 2))
        dn = nx * dx + nz * dz
        t2 = 2.0 * dn
        ox, oz = dx - t2 * nx, dz - t2 * nz
        if oz == 0.0:
            continue
        c = state(ox, abs(oz))
        if c >= 0:
            reach(c, 1 if oz < 0.0 else 0)
    return states, low, full


def off_table_case(name):
    if name == "normal_incidence":
        w = inputs.small_variant("diff_1200", lambdas_nm=(460.0,), n_layers=5, rays_per_point=200, center_x_mm=4.0,
                                 pitch_mm=1.0)
        inp = inputs.make_inputs(w)
        ng = inp["n_re"][0, MAT_GLASS]
        th = math.degrees(math.asin(ng * math.sin(math.radians(w.tilt_deg))))
        fov = [(-th, 0.0), (-th + 3e-3, 0.0), (-th + 6e-3, 0.0), (-th + 2e-2, 0.0), (-th, 4e-3), (0.0, 0.0)]
    else:
        w = inputs.small_variant("diff_1200", lambdas_nm=(460.0,), n_layers=3, rays_per_point=1500, n_mirrors=16, pitch_mm=0.4,
                                 center_x_mm=6.0, max_events=256)
        inp = inputs.make_inputs(w)
        ng = inp["n_re"][0, MAT_GLASS]
        fov = [(0.0, 0.0), (-15.0, 15.0)]
    inp["fov"] = np.array(fov)
    inp["eyebox"] = (-20.0, -10.0, 45.0, 20.0)
    return w, inp, ng, fov

"""What the FP64 forward keeps of its sweeps for the adjoint, and how much.

The sorted adjoint reads segment matrices (states of reflected hits) of 48
layers, 24 for hits that meet an evanescent layer.  Where the forward did not
keep an entry's, the adjoint sweeps itself, with the same arithmetic: gradients
are the same bit for bit whatever is kept.  With less memory than the entries
want, evanescent hits go without, then the entries of the later items.  While a
stream captures nothing is allocated, so the memory is what an earlier call
left: that makes the reduced forms here (test_host_segments_cpu.py shows that
these scenes take them).
"""
import numpy as np
import pytest
import torch

import inputs
import paper_2601_04370_amd as gwg

pytestmark = pytest.mark.gpu

KW = dict(lambdas_nm=(430.0, 640.0), fov_n=3, rays_per_point=200)


def _scene(n_layers):
    w = inputs.small_variant("diff_1200", n_layers=n_layers, **KW)
    inp = inputs.make_inputs(w)
    return w, inp, gwg.SceneSpec.from_workload(w, inp), torch.tensor(inp["thk"], dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("n_layers", [23, 24, 25, 47, 48, 49, 71, 72, 73, 95, 96, 97])
def test_kept_and_swept_segments_at_their_boundaries(gctx, orc, n_layers):
    """Layer counts around the ends of one to four segments of either length."""
    w, inp, scene, thk = _scene(n_layers)
    print(f"segments L={n_layers}", flush=True)
    dLdI = np.random.default_rng(5).standard_normal(scene.shape)
    out, stored = [], []
    for per in (-1, 0, 1):
        gctx.set_tuning(ck_entries_per_ray=per)
        try:
            gctx.trace_forward(scene, thk, w.seed, 0, 0, grad=True)
            g, st = gctx.trace_backward(torch.tensor(dLdI), scene, stats=True)
        finally:
            gctx.set_tuning()
        out.append(g.cpu().numpy())
        stored.append(st["adjoint_stored_layer_steps"])
    assert stored[0] == 0 < stored[2] < stored[1]
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    og = orc.OracleScene(w, inp).backward(dLdI, 1)
    assert np.max(np.abs(out[0] - og)) <= 1e-9 * np.max(np.abs(og))


@pytest.mark.parametrize("earlier,n_layers", [(80, 97), (30, 97), (5, 97), (80, 200), (200, 97)])
def test_reduced_storage_gives_the_same_gradient(earlier, n_layers):
    """earlier: layers of the call that sized the memory for what is kept."""
    w, _, scene, thk = _scene(n_layers)
    print(f"reduced storage: sized by {earlier} layers, {n_layers} traced", flush=True)
    dLdI = torch.tensor(np.random.default_rng(5).standard_normal(scene.shape), device="cuda:0")

    def step(ctx):
        ctx.trace_forward(scene, thk, w.seed, 0, 0, grad=True)
        return ctx.trace_backward(dLdI, scene)

    full = gwg.Context(0)
    want = step(full).clone()
    ctx = gwg.Context(0)
    w0, _, scene0, thk0 = _scene(earlier)
    ctx.trace_forward(scene0, thk0, w0.seed, 0, 0, grad=True)
    ctx.set_tuning(ck_entries_per_ray=-1)                    # sizes every other buffer
    assert torch.equal(step(ctx), want)
    ctx.set_tuning()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = step(ctx)
    for k in range(3):
        got.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want), k
    full.close()
    ctx.close()

"""The CFL step is the one of the state the solver holds, however the state got
there: set from the device or the host, left by a step, replayed from a
captured graph, or corrected."""
import numpy as np
import pytest

import paper_2512_13403_amd as mh
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _name(request):
    print(f"\n[gpu case] {request.node.nodeid}", flush=True)
    yield


@pytest.mark.parametrize("where", ["device", "host"])
@pytest.mark.parametrize("dtype,flags", [("f32", mh.SRC_FORCING | mh.SRC_COOLING), ("f64", 0)])
def test_captured_cfl_step_replays_like_plain_steps(dtype, flags, where):
    """One CFL step captured right after a state was set: every replay takes its
    dt from the state it starts from, also after another state was set, with
    eager work between the replays."""
    import torch

    shape = (16, 24, 40)
    grid = mh.grid_desc(shape, (1.0 / 40, 1.0 / 24, 1.0 / 16), dtype=dtype)
    phys = mh.physics_desc(flags=flags)
    td = torch.float64 if dtype == "f64" else torch.float32
    host = [wl.random_state(shape, seed=21 + k, vmax=0.4 + 0.5 * k).astype(
        np.float64 if dtype == "f64" else np.float32) for k in range(3)]
    U = [torch.tensor(h, dtype=td, device="cuda:0") for h in host]
    put = lambda s, k: s.set_state(U[k] if where == "device" else host[k])
    side = torch.cuda.Stream()
    plain = mh.Solver(grid, phys)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        s = mh.Solver(grid, phys)
    for t in (s, plain):
        put(t, 0)
        t.step(1)  # (its kernels are loaded before the capture)
        put(t, 0)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        s.step(1)
    for k in range(6):
        if k in (3, 5):
            for t in (s, plain):
                put(t, k // 2)
            torch.cuda.synchronize()
        with torch.cuda.stream(side):
            g.replay()
        plain.step(1)
        torch.cuda.synchronize()
        assert s.clock() == plain.clock(), k
        got, want = s.get_state_device(), plain.get_state_device()
        torch.cuda.synchronize()
        assert torch.equal(got, want), k

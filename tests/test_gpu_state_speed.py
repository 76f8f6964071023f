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


def corrected_case(B, dtype, kinds, scale, flags=0, **phys):
    """B solvers at 16^3 (twice, alike pairwise), their states and a corrector;
    kinds: grid options by member."""
    import torch

    n = 16
    td = torch.float64 if dtype == "f64" else torch.float32
    mk = lambda: [mh.Solver(mh.grid_desc((n,) * 3, (1.0 / n,) * 3, dtype=dtype, **kinds(b)),
                            mh.physics_desc(flags=flags, ou_seed=3 * b, **phys)) for b in range(B)]
    U = torch.tensor(np.stack([wl.smooth_random_state((n,) * 3, seed=60 + b) for b in range(B)]),
                     dtype=td, device="cuda:0")
    mean = [float(v) for v in U.mean(dim=(0, 2, 3, 4))]
    std = [float(v) + 1e-3 for v in U.std(dim=(0, 2, 3, 4))]
    corr = mh.Corrector(mh.corr_desc(n, B, dtype, 5.0 / 3.0, mean, std, (scale,) * 5,
                                     fallback_frac=1.0))
    corr.set_params(wl.corrector_init_params(seed=12, out_scale=1.0).astype(np.float32))
    a, b = mk(), mk()
    for s, t, u in zip(a, b, U):
        s.set_state(u)
        t.set_state(u)
    return a, b, corr


def host_driven(solvers, corr, steps, dts):
    """The corrected steps driven from the host: the reference of mh_step_corrected."""
    import torch

    for k in range(steps):
        for q, t in enumerate(solvers):
            t.step(1, 0.0 if dts is None else float(dts[k, q]))
        out, _, _ = corr.apply(torch.stack([t.get_state_device() for t in solvers]))
        for t, u in zip(solvers, out):
            t.set_state(u)


def schedule(steps, B):
    import torch

    return torch.tensor(1e-3 * (1.0 + np.arange(steps * B).reshape(steps, B) % 4),
                        dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("B", [2, 8])
@pytest.mark.parametrize("cfl", [False, True])
def test_unlike_contexts_step_without_a_graph(B, cfl):
    """Contexts that differ in more than the forcing's seed, with use_graph set:
    bitwise the host-driven loop, clocks too, in two calls."""
    import torch

    steps = 3
    a, b, corr = corrected_case(B, "f32", lambda q: dict(cfl=0.2 + 0.02 * q,
                                                         limiter=q % 2), 1e-3, mh.SRC_FORCING)
    dts = None if cfl else schedule(steps, B)
    for _ in range(2):
        mh.step_corrected(a, corr, steps, dts, use_graph=True)
        host_driven(b, corr, steps, dts)
        for s, t in zip(a, b):
            assert torch.equal(s.get_state_device(), t.get_state_device())
            assert s.clock() == t.clock()


@pytest.mark.parametrize("alike", [True, False])
@pytest.mark.parametrize("after", ["step", "corrected"])
def test_cfl_step_after_scheduled_corrected_steps(alike, after):
    """The CFL step that follows corrected steps on a schedule is the one of the
    corrected states, whose signal speed a strong correction moves away from
    the stepped states'."""
    import torch

    B, steps = 3, 2
    a, b, corr = corrected_case(B, "f64", lambda q: dict(cfl=0.2 + (not alike) * 0.05 * q), 0.1,
                                mh.SRC_FORCING)
    dts = schedule(steps, B)
    fell = mh.step_corrected(a, corr, steps, dts, count_fallbacks=True)
    host_driven(b, corr, steps, dts)
    assert fell == 0
    if after == "step":
        got = [float(s.step(1, record=True)[0]) for s in a]
        want = [float(t.step(1, record=True)[0]) for t in b]
        assert got == want
    else:
        mh.step_corrected(a, corr, 1)
        host_driven(b, corr, 1, None)
    for s, t in zip(a, b):
        assert s.clock() == t.clock()
        assert torch.equal(s.get_state_device(), t.get_state_device())


@pytest.mark.parametrize("cfl", [False, True])
def test_cooling_limit_of_corrected_states(cfl):
    """Tabulated cooling with a cooling-time limit: the corrected CFL steps, and
    the plain one after corrected steps of either kind, are limited by the
    rate of the state they start from."""
    import torch

    B, steps = 2, 3
    table = dict(cool_model=mh.COOL_TABLE, cool_table=wl.synthetic_cie_table(),
                 **wl.COOLING_TABLE_MODEL)
    a, b, corr = corrected_case(B, "f64", lambda q: {}, 0.02, mh.SRC_COOLING, cool_ccool=1e-3,
                                **table)
    free = mh.Solver(a[0].grid, mh.physics_desc(flags=mh.SRC_COOLING, **table))
    free.set_state(a[0].get_state_device())
    dts = None if cfl else schedule(steps, B)
    mh.step_corrected(a, corr, steps, dts)
    host_driven(b, corr, steps, dts)
    for s, t in zip(a, b):
        assert s.clock() == t.clock()
        assert torch.equal(s.get_state_device(), t.get_state_device())
    got = [float(s.step(1, record=True)[0]) for s in a]
    assert got == [float(t.step(1, record=True)[0]) for t in b]
    # (the limit is the cooling time's, not the signal speed's)
    assert got[0] < 0.5 * float(free.step(1, record=True)[0])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("source", ["tensor", "pinned", "byte offset", "last bytes", "other gpu"])
def test_set_state_from_any_device_memory(source, dtype):
    """mh_set_state(MH_DEVICE) takes what the runtime's copy takes: the state and
    its CFL step are those of the same values set from a tensor."""
    import ctypes

    import torch

    if source == "other gpu" and torch.cuda.device_count() < 2:
        pytest.skip("one GPU")
    shape = (6, 10, 24)
    s = mh.Solver(mh.grid_desc(shape, (1.0 / 24, 0.1, 1.0 / 6), dtype=dtype))
    host = torch.tensor(wl.random_state(shape, seed=31, vmax=0.5), dtype=s.torch_dtype)
    s.set_state(host.to("cuda:0"))
    want = s.get_state_device()
    dt = float(s.step(1, record=True)[0])
    if source == "pinned":
        keep = host.pin_memory()
        ptr = keep.data_ptr()
    elif source == "byte offset":  # not a multiple of the value's size
        raw = torch.frombuffer(bytearray(host.numpy().tobytes()), dtype=torch.uint8)
        keep = torch.empty(raw.numel() + 1, dtype=torch.uint8, device="cuda:0")
        keep[1:].copy_(raw)
        ptr = keep.data_ptr() + 1
    elif source == "last bytes":  # the end of an allocation of its own (over 10 MiB)
        keep = torch.empty(12 * 2 ** 20 // host.element_size(), dtype=host.dtype, device="cuda:0")
        keep[-host.numel():].copy_(host.reshape(-1))
        ptr = keep.data_ptr() + (keep.numel() - host.numel()) * host.element_size()
    else:
        keep = host.to("cuda:1" if source == "other gpu" else "cuda:0")
        torch.cuda.synchronize(keep.device)
        ptr = keep.data_ptr()
    torch.cuda.synchronize()
    assert s.lib.mh_set_state(s.ctx, ctypes.c_void_p(ptr), mh.DEVICE) == mh.OK
    assert torch.equal(s.get_state_device(), want)
    assert float(s.step(1, record=True)[0]) == dt


def test_set_state_inside_a_capture():
    """A captured set_state and CFL step: every replay starts from what the tensor
    holds then."""
    import torch

    shape = (6, 10, 24)
    grid = mh.grid_desc(shape, (1.0 / 24, 0.1, 1.0 / 6))
    U = [torch.tensor(wl.random_state(shape, seed=41 + k, vmax=0.3 * (k + 1)),
                      dtype=torch.float32, device="cuda:0") for k in range(3)]
    plain = mh.Solver(grid)
    side = torch.cuda.Stream()
    room = U[0].clone()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        s = mh.Solver(grid)
    s.set_state(room)
    s.step(1)
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        s.set_state(room)
        s.step(1)
    for k in (1, 0, 2, 1):
        room.copy_(U[k])
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            g.replay()
        plain.set_state(U[k])
        plain.step(1)
        torch.cuda.synchronize()
        got, want = s.get_state_device(), plain.get_state_device()
        torch.cuda.synchronize()
        assert torch.equal(got, want), k


@pytest.mark.parametrize("where", ["device", "host"])
def test_timing_includes_the_reduction_of_a_set_state(where):
    """The signal speed of a set state is a timed launch of kind MH_TIME_OTHER, once
    a state, wherever it is measured."""
    import torch

    shape = (16, 16, 64)
    s = mh.Solver(mh.grid_desc(shape, (1.0 / 64, 1.0 / 16, 1.0 / 16)))
    U = wl.random_state(shape, seed=3, vmax=0.5).astype(np.float32)
    if where == "device":
        U = torch.tensor(U, device="cuda:0")
    s.set_timing(True)
    for _ in range(2):
        s.set_state(U)
        s.step(2)
    ms, launches = s.timing()
    assert launches[mh.TIME_OTHER] == 2 and ms[mh.TIME_OTHER] > 0.0
    assert list(launches[[mh.TIME_STAGE1, mh.TIME_STAGE2, mh.TIME_PROLOGUE]]) == [4, 4, 4]


@pytest.mark.parametrize("solver", [mh.GRAV_MG, mh.GRAV_FFT])
def test_multigrid_is_refused_inside_a_capture(solver):
    """The multigrid solve waits for its convergence tests on the host, so a captured
    step with it is refused, and the solver steps on afterwards; the spectral
    solve is captured."""
    import torch

    n = 16
    grid = mh.grid_desc((n,) * 3, (1.0 / n,) * 3)
    phys = mh.physics_desc(flags=mh.SRC_GRAVITY, grav_G=2.0, mg_tol=1e-5, grav_solver=solver)
    U = torch.tensor(wl.grf_density_state(n, seed=5), dtype=torch.float32, device="cuda:0")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    plain = mh.Solver(grid, phys)
    with torch.cuda.stream(side):
        s = mh.Solver(grid, phys)
    for t in (s, plain):
        t.set_state(U)
        t.step(1, 1e-3)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    refused = False
    with torch.cuda.graph(g, stream=side):
        try:
            s.step(1, 1e-3)
        except mh.MHError:
            refused = True
    assert refused == (solver == mh.GRAV_MG)
    s.set_state(plain.get_state_device())
    s.set_potential(plain.potential_device())
    for k in range(3):
        if refused:
            s.step(1, 1e-3)
        else:
            with torch.cuda.stream(side):
                g.replay()
        plain.step(1, 1e-3)
        torch.cuda.synchronize()
        got, want = s.get_state_device(), plain.get_state_device()
        torch.cuda.synchronize()
        assert torch.equal(got, want), k

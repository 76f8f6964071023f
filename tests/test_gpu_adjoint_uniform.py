"""Reverse of an Euler step at states whose velocity is uniform and whose
pressure is, or is constant over blocks of cells: those slopes are exactly
zero, so no limiter branch may be taken from a rounding error, along any axis
and on any path of the reverse."""
import numpy as np
import pytest

import oracle
from parity import TOL, as_input, pair

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _name(request):
    print(f"\n[gpu case] {request.node.nodeid}", flush=True)
    yield


def contact_state(shape, seed, run=None):
    """Densities of powers of two, velocity uniform, pressure uniform or
    constant over blocks of `run` cells along each axis (the last takes the
    remainder), all exact in fp32: every conserved and primitive value is, but
    for the one rounding of P = (gamma - 1) e, which is the same in every cell
    of that e."""
    rng = np.random.default_rng(seed)
    rho = 2.0 ** rng.integers(-1, 2, shape)
    v = (0.5, -0.25, 0.125)
    e = 3.75 * np.ones(shape)  # P = 2.5 at gamma = 5/3
    if run:
        blocks = rng.choice([3.75, 5.25, 8.25], size=[max(n // run, 1) for n in shape])
        e = blocks[np.ix_(*(np.minimum(np.arange(n) // run, max(n // run, 1) - 1)
                            for n in shape))]
    return np.stack([rho, *(rho * c for c in v), e + 0.5 * rho * sum(c * c for c in v)])


# rows and columns of the fused kernels: whole rows, rows in pieces, a single
# segment and several; the general path: an outflow axis, other schemes
@pytest.mark.parametrize("shape,bc,limiter,riemann", [
    ((8, 9, 70), (0, 0, 0), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((4, 5, 600), (0, 0, 0), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((70, 12, 5), (0, 0, 0), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((5, 140, 6), (0, 0, 0), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((9, 11, 33), (1, 1, 1), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((3, 2, 33), (0, 0, 1), oracle.LIM_MINMOD, oracle.RS_HLLC),
    ((9, 11, 33), (0, 1, 0), oracle.LIM_VANLEER, oracle.RS_HLLC),
    ((9, 11, 33), (0, 0, 0), oracle.LIM_SUPERBEE, oracle.RS_HLLC),
    ((9, 11, 33), (0, 0, 0), oracle.LIM_MC, oracle.RS_HLLC),
])
@pytest.mark.parametrize("dtype,run", [("f32", None), ("f64", None), ("f32", 2), ("f32", 3), ("f64", 2)])
def test_adjoint_where_velocity_and_pressure_are_uniform(shape, bc, limiter, riemann, dtype, run):
    import torch

    nz, ny, nx = shape
    s, oc = pair(shape, (1.0 / nx, 1.0 / ny, 1.0 / nz), bc, dtype, integrator=oracle.RK_EULER,
                 limiter=limiter, riemann=riemann)
    U = contact_state(shape, 13, run)
    assert np.array_equal(as_input(U, dtype), U)
    lam = as_input(np.random.default_rng(14).standard_normal(U.shape), dtype)
    dt = float(np.float32(0.5 * oracle.cfl_dt(oc, U)))
    ref = oracle.step_vjp(oc, U, dt, 0, np.zeros((0, 3), np.int32), np.zeros(6), np.zeros(shape),
                          lam)
    dev = lambda a: torch.tensor(a, dtype=s.torch_dtype, device="cuda:0")
    got = s.adjoint_step(dev(U), dt, 0, dev(lam)).cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() / np.abs(ref).max() < TOL[dtype]

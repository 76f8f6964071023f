"""The fp32 multigrid's residual at its round-off floor, where the stall rule ends
a solve, is that of sweeps that divide by six."""
import numpy as np
import pytest

import paper_2512_13403_amd as mh

pytestmark = pytest.mark.gpu


def neighbours(p):
    s = np.roll(p, 1, 2) + np.roll(p, -1, 2)
    for d, axis in ((1, 1), (-1, 1), (1, 0), (-1, 0)):
        s = s + np.roll(p, d, axis)
    return s


# 64^3: pairs of sweeps on the small tiles; 96^3: single ones on the large.  The
# same cycle emulated in numpy (32^3, 64^3, 96^3) leaves 1.03 to 1.04 times the
# residual that four more dividing sweeps do where its own sweeps divide, and 1.22
# to 1.24 times where they multiply by the rounded 1/6; the bound lies half way
@pytest.mark.parametrize("n", [64, 96])
@pytest.mark.parametrize("seed", [1, 2])
def test_fp32_residual_at_the_floor(n, seed):
    f32 = np.float32
    rho = (1.0 + 0.1 * np.random.default_rng(seed).standard_normal((n,) * 3)).astype(f32)
    U = np.zeros((5, n, n, n), dtype=f32)
    U[0], U[4] = rho, 1.5  # at rest, uniform pressure: the step leaves the density as it is
    G = 1.0 / (4.0 * np.pi)
    s = mh.Solver(mh.grid_desc((n,) * 3, (1.0 / n,) * 3, dtype="f32"),
                  mh.physics_desc(flags=mh.SRC_GRAVITY, grav_G=G, mg_tol=0.0, mg_max_cycles=12))
    s.set_state(U)
    s.step(1, 1e-6)
    assert s.mg_cycles() == 12
    assert np.array_equal(s.get_state()[0], rho)
    r64 = rho.astype(np.float64)
    F = (4.0 * np.pi * G * (r64 - r64.mean())).astype(f32)
    h2 = f32(1.0 / n ** 2)

    def residual(p):
        p = p.astype(np.float64)
        r = F - (neighbours(p) - 6.0 * p) * n * n
        return np.linalg.norm(r - r.mean())

    phi = s.potential().astype(f32)
    p = phi
    even = np.indices((n,) * 3).sum(axis=0) % 2 == 0
    for _ in range(4):
        for colour in (even, ~even):
            g = (neighbours(p).astype(np.float64) - np.float64(h2) * F).astype(f32)  # one rounding
            p = np.where(colour, g / f32(6), p)
    assert residual(phi) < 1.13 * residual(p)

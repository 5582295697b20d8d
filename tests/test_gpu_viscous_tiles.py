"""GPU parity of the viscous path at the edges of its kernels' tiles: element
counts that fill the gradient kernel's blocks (64, 32 or 16 elements) exactly,
leave a remainder or stay below one block, straight and curved elements, every
boundary, P = 1..5.

Bars: FP64 1e-12 relative L2 of the rhs; FP32 2e-5 (unit roundoff 6e-8 times
the cancellation of the flux derivatives, 10-100 on these meshes, with a
factor of four).
"""
import numpy as np
import pytest

import meshgen
from oracle import oracle as orc
from oracle.refelem import ref

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32": 2e-5}


def viscous_state(c, seed):
    """The case's start, disturbed down to the element scale so that the
    sensor switches on."""
    rng = np.random.default_rng(seed)
    rho, u, v = c.U0[:, 0], c.U0[:, 1] / c.U0[:, 0], c.U0[:, 2] / c.U0[:, 0]
    p = 0.4 * (c.U0[:, 3] - 0.5 * rho * (u * u + v * v))
    f = 1 + 0.05 * rng.uniform(-1, 1, (4,) + rho.shape)
    return np.ascontiguousarray(meshgen.primitive_to_conserved(rho * f[0], u * f[1], v * f[2], p * f[3]))


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mesh,scale,K", [("vortex", 9 / 256, 18), ("cylinder", 0.0016, 32),
                                          ("airfoil", 0.0011, 160), ("cylinder", 0.0064, 128)])
def test_viscous_rhs_at_tile_edges(mesh, scale, K, precision, P):
    from paper_1208_4772_amd import dg
    R = ref(P)
    c = meshgen.make_case(mesh, R.r, R.s, scale=scale, P=P)
    assert c.K == K
    kw = dict(av=True, av_kappa=4.0, av_eps0=0.3)
    U0 = viscous_state(c, 7 + P)
    o = orc.Oracle.for_case(c, **kw)
    assert (o.sensor(U0) > 0).mean() > 0.2   # (P = 1 has the highest threshold)
    want = o.rhs(U0)
    s = dg.Solver.from_case(c, precision, **kw)
    got = s.rhs(s.state(U0)).double().cpu().numpy()
    s.close()
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"{mesh} K={c.K} P={P} {precision}: {err:.2e}")
    assert err <= TOL[precision]

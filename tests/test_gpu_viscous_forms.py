"""GPU parity of the viscous path with either numerical flux and each FP32
product, at the edges of its kernels' blocks: element counts of one block of 8
(the FP64 gradient at P = 5), 16 or 32 elements, of fewer, and with remainders
of a part of a group of four, straight and curved, every boundary.

Bars as for the inviscid right-hand side: FP64 1e-12 relative L2; FP32 2e-5;
BF16x3 the three-term split's roundoff 3 x 2^-16 times the cancellation of the
flux derivatives.
"""
import numpy as np
import pytest

import meshgen
from oracle import oracle as orc
from oracle.refelem import ref
from test_gpu_parity import TOL
from test_gpu_viscous_tiles import viscous_state

pytestmark = pytest.mark.gpu


def check(c, precision, riemann):
    from paper_1208_4772_amd import dg
    kw = dict(av=True, av_kappa=4.0, av_eps0=0.3, riemann=riemann)
    U0 = viscous_state(c, 7 + c.P)
    o = orc.Oracle.for_case(c, **kw)
    assert (o.sensor(U0) > 0).mean() > 0.2
    want = o.rhs(U0)
    s = dg.Solver.from_case(c, precision, **kw)
    got = s.rhs(s.state(U0)).double().cpu().numpy()
    s.close()
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"{c.name} K={c.K} P={c.P} {precision} {riemann}: {err:.2e}", flush=True)
    assert err <= TOL[precision]


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("precision,riemann", [("fp64", "hllc"), ("fp32", "hllc"), ("bf16x3", "lf"),
                                               ("bf16x3", "hllc")])
@pytest.mark.parametrize("mesh,scale,K", [("vortex", 9 / 256, 18), ("airfoil", 0.0011, 160),
                                          ("cylinder", 0.0064, 128)])
def test_viscous_rhs_in_each_flux_and_product(mesh, scale, K, precision, riemann, P):
    R = ref(P)
    c = meshgen.make_case(mesh, R.r, R.s, scale=scale, P=P)
    assert c.K == K
    check(c, precision, riemann)


@pytest.mark.parametrize("riemann", ["lf", "hllc"])
@pytest.mark.parametrize("nt,nr", [(9, 2), (11, 3), (10, 2), (51, 31)])
def test_viscous_fp64_at_the_gradients_block_of_eight(nt, nr, riemann):
    """P = 5: 36, 66, 40 and 3,162 elements (remainders 4, 2, 0 and 2 of 8)."""
    R = ref(5)
    c = meshgen.make_case("cylinder", R.r, R.s, scale=0.0016, P=5)
    m = meshgen.cylinder_annulus(nt, nr, 1.0, 20.0, 0.1, 38, True)
    x, y = meshgen.node_coordinates(m, R.r, R.s)
    c.mesh, c.x, c.y = m, x, y
    c.U0 = np.ascontiguousarray(np.broadcast_to(c.freestream[None, :, None], (m.K, 4, x.shape[1])))
    assert c.K == 2 * nt * nr
    check(c, "fp64", riemann)

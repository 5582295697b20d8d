"""The FP32 weak form's error against FP64 on meshes with curved elements is no
larger than a plain evaluation's: per node the two products of a cubature point
first, then the running sum, then the inverse mass matrix.

`PLAIN` holds that evaluation's relative L2 errors of the right-hand side (on
the VALUs, one thread a node, each operator entry in FP32).  Bar: 1.15 times
it, what the order of the sums may change; a single sum over all the products
with the inverse folded into the operator is 1.17 to 1.44 times as far off.
"""
import pytest

from oracle import oracle as orc
from test_gpu_curved64 import curved_case, rel

pytestmark = pytest.mark.gpu

PLAIN = [("cylinder", 0.0081, 5, "lf", 1.101e-05), ("cylinder", 0.0081, 5, "hllc", 1.170e-05),
         ("cylinder", 0.09, 3, "lf", 1.243e-05), ("cylinder", 0.09, 4, "lf", 1.394e-05),
         ("cylinder", 0.09, 5, "lf", 1.496e-05),
         ("roofline_curved", 2e-4, 3, "lf", 2.900e-05), ("roofline_curved", 2e-4, 4, "lf", 5.783e-05),
         ("roofline_curved", 2e-4, 5, "lf", 8.342e-05), ("roofline_curved", 2e-4, 5, "hllc", 8.461e-05),
         ("airfoil", 0.02, 3, "lf", 2.121e-06), ("airfoil", 0.02, 4, "lf", 2.370e-06),
         ("airfoil", 0.02, 5, "lf", 2.535e-06)]


@pytest.mark.parametrize("mesh,scale,P,riemann,plain", PLAIN)
def test_fp32_weak_error_on_curved_meshes(mesh, scale, P, riemann, plain):
    from paper_1208_4772_amd import dg
    c, U0 = curved_case(mesh, scale, P)
    want = orc.Oracle.for_case(c, weak=True, riemann=riemann, av=False).rhs(U0)
    s = dg.Solver.from_case(c, "fp32", form="weak", riemann=riemann, av=False)
    err = rel(s.rhs(s.state(U0)).double().cpu().numpy(), want)
    s.close()
    print(f"{mesh} K={c.K} P={P} {riemann}: {err:.3e}, plain {plain:.3e}", flush=True)
    assert err <= 1.15 * plain

"""GPU parity of the weak form's stage at the edges of its tiles: groups of
four elements (a last group of two, one that holds straight and curved
elements), meshes below and above the block-size rule (2,048 groups) and large
enough that a wavefront walks several groups.

Bar: FP64 1e-12 relative L2 against the FP64 oracle, or twice the spread of
the oracle's own valid evaluations where that is larger; FP32 2e-5, or 2^29
times the FP64 kernel's distance (the conditioning of V - S).
"""
import numpy as np
import pytest

import meshgen
from oracle import oracle as orc
from oracle.refelem import ref
from test_gpu_curved64 import rel
from test_gpu_parity import FP32_RHS_TOL, perturbed_state

pytestmark = pytest.mark.gpu


def spread(mesh, P, x, y, q, U, riemann):
    kw = dict(freestream=q, riemann=riemann, weak=True)
    got = [orc.Oracle(mesh, P, x, y, **kw).rhs(U), orc.Oracle(mesh, P, x, y, fma=True, **kw).rhs(U),
           orc.Oracle(mesh, P, x - x[:, :1], y - y[:, :1], **kw).rhs(U)]
    return max(rel(a, b) for i, a in enumerate(got) for b in got[:i])


MESHES = {
    "channel_18": lambda: meshgen.channel(3, 3, perm_seed=5),
    "curved_18": lambda: meshgen.periodic_square(3, perm_seed=11, curved_amplitude=0.05),
    "cylinder_54": lambda: meshgen.cylinder_annulus(9, 3),
    "channel_8450": lambda: meshgen.channel(65, 65, perm_seed=5),
    "cylinder_17030": lambda: meshgen.cylinder_annulus(131, 65),
    "channel_33282": lambda: meshgen.channel(129, 129, perm_seed=5),
}


@pytest.mark.parametrize("name,P", [(n, P) for n in ("channel_18", "curved_18", "cylinder_54") for P in range(1, 6)]
                         + [("channel_8450", 2), ("channel_8450", 5), ("cylinder_17030", 3),
                            ("cylinder_17030", 4), ("channel_33282", 2)])
@pytest.mark.parametrize("riemann", ["lf", "hllc"])
def test_weak_rhs_at_tile_edges(name, P, riemann):
    from paper_1208_4772_amd import dg
    mesh = MESHES[name]()
    R = ref(P)
    x, y = meshgen.node_coordinates(mesh, R.r, R.s)
    q = meshgen.freestream_state(0.38, 1.25)
    U = perturbed_state(x, y, q)
    want = orc.Oracle(mesh, P, x, y, freestream=q, riemann=riemann, weak=True).rhs(U)
    err = {}
    for precision in ("fp64", "fp32"):
        s = dg.Solver(mesh.EToE, mesh.EToF, mesh.bc, x, y, P, precision, freestream=q, riemann=riemann,
                      form="weak")
        err[precision] = rel(s.rhs(s.state(U)).double().cpu().numpy(), want)
        s.close()
    tol = 1e-12
    if err["fp64"] > tol:
        tol = max(tol, 2.0 * spread(mesh, P, x, y, q, U, riemann))
    print(f"{name} P={P} {riemann}: fp64 {err['fp64']:.2e} (bar {tol:.1e}) fp32 {err['fp32']:.2e}")
    assert err["fp64"] <= tol
    assert err["fp32"] <= max(FP32_RHS_TOL, 2.0 ** 29 * err["fp64"])

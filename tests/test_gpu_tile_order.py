"""FP64 right-hand sides beyond the last-level cache, where the VALU stage and
the viscous gradient take their tiles in block order instead of XCD by XCD
(399,618 all-curved elements at P = 2; a count that leaves a remainder in
every block)."""
import numpy as np
import pytest

import meshgen
from oracle import oracle as orc
from oracle.refelem import ref
from test_gpu_viscous_tiles import viscous_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("av", [False, True])
def test_fp64_rhs_beyond_the_cache(av):
    from paper_1208_4772_amd import dg
    R = ref(2)
    c = meshgen.make_case("roofline_curved", R.r, R.s, scale=(447 / 707) ** 2, P=2)
    assert c.K == 2 * 447 ** 2
    kw = dict(av=av, av_kappa=4.0, av_eps0=0.3)
    U0 = viscous_state(c, 5)
    want = orc.Oracle.for_case(c, **kw).rhs(U0)
    s = dg.Solver.from_case(c, "fp64", **kw)
    got = s.rhs(s.state(U0)).cpu().numpy()
    s.close()
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    # FP64: 1e-12, or twice what the oracle's own valid evaluations differ by
    # (its fused build, and the coordinates relative to each element)
    tol = 1e-12
    if err > tol:
        other = [orc.Oracle.for_case(c, fma=True, **kw).rhs(U0)]
        c.x, c.y = c.x - c.x[:, :1], c.y - c.y[:, :1]
        other.append(orc.Oracle.for_case(c, **kw).rhs(U0))
        tol = max(tol, 2.0 * max(np.linalg.norm(o - want) for o in other) / np.linalg.norm(want))
    print(f"K={c.K} av={av}: {err:.2e} (bar {tol:.1e})")
    assert err <= tol

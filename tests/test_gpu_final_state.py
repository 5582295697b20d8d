"""A run (and a slot of a batch) whose last step goes bad reports it, on every
path of the stage: the VALUs and the matrix cores in FP64, FP32, with and
without viscosity, and the weak form.  The step size that does it (the states
before are sound, the last is not) is found with the oracle."""
import numpy as np
import pytest

from oracle import oracle as orc
from test_gpu_curved64 import curved_case

pytestmark = pytest.mark.gpu

AV = dict(av=True, av_kappa=4.0)
CASES = {   # mesh, scale, P, precision, options
    "fp64 VALU": ("cylinder", 0.0081, 2, "fp64", {}),
    "fp64 VALU small": ("cylinder", 0.0081, 4, "fp64", {}),
    "fp64 matrix curved": ("cylinder", 0.0081, 3, "fp64", {}),
    "fp64 matrix straight": ("vortex", 0.1, 3, "fp64", {}),
    "fp64 viscous VALU": ("airfoil", 0.002, 2, "fp64", AV),
    "fp64 viscous matrix": ("airfoil", 0.002, 3, "fp64", AV),
    "fp32": ("cylinder", 0.0081, 3, "fp32", {}),
    "fp32 viscous": ("airfoil", 0.002, 3, "fp32", AV),
    "weak fp64": ("cylinder", 0.0081, 3, "fp64", dict(weak=True)),
    "weak fp32": ("cylinder", 0.0081, 3, "fp32", dict(weak=True)),
    "weak fp64 P1": ("cylinder", 0.0081, 1, "fp64", dict(weak=True)),
    "weak fp32 P1": ("cylinder", 0.0081, 1, "fp32", dict(weak=True)),
}


def smallest(U):
    """Smallest density and pressure (-inf for a state that is not finite)."""
    if not np.isfinite(U).all():
        return -np.inf
    p = 0.4 * (U[:, 3] - 0.5 * (U[:, 1] ** 2 + U[:, 2] ** 2) / U[:, 0])
    return min(U[:, 0].min(), p.min())


def bad_last_step(c, U0, steps, kw):
    for cfl in 0.5 * 1.1 ** np.arange(60):
        o = orc.Oracle.for_case(c, cfl=cfl, **{"av": False, **kw})
        m = [smallest(o.run(U0, n)[0]) for n in range(steps + 1)]
        if min(m[:-1]) > 0.05 and m[-1] == -np.inf:
            return cfl
    raise AssertionError("no such step size")


def make(name, steps):
    from paper_1208_4772_amd import dg
    mesh, scale, P, precision, kw = CASES[name]
    c, U0 = curved_case(mesh, scale, P)
    cfl = bad_last_step(c, U0, steps, kw)
    opts = {"av": False, **kw}
    opts["form"] = "weak" if opts.pop("weak", False) else "nodal"
    s = dg.Solver.from_case(c, precision, cfl=cfl, **opts)
    return s, U0, dg


@pytest.mark.parametrize("name,steps", [(n, 1) for n in CASES] + [
    (n, 2) for n in ("fp64 VALU small", "fp64 matrix curved", "fp64 viscous VALU", "fp32", "weak fp64", "weak fp32",
                     "weak fp64 P1", "weak fp32 P1")])
def test_run_reports_a_bad_final_state(name, steps):
    s, U0, dg = make(name, steps)
    U = s.state(U0)
    assert s.run(U.clone(), steps - 1).status == 0
    st = s.run(U, steps, check=False)
    assert st.status == dg.DG_ENONFINITE and st.steps == steps
    with pytest.raises(dg.DGError):
        s.run(s.state(U0), steps)
    # no steps: a state that the caller holds is not the run's to refuse
    bad = s.state(U0)
    bad[0, 0, 0] = -1.0
    assert s.run(bad, 0).status == 0
    s.close()


@pytest.mark.parametrize("name", list(CASES))
def test_batch_slot_reports_a_bad_final_state(name):
    s, U0, dg = make(name, 1)
    b = dg.Batch(1 << 32, 2)
    slot = b.admit(s, s.state(U0), 1)
    assert b.advance(1) == 1
    assert b.poll() == [slot]
    assert b.stats(slot).status == dg.DG_ENONFINITE
    b.release(slot)
    b.close()
    s.close()

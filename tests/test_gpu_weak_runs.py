"""The weak form's run, whose steps take their time step from the bound the
step before left, against single steps, which reduce it from the state: the
same bits in state, time and step sizes, at every order, for one, two and
several steps, with straight and with curved elements."""
import numpy as np
import pytest

import meshgen
from oracle.refelem import ref
from test_gpu_parity import perturbed_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("mk", [lambda: meshgen.channel(3, 3, perm_seed=5), lambda: meshgen.cylinder_annulus(24, 6),
                                lambda: meshgen.cylinder_annulus(131, 17)], ids=["channel", "cylinder", "cylinder4k"])
def test_weak_run_is_its_steps(mk, P, precision):
    import torch
    from paper_1208_4772_amd import dg
    mesh = mk()
    R = ref(P)
    x, y = meshgen.node_coordinates(mesh, R.r, R.s)
    q = meshgen.freestream_state(0.38)
    s = dg.Solver(mesh.EToE, mesh.EToF, mesh.bc, x, y, P, precision, freestream=q, form="weak")
    U0 = perturbed_state(x, y, q)
    for n in (1, 2, 5):
        a, b = s.state(U0), s.state(U0)
        st = s.run(a, n)
        for _ in range(n):
            s.step(b)
        assert st.status == 0 and st.steps == n
        assert torch.equal(a, b), (n, float((a - b).abs().max()))
        # a second run carries on where the first ended
        st2 = s.run(b, 1)
        c = s.state(U0)
        st3 = s.run(c, n + 1)
        assert torch.equal(b, c)
        assert st3.t == pytest.approx(st.t + st2.t, rel=1e-14) and st3.dt_min == min(st.dt_min, st2.dt_min)
    s.close()


def test_weak_run_flags_a_bad_state():
    """A step that starts from a non-physical state is reported, as before."""
    from paper_1208_4772_amd import dg
    mesh = meshgen.channel(3, 3)
    R = ref(3)
    x, y = meshgen.node_coordinates(mesh, R.r, R.s)
    q = meshgen.freestream_state(0.38)
    s = dg.Solver(mesh.EToE, mesh.EToF, mesh.bc, x, y, 3, "fp64", freestream=q, form="weak")
    U0 = np.array(perturbed_state(x, y, q))
    U0[5, 0, 2] = -1.0
    for n in (1, 3):
        with pytest.raises(dg.DGError):
            s.run(s.state(U0), n)
    s.close()

"""The bench's description of the launches: the FP64 and weak-form kernels'
names on both sides of the rules that pick them, the sources a traffic record
is tied to, and the viscous stage's bytes on a periodic straight mesh (no GPU).
"""
import pytest

import bench
import meshgen
from paper_1208_4772_amd import dg


def case(mesh, P, scale, av=False):
    c = meshgen.make_case(mesh, *dg.reference_nodes(P), P=P, scale=scale)
    c.av = av
    return c


def label(c, precision="fp64", form="nodal"):
    return bench.stage_kernel_label(c, precision, 0, form, bench.fp64_on_matrix_cores(c))


@pytest.mark.parametrize("mesh,P,scale,av,kernel", [
    ("roofline", 5, 0.01, False, "k_stage_mfma64<5,false,false>"),
    ("vortex", 1, 1.0, False, "k_stage_mfma64<1,false,false>"),
    ("cylinder", 2, 0.2, False, "k_stage<double,2,false>"),
    ("cylinder", 3, 0.0081, False, "k_stage_mfma64<3,false,true>"),
    ("cylinder", 4, 0.09, False, "k_stage<double,4,false>"),
    ("cylinder", 4, 0.1225, False, "k_stage_mfma64<4,false,true>"),
    ("cylinder", 5, 0.25, False, "k_stage<double,5,false>"),
    ("cylinder", 5, 0.36, False, "k_stage_mfma64<5,false,true>"),
    ("vortex", 2, 1.0, True, "k_sensor_elem<2> + k_avgrad<2> + k_stage<double,2,true>"),
    ("vortex", 3, 1.0, True, "k_sensor_elem<3> + k_avgrad<3> + k_stage_mfma64<3,true,true>")])
def test_fp64_label_names_the_kernel_that_runs(mesh, P, scale, av, kernel):
    assert label(case(mesh, P, scale, av)) == kernel


def test_weak_label():
    assert label(case("vortex", 1, 1.0), "fp32", "weak") == "k_stage_weak1<float>"
    assert label(case("vortex", 4, 1.0), "fp64", "weak") == "k_stage_weak<double,4>"


def test_traffic_records_are_tied_to_the_stage_sources(tmp_path, monkeypatch):
    """A change of the file a precision's stage lives in changes its hash."""
    import os
    import shutil
    src = os.path.join(bench.ROOT, "paper_1208_4772_amd", "csrc")
    dst = tmp_path / "paper_1208_4772_amd" / "csrc"
    shutil.copytree(src, dst)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    for precision, av, name in (("fp64", False, "stage64.hip"), ("fp64", False, "kernels.hip"),
                                ("fp64", True, "stage64.hip"), ("fp32", False, "stage_mfma.hip"),
                                ("fp32", True, "kernels.hip")):
        before = bench.kernel_source_hash(precision, av)
        with open(dst / name, "a") as fh:
            fh.write("\n")
        assert bench.kernel_source_hash(precision, av) != before, (precision, av, name)


@pytest.mark.parametrize("s", [4, 8])
def test_viscous_bytes_per_element(s):
    c = case("roofline", 3, 0.01, True)
    b, info = bench.algorithmic_stage_bytes(c, s)
    assert info == dict(curved=0, interior_sides=3 * c.K)
    Np, F = 10, 3 * 4
    stage = 4 * Np * 3.8 + F * 4 + 13              # state, register, traces, geometry
    sensor = Np + 2
    gradient = 4 * Np + 1 + 8 * Np + 13 + F * 4 + 3 + (F / 5 if s == 4 else 0)
    viscous = 8 * Np + F * 8                       # sigma Q, and its traces
    per_el = (stage + sensor + gradient + viscous) * s + 12 + 16
    assert abs(b / c.K - per_el) < 1e-9

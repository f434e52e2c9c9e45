"""The batched solver's code compiled for the CPU (tests/host/batched_host.cpp)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2001_01978_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2001_01978_amd", "csrc")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """The program, with a stand-in for the kernel's row code beside batched.hip."""
    d = tmp_path_factory.mktemp("batched_host")
    for f in (os.path.join(HOST, "batched_host.cpp"), os.path.join(HOST, "sigma_impl.h"),
              os.path.join(CSRC, "batched.hip")):
        shutil.copy(f, d)
    exe = str(d / "batched_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", str(d), "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include", "-o", exe,
                    str(d / "batched_host.cpp"), "-lpthread"], check=True, timeout=120)
    return exe


@pytest.mark.parametrize("om,n,block,team", [(6, 2, 256, 1), (8, 4, 256, 1), (11, 3, 512, 1), (8, 4, 256, 2),
                                             (8, 4, 128, 4)])
def test_result_does_not_depend_on_the_order_of_the_waves(host, oracle_mod, om, n, block, team):
    """Spaces of fewer rows than lanes, alone and on a team with members that
    have none: waves without rows pass through a product at once, and what the
    steps hand over in LDS may not depend on who is first."""
    _, _, eps, V = inputs.c5_instance(om, n, seed=3)
    text = " ".join(repr(float(v)) for v in (*(2 * eps + np.diag(V)), *V.ravel()))
    out = []
    for seed in (0, 1, 2, 3, 4):   # first wave first, last wave first, three at random
        r = subprocess.run([host, "solve", str(block), str(team), str(seed)], input=f"{om} {n} 20 1e-10 {text}",
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, (seed, r.stdout)
        out.append(r.stdout.split())
    assert all(o == out[0] for o in out), out
    e0, _, occ0, _ = oracle_mod.dense_ground(om, n, eps, V)
    assert out[0][4] == "1" and abs(float(out[0][0]) - e0) <= 1e-10 * abs(e0)
    assert np.allclose([float(v) for v in out[0][5:]], occ0, atol=1e-8)


@pytest.mark.parametrize("krylov,kinds", [
    (20, [(32, 3, 4), (15, 6, 400)]),    # 4960 and 5005 states: the smaller ones are the costlier
    (8, [(32, 3, 16), (15, 6, 220)]),
    (2, [(32, 3, 16), (15, 6, 220)]),
    (20, [(16, 8, 64)]),                 # teams of 8 only, all alike
    (20, [(22, 11, 6), (12, 6, 100)]),   # large teams
    (20, [(10, 5, 300)]),                # single workgroups
])
def test_every_launch_fits_its_slots(host, krylov, kinds):
    """The tuner's trials and the solve: an instance goes to a level whose slots
    hold its Krylov vectors."""
    text = f"{krylov} {len(kinds)} " + " ".join(f"{o} {n} {c}" for o, n, c in kinds)
    r = subprocess.run([host, "tune"], input=text, capture_output=True, text=True, timeout=120)
    last = r.stdout.splitlines()[-1].split()
    assert r.returncode == 0 and last[:4] == ["status", "0", "launches", "4"], r.stdout
    assert last[-2:] == ["bad", "0"], r.stdout

"""FBP's unclamped sample index on the host: its range over the workloads' geometries and just inside
the limit of fbp_window_holds, where FP32 distances leave the least room."""
import os
import subprocess

import pytest

from paper_1304_2017_amd import synth
from test_abi import _fbp_window_workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("fbp") / "fbp_index_check"
    # (no contraction: the kernel's file has none, fmaf stands where it fuses)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_1304_2017_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "fbp_index_check.cpp"), "-o", str(exe)], check=True)

    def run(geom, *args):
        lines = [" ".join(repr(v) for v in (geom.nx, geom.ny, geom.nz, float(geom.dx), float(geom.x0),
                                            float(geom.y0), float(geom.z0), float(geom.c0), float(geom.dt),
                                            float(geom.t0), geom.n_t, geom.n_det))]
        lines += [" ".join(repr(float(c)) for c in r) for r in geom.det_xyz]
        r = subprocess.run([str(exe), *args], input="\n".join(lines) + "\n", capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0 and r.stdout.startswith("OK"), (geom.name, r.stdout + r.stderr)
        held, indices, least, room = map(int, r.stdout.split()[1:])
        print(f"{geom.name or geom.shape}: held {held}, {indices} indices, least {least}, room {room}")
        return held

    return run


def test_workloads(check):
    # a few hundred of a workload's transducers, spread over it
    for geom in _fbp_window_workloads():
        step = max(1, geom.n_det // 256)
        assert check(geom.with_detectors(range(0, geom.n_det, step)))
    small = synth.Geometry(21, 37, 11, 0.45, 1.0, -3.0, 0.2, synth.fibonacci_sphere(24, 40.0), 300, 0.08, 0.0, 1.5, 1.0)
    assert check(small, "all")


@pytest.mark.parametrize("sigma", [0.05, 0.8, 1.3, 20.0, 180.0])
@pytest.mark.parametrize("recorded", [False, True])
def test_at_the_limit(check, sigma, recorded):
    """16 2^-24 ((reach + 36) sigma + |tau|) a hair below 1/2 (and above it: not held), with tau = 0 or
    the transducers' own distance."""
    n, dx, c0 = (37, 21, 30), 1.0, 1.5
    dt = dx / (c0 * sigma)
    limit = 0.5 / 16.0 * 2.0 ** 24
    o = [synth.centred_origin(k, dx) for k in n]

    def geom(dist):
        xyz = synth.fibonacci_sphere(24, dist)
        xyz[0] = (dist, 0.0, 0.0)
        return synth.Geometry(*n, dx, *o, xyz, 64, dt, (dist - 20.0) / c0 if recorded else 0.0, c0, 1.0)

    # reach = dist + 18 (the origin's offset) + 37 + 16 grid units along x
    dist = (limit / sigma - 36.0 - 71.0) / (2.0 if recorded else 1.0)
    assert check(geom(0.9999 * dist), "all")
    assert not check(geom(1.001 * dist + 25.0))

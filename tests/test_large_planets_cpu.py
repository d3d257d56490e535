"""The direct rules of one sub-sample over the whole range of planets that the
interface accepts (semi-axes up to the star's), against the general path on the
same samples (host build), and the oracle where the two differ most.

Samples: ellipses anywhere on the disk, within 1e-9 to 0.3 of touching the limb
from inside, and about the star's centre, where a large planet is close to the
limb on both sides.

Tolerance: the exact path's bar of 1e-9 on every accepted sample.  The rules'
orders aim at exp(-31) and better; the general path's own error is below 1e-9.
"""
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest

from paper_2410_05408_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIP_INC = "/opt/rocm/include"
TOL = 1e-9
ARS, PERIOD = 200.0, 500.0


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(HIP_INC, "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("host") / "gl_direct_check")
    subprocess.run([cxx, "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INC,
                    "-I", os.path.join(ROOT, "paper_2410_05408_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "tests", "host", "gl_direct_check.cpp"), "-o", exe], check=True)
    return exe


def run(check, tmp_path, p, t):
    pf, tf, of = (str(tmp_path / f) for f in ("p.bin", "t.bin", "o.bin"))
    np.ascontiguousarray(p).tofile(pf)
    np.ascontiguousarray(t).tofile(tf)
    subprocess.run([check, pf, tf, of], check=True)
    return np.fromfile(of).reshape(3, t.size)


def oracle_flux(p, t):
    # in a process of its own: the oracle counts integrals that stop above
    # their target, which other tests read
    code = ("import sys, numpy as np; from oracle import glo; a = np.load(sys.argv[1]); n = a.shape[1]; "
            "f = glo.flux_batch if a.shape[0] == 11 else glo.flux_batch_ell; "
            "np.save(sys.argv[1], f(np.ascontiguousarray(a[:-1]), np.ascontiguousarray(a[-1]), offsets=np.arange(n + 1), "
            "n_ss=np.ones(n, np.int32), t_exp=np.zeros(n)).reshape(-1))")
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "a.npy")
        np.save(path, np.concatenate([p, t[None, :]]))
        subprocess.run([sys.executable, "-c", code, path], check=True, cwd=ROOT)
        return np.load(path)


def planets(rng, n, k_lo, k_hi):
    p = np.zeros((10, n))
    p[W.K], p[W.F] = rng.uniform(k_lo, k_hi, n), rng.uniform(0.0, 0.95, n)
    p[W.THETA], p[W.PHI] = rng.uniform(0.0, np.pi, n), rng.uniform(0.0, 2.0 * np.pi, n)
    p[W.ARS], p[W.P] = ARS, PERIOD
    p[W.Q1], p[W.Q2] = rng.uniform(0.0, 1.0, n), rng.uniform(0.0, 1.0, n)
    return p


def semi_axes(p):
    """Projected semi-axes and the minor axis' direction on the sky."""
    k, f, th, ph = p[W.K], p[W.F], p[W.THETA], p[W.PHI]
    minor = k * np.sqrt(np.cos(th) ** 2 + (1.0 - f) ** 2 * np.sin(th) ** 2)
    return k, minor, np.cos(ph), -np.sin(ph)


def placed(p, x, y):
    """Impact parameters and times that put the centres at (x, y)."""
    al = np.arcsin(y / ARS)
    p[W.B] = x / np.cos(al)
    return p, al * PERIOD / (2.0 * np.pi)


def samples(kind, n, k_lo, k_hi, seed=41):
    rng = np.random.default_rng(seed)
    p = planets(rng, n, k_lo, k_hi)
    a = rng.uniform(0.0, 2.0 * np.pi, n)
    ca, sa = np.cos(a), np.sin(a)
    if kind == "disk":
        r = rng.uniform(0.0, 1.0, n) * (1.0 + p[W.K])
    elif kind == "centre":
        r = 10.0 ** rng.uniform(-9.0, -1.0, n)
    else:  # the farthest point of the ellipse at 1 - eps
        eps = 10.0 ** rng.uniform(-9.0, -0.5, n)
        maj, mnr, ux, uy = semi_axes(p)
        th = np.linspace(0.0, 2.0 * np.pi, 257)[:-1, None]
        ex = maj * np.cos(th) * -uy + mnr * np.sin(th) * ux
        ey = maj * np.cos(th) * ux + mnr * np.sin(th) * uy
        lo, hi = np.zeros(n), np.ones(n)
        for _ in range(40):
            m = 0.5 * (lo + hi)
            out = np.max((m * ca + ex) ** 2 + (m * sa + ey) ** 2, axis=0) > (1.0 - eps) ** 2
            lo, hi = np.where(out, lo, m), np.where(out, m, hi)
        r = lo
    return placed(p, r * ca, r * sa)


def compare(check, tmp_path, p, t):
    direct, general, cls = run(check, tmp_path, p, t)
    assert np.all(np.isfinite(general))
    took = np.isfinite(direct) & (cls != -2)
    diff = np.where(took, np.abs(direct - general), 0.0)
    assert diff.max() <= TOL
    worst = np.argsort(diff)[-50:]
    ref = oracle_flux(np.ascontiguousarray(p[:, worst]), t[worst])
    assert np.abs(direct[worst] - ref)[took[worst]].max() <= TOL
    return took, cls


@pytest.mark.parametrize("kind", ["disk", "limb", "centre"])
@pytest.mark.parametrize("k_lo,k_hi", [(0.5, 0.8), (0.8, 0.95), (0.95, 0.999)])
def test_large_planets(check, tmp_path, kind, k_lo, k_hi):
    p, t = samples(kind, 20000, k_lo, k_hi)
    took, cls = compare(check, tmp_path, p, t)
    assert took.sum() > 2000
    if kind == "disk":
        # outlines around the star's centre are accepted (they and those near
        # it, which can take too long an order, are 0.15 to 0.65 of the samples)
        assert np.sum(cls[~took] == -1) <= 0.15 * np.sum(cls != -2)


@pytest.mark.parametrize("k_lo,k_hi", [(0.5, 0.7), (0.7, 0.9), (0.9, 0.999)])
def test_crossing_arcs(check, tmp_path, k_lo, k_hi):
    # no further from the oracle than the general path, which they replace
    p, t = samples("disk", 12000, k_lo, k_hi, seed=7)
    direct, general, cls = run(check, tmp_path, p, t)
    m = np.isfinite(direct) & (cls == -1)
    assert m.sum() > 2000
    ref = oracle_flux(np.ascontiguousarray(p[:, m]), t[m])
    rms = lambda f: np.sqrt(np.mean((f[m] - ref) ** 2))
    assert rms(direct) <= rms(general)


@pytest.mark.parametrize("locked", [False, True])
def test_large_ellipsoids(check, tmp_path, locked):
    rng = np.random.default_rng(43)
    n = 20000
    p = W.draw_ellipsoids(rng, n, locked)
    p[:3] = 10.0 ** rng.uniform(-1.0, np.log10(0.99), (3, n))
    k = np.max(p[:3], axis=0)
    p[W.E_ARS] = rng.uniform(2.5, 20.0, n)
    p[W.E_B] = rng.uniform(0.0, 1.0, n)
    reach = np.arcsin(np.minimum(1.0, (1.0 + k) / p[W.E_ARS])) / (2.0 * np.pi) * p[W.E_P]
    took, cls = compare(check, tmp_path, p, p[W.E_T0] + rng.uniform(-1.0, 1.0, n) * reach)
    assert took.sum() > 4000


def test_known_samples(check, tmp_path):
    # close to the limb on both sides: off by 4.0e-7 with an order from the near
    # side's zeros alone; a needle (f = 0.999996), off by 3.8e-10 with an order
    # without the quartic's complex pair
    p = np.array([[0.960440290366926, 0.47358153665846714, 1.7029063907121635, 6.160755649334051, 0.0034152288856442643,
                   201.77358757001537, 500.0, 0.0, 0.81225802445182, 0.028127730765128867],
                  [0.19752358398605882, 0.99999579031346308, 1.5853178409309001, 4.2426871421488102, 0.0, 200.0, 500.0, 0.0,
                   1.0, 0.5]]).T
    q, t1 = placed(np.ascontiguousarray(p[:, 1:]), np.array([-0.4746243309247809]), np.array([0.85719980323387412]))
    p = np.concatenate([p[:, :1], q], axis=1)
    t = np.array([0.008177178922197671, t1[0]])
    direct, general, _ = run(check, tmp_path, p, t)
    assert np.abs(direct - oracle_flux(p, t)).max() <= 1e-11


# rounding of fluxes near 1, and the oracle's own error, which both sides share
@pytest.mark.parametrize("kind", ["disk", "limb"])
@pytest.mark.parametrize("k_lo,k_hi", [(0.005, 0.05), (0.05, 0.12), (0.12, 0.2), (0.2, 0.35)])
def test_no_further_off_than_the_general_path(check, tmp_path, kind, k_lo, k_hi):
    p, t = samples(kind, 8000, k_lo, k_hi, seed=79)
    direct, general, cls = run(check, tmp_path, p, t)
    ref = oracle_flux(p, t)
    for m in (np.isfinite(direct) & (cls >= 0), np.isfinite(direct) & (cls == -1)):
        assert m.sum() > 200
        rms = lambda f: np.sqrt(np.mean((f[m] - ref[m]) ** 2))
        assert rms(direct) <= 1.05 * rms(general) + 1e-15

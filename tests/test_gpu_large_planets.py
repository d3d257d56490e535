"""The fused pass on large planets, where the direct rules decline samples: units
that hold declined and accepted samples, more declined ones than a wavefront or
a workgroup has lanes, and crossings around the star's centre."""
import os
import subprocess
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu
TOL = 1e-9  # the exact path's bar


def planets(n, k_lo, k_hi):
    from paper_2410_05408_amd import workloads as W
    rng = np.random.default_rng(17)
    p = W.walker_batch(n_sets=n).params
    p[W.K], p[W.F], p[W.B] = rng.uniform(k_lo, k_hi, n), rng.uniform(0.0, 0.9, n), rng.uniform(0.0, 0.9, n)
    p[W.T0] = 0.0
    return np.ascontiguousarray(p)


def oracle(tmp_path, p, times, ss, te):
    # in a process of its own: the oracle counts integrals that stop above
    # their target, which other tests read
    code = ("import sys, numpy as np; from oracle import glo; a = np.load(sys.argv[1]); p = a['p']; "
            "f = glo.flux_batch if p.shape[0] == 10 else glo.flux_batch_ell; "
            "np.save(sys.argv[2], f(p, a['t'], n_ss=a['ss'], t_exp=a['te']))")
    a, b = str(tmp_path / "in.npz"), str(tmp_path / "out.npy")
    np.savez(a, p=p, t=times, ss=ss, te=te)
    subprocess.run([sys.executable, "-c", code, a, b], check=True, cwd=ROOT)
    return np.load(b).reshape(p.shape[1], -1)


def check(gl, ctx, p, times, n_ss, t_exp, tmp_path):
    import torch
    n = p.shape[1]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ss, te = np.full(n, n_ss, np.int32), np.full(n, t_exp)
    got = ctx.batch(dev(p), dev(times), n_ss=dev(ss), t_exp=dev(te))
    torch.cuda.synchronize()
    assert gl.gl_ctx_sync_status(ctx.handle) == gl.GL_OK
    got = got.cpu().numpy().reshape(n, -1)
    ref = oracle(tmp_path, p, times, ss, te)
    assert np.abs(got - ref).max() <= TOL
    return got


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("k_lo,k_hi", [(0.3, 0.5), (0.5, 0.8), (0.8, 0.999)])
@pytest.mark.parametrize("n_times,n_ss", [(65, 1), (700, 1), (257, 5), (40, 64)])
def test_mixed_units(gpu_lib, ctx, tmp_path, k_lo, k_hi, n_times, n_ss):
    print(f"case: k {k_lo} to {k_hi}, 6 sets of {n_times} outputs of {n_ss} sub-samples", flush=True)
    check(gpu_lib, ctx, planets(6, k_lo, k_hi), np.linspace(-0.6, 0.6, n_times), n_ss, 0.01, tmp_path)


def test_whole_units_declined(gpu_lib, ctx, tmp_path):
    # every sample of the middle units declined, more than a workgroup's threads
    from paper_2410_05408_amd import workloads as W
    print("case: concentric spheres of nearly the star's size, 3 sets of 1500 outputs of 1 sub-sample", flush=True)
    p = planets(3, 0.9, 0.95)
    p[W.K], p[W.F], p[W.B] = [0.999, 0.9995, 0.99], 0.02, 0.0
    check(gpu_lib, ctx, p, np.linspace(-4e-3, 4e-3, 1500), 1, 0.0, tmp_path)


def test_a_set_alone(gpu_lib, ctx, tmp_path):
    # an output is the same whatever shares its batch, by the largest order and
    # by the general path alike
    print("case: 5 sets of 300 outputs of 3 sub-samples, together and one by one", flush=True)
    p, t = planets(5, 0.4, 0.95), np.linspace(-0.6, 0.6, 300)
    got = check(gpu_lib, ctx, p, t, 3, 0.01, tmp_path)
    for s in range(5):
        one = check(gpu_lib, ctx, np.ascontiguousarray(p[:, s:s + 1]), t, 3, 0.01, tmp_path)
        assert np.abs(one - got[s:s + 1]).max() <= 64 * 2.3e-16


@pytest.mark.parametrize("locked", [0, 1])
def test_ellipsoids(gpu_lib, ctx, tmp_path, locked):
    import torch
    from paper_2410_05408_amd import workloads as W
    print(f"case: 8 ellipsoids of semi-axes to 0.99, locked {locked}", flush=True)
    rng = np.random.default_rng(19)
    p = W.draw_ellipsoids(rng, 8, bool(locked))
    p[:3] = rng.uniform(0.3, 0.99, (3, 8))
    p[W.E_ARS], p[W.E_P] = 4.0, 2.0
    t, ss, te = np.linspace(-0.2, 0.2, 301), np.array([1, 3] * 4, np.int32), np.full(8, 1e-3)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = torch.empty(8 * t.size, dtype=torch.float64, device="cuda")
    gpu_lib.gl_lightcurve_batch_ellipsoid(ctx.handle, dev(p), dev(t), out, n_ss=dev(ss), t_exp=dev(te))
    torch.cuda.synchronize()
    assert gpu_lib.gl_ctx_sync_status(ctx.handle) == gpu_lib.GL_OK
    assert np.abs(out.cpu().numpy().reshape(8, -1) - oracle(tmp_path, p, t, ss, te)).max() <= TOL

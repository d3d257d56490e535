"""The fused pass at the edges of its splits: outputs per workgroup, outputs and
sub-samples per sorted unit, tiles of a wavefront, sets without outputs, and a
workgroup whose outputs all need the general path."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL = 1e-9  # the exact path's bar


@pytest.fixture(scope="module")
def ctx(gpu_lib):
    c = gpu_lib.Context(0)
    yield c
    c.close()


def flux(gl, ctx, w):
    import torch
    d = gl.to_device(w, "cuda:0")
    kw = dict(offsets=d["offsets"], n_ss=d["n_ss"], t_exp=d["t_exp"])
    a = ctx.batch(d["params"], d["times"], **kw)
    torch.cuda.synchronize()
    assert gl.gl_ctx_sync_status(ctx.handle) == gl.GL_OK
    assert gl.gl_ctx_get_unconverged(ctx.handle) == 0
    return a.cpu().numpy().reshape(-1)


@pytest.mark.parametrize("n_sets,n_times,n_ss", [
    (1, 1, 1), (3, 63, 64), (2, 64, 1), (5, 65, 3), (1, 127, 2), (2, 128, 64), (3, 129, 17), (1, 1023, 1), (1, 1024, 1),
    (1, 1025, 1), (2, 2049, 2), (1000, 640, 1), (1200, 2047, 1), (700, 4096, 1), (300, 4097, 3), (130, 16385, 1)])
def test_shared_grid(gpu_lib, ctx, oracle, n_sets, n_times, n_ss):
    from paper_2410_05408_amd import workloads as W
    print(f"case: {n_sets} sets of {n_times} outputs of {n_ss} sub-samples", flush=True)
    p = W.walker_batch(n_sets=max(n_sets, 2)).params[:, :n_sets]
    p[W.B] *= 0.8
    w = W.Workload("edge", np.ascontiguousarray(p), np.linspace(-0.25, 0.3, n_times) if n_times > 1 else np.array([0.01]), None,
                   np.full(n_sets, n_ss, np.int32), np.full(n_sets, 0.01), {})
    got = flux(gpu_lib, ctx, w).reshape(n_sets, n_times)
    pick = np.unique(np.linspace(0, n_sets - 1, min(n_sets, 12)).astype(int))
    ref = oracle.flux_batch(np.ascontiguousarray(p[:, pick]), w.times, n_ss=w.n_ss[pick], t_exp=w.t_exp[pick])
    assert np.abs(got[pick] - ref.reshape(pick.size, -1)).max() <= TOL
    assert np.isfinite(got).all() and got.max() <= 1.0 + 1e-12


@pytest.mark.parametrize("lens", [[0, 127, 0, 0, 128, 129, 1], [2048, 2049, 4095, 0, 4097], [20000, 1, 9000, 9001]])
def test_own_grids(gpu_lib, ctx, oracle, lens):
    from paper_2410_05408_amd import workloads as W
    print(f"case: own grids of {lens}", flush=True)
    n = len(lens)
    p = W.walker_batch(n_sets=n).params
    p[W.B] *= 0.8
    w = W.Workload("own", p, np.concatenate([np.linspace(-0.2, 0.2, m) for m in lens]),
                   np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), np.array([1, 64, 15, 2, 3, 1, 5][:n], np.int32),
                   np.full(n, 0.01), {})
    got = flux(gpu_lib, ctx, w)
    ref = oracle.flux_batch(w.params, w.times, offsets=w.offsets, n_ss=w.n_ss, t_exp=w.t_exp)
    assert np.abs(got - ref.reshape(-1)).max() <= TOL


def test_every_sample_declined(gpu_lib, ctx, oracle):
    # a sphere of nearly the star's size concentric with it at mid-transit:
    # its limb and the star's are close everywhere, which no direct rule takes
    from paper_2410_05408_amd import workloads as W
    p = W.walker_batch(n_sets=2).params
    p[W.K] = [0.999, 0.9995]
    p[W.F] = 0.02
    p[W.B] = 0.0
    w = W.Workload("declined", p, np.linspace(-2e-4, 2e-4, 200), None, np.full(2, 3, np.int32), np.full(2, 1e-5), {})
    got = flux(gpu_lib, ctx, w).reshape(2, -1)
    ref = oracle.flux_batch(w.params, w.times, n_ss=w.n_ss, t_exp=w.t_exp)
    assert np.abs(got - ref.reshape(2, -1)).max() <= TOL


@pytest.mark.parametrize("lens", [[1, 0, 129, 63], [1500, 2049, 128, 1023]])
def test_ellipsoids_own_grids(gpu_lib, ctx, oracle, lens):
    # locked and free sets of one batch, single and several sub-samples
    import torch
    from paper_2410_05408_amd import workloads as W
    print(f"case: ellipsoids on own grids of {lens}", flush=True)
    rng = np.random.default_rng(31)
    n = len(lens)
    p = np.concatenate([W.draw_ellipsoids(rng, 1, i % 2 == 0) for i in range(n)], axis=1)
    reach = np.arcsin(np.minimum(1.0, 1.3 / p[W.E_ARS])) / (2.0 * np.pi) * p[W.E_P]
    times = np.concatenate([p[W.E_T0, i] + reach[i] * np.linspace(-1, 1, m) for i, m in enumerate(lens)])
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ss, te = np.array([1, 3, 64, 2], np.int32), 0.01 * reach
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    out = ctx.batch_ellipsoid(dev(p), dev(times), offsets=dev(off), n_ss=dev(ss), t_exp=dev(te))
    torch.cuda.synchronize()
    assert gpu_lib.gl_ctx_sync_status(ctx.handle) == gpu_lib.GL_OK
    ref = oracle.flux_batch_ell(p, times, offsets=off, n_ss=ss, t_exp=te)
    assert np.abs(out.cpu().numpy().reshape(-1) - ref.reshape(-1)).max() <= TOL


def test_more_outputs_than_one_row_of_workgroups(gpu_lib, ctx, oracle):
    # own grids of 2^31 outputs and more: their workgroups, counted at their
    # smallest, pass what one dimension of a launch holds
    import torch
    from paper_2410_05408_amd import workloads as W
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    n, tail = (1 << 31) + 4097, 301
    print(f"case: own grids of {n} outputs in three sets", flush=True)
    p = W.walker_batch(n_sets=3).params
    p[W.B] *= 0.8
    off = np.array([0, 1 << 30, n - tail, n], np.int64)
    ss, te = np.array([1, 5, 3], np.int32), np.full(3, 0.01)
    t = np.linspace(-0.2, 0.2, tail)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    times = torch.full((n,), 50.0, dtype=torch.float64, device="cuda")  # out of transit
    times[-tail:] = dev(t)
    out = torch.zeros(n, dtype=torch.float64, device="cuda")
    ctx.batch(dev(p), times, offsets=dev(off), n_ss=dev(ss), t_exp=dev(te), out=out)
    torch.cuda.synchronize()
    assert gpu_lib.gl_ctx_sync_status(ctx.handle) == gpu_lib.GL_OK
    assert all(bool((c == 1.0).all()) for c in out[:-tail].split(1 << 28))
    ref = oracle.flux_batch(np.ascontiguousarray(p[:, 2:]), t, n_ss=ss[2:], t_exp=te[2:]).reshape(-1)
    assert np.abs(out[-tail:].cpu().numpy() - ref).max() <= TOL


@pytest.mark.parametrize("n_times,shift", [(1, 0), (127, 1), (128, 0), (2047, 1), (2048, 0), (2049, 1), (4095, 0), (6145, 1)])
def test_window_edges_and_values(gpu_lib, ctx, oracle, n_times, shift):
    # ends of the 128 and 2048 outputs the window test takes together, times
    # that are not finite, an invalid set, rows and tensors on 8-byte
    # boundaries only
    import torch
    from paper_2410_05408_amd import workloads as W
    print(f"case: window test of {n_times} outputs, tensors {8 * shift} bytes on", flush=True)
    p = W.walker_batch(n_sets=5).params
    p[W.B] *= 0.8
    p[W.K, 3] = -1.0
    t = np.linspace(-4.0, 0.02, n_times) if n_times > 1 else np.array([0.01])
    bad = np.array([0, n_times // 2, n_times - 1]) if n_times > 1 else np.array([], int)
    te, ss = np.full(5, 0.01), np.array([1, 2, 3, 1, 5], np.int32)
    good = [0, 1, 2, 4]
    ref = np.full((5, n_times), np.nan)
    ref[good] = oracle.flux_batch(np.ascontiguousarray(p[:, good]), t, n_ss=ss[good], t_exp=te[good]).reshape(4, -1)
    tv = t.copy()
    tv[bad] = np.array([np.nan, np.inf, -np.inf])[:bad.size]
    ref[:, bad] = np.nan
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    times = torch.zeros(n_times + 1, dtype=torch.float64, device="cuda")[shift:shift + n_times]
    times.copy_(dev(tv))
    out = torch.full((5 * n_times + 2,), 7.0, dtype=torch.float64, device="cuda")
    res = out[shift:shift + 5 * n_times]
    ctx.batch(dev(p), times, out=res, n_ss=dev(ss), t_exp=dev(te))
    torch.cuda.synchronize()
    assert gpu_lib.gl_ctx_sync_status(ctx.handle) == gpu_lib.GL_ERR_DOMAIN  # the invalid set, and the times
    got = res.cpu().numpy().reshape(5, n_times)
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    if not np.isnan(ref).all():
        assert np.nanmax(np.abs(got - ref)) <= TOL
    assert bool((out[:shift] == 7.0).all()) and bool((out[shift + 5 * n_times:] == 7.0).all())


@pytest.mark.parametrize("n_sets", [1, 63, 65, 255, 256, 257])
def test_own_grids_by_number_of_sets(gpu_lib, ctx, oracle, n_sets):
    # up to 256 sets their workgroups are counted and placed by one workgroup
    from paper_2410_05408_amd import workloads as W
    print(f"case: {n_sets} own grids", flush=True)
    rng = np.random.default_rng(n_sets)
    lens = rng.integers(0, 400, n_sets)
    lens[rng.random(n_sets) < 0.2] = 0
    lens[-1] = 129
    p = W.walker_batch(n_sets=max(n_sets, 2)).params[:, :n_sets].copy()
    p[W.B] *= 0.8
    w = W.Workload("own", p, np.concatenate([np.linspace(-0.2, 0.2, max(m, 1))[:m] for m in lens]),
                   np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), rng.integers(1, 6, n_sets).astype(np.int32),
                   np.full(n_sets, 0.01), {})
    got = flux(gpu_lib, ctx, w)
    ref = oracle.flux_batch(w.params, w.times, offsets=w.offsets, n_ss=w.n_ss, t_exp=w.t_exp)
    assert np.abs(got - ref.reshape(-1)).max() <= TOL


def test_bits_of_a_sample_alone(gpu_lib, ctx):
    # long arcs (near the inner tangency) by the hundred in a unit, and each one
    # the only output of a set: 1 and 4 lanes per sample, the same bits
    from paper_2410_05408_amd import workloads as W
    print("case: 4 sets of 900 grazing outputs, together and one by one", flush=True)
    rng = np.random.default_rng(29)
    p = W.walker_batch(n_sets=4).params
    p[W.K], p[W.F], p[W.T0] = [0.06, 0.1, 0.12, 0.3], [0.1, 0.0, 0.3, 0.2], 0.0
    p[W.B] = 1.0 - 0.97 * p[W.K]
    t = rng.uniform(-0.06, 0.06, 900)
    one = np.ones(4, np.int32)
    got = flux(gpu_lib, ctx, W.Workload("together", np.ascontiguousarray(p), t, None, one, np.zeros(4), {})).reshape(4, -1)
    n = 4 * t.size
    alone = W.Workload("alone", np.ascontiguousarray(np.repeat(p, t.size, axis=1)), np.tile(t, 4),
                       np.arange(n + 1, dtype=np.int64), np.ones(n, np.int32), np.zeros(n), {})
    assert np.array_equal(got, flux(gpu_lib, ctx, alone).reshape(4, -1))


def _many(n, seed):
    # planets up to k = 0.9, some of whose samples the direct rules decline
    from paper_2410_05408_amd import workloads as W
    rng = np.random.default_rng(seed)
    p = W.walker_batch(n_sets=n).params
    p[W.B], p[W.T0] = rng.uniform(0.0, 1.0, n), 0.0
    p[W.K, ::7] = rng.uniform(0.2, 0.9, p[W.K, ::7].size)
    p[W.P, 11] = -1.0  # an invalid set
    return np.ascontiguousarray(p)


def _in_parts(run, n, *cols):
    # the same sets in batches too small for workgroups of one wavefront
    return np.concatenate([run(*(None if c is None else np.ascontiguousarray(c[..., a:a + 1500]) for c in cols))
                           for a in range(0, n, 1500)])


@pytest.mark.parametrize("n_sets,n_times,n_ss", [(4096, 1, 64), (4100, 4, 0), (4097, 128, None), (4099, 65, None),
                                                 (16384, 16, 15), (16385, 13, 0), (33000, 32, 5)])
def test_many_small_sets_shared(gpu_lib, ctx, n_sets, n_times, n_ss):
    import torch
    print(f"case: {n_sets} sets of {n_times} shared outputs of {n_ss} sub-samples", flush=True)
    p, t = _many(n_sets, 3), np.linspace(-0.3, 0.35, n_times) if n_times > 1 else np.array([0.05])
    if n_times > 2:
        t[1] = np.nan
    ss = None if n_ss is None else np.random.default_rng(5).integers(1, 65, n_sets).astype(np.int32) if n_ss == 0 else \
        np.full(n_sets, n_ss, np.int32)
    te = np.full(n_sets, 0.02)
    dev = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()

    def run(p, ss, te):
        out = ctx.batch(dev(p), dev(t), n_ss=dev(ss), t_exp=dev(te)).cpu().numpy().reshape(p.shape[1], -1)
        gpu_lib.gl_ctx_sync_status(ctx.handle)
        return out

    got = run(p, ss, te)
    assert np.array_equal(got, _in_parts(run, n_sets, p, ss, te), equal_nan=True)
    ok = np.delete(got, 11, axis=0)
    assert np.isnan(got[11]).all() and np.isfinite(np.delete(ok, 1, axis=1) if n_times > 2 else ok).all()


@pytest.mark.parametrize("kind", ["oblate", "ellipsoid"])
def test_many_small_sets_own(gpu_lib, ctx, kind):
    import torch
    from paper_2410_05408_amd import workloads as W
    print(f"case: 5000 own grids of 0 to 7 outputs and two of 300 and 129, {kind}", flush=True)
    n, rng = 5000, np.random.default_rng(8)
    p = _many(n, 4) if kind == "oblate" else np.concatenate([W.draw_ellipsoids(rng, n // 2, True), W.draw_ellipsoids(rng, n // 2, False)], axis=1)
    lens = rng.integers(0, 8, n)
    lens[[17, 4000]] = 300, 129
    ss, te = rng.integers(1, 20, n).astype(np.int32), np.full(n, 0.01)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    t = rng.uniform(-0.3, 0.3, off[-1])
    t[off[17] + 150] = np.inf
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    call = ctx.batch if kind == "oblate" else ctx.batch_ellipsoid

    def run(a, e):
        out = call(dev(p[:, a:e]), dev(t[off[a]:off[e]]), offsets=dev(off[a:e + 1] - off[a]), n_ss=dev(ss[a:e]), t_exp=dev(te[a:e]))
        out = out.cpu().numpy()
        gpu_lib.gl_ctx_sync_status(ctx.handle)
        return out

    got = run(0, n)
    assert np.array_equal(got, np.concatenate([run(a, min(n, a + 1500)) for a in range(0, n, 1500)]), equal_nan=True)
    assert np.isnan(got[off[17] + 150]) and np.isfinite(np.delete(got[off[12]:], off[17] + 150 - off[12])).all()


def test_many_small_sets_other_calls(gpu_lib, ctx):
    # the allocation-free call, a timed batch and a census give the same bits
    import torch
    gl = gpu_lib
    print("case: 4500 sets of 4 shared outputs of 3 sub-samples by every call", flush=True)
    n, t = 4500, np.linspace(-0.2, 0.2, 4)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    d, td, ss, te = dev(_many(n, 6)), dev(t), dev(np.full(n, 3, np.int32)), dev(np.full(n, 0.01))
    new = lambda: torch.full((n * 4,), -1.0, dtype=torch.float64, device="cuda")
    outs = [new() for _ in range(4)]
    gl.gl_lightcurve_batch(ctx.handle, d, td, outs[0], n_ss=ss, t_exp=te)
    gl.gl_lightcurve_batch_noalloc(d, td, outs[1], n_ss=ss, t_exp=te)
    gl.gl_ctx_set_timing(ctx.handle, 1)
    gl.gl_lightcurve_batch(ctx.handle, d, td, outs[2], n_ss=ss, t_exp=te)
    gl.gl_ctx_set_timing(ctx.handle, 0)
    census = gl.gl_census(ctx.handle, d, td, outs[3], n_ss=ss, t_exp=te)
    torch.cuda.synchronize()
    gl.gl_ctx_sync_status(ctx.handle)
    assert census["sub_in_window"] > 4 * n
    for o in outs[1:]:
        assert np.array_equal(outs[0].cpu().numpy(), o.cpu().numpy(), equal_nan=True)


@pytest.mark.parametrize("own", [False, True])
@pytest.mark.parametrize("n_sets,n_times", [(1, 100), (3, 1009), (16, 130), (40, 300)])
def test_few_sets_of_many_sub_samples(gpu_lib, ctx, n_sets, n_times, own):
    # ranges halved by each set's n_ss: the same bits as each output on its own
    from paper_2410_05408_amd import workloads as W
    print(f"case: {n_sets} sets of {n_times} outputs of 1 to 64 sub-samples, own grids {own}", flush=True)
    rng = np.random.default_rng(12)
    p = W.walker_batch(n_sets=max(2, n_sets)).params[:, :n_sets]
    p[W.T0] = 0.0
    t = np.linspace(-0.25, 0.25, n_times)
    ss, te = rng.integers(1, 65, n_sets).astype(np.int32), np.full(n_sets, 0.004)
    ss[0] = 64
    off = np.arange(n_sets + 1, dtype=np.int64) * n_times
    w = W.Workload("few", np.ascontiguousarray(p), np.tile(t, n_sets) if own else t, off if own else None, ss, te, {})
    got = flux(gpu_lib, ctx, w)
    n = n_sets * n_times
    alone = W.Workload("alone", np.ascontiguousarray(np.repeat(p, n_times, axis=1)), np.tile(t, n_sets), np.arange(n + 1, dtype=np.int64),
                       np.repeat(ss, n_times), np.repeat(te, n_times), {})
    assert np.array_equal(got, flux(gpu_lib, ctx, alone))

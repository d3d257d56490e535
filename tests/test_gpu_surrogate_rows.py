"""The network's rows of a gated batch: in order and complete over tile and unit
edges, and exact outputs for the units that find no room for theirs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _surrogate(gl, ctx, path):
    from paper_2410_05408_amd import surrogate
    rng = np.random.default_rng(3)
    w = (0.05 * rng.standard_normal(gl.gl_mlp_num_params())).astype(np.float32)
    bins = 24 * 8
    gl.gl_surrogate_file_write(path, gl.gl_surrogate_config_default(), w, np.zeros_like(w), np.zeros_like(w), 0,
                               np.full(bins, 1e-9, np.float32), np.zeros(bins, np.uint8), np.full(bins, 5000, np.int32))
    return surrogate.Surrogate.load(ctx, path)


# rows: fewer than a tile, several units, more than the first batch makes room for
@pytest.mark.parametrize("n_sets,n_times,n_ss", [(1, 1, 1), (2, 65, 3), (5, 700, 2), (3, 100, 64)])
def test_rows_complete(gpu_lib, tmp_path, n_sets, n_times, n_ss):
    import torch
    from paper_2410_05408_amd import workloads as W
    gl = gpu_lib
    print(f"case: {n_sets} sets of {n_times} outputs of {n_ss} sub-samples", flush=True)
    p = W.walker_batch(n_sets=max(2, n_sets)).params[:, :n_sets]
    p[W.B] = 0.3
    p[W.T0] = 0.0
    times, te = np.linspace(-0.05, 0.06, n_times), 1e-3
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()

    def run(ctx, sur, t, nss, texp):
        d = {"params": dev(p), "times": dev(t), "offsets": None, "n_ss": dev(np.full(n_sets, nss, np.int32)),
             "t_exp": dev(np.full(n_sets, texp))}
        out = torch.empty(n_sets * t.size, dtype=torch.float64, device="cuda")
        n_sub, n_fb = sur.lightcurve(d, out, tol=1e-6)
        assert (n_sub, n_fb) == (n_sets * t.size * nss, 0)
        return out.cpu().numpy().reshape(n_sets, t.size), d

    ctx = gl.Context(0)
    sur = _surrogate(gl, ctx, str(tmp_path / "s.bin"))
    first, d = run(ctx, sur, times, n_ss, te)
    again, _ = run(ctx, sur, times, n_ss, te)
    exact = ctx.batch(d["params"], d["times"], n_ss=d["n_ss"], t_exp=d["t_exp"]).cpu().numpy().reshape(n_sets, -1)
    # every sub-sample as an output of its own, on a context with room
    ctx1 = gl.Context(0)
    sur1 = _surrogate(gl, ctx1, str(tmp_path / "s.bin"))
    j = (np.arange(n_ss) + 0.5) / n_ss - 0.5
    single, _ = run(ctx1, sur1, (times[:, None] + te * j[None, :]).reshape(-1), 1, 0.0)
    want = single.reshape(n_sets, n_times, n_ss).mean(axis=2)
    assert np.abs(want - exact).max() > 1e-9          # the network does something
    # (sums of at most 64 fluxes of about 1)
    assert np.abs(again - want).max() <= 64 * 2.3e-16 * 2
    one = np.minimum(np.abs(first - want), np.abs(first - exact))
    assert one.max() <= 64 * 2.3e-16 * 2
    if n_ss == 64:
        assert np.any(np.abs(first - exact) <= 64 * 2.3e-16 * 2)
    else:
        assert np.array_equal(first, again)


def test_first_batch_of_two_million_rows(gpu_lib, tmp_path):
    # every sub-sample a network row, 15 per output: the first batch on a context
    # has room for all of them
    import torch
    from paper_2410_05408_amd import workloads as W
    gl = gpu_lib
    n_sets, n_times, n_ss = 70, 2000, 15
    print(f"case: {n_sets} sets of {n_times} outputs of {n_ss} sub-samples", flush=True)
    p = W.walker_batch(n_sets=n_sets).params
    p[W.B], p[W.T0] = 0.3, 0.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = gl.Context(0)
    sur = _surrogate(gl, ctx, str(tmp_path / "s.bin"))
    d = {"params": dev(p), "times": dev(np.linspace(-0.05, 0.06, n_times)), "offsets": None,
         "n_ss": dev(np.full(n_sets, n_ss, np.int32)), "t_exp": dev(np.full(n_sets, 1e-3))}
    outs = []
    for _ in range(2):
        out = torch.empty(n_sets * n_times, dtype=torch.float64, device="cuda")
        assert sur.lightcurve(d, out, tol=1e-6) == (n_sets * n_times * n_ss, 0)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])


def test_many_small_sets(gpu_lib, tmp_path):
    # workgroups of one wavefront: the same bits as in batches of fewer sets
    import torch
    from paper_2410_05408_amd import workloads as W
    gl = gpu_lib
    print("case: 4200 sets of 4 outputs of 5 sub-samples", flush=True)
    n = 4200
    p = W.walker_batch(n_sets=n).params
    p[W.B], p[W.T0] = 0.3, 0.0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    t = np.linspace(-0.3, 0.3, 4)
    ctx = gl.Context(0)
    sur = _surrogate(gl, ctx, str(tmp_path / "s.bin"))

    def run(q):
        m = q.shape[1]
        out = torch.empty(m * t.size, dtype=torch.float64, device="cuda")
        sur.lightcurve({"params": dev(q), "times": dev(t), "offsets": None, "n_ss": dev(np.full(m, 5, np.int32)),
                        "t_exp": dev(np.full(m, 0.02))}, out, tol=1e-6)
        return out.cpu().numpy()

    assert np.array_equal(run(p), np.concatenate([run(p[:, a:a + 1400]) for a in range(0, n, 1400)]))

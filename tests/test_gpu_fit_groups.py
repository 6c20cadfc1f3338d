"""The full grid on both sides of the line between shared knots and one thread
per point, which counts groups of 64 points: 11 x 11 points (two groups) with
2,376 and 2,377 sources, 81 x 81 with 48 and 49; against the oracle.  And the
two kernels against each other: the refit of a source (shared knots) and the
grid of a large catalogue have the same bits, in the mixed form at the points
its FP64 recheck leaves alone.  The mixed form with 20 knots, which one of them
sums in two passes over the cells, is left out: equal to rounding only."""
import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _world(n_src, mixed, seed=5, **kw):
    cfg = synth.small_config(0, n_ant=8, n_time=10, n_src=n_src)
    o = synth.observation(0, cfg)
    o.weight = o.weight.astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(seed)
    cat = synth.catalogue(cfg, rng)
    resid = cfg.noise_sigma_jy * (rng.standard_normal(o.n_rows) + 1j * rng.standard_normal(o.n_rows))
    resid = resid.astype(np.complex64).astype(np.complex128)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64, **kw))
    obs = G.make_obs(o, resid, mixed=mixed)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    return o, cat, resid, ctx, f


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n_src,n_e,step,num_r", [(2376, 11, 0.125, 20), (2377, 11, 0.125, 20), (2377, 11, 0.125, 9),
                                                  (48, 81, 0.02, 23), (49, 81, 0.02, 23), (1, 11, 0.125, 20),
                                                  (300, 5, 0.25, 20)])
def test_grid_matches_oracle(n_src, n_e, step, num_r, mixed):
    o, cat, resid, ctx, f = _world(n_src, mixed, n_e=n_e, e_step=step, num_r=num_r)
    out = G.fit_out_tensors(n_src, n_e)
    ctx.fit_sources(f, out, want_surface=True)
    ctx.sync()
    h = G.host(out)
    p = oracle.Params(n_e=n_e, e_step=step, num_r=num_r)
    for s in sorted({0, n_src // 2, n_src - 1}):
        surf, est = oracle.fit_source(G.oracle_facet(o, resid, cat, s), cat.flux_jy[s], p)
        fin = np.isfinite(surf)
        assert np.array_equal(fin, np.isfinite(h["surface"][s])), s
        d = np.abs(h["surface"][s][fin] - surf[fin])
        tol = G.mixed_delta(est.lmax) if mixed else G.LL_RTOL * np.maximum(1.0, np.abs(surf[fin]))
        assert np.all(d <= tol), (s, d.max())
    f.free()
    ctx.close()


@pytest.mark.parametrize("mixed,num_r", [(False, 20), (False, 23), (False, 7), (True, 23), (True, 7), (True, 31)])
def test_refit_has_the_grids_bits(mixed, num_r):
    torch = G.torch_cuda()
    n = 700
    o, cat, resid, ctx, f = _world(n, mixed, num_r=num_r)
    full = G.fit_out_tensors(n)
    ctx.fit_sources(f, full, want_surface=True)
    redo = np.arange(0, n, 7)
    win = np.tile(np.array([0, 80, 0, 80], np.int32), (n, 1))
    win[redo] = (0, 0, 0, 0)                                  # no valid grid point: refitted
    out = G.fit_out_tensors(n)
    ctx.fit_sources(f, out, mode=1, window=torch.from_numpy(win).to("cuda:0"), want_surface=True, fallback=True)
    ctx.sync()
    a, b = G.host(full), G.host(out)
    assert np.array_equal(np.flatnonzero(b["flags"] & rlf.RLF_FLAG_FALLBACK), redo)
    left = 0
    for s in redo:
        x, y = a["surface"][s], b["surface"][s]
        take = np.isfinite(x)
        if mixed:                                             # not the points either fit evaluated again in FP64
            band = 4.0 * G.mixed_delta(a["lmax"][s])
            take &= (x < a["lmax"][s] - band) & (np.abs(x - a["lmax"][s] - np.log(0.05)) > band)
        assert np.array_equal(np.isfinite(x), np.isfinite(y))
        assert np.array_equal(x[take], y[take]), s
        left += int(take.sum())
    assert left > 1000 * len(redo)
    f.free()
    ctx.close()

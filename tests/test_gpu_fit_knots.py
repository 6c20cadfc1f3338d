"""The likelihood grid with the knots shared by waves (small catalogues, and
the full refit of flagged sources) against the oracle and against the grid of
larger catalogues: the largest catalogue it takes and the first it does not,
grids whose point count is not a multiple of a block's 64 points, knot numbers
that do not fill the waves' blocks of five, and refits of none, of some and of
all sources.  Both kernels add the same terms in another order, so
their ln L agree to the oracle's tolerance."""
import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


def _facets(n_src, p=None, seed=5):
    cfg = synth.small_config(0, n_ant=10, n_time=12, n_src=n_src)
    o = synth.observation(0, cfg)
    rng = np.random.default_rng(seed)
    cat = synth.catalogue(cfg, rng)
    resid = cfg.noise_sigma_jy * (rng.standard_normal(o.n_rows) + 1j * rng.standard_normal(o.n_rows))
    ctx = rlf.Context(0, None, p or rlf.params())
    obs = G.make_obs(o, resid)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    return o, cat, resid, ctx, f


@pytest.mark.parametrize("n_src,n_e,step,num_r", [(1, 81, 0.02, 20), (48, 81, 0.02, 20), (49, 81, 0.02, 20),
                                                  (3, 21, 0.1, 20), (2, 3, 0.5, 20), (2, 81, 0.02, 7),
                                                  (2, 81, 0.02, 23), (2, 81, 0.02, 32), (2, 81, 0.02, 2)])
def test_small_catalogue_grid(n_src, n_e, step, num_r):
    o, cat, resid, ctx, f = _facets(n_src, rlf.params(n_e=n_e, e_step=step, num_r=num_r))
    out = G.fit_out_tensors(n_src, n_e)
    ctx.fit_sources(f, out, want_surface=True)
    ctx.sync()
    h = G.host(out)
    p = oracle.Params(n_e=n_e, e_step=step, num_r=num_r)
    for s in sorted({0, n_src // 2, n_src - 1}):
        surf, est = oracle.fit_source(G.oracle_facet(o, resid, cat, s), cat.flux_jy[s], p)
        G.check_fit(h, s, surf, [est] if n_e < 81 else G.oracle_estimate_variants(surf), h["surface"][s])
    f.free()
    ctx.close()


@pytest.mark.parametrize("n_src,redo", [(6, []), (6, [0, 5]), (700, [0, 255, 256, 511, 699]), (40, list(range(40)))])
def test_refit_of_flagged_sources(n_src, redo):
    import torch
    o, cat, resid, ctx, f = _facets(n_src)
    full = G.fit_out_tensors(n_src)
    ctx.fit_sources(f, full, want_surface=True)
    win = np.tile(np.array([0, 80, 0, 80], np.int32), (n_src, 1))
    win[redo] = (0, 0, 0, 0)                                  # no valid grid point: refitted
    out = G.fit_out_tensors(n_src)
    ctx.fit_sources(f, out, mode=1, window=torch.from_numpy(win).to("cuda:0"), want_surface=True, fallback=True)
    ctx.sync()
    a, b = G.host(full), G.host(out)
    again = (b["flags"] & rlf.RLF_FLAG_FALLBACK) != 0
    assert np.array_equal(np.flatnonzero(again), np.array(redo, dtype=np.int64))
    assert np.array_equal(a["argmax"], b["argmax"]) and np.array_equal(a["n_above"], b["n_above"])
    fin = np.isfinite(a["surface"])
    assert np.array_equal(fin, np.isfinite(b["surface"]))
    d = np.abs(a["surface"][fin] - b["surface"][fin])
    assert np.all(d <= G.LL_RTOL * np.maximum(1.0, np.abs(a["surface"][fin])))
    for k in ("e1", "e2", "s1", "s2", "c12"):
        assert np.max(np.abs(a[k] - b[k])) <= G.E_TOL, k
    f.free()
    ctx.close()

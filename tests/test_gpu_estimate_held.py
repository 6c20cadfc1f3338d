"""The estimate with its grid values held in registers against the oracle: the
smallest grid, grids just below and just above the number a block can hold
(7,168), and the largest, in FP64 and in the mixed form, whose recheck
changes values between the passes."""
import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_e,inv_step", [(3, 2), (87, 50), (89, 50), (101, 50), (255, 127)])
@pytest.mark.parametrize("mixed", [False, True])
def test_estimate_of_held_and_reread_grids(n_e, inv_step, mixed):
    step = 1.0 / inv_step
    cfg = synth.small_config(0, n_ant=8, n_time=8, n_src=2)
    o = synth.observation(0, cfg)
    rng = np.random.default_rng(11)
    cat = synth.catalogue(cfg, rng)
    resid = cfg.noise_sigma_jy * (rng.standard_normal(o.n_rows) + 1j * rng.standard_normal(o.n_rows))
    d = resid
    if mixed:
        d = resid.astype(np.complex64)
        o.weight = o.weight.astype(np.float32).astype(np.float64)
    ctx = rlf.Context(0, None, rlf.params(n_e=n_e, e_step=step,
                                              precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    obs = G.make_obs(o, d, mixed=mixed)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    out = G.fit_out_tensors(2, n_e)
    ctx.fit_sources(f, out, want_surface=True)
    ctx.sync()
    h = G.host(out)
    p = oracle.Params(n_e=n_e, e_step=step)
    i1, i2, e1, e2, valid = oracle.e_grid(n_e, step)
    for s in range(2):
        surf = h["surface"][s]
        assert np.array_equal(np.isfinite(surf), valid)
        est = oracle.estimate(surf, e1, e2, valid, n_e, p.frac, p.bad_sigma, p.bad_sqrtdet)
        # the surface handed out is the one estimated: the same set, sums in another order
        assert int(h["argmax"][s]) == est.argmax and int(h["n_above"][s]) == est.n_above
        assert int(h["flags"][s]) == est.flags and h["lmax"][s] == est.lmax
        for k in ("e1", "e2", "s1", "s2", "c12"):
            assert abs(h[k][s] - getattr(est, k)) <= 1e-9, (s, k)
    f.free()
    ctx.close()

"""Sequential refinement with chunks whose tables are too large for the one
launch that uploads a small chunk's (450 sources: the scale weights; 3,300:
every table and the results), against the same refinement put together from
the public calls: residual of the starting model, then per chunk extraction,
fit and swap of the reliable shapes' models.  Both add the same FP64 terms;
the tolerance is that of the sequential tests against the oracle."""
import dataclasses

import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src,chunk", [(900, 450), (3310, 3300)])
def test_chunks_with_large_tables(n_src, chunk):
    torch = G.torch_cuda()
    cfg = dataclasses.replace(synth.small_config(0, n_ant=6, n_time=4, n_src=n_src), field_deg=0.5)
    o = synth.observation(0, cfg)
    cat = synth.catalogue(cfg, np.random.default_rng(31))
    rng = np.random.default_rng(32)
    vis = cfg.noise_sigma_jy * (rng.standard_normal(o.n_rows) + 1j * rng.standard_normal(o.n_rows))
    ctx = rlf.Context(0)
    obs = G.make_obs(o, vis)
    ctx.model_vis(obs, cat, obs.vis, mode=rlf.RLF_MODEL_ACCUMULATE)
    start = G.circular(cat)
    out = G.fit_out_tensors(n_src, surface=False)
    e1, e2 = ctx.fit_sequential(obs, start, chunk, out, refit_bad=False)
    got = G.host(out)
    cur1, cur2 = np.zeros(n_src), np.zeros(n_src)
    resid = torch.empty_like(obs.vis)
    ctx.model_vis(obs, start, resid, mode=rlf.RLF_MODEL_RESIDUAL)
    n_good = 0
    for c0 in range(0, n_src, chunk):
        idx = np.arange(c0, min(n_src, c0 + chunk))
        sub = start.subset(idx)
        f = ctx.facets_create(obs, sub)
        ctx.extract_facets(obs, sub, resid, f)
        want = G.fit_out_tensors(len(idx), surface=False)
        ctx.fit_sources(f, want)
        ctx.sync()
        f.free()
        w = G.host(want)
        assert np.array_equal(got["flags"][idx], w["flags"]) and np.array_equal(got["argmax"][idx], w["argmax"])
        for k in ("e1", "e2", "s1", "s2"):
            assert np.allclose(got[k][idx], w[k], rtol=0, atol=1e-8, equal_nan=True), k
        ok = (w["flags"] & (rlf.RLF_FLAG_BAD_VAR | rlf.RLF_FLAG_EMPTY)) == 0
        good = idx[ok & np.isfinite(w["e1"]) & np.isfinite(w["e2"]) & (w["e1"] ** 2 + w["e2"] ** 2 < 1)]
        n_good += len(good)
        cur1[good], cur2[good] = w["e1"][good - c0], w["e2"][good - c0]
        if len(good):
            old = start.subset(good)
            ctx.model_vis(obs, old, resid, mode=rlf.RLF_MODEL_ACCUMULATE)
            new = dataclasses.replace(old, e1=cur1[good], e2=cur2[good])
            minus = torch.empty_like(resid)
            ctx.model_vis(obs, new, minus, mode=rlf.RLF_MODEL_WRITE)
            resid -= minus
    assert n_good > 0
    assert np.allclose(e1, cur1, rtol=0, atol=1e-8) and np.allclose(e2, cur2, rtol=0, atol=1e-8)
    ctx.close()

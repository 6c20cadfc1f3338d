"""A facet cell that is NaN (a visibility without a value but with a weight):
ln L is NaN at every valid grid point, with the position fixed and marginalised
alike, and the source is flagged as the fixed-position fit flags it."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n_side", [1, 3, 5, 7])
@pytest.mark.parametrize("n_src", [2, 60])
def test_surface_is_nan(n_src, n_side, mixed):
    rng = np.random.default_rng(n_src)
    rows = 3000
    uvw = [rng.normal(0.0, 3000.0, rows) for _ in range(3)]
    vis = 1e-4 * (rng.standard_normal(rows) + 1j * rng.standard_normal(rows))
    vis[rows // 3] = np.nan
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=n_src), rng)
    obs = G.make_obs(synth.Observation(*uvw, np.array([1.4e9]), np.ones(rows)), vis, mixed=mixed)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    ctx.set_positions(f, n_side, 0.1 if n_side > 1 else 0.0)
    out = G.fit_out_tensors(n_src)
    ctx.fit_sources(f, out, want_surface=True)
    ctx.sync()
    g = G.host(out)
    valid = oracle.e_grid(81, 0.02)[4].reshape(-1)
    assert np.all(np.isnan(g["surface"][:, valid]))
    assert np.all(g["surface"][:, ~valid] == -np.inf)
    assert np.all((g["flags"] & rlf.RLF_FLAG_EMPTY) != 0) and np.all(np.isnan(g["e1"])) and np.all(g["argmax"] == -1)
    f.free()
    ctx.close()

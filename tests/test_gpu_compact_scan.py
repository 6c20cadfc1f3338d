"""Compaction offsets around the numbers of sources where the scan changes (a
block's own up to 1,024 sources) and where a thread starts its second load:
each source's cells, and its likelihood from the folded records, are those of
the source alone."""
import dataclasses

import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src", [1, 2, 256, 258, 1024, 1025])
@pytest.mark.parametrize("mixed", [False, True])
def test_cells_of_a_source_do_not_depend_on_the_others(n_src, mixed):
    rng = np.random.default_rng(n_src)
    rows = 700
    u, v, w = (rng.normal(0.0, s, rows) for s in (4000.0, 4000.0, 50.0))
    resid = (1e-4 * (rng.standard_normal(rows) + 1j * rng.standard_normal(rows))).astype(np.complex64)
    o = synth.Observation(u, v, w, np.array([1.4e9]), np.full(rows, 1e8))
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=n_src), rng)
    obs = G.make_obs(o, resid if mixed else resid.astype(np.complex128), mixed=mixed)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))

    def run(c):
        f = ctx.facets_create(obs, c)
        ctx.extract_facets(obs, c, obs.vis, f)
        out = G.fit_out_tensors(c.n_src, surface=False)
        ctx.fit_sources(f, out)
        ctx.sync()
        got, fit = f.copy(), G.host(out)
        f.free()
        return got, fit

    got, fit = run(cat)
    assert got["offsets"][0] == 0 and len(got["ix"]) >= got["offsets"][n_src]
    for s in sorted({0, n_src // 2, n_src - 1}):
        one, alone = run(cat.subset(np.array([s])))
        a, b = int(got["offsets"][s]), int(got["offsets"][s + 1])
        assert b - a == int(one["offsets"][1])
        for k in ("ix", "iy", "count"):
            assert np.array_equal(got[k][a:b], one[k][:b - a]), (s, k)
        assert np.allclose(got["wsum"][a:b], one["wsum"][:b - a], rtol=1e-12, atol=0)
        assert abs(fit["lmax"][s] - alone["lmax"][0]) <= (1e-4 if mixed else 1e-9) * max(1.0, abs(alone["lmax"][0]))
    ctx.close()

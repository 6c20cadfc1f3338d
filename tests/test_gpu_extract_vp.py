"""The visibility-parallel extraction (small catalogues and observations)
against the oracle at its edges: fewer visibilities than a wave, whole and
ragged steps of 64, odd source numbers (a source group half empty), the
largest catalogue it takes and the first of the source-parallel kernel, small
observations of many sources, flagged visibilities with unusable residuals,
facets entered cell by cell (every visibility in another cell) and a single
cell."""
import dataclasses

import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

CASES = [(1, 1), (63, 2), (64, 1), (65, 3), (129, 2), (1000, 5), (4500, 128), (4500, 129), (9000, 64)]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("rows,n_src", CASES)
@pytest.mark.parametrize("spread", ["cells", "one"])
def test_small_extraction_against_oracle(rows, n_src, mixed, spread):
    rng = np.random.default_rng(rows + n_src)
    scale = 6000.0 if spread == "cells" else 1.0
    u, v, w = (rng.normal(0.0, scale, rows) for _ in range(3))
    weight = rng.uniform(0.5, 1.5, rows) * 1e8
    flagged = rng.random(rows) < 0.1
    if rows > 200:
        flagged[64:192] = True                                # whole steps without a usable visibility
    weight[flagged] = np.where(rng.random(rows) < 0.5, 0.0, -1.0)[flagged]
    weight = weight.astype(np.float32).astype(np.float64)
    resid = 1e-4 * (rng.standard_normal(rows) + 1j * rng.standard_normal(rows))
    resid = resid.astype(np.complex64).astype(np.complex128)
    o = synth.Observation(u, v, w, np.array([1.4e9]), weight)
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=n_src), rng)
    given = resid.copy()
    given[flagged] = np.nan
    obs = G.make_obs(o, given, mixed=mixed)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    got = f.copy()
    big = np.max(np.abs(resid))
    for s in sorted({0, n_src // 2, n_src - 1}):
        ref = G.oracle_facet(o, resid, cat, s)
        if not mixed:
            G.check_facet(got, s, ref, big, cat.flux_jy[s])
            continue
        a, b = int(got["offsets"][s]), int(got["offsets"][s + 1])
        assert np.array_equal(got["ix"][a:b], ref.ix) and np.array_equal(got["iy"][a:b], ref.iy), s
        assert np.array_equal(got["count"][a:b], ref.count), s
        assert np.all(np.abs(got["wsum"][a:b] - ref.wsum) <= np.maximum(1e-15, 2.3e-16 * ref.count) * ref.wsum), s
        assert b == a or np.max(np.abs(got["vbar"][a:b] - ref.vbar)) <= 2e-5 * (big + cat.flux_jy[s]), s
    f.free()
    ctx.close()

"""The facet sizing's maximum over u and v: an outlier at the first, a middle
and the last row, in numbers of rows around one pass of the unrolled loop
(524,288 rows) and far below; with a maximum missed, the outlier's visibility
would fall outside its facet."""
import dataclasses

import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 3, 65537, 524287, 524289])
@pytest.mark.parametrize("where", [0.0, 0.37, 1.0])
@pytest.mark.parametrize("axis", [0, 1])
def test_outlier_is_inside_its_facet(rows, where, axis):
    rng = np.random.default_rng(rows)
    uvw = [rng.uniform(-1.0, 1.0, rows) for _ in range(3)]
    uvw[axis][int(where * (rows - 1))] = -5000.0
    o = synth.Observation(*uvw, np.array([1.4e9]), np.ones(rows))
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=1), rng)
    obs = G.make_obs(o, np.ones(rows, dtype=np.complex128))
    ctx = rlf.Context(0)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    got = f.copy()
    assert int(np.sum(got["count"])) == rows
    cell = np.abs(got["iy" if axis else "ix"])
    theta = rlf.params().K * cat.alpha_arcsec[0] * np.pi / (180.0 * 3600.0)
    assert got["count"][np.argmax(cell)] == 1 and cell.max() == np.rint(5000.0 * (1.4e9 / 299792458.0) * theta)
    f.free()
    ctx.close()

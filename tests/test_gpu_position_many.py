"""The mixed form's position-marginalised grid on both sides of the line between
the kernel whose waves share the knots and the one with all knots in a thread
(15 and 16 sources on the 81 x 81 grid), with numbers of knots that fill and do
not fill the last block of them, against the oracle; tolerance that of the
mixed position test."""
import numpy as np
import pytest

import oracle
from oracle.position import fit_source_pos
from paper_2203_14071_amd import rlf
from tests import gpu_common as G
from tests.test_gpu_position import _field, _gpu_fit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_src", [15, 16])
@pytest.mark.parametrize("n_side,num_r", [(3, 20), (3, 7), (5, 20), (5, 9), (7, 7)])
def test_mixed_surface_matches_oracle(n_side, num_r, n_src):
    o, cat, vis = _field(12, n_src=n_src)
    o.weight = o.weight.astype(np.float32).astype(np.float64)
    vis = vis.astype(np.complex64).astype(np.complex128)
    catc = G.circular(cat)
    resid = vis - oracle.sky_model(o.u_m, o.v_m, o.w_m, o.freq_hz, catc)
    p = oracle.Params(num_r=num_r)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED, num_r=num_r))
    h, _ = _gpu_fit(ctx, o, vis, catc, n_side, 0.15, mixed=True)
    for s in (0, n_src - 1):
        surf, _ = fit_source_pos(G.oracle_facet(o, resid, catc, s), cat.flux_jy[s], n_side, 0.15, p)
        fin = np.isfinite(surf)
        assert np.array_equal(fin, np.isfinite(h["surface"][s]))
        assert np.all(np.abs(h["surface"][s][fin] - surf[fin]) <= 1e-4 * np.maximum(1.0, np.abs(surf[fin]))), s
    ctx.close()

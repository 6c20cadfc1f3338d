"""Refinement on the position-marginalised likelihood with the knots shared by
the waves of a block, against the oracle: every offset grid, with numbers of
knots that leave waves without a knot, fill one walk exactly, and need a
second.  Sources whose oracle result hangs on the last digits (other numbers
of points within the grid's rounding of the threshold) are left out, as in the
position tests; tolerances are theirs."""
import pytest

import oracle
from oracle.position import fit_source_pos
from paper_2203_14071_amd import rlf
from tests import gpu_common as G
from tests.test_gpu_position import _field, _gpu_fit, _robust_refine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_side,num_r", [(3, 7), (3, 20), (5, 20), (5, 23), (7, 9), (7, 20)])
def test_refined_sources_match_oracle(n_side, num_r):
    o, cat, vis = _field(21, n_src=4, noise_scale=0.05)
    catc = G.circular(cat)
    resid = vis - oracle.sky_model(o.u_m, o.v_m, o.w_m, o.freq_hz, catc)
    p = oracle.Params(num_r=num_r)
    ctx = rlf.Context(0, None, rlf.params(num_r=num_r))
    coarse, h = _gpu_fit(ctx, o, vis, catc, n_side, 0.1, refine=True)
    checked = 0
    for s in range(cat.n_src):
        fac = G.oracle_facet(o, resid, catc, s)
        surf, est = fit_source_pos(fac, cat.flux_jy[s], n_side, 0.1, p)
        ref = _robust_refine(fac, cat.flux_jy[s], surf, est, p, (n_side, 0.1))
        if ref is None or int(coarse["n_above"][s]) != est.n_above:
            continue
        checked += 1
        assert int(h["flags"][s]) == ref.flags and int(h["n_above"][s]) == ref.n_above, s
        for k in ("e1", "e2", "s1", "s2", "c12"):
            assert abs(h[k][s] - getattr(ref, k)) <= G.E_TOL, (s, k)
        assert abs(h["lmax"][s] - ref.lmax) <= G.LL_RTOL * max(1.0, abs(ref.lmax))
    assert checked >= 2
    ctx.close()

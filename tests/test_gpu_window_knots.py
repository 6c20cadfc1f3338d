"""Narrowed fits with the knots shared by waves against the full grid: boxes of
one point, ragged in the 64 positions of a block, partly off the grid, empty
and whole, with and without the lattice outside the box, for catalogues on
both sides of the numbers that choose the kernel and with boxes on both sides
of the size that splits a launch.  All kernels add the same terms in the same
order, so every evaluated point has the full grid's bits."""
import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu

N_E = 81


@pytest.mark.parametrize("n_src,num_r", [(1, 20), (40, 20), (40, 7), (80, 20), (81, 20), (1001, 20), (1501, 20)])
@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("stride", [0, 4])
def test_window_points_are_those_of_the_full_grid(n_src, num_r, mixed, stride):
    import torch
    cfg = synth.small_config(0, n_ant=8, n_time=8, n_src=n_src)
    o = synth.observation(0, cfg)
    rng = np.random.default_rng(n_src)
    cat = synth.catalogue(cfg, rng)
    resid = cfg.noise_sigma_jy * (rng.standard_normal(o.n_rows) + 1j * rng.standard_normal(o.n_rows))
    if mixed:
        resid = resid.astype(np.complex64)
        o.weight = o.weight.astype(np.float32).astype(np.float64)
    ctx = rlf.Context(0, None, rlf.params(num_r=num_r, precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    obs = G.make_obs(o, resid, mixed=mixed)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, obs.vis, f)
    full, out = G.fit_out_tensors(n_src), G.fit_out_tensors(n_src)
    ctx.fit_sources(f, full, want_surface=True)
    boxes = np.array([[40, 40, 40, 40], [30, 37, 50, 58], [-5, 6, 30, 90], [20, 19, 0, 80], [0, 80, 0, 80],
                      [33, 40, 33, 41], [10, 30, 10, 29]], np.int32)
    win = boxes[np.arange(n_src) % len(boxes)]
    ctx.fit_sources(f, out, mode=1, window=torch.from_numpy(win).to("cuda:0"), want_surface=True,
                    fallback=stride > 0, check_stride=stride)
    ctx.sync()
    a, b = G.host(full), G.host(out)
    i1, i2 = np.divmod(np.arange(N_E * N_E), N_E)
    valid = (i1 - 40) ** 2 + (i2 - 40) ** 2 < 2500
    for s in range(0, n_src, max(1, n_src // 60)):
        w = win[s]
        again = bool(b["flags"][s] & rlf.RLF_FLAG_FALLBACK)
        inside = valid & (i1 >= w[0]) & (i1 <= w[1]) & (i2 >= w[2]) & (i2 <= w[3]) | (valid & again)
        sf, sb = a["surface"][s].reshape(-1), b["surface"][s].reshape(-1)
        assert np.array_equal(np.isfinite(sb), inside), s
        same = sf[inside] == sb[inside]
        # the mixed form re-evaluates in FP64 the points that decide its own maximum and threshold
        assert np.all(same) if not mixed else np.all(
            np.abs(sf[inside] - sb[inside])[~same] <= G.mixed_delta(np.max(np.abs(sf[inside]), initial=0.0))), s
    f.free()
    ctx.close()

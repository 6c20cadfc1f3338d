"""What a captured pass runs: on facets with position offsets its likelihood is
the marginalised one, as rlf_fit_sources' on the same facets; where the work
queue is captured (mixed form, 400 sources and more, knot numbers other than 20
above 8) it gives the fit's numbers.  With every tile in the table creation
times nothing and leaves the output arrays alone."""
import numpy as np
import pytest

from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G

pytestmark = pytest.mark.gpu



def _tol(lmax, mixed):
    """Between two extractions of the same data: their atomic sums differ in
    the last bits, the mixed form's FP32 records by at most one unit (2^-24
    relative), which moves ln L by a few 2^-24 of its terms (16 of the bound
    mixed_delta puts on all of its rounding)."""
    return G.mixed_delta(lmax) / 16.0 if mixed else G.LL_RTOL * np.maximum(1.0, np.abs(lmax))


def _world(n_src, mixed):
    cfg = synth.small_config(1, n_ant=14, n_time=60, n_src=n_src)
    o = synth.observation(1, cfg)
    rng = np.random.default_rng(n_src)
    cat = synth.catalogue(cfg, rng)
    n = o.n_rows * o.n_chan
    vis = cfg.noise_sigma_jy * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
    obs = G.make_obs(o, vis, mixed=mixed)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED if mixed else rlf.RLF_FP64))
    ctx.model_vis(obs, cat, obs.vis, rlf.RLF_MODEL_ACCUMULATE)
    return ctx, obs, cat, ctx.facets_create(obs, cat)


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n_src", [3, 70])
@pytest.mark.parametrize("n_side", [3, 5])
def test_pass_marginalises_positions(n_side, n_src, mixed):
    ctx, obs, cat, f = _world(n_src, mixed)
    fits = []
    for side in (1, n_side):
        ctx.set_positions(f, side, 0.3 if side > 1 else 0.0)
        ctx.extract_facets(obs, cat, None, f)
        out = G.fit_out_tensors(n_src, surface=False)
        ctx.fit_sources(f, out)
        ctx.sync()
        fits.append(G.host(out))
    out = G.fit_out_tensors(n_src, surface=False)
    ps = ctx.pass_create(obs, cat, f, out)
    for _ in range(3):
        for t in out.values():
            t.fill_(-3)
        ps.launch()
        ctx.sync()
        got = G.host(out)
        assert np.all(np.abs(got["lmax"] - fits[1]["lmax"]) <= _tol(fits[1]["lmax"], mixed))
    # the fixed-position likelihood is far from it
    assert np.max(np.abs(fits[0]["lmax"] - fits[1]["lmax"]) / _tol(fits[1]["lmax"], mixed)) > 100
    ps.free()
    f.free()
    ctx.close()


@pytest.mark.parametrize("mixed", [False, True])
def test_creation_with_a_full_table_writes_no_outputs(mixed, tmp_path):
    ctx, obs, cat, f = _world(30, mixed)
    table = str(tmp_path / "tiles.txt")
    out = G.fit_out_tensors(30, surface=False)
    ps = ctx.pass_create(obs, cat, f, out, tune_path=table)
    assert 1 in ps.tiles()[1]
    ps.launch()
    ctx.sync()
    ref = G.host(out)
    ps.free()
    for t in out.values():
        t.fill_(-3)
    ps = ctx.pass_create(obs, cat, f, out, tune_path=table)
    ctx.sync()
    assert 1 not in ps.tiles()[1] and 2 in ps.tiles()[1]
    assert all(np.all(v == -3) for v in G.host(out).values())
    ps.launch()
    ctx.sync()
    got = G.host(out)
    assert np.array_equal(got["argmax"], ref["argmax"])
    assert np.all(np.abs(got["lmax"] - ref["lmax"]) <= _tol(ref["lmax"], mixed))
    ps.free()
    f.free()
    ctx.close()


@pytest.mark.parametrize("num_r", [8, 9, 20, 23, 32])
@pytest.mark.parametrize("n_src", [399, 400])
def test_queue_and_grid_passes_match_the_fit(n_src, num_r):
    cfg = synth.small_config(1, n_ant=8, n_time=30, n_src=n_src)
    o = synth.observation(1, cfg)
    rng = np.random.default_rng(num_r)
    cat = synth.catalogue(cfg, rng)
    n = o.n_rows * o.n_chan
    vis = cfg.noise_sigma_jy * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
    obs = G.make_obs(o, vis, mixed=True)
    p = rlf.params(precision=rlf.RLF_MIXED, num_r=num_r, n_e=21, e_step=0.1)
    ctx = rlf.Context(0, None, p)
    f = ctx.facets_create(obs, cat)
    ctx.extract_facets(obs, cat, None, f)
    ref = G.fit_out_tensors(n_src, n_e=21)
    ctx.fit_sources(f, ref, want_surface=True)
    ctx.sync()
    ref = G.host(ref)
    out = G.fit_out_tensors(n_src, n_e=21)
    ps = ctx.pass_create(obs, cat, f, out, want_surface=True)
    for _ in range(3):
        for t in out.values():
            t.fill_(-3)
        ps.launch()
        ctx.sync()
        got = G.host(out)
        fin = np.isfinite(ref["surface"])
        assert np.array_equal(fin, np.isfinite(got["surface"]))
        tol = _tol(ref["lmax"], True)[:, None] * np.ones_like(ref["surface"])
        d = np.abs(got["surface"][fin] - ref["surface"][fin])
        assert np.all(d <= np.maximum(tol[fin], _tol(ref["surface"][fin], True)))
    ps.free()
    f.free()
    ctx.close()

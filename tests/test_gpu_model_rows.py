"""The mixed-form sky model with the channels of a row in one thread against
the oracle: every group size, last groups with idle channels, the channel
number that keeps one thread per visibility, ragged row numbers just above and
below the number that chooses between the two, the three modes, and fluxes
from none to bright.  Tolerance: the mixed form's, per unit of total flux,
plus the FP32 rounding of the data it is added to."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G
from tests.test_gpu_mixed import VIS_MIXED_L1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,chan", [(196545, 2), (196544, 2), (196601, 3), (196601, 4), (98273, 5), (98273, 6),
                                       (98273, 7), (98241, 8), (65537, 9), (65537, 10), (49153, 16)])
def test_rows_of_channels_against_oracle(rows, chan):
    torch = G.torch_cuda()
    rng = np.random.default_rng(rows + chan)
    u, v, w = (rng.normal(0.0, s, rows) for s in (6000.0, 6000.0, 500.0))
    freq = 1.4e9 - 2.5e7 * np.arange(chan) * rng.uniform(0.9, 1.1, chan)
    o = synth.Observation(u, v, w, freq, np.ones(rows * chan))
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=5), rng)
    cat.flux_jy[0], cat.flux_jy[1] = 0.0, 10.0
    data = (rng.standard_normal(rows * chan) + 1j * rng.standard_normal(rows * chan)).astype(np.complex64)
    obs = G.make_obs(o, data, mixed=True)
    ref = oracle.sky_model(u, v, w, freq, cat).reshape(-1)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED))
    tol = VIS_MIXED_L1 * np.sum(cat.flux_jy) + 1.2e-7 * (np.abs(data) + np.abs(ref))
    for mode, want in ((rlf.RLF_MODEL_WRITE, ref), (rlf.RLF_MODEL_ACCUMULATE, data + ref),
                       (rlf.RLF_MODEL_RESIDUAL, data - ref)):
        out = torch.as_tensor(data.copy(), device="cuda:0").reshape(obs.vis.shape)
        ctx.model_vis(obs, cat, out, mode=mode)
        ctx.sync()
        assert np.all(np.abs(out.cpu().numpy().reshape(-1) - want) <= tol), mode
    ctx.close()

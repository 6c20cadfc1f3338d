"""The mixed sky model on both sides of the lines between one thread per
visibility and one per row and group of channels: the number of waves (4,600)
for three and four channels, the number of sources for six to sixteen, channel
numbers that fit no group, and a range of the catalogue's sources; a sample of
the rows, the first and the last among them, against the oracle with the
tolerance of the other mixed tests."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2203_14071_amd import rlf, synth
from tests import gpu_common as G
from tests.test_gpu_mixed import VIS_MIXED_L1

pytestmark = pytest.mark.gpu


# rows, channels, sources
CASES = [(294336, 4, 3), (294337, 4, 3), (294399, 3, 40), (294400, 3, 1), (147137, 8, 30), (147137, 8, 29),
         (147137, 6, 30), (98177, 9, 45), (98177, 9, 44), (73601, 16, 80), (147137, 10, 60), (147137, 2, 60),
         (1158400, 4, 1)]


@pytest.mark.parametrize("rows,chan,n_src", CASES)
def test_both_kernels_against_oracle(rows, chan, n_src):
    torch = G.torch_cuda()
    rng = np.random.default_rng(rows + chan + n_src)
    uvw = [rng.normal(0.0, s, rows) for s in (6000.0, 6000.0, 500.0)]
    freq = 1.4e9 - 2.5e7 * np.arange(chan) * rng.uniform(0.9, 1.1, chan)
    cat = synth.catalogue(dataclasses.replace(synth.CONFIGS[1], n_src=n_src + 2), rng)
    data = (rng.standard_normal((rows, chan)) + 1j * rng.standard_normal((rows, chan))).astype(np.complex64)
    obs = G.make_obs(synth.Observation(*uvw, freq, np.ones(rows * chan)), data.reshape(-1), mixed=True)
    pick = np.unique(np.concatenate([rng.integers(0, rows, 3000), [0, 1, rows - 2, rows - 1]]))
    sub = cat.subset(np.arange(1, n_src + 1))                # sources 1 .. n_src of n_src + 2
    ref = oracle.sky_model(*(a[pick] for a in uvw), freq, sub).reshape(-1, chan)
    ctx = rlf.Context(0, None, rlf.params(precision=rlf.RLF_MIXED))
    given = data[pick]
    tol = VIS_MIXED_L1 * np.sum(sub.flux_jy) + 1.2e-7 * (np.abs(given) + np.abs(ref))
    for mode, want in ((rlf.RLF_MODEL_WRITE, ref), (rlf.RLF_MODEL_ACCUMULATE, given + ref),
                       (rlf.RLF_MODEL_RESIDUAL, given - ref)):
        out = torch.as_tensor(data.reshape(-1).copy(), device="cuda:0")
        ctx.model_vis(obs, cat, out, mode=mode, src_begin=1, src_end=n_src + 1)
        ctx.sync()
        got = out.cpu().numpy().reshape(rows, chan)[pick]
        assert np.all(np.abs(got - want) <= tol), mode
    ctx.close()

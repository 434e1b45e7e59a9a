"""Power-of-two columns of 256 and more with rows whose length is no multiple
of the column tile (the last tile is ragged, or the row is shorter than one):
sampler and Wiener filter against the oracle."""
import numpy as np
import pytest

from gpu_common import REL_TOL, banner, rel
from oracle import messenger as om
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(256, 18), (256, 36), (512, 54), (1024, 18), (2048, 162)])
def test_ragged_column_tiles_match_oracle(H, W):
    import paper_1810_02821_amd as mf
    banner(f"ragged column tiles {H} x {W}")
    rng = np.random.default_rng(H + W)
    prob = synth.make_problem(H, W, synth.spectrum_powerlaw(1.0, 1.0, 2.0), np.full((H, W), 0.7),
                              synth.tile_mask(H, W, 0.1, rng), rng)
    plan = mf.Plan([prob])
    d = plan.concat([prob.d])
    x, _ = plan.sample(d, 5, chains=4, burn_in=2, n_samples=1)
    x = plan.sample_view(x, 0, 4, 1).cpu().numpy()
    for pair in range(2):
        smp, _ = om.sample_pair(prob, 5, 0, pair, 2, 1)
        for h in range(2):
            assert rel(x[2 * pair + h, 0], smp[h, 0]) < REL_TOL
    wf, _ = plan.wiener(d, mf.Schedule([10.0, 1.0], [3, 6]))
    ref, _ = om.wiener(prob, om.Schedule((10.0, 1.0), (3, 6)))
    assert rel(plan.split(wf)[0], ref) < REL_TOL

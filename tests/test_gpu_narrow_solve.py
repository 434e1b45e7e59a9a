"""Wiener solves that still take the complex row and column kernels and their
selectable shapes (one side a power of two from 256, the other below): forcing
the wide shapes on a single image, which would take the narrow ones, gives the
same filter bit for bit."""
import numpy as np
import pytest

from gpu_common import REL_TOL, banner, rel
from oracle import messenger as om
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,narrow,wide,lines", [
    # columns of 256: tiles of 4 x 128 against 16 x 256
    (256, 128, (4, 128, 0), (16, 256, 0), "gfx950 256 128 16 256\ngfx950-narrow 256 128 16 256 0\n"),
    # rows of 256: 4 rows a block against 16
    (128, 256, (16, 256, 4), (16, 256, 16), "gfx950-rows 128 256 16\ngfx950-narrow 128 256 16 256 16\n"),
    # both, the columns of a length with a factor 3 in their only tile
    (324, 256, (8, 256, 4), (8, 256, 16), "gfx950-rows 324 256 16\ngfx950-narrow 324 256 8 256 16\n"),
])
def test_narrow_and_wide_shapes_solve_alike(tmp_path, monkeypatch, H, W, narrow, wide, lines):
    import torch
    import paper_1810_02821_amd as mf
    banner(f"narrow solve {H}x{W}")
    rng = np.random.default_rng(4)
    prob = synth.make_problem(H, W, synth.spectrum_powerlaw(1.0, 1.0, 2.0), rng.uniform(0.5, 2.0, (H, W)),
                              synth.tile_mask(H, W, 0.3, rng), rng)
    levels = ((100.0, 10.0, 1.0), (5, 5, 20))
    base = mf.Plan([prob])
    assert base.narrow_shape(H, W) == narrow
    d = base.concat([prob.d])
    s_n, _ = base.wiener(d, mf.Schedule(*levels))
    cache = tmp_path / "wide.txt"
    cache.write_text(lines)
    monkeypatch.setenv("MF_TUNE_CACHE", str(cache))
    plan = mf.Plan([prob], autotune=True)
    assert plan.narrow_shape(H, W) == wide
    s_w, _ = plan.wiener(d, mf.Schedule(*levels))
    assert torch.equal(s_n, s_w)
    ref, _ = om.wiener(prob, om.Schedule(*levels))
    assert rel(base.split(s_n)[0], ref) < REL_TOL
    base.close()
    plan.close()

"""Lines of a tuning cache file that name a shape this library has no kernel
for (a file written by another version) are passed over: the plan runs, draws
the default shapes' samples bit for bit, and adds the choice it makes instead."""
import numpy as np
import pytest

from gpu_common import banner
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


def _problem(H, W):
    rng = np.random.default_rng(7)
    return synth.make_problem(H, W, synth.spectrum_powerlaw(1.0, 1.0, 2.0), rng.uniform(0.5, 1.0, (H, W)),
                              synth.tile_mask(H, W, 0.2, rng), rng)


@pytest.mark.parametrize("H,W,line", [
    (324, 256, "gfx950-narrow 324 256 16 256 4"),  # a column tile that is not built
    (54, 256, "gfx950-narrow 54 256 16 256 4"),
    (324, 256, "gfx950-narrow 324 256 8 256 5"),   # rows per block that are not built
    (324, 256, "gfx950 324 256 16 512"),
    (256, 256, "gfx950 256 256 32 256"),
    (324, 256, "gfx950-rows 324 256 3"),
])
def test_unknown_shapes_in_the_cache_are_passed_over(tmp_path, monkeypatch, H, W, line):
    import torch
    import paper_1810_02821_amd as mf
    banner(f"cache line {line}")
    prob = _problem(H, W)
    base = mf.Plan([prob])
    d = base.concat([prob.d])
    kw = dict(chains=2, burn_in=2, n_samples=2, form="streamed")
    ref, _ = base.sample(d, 3, **kw)
    sch = mf.Schedule([10.0, 1.0], [3, 3])
    ref_w, _ = base.wiener(d, sch)
    cache = tmp_path / "tune.txt"
    cache.write_text(line + "\n")
    monkeypatch.setenv("MF_TUNE_CACHE", str(cache))
    for _ in range(2):  # the file as given, then with the lines the first plan added
        plan = mf.Plan([prob], autotune=True)
        out, _ = plan.sample(d, 3, **kw)
        w, _ = plan.wiener(d, sch)
        assert torch.equal(out, ref) and torch.equal(w, ref_w)
        plan.close()
    assert cache.read_text().startswith(line + "\n")


def test_known_shapes_in_the_cache_are_kept(tmp_path, monkeypatch):
    import paper_1810_02821_amd as mf
    banner("cache lines of built shapes")
    prob = _problem(324, 256)
    base = mf.Plan([prob])
    tc, nth = base.tile_shape(324, 256)
    text = f"gfx950-rows 324 256 16\ngfx950-narrow 324 256 {tc} {nth} 16\n"
    cache = tmp_path / "tune.txt"
    cache.write_text(text)
    monkeypatch.setenv("MF_TUNE_CACHE", str(cache))
    plan = mf.Plan([prob], autotune=True)
    assert plan.row_shape(324, 256) == 16
    assert plan.narrow_shape(324, 256) == (tc, nth, 16)
    assert cache.read_text() == text
    plan.close()

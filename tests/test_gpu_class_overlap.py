"""Size classes of one mf_sample call side by side: a caller's captured graph
keeps them in sequence, so its replays give the reference for the eager calls,
bit for bit (same kernels, same order within a class)."""
import numpy as np
import pytest

from gpu_common import banner
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


def _plan(seed):
    import paper_1810_02821_amd as mf
    # five classes: the fifth shares the caller's stream with the first
    sizes = [(64, 64), (256, 256), (54, 72), (128, 128), (256, 128)]
    rng = np.random.default_rng(seed)
    spec = synth.spectrum_powerlaw(1.0, 1.0, 2.0)
    probs = [synth.make_problem(H, W, spec, np.full((H, W), 0.5), synth.tile_mask(H, W, 0.2, rng), rng)
             for H, W in sizes for _ in range(3)]
    plan = mf.Plan(probs)
    return mf, plan, plan.concat([p.d for p in probs])


@pytest.mark.parametrize("chains,storage", [(1, "fp32"), (4, "fp32"), (3, "bf16")])
def test_classes_side_by_side_equal_the_sequence(chains, storage):
    import torch
    banner(f"class overlap chains={chains} {storage}")
    mf, plan, d = _plan(4)
    plan.reserve(["sample"], chains=chains, storage=storage)
    kw = dict(chains=chains, burn_in=4, n_samples=2, storage=storage, check_finite=False)
    out = plan.samples_buffer(chains, 2)
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.sample(d, 9, out=out, **kw)
    for rep in range(2):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        # back to back on another stream, the inputs made there just before
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            d2 = d + 0.0
            other, _ = plan.sample(d2, 8, **kw)
            a, _ = plan.sample(d2, 9, **kw)
            b = a.clone()
        side.synchronize()
        assert torch.equal(b, out), f"replay {rep}"
        assert not torch.equal(other, out)


def test_non_finite_class_on_a_side_stream_is_reported():
    import torch
    banner("class overlap, non-finite state")
    mf, plan, d = _plan(5)
    views = plan.split(d.clone())
    for i in (7, 10):  # problems of two classes
        views[i][:] = float("nan")
    with pytest.raises(mf.MFError, match="problem 7"):
        plan.sample(plan.concat(views), 3, chains=1, burn_in=2, n_samples=1)
    out, _ = plan.sample(d, 3, chains=1, burn_in=2, n_samples=1)
    assert torch.isfinite(out).all()

"""MF_FLAG_GRAPH with several size classes: each class's sweep loop is replayed
on the stream the class runs on, side by side with the others; replays with
eager work between them equal the eager plan bit for bit."""
import numpy as np
import pytest

from gpu_common import banner
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chains,storage", [(1, "fp32"), (4, "fp32"), (3, "bf16")])
def test_replayed_classes_equal_eager_ones(chains, storage):
    import torch
    import paper_1810_02821_amd as mf
    banner(f"graphs of several classes, chains={chains} {storage}")
    # persistent and streamed classes; the fifth shares a stream with the first
    sizes = [(64, 64), (256, 256), (54, 72), (512, 256), (256, 128)]
    rng = np.random.default_rng(6)
    spec = synth.spectrum_powerlaw(1.0, 1.0, 2.0)
    probs = [synth.make_problem(H, W, spec, np.full((H, W), 0.5), synth.tile_mask(H, W, 0.2, rng), rng)
             for H, W in sizes for _ in range(3)]
    eager, graph = mf.Plan(probs), mf.Plan(probs, graph=True)
    d = eager.concat([p.d for p in probs])
    kw = dict(chains=chains, burn_in=3, n_samples=2, storage=storage)
    ref = {seed: eager.sample(d, seed, **kw)[0] for seed in (9, 10)}
    out = graph.samples_buffer(chains, 2)
    state, want = graph.state_buffer(chains), eager.state_buffer(chains)
    eager.sample(d, 9, state_out=want, out=torch.empty_like(out), **kw)
    for rep in range(3):
        for seed in (9, 10):  # four streamed classes and two seeds: the plan's eight graphs
            out.fill_(float("nan"))
            graph.sample(d, seed, state_out=state, out=out, **kw)
            torch.cuda.synchronize()
            assert torch.equal(out, ref[seed]), f"replay {rep} seed {seed}"
            if seed == 9:
                assert torch.equal(state, want), f"replay {rep}"
            eager.sample(d, 11, **kw)
            torch.cuda.synchronize()
    eager.close()
    graph.close()

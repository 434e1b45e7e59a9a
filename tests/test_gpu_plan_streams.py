"""Plans of several size classes hand their side streams on: more plans alive
together than the idle sets that are kept, made and closed from several threads
on streams of their own, draw what one plan alone draws, bit for bit."""
import threading

import numpy as np
import pytest

from gpu_common import banner
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


def test_plans_that_share_side_streams_in_turn():
    import torch
    import paper_1810_02821_amd as mf
    banner("side streams of many plans")
    rng = np.random.default_rng(3)
    spec = synth.spectrum_powerlaw(1.0, 1.0, 2.0)
    probs = [synth.make_problem(H, W, spec, np.full((H, W), 0.5), synth.tile_mask(H, W, 0.2, rng), rng)
             for H, W in [(32, 32), (64, 64), (48, 36), (64, 32), (32, 128)]]
    few = probs[:2]  # sets of one stream, later taken by plans that need three
    one = mf.Plan(probs)
    d = one.concat([p.d for p in probs])
    kw = dict(chains=2, burn_in=4, n_samples=1)
    ref = one.sample(d, 9, **kw)[0].clone()
    one.close()
    torch.cuda.synchronize()
    wrong = []

    def worker():
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(6):
                small = mf.Plan(few)
                small.sample(d, 9, **kw)
                small.close()
                a, b = mf.Plan(probs), mf.Plan(probs)
                x, _ = a.sample(d, 9, check_finite=False, **kw)
                y, _ = b.sample(d, 9, check_finite=False, **kw)
                a.close()
                z, _ = b.sample(d, 9, check_finite=False, **kw)
                torch.cuda.current_stream().synchronize()
                wrong.extend(t for t in (x, y, z) if not torch.equal(t, ref))
                b.close()

    threads = [threading.Thread(target=worker) for _ in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong

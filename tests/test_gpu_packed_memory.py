"""Workspace of single-chain calls: two problems of a streamed size class share
the first one's place in the work field, so that a call takes one field whether
or not it is given state_out, and gives the same samples."""
import pytest

from gpu_common import banner
from paper_1810_02821_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_state", [False, True])
def test_single_chains_take_one_field(with_state):
    import torch
    import paper_1810_02821_amd as mf
    banner(f"single-chain workspace, state {with_state}")
    # 24 problems of 1024^2 and one of 256^2: a field is 202 MB
    probs = [synth.config_128(1, 256)] + [synth.config_128(2, 1024)] * 24
    plan = mf.Plan(probs)
    d = plan.concat([p.d for p in probs])
    field = 8 * plan.total_pixels
    out = plan.samples_buffer(1, 1)
    state = plan.state_buffer(1) if with_state else None
    kw = dict(chains=1, burn_in=1, n_samples=1, form="streamed")
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    plan.sample(d, 5, out=out, state_out=state, **kw)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 1.1 * field
    # a second call from the state of the first equals one longer call
    if with_state:
        out2, long = plan.samples_buffer(1, 1), plan.samples_buffer(1, 1)
        plan.sample(d, 5, chains=1, burn_in=0, n_samples=1, sweep_offset=2, form="streamed", state_in=state,
                    state_out=state, out=out2)
        plan.sample(d, 5, chains=1, burn_in=2, n_samples=1, form="streamed", out=long)
        assert torch.equal(out2, long)
    plan.close()

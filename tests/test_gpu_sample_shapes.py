"""The persistent sampler's workgroup shapes (8 or 16 values per thread, by size
and by how many items a launch has) draw the same chains bit for bit."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,chains", [(32, 3), (64, 1), (64, 1024), (64, 1025), (64, 1026)])
def test_a_chain_does_not_depend_on_how_many_run_beside_it(N, chains):
    import torch
    import paper_1810_02821_amd as mf
    from paper_1810_02821_amd import synth
    prob = synth.config_small(5, N)
    plan = mf.Plan([prob])
    d = plan.concat([prob.d])

    def run(n):
        st = plan.state_buffer(n)
        out, _ = plan.sample(d, 11, chains=n, burn_in=2, n_samples=2, thin=2, init_scale=2.0, form="persistent",
                             state_out=st)
        return plan.sample_view(out, 0, n, 2), plan.state_view(st, 0, n)

    few, few_state = run(2)
    many, many_state = run(chains)
    k = min(2, chains)
    assert torch.equal(few[:k], many[:k])
    assert torch.equal(few_state[0], many_state[0])
    assert bool(torch.isfinite(many).all()) and bool(many.abs().sum(dim=(1, 2, 3)).min() > 0)
    plan.close()

"""The streamed solve of real fields (power-of-two sides from 256) folds columns
in two and recombines each mode with its mirror: every mode of a few sweeps for
every row and column length, and the residual of rows longer than a wave,
against the FP64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _problem(H, W, seed):
    from paper_1810_02821_amd import synth
    rng = np.random.default_rng(seed)
    # n P / tau from about 12 (k = 0) down to 0.1 or less in the corners
    spec = synth.spectrum_powerlaw(12.0 * 0.25 / (H * W), 1.0, 0.8)
    sigma = rng.uniform(0.5, 1.0, (H, W))
    prob = synth.make_problem(H, W, spec, sigma, synth.tile_mask(H, W, 0.1, rng), rng)
    prob.d = np.where(prob.mask, 0.0, rng.standard_normal((H, W))).astype(np.float32).astype(np.float64)
    prob.noise_var = prob.noise_var.astype(np.float32).astype(np.float64)
    return prob, rng.standard_normal((H, W)).astype(np.float32)


@pytest.mark.parametrize("H,W", [(256, 256), (512, 256), (256, 512), (1024, 256), (256, 1024), (2048, 256),
                                 (256, 2048)])
def test_every_mode_of_the_streamed_solve(H, W):
    import paper_1810_02821_amd as mf
    from oracle import messenger as om
    probs = [_problem(H, W, 1), _problem(H, W, 2)]
    plan = mf.Plan([p for p, _ in probs])
    levels = ((8.0, 1.0), (2, 1))
    s, _ = plan.wiener(plan.concat([p.d for p, _ in probs]), mf.Schedule(*levels),
                       s_init=plan.concat([s0 for _, s0 in probs]))
    for (prob, s0), got in zip(probs, plan.split(s)):
        ref, _ = om.wiener(prob, om.Schedule(*levels), s0=s0.astype(np.float64))
        # rounding spreads over the modes as white noise: well under 80 units of
        # 2^-24 of a pixel per transform pair in the worst mode
        unit = 2.0 ** -24 * np.sqrt((np.mean(ref ** 2) + 1.0) * H * W)
        assert np.max(np.abs(np.fft.fft2(got.astype(np.float64)) - np.fft.fft2(ref))) < 80 * unit
    plan.close()


@pytest.mark.parametrize("H,W", [(256, 256), (256, 1024)])
def test_the_residual_stops_where_the_oracle_stops(H, W):
    import paper_1810_02821_amd as mf
    from oracle import messenger as om
    prob, _ = _problem(H, W, 3)
    plan = mf.Plan([prob])
    kw = dict(tol=2e-3, max_sweeps=60, check_every=3)
    s, info = plan.wiener(plan.concat([prob.d]), mf.Schedule([4.0, 1.0], [2, 1], **kw))
    ref, oi = om.wiener(prob, om.Schedule((4.0, 1.0), (2, 1), **kw))
    assert oi.converged and info[0].converged == 1 and info[0].sweeps == oi.sweeps
    # the residual is a difference of fields of relative rounding 1e-6 over a tolerance of 2e-3
    assert abs(info[0].residual - oi.residual) < 1e-2 * oi.residual
    got = plan.split(s)[0]
    assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref)
    plan.close()


@pytest.mark.parametrize("H,W,bands", [(24, 18, 2), (64, 128, 64), (256, 256, 32)])
def test_new_amplitudes_on_the_same_bands_equal_a_new_plan(H, W, bands):
    """mf_plan_set_spectrum rewrites the tables on the device when the band edges
    stay; solves, gradients and the loss see the same values as a plan made with
    the new spectrum, and as after a change of edges (the host path)."""
    import types
    import torch
    import paper_1810_02821_amd as mf
    from paper_1810_02821_amd import synth
    prob = synth.config_bands(1, H, bands, W)
    rng = np.random.default_rng(2)
    amps = prob.spectrum.amps * rng.uniform(0.5, 2.0, bands)
    new = types.SimpleNamespace(kind="bands", edges=prob.spectrum.edges, amps=amps)
    wide = types.SimpleNamespace(kind="bands", edges=np.append(prob.spectrum.edges[:-1], 1e4), amps=amps)
    fresh = synth.config_bands(1, H, bands, W)
    fresh.spectrum = new
    same, moved, made = mf.Plan([prob]), mf.Plan([prob]), mf.Plan([fresh])
    same.set_spectrum(0, new)
    moved.set_spectrum(0, wide)  # other edges, the same band for every mode
    d, t = made.concat([prob.d]), made.concat([prob.s_true])
    sch = mf.Schedule([10.0, 1.0], [3, 5])
    out = []
    for plan in (made, same, moved):
        s, _ = plan.wiener(d, sch)
        loss, gd, gb, _ = plan.band_loss(d, s, t, sch)
        out.append((s, loss, gd, gb))
        plan.close()
    for got in out[1:]:
        for a, b in zip(out[0], got):
            if a.dtype == torch.float64:  # sums in an order that varies
                assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max())
            else:
                assert torch.equal(a, b)

"""The persistent solve folds the real field's rows in two and recombines each
mode with its mirror: every mode of a few sweeps, those that mirror themselves
(k_x, k_y in {0, N/2}) among them, against the FP64 oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [32, 64, 128])
@pytest.mark.parametrize("levels", [((1.0,), (1,)), ((8.0, 1.0), (2, 1))])
def test_every_mode_of_the_persistent_solve(N, levels):
    import paper_1810_02821_amd as mf
    from oracle import messenger as om
    from paper_1810_02821_amd import synth
    rng = np.random.default_rng(N)
    # n P / tau from about 12 (k = 0) down to 0.1 in the corners: every mode's
    # filter differs from its neighbours' and none is negligible
    spec = synth.spectrum_powerlaw(12.0 * 0.25 / (N * N), 1.0, 1.0)
    sigma = rng.uniform(0.5, 1.0, (N, N))
    prob = synth.make_problem(N, N, spec, sigma, synth.tile_mask(N, N, 0.1, rng), rng)
    prob.d = np.where(prob.mask, 0.0, rng.standard_normal((N, N))).astype(np.float32).astype(np.float64)
    prob.noise_var = prob.noise_var.astype(np.float32).astype(np.float64)
    s0 = rng.standard_normal((N, N)).astype(np.float32)
    plan = mf.Plan([prob])
    s, _ = plan.wiener(plan.concat([prob.d]), mf.Schedule(*levels), s_init=plan.concat([s0]))
    got = np.fft.fft2(plan.split(s)[0].astype(np.float64))
    ref, _ = om.wiener(prob, om.Schedule(*levels), s0=s0.astype(np.float64))
    ref = np.fft.fft2(ref)
    # FP32 rounding spreads over the modes as white noise: about sqrt(log2 n)
    # roundings of 2^-24 of a pixel per transform, two transforms a sweep, so
    # well under 20 units of the pixels' rms (times N) in the worst of n modes
    unit = 2.0 ** -24 * np.sqrt(np.mean(np.abs(np.fft.ifft2(ref)) ** 2) + 1.0) * N
    assert np.max(np.abs(got - ref)) < 4 * 20 * unit
    plan.close()


@pytest.mark.parametrize("N", [32, 64, 128])
@pytest.mark.parametrize("b_ratio", [0.0, 0.5])
def test_every_mode_of_the_persistent_mass_mapping_step(N, b_ratio):
    """The Fourier step takes each mode with its mirror from one thread, and the
    modes that mirror themselves by way of LDS: every mode of kappa after a few
    sampled sweeps, of the last state, and of the filter, against the oracle."""
    import paper_1810_02821_amd as mf
    from oracle import messenger as om
    from oracle import shear as osh
    from paper_1810_02821_amd import synth
    prob = synth.config_shear(3, N, b_ratio)
    prob.spectrum = synth.spectrum_powerlaw(12.0 * 0.25 / (N * N), 1.0, 1.0)  # no mode negligible
    prob.noise_var = prob.noise_var.astype(np.float32).astype(np.float64)
    prob.gamma = prob.gamma.astype(np.complex64).astype(np.complex128)
    plan = mf.Plan([prob])
    g = plan.concat_complex([prob.gamma])
    st = plan.shear_state_buffer(2)
    out, _ = plan.shear_sample(g, 7, chains=2, burn_in=1, n_samples=1, thin=2, b_ratio=b_ratio, state_out=st)
    ref, state = osh.sample_shear_chain(prob, 7, 0, 1, 1, 1, 2, b_ratio)
    filt = plan.shear_wiener(g, mf.Schedule([4.0, 1.0], [1, 1]), b_ratio)
    fref = osh.wiener_shear(prob, om.Schedule([4.0, 1.0], [1, 1]), b_ratio)
    for got, want in ((out.cpu().numpy().reshape(2, N, N)[1], ref[0]), (st.cpu().numpy().reshape(2, N, N)[1], state),
                      (filt.cpu().numpy().reshape(N, N), fref)):
        # the bound of the test above, with the normals' hardware log, sine and
        # cosine (about 2^-21 of the noise's unit variance) beside the transforms
        unit = 2.0 ** -24 * np.sqrt(np.mean(np.abs(want) ** 2) + 1.0) * N
        assert np.max(np.abs(np.fft.fft2(got.astype(np.complex128)) - np.fft.fft2(want))) < 8 * 20 * unit
    plan.close()

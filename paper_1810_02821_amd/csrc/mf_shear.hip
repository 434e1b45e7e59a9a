// Mass mapping (Sec. 5): the messenger Wiener filter and sampler for complex
// shear data gamma = A kappa + n with the spin-2 operator A = F^-1 D F,
// D_k = (k_1 + i k_2)^2 / |k|^2 (D_0 = 0), and a complex convergence
// kappa = kappa_E + i kappa_B with spectra P_E and P_B = r P_E.  One
// workgroup owns one chain of an N x N problem for every sweep, on chip.
//
// The state between sweeps is the model shear A kappa (pixel space):
//   t      = (1 - a) A kappa + a gamma + sqrt(T (1 - a)) xi        (shear space)
//   u(k)   = conj(D_k) F(t)(k)
//   kappa^ = f_+ u(k) + f_- conj(u(-k)) + w_+ eta(k) + w_- conj(eta(-k))
// with f_+- = (f_E +- f_B)/2, w_+- = (w_E +- w_B)/2: the E and B parts of u are
// the spectra of the real fields Re and Im of F^-1 u, and each gets its own
// Wiener-sampler step.  At k = 0 (no data) f = 0 and w draws the prior.  The
// next state is F^-1(D kappa^); on sweeps that emit a sample (and after the
// last sweep of a filter) kappa itself is F^-1(kappa^), written out before the
// field is transformed back.
#include "mf_device.hpp"
#include "mf_resident.hpp"
#include "mf_resident_fft.hpp"
#include "mf_shear.hpp"

namespace mf {

namespace {

template <int N>
__device__ __forceinline__ int signed_freq(unsigned k) {
    return k < (unsigned)(N / 2) ? (int)k : (int)k - N;  // numpy fftfreq * N
}

// D at mode (ky, kx) in unshifted FFT order (D_0 = 0 falls out of x = y = 0).
template <int N>
__device__ __forceinline__ float2 ks(unsigned ky, unsigned kx) {
    const float x = (float)signed_freq<N>(kx), y = (float)signed_freq<N>(ky);
    const float r = __builtin_amdgcn_rcpf(fmaxf(fmaf(x, x, y * y), 1.f));
    return make_float2((x * x - y * y) * r, 2.f * x * y * r);
}

template <int N>
__device__ __forceinline__ unsigned mirror_index(unsigned ky, unsigned kx) {
    return ((N - ky) & (N - 1)) * N + ((N - kx) & (N - 1));
}

__device__ __forceinline__ float2 mulc(float2 z, float2 d) {  // conj(d) z
    return make_float2(fmaf(d.x, z.x, d.y * z.y), fmaf(d.x, z.y, -d.y * z.x));
}

struct Filt {
    float fp, fm, wp, wm;
};

// (f_+, f_-, w_+, w_-) of one mode, the 1/n of the inverse transform and the
// normals' sqrt(2 ln 2) folded in: f / 2n, and w / 2n = sqrt(nP T / (nP + T)) / 2N.
// Scaled only after the ratios nP / (nP + T) and T / (nP + T) are formed, and by
// N = sqrt(n) outside the root: with 1/n on nP or T first, variances below 1e-33
// leave the normal numbers (which the root takes as zero).
template <int N>
__device__ __forceinline__ Filt filt(float nP, float r, float T) {
    constexpr float c = 0.5f / (float)(N * N), cw = 0.5f / (float)N;
    const float nB = r * nP, g = kBoxMuller2 * T;
    const float rE = __builtin_amdgcn_rcpf(nP + T), rB = __builtin_amdgcn_rcpf(nB + T);
    const float fE = nP * rE, hB = c * (nB * rB);
    const float wE = __builtin_amdgcn_sqrtf(nP * (g * rE)), vB = cw * __builtin_amdgcn_sqrtf(nB * (g * rB));
    return {fmaf(c, fE, hB), fmaf(c, fE, -hB), fmaf(cw, wE, vB), fmaf(cw, wE, -vB)};
}
// The same at k = 0, which has no data: f = 0 and the prior w = sqrt(n nP).  Not
// filt at a large stand-in for T, which is exact only for nP far below it.
template <int N>
__device__ __forceinline__ Filt prior_filt(float nP, float r) {
    constexpr float c = 0.5f / (float)N;
    const float wE = c * __builtin_amdgcn_sqrtf(kBoxMuller2 * nP), wB = c * __builtin_amdgcn_sqrtf(kBoxMuller2 * (r * nP));
    return {0.f, 0.f, wE + wB, wE - wB};
}
// The Fourier step kappa^(k) = f_+ u(k) + f_- conj(u(-k)) + w_+ eta(k) + w_- conj(eta(-k)),
// u = conj(D) Z, times D unless the sweep emits kappa.  eta: the mode variates
// in LDS.  D(-k) equals D(k), except that on exactly one Nyquist line (where -k
// aliases to the same frequency in that component) the mixed term changes sign.
template <int N, bool NOISE, bool TIMES_D>
struct ShearStep {
    using S = typename SquareShape<N>::type;
    const float* nP;
    const float2* eta;
    float r, T;
    float x, x2, y1;  // k_1 of task a, its square, and its ky mod RC
    bool nyq_x;       // task a lies on the Nyquist column
    __device__ __forceinline__ ShearStep(const float* nP_, const float2* eta_, float r_, float T_, const DPair& dp)
        : nP(nP_), eta(eta_), r(r_), T(T_), x((float)signed_freq<N>(dp.kxa)), x2(x * x), y1((float)dp.k1a),
          nyq_x(dp.kxa == (unsigned)(N / 2)) {}
    // kappa^ of a mode from u, u of its mirror, and both variates
    __device__ __forceinline__ float2 mode(const Filt& c, float2 u, float2 um, float2 e, float2 em, float2 d) const {
        float2 k = make_float2(fmaf(c.fp, u.x, c.fm * um.x), fmaf(c.fp, u.y, -c.fm * um.y));
        if constexpr (NOISE) {
            k = make_float2(fmaf(c.wp, e.x, k.x), fmaf(c.wp, e.y, k.y));
            k = make_float2(fmaf(c.wm, em.x, k.x), fmaf(-c.wm, em.y, k.y));
        }
        return TIMES_D ? cmul(k, d) : k;
    }
    __device__ __forceinline__ void pair(int k2, unsigned ky, unsigned kx, float2 za, float2 zb, float2& sa,
                                         float2& sb) const {
        const Filt c = filt<N>(nP[ky * N + kx], r, T);
        // ky = k1 + RC k2 is below the Nyquist row exactly for k2 < RD/2
        const float y = y1 + (float)(S::RC * k2 - (k2 >= S::RD / 2 ? N : 0));
        const float q = __builtin_amdgcn_rcpf(fmaf(y, y, x2));  // k = 0 mirrors itself: never here
        const float2 d = make_float2(fmaf(-y, y, x2) * q, 2.f * x * y * q);
        const bool flip = k2 == S::RD / 2 ? (y1 == 0.f) != nyq_x : nyq_x;
        const float2 dm = make_float2(d.x, flip ? -d.y : d.y);
        const float2 u = mulc(za, d), um = mulc(zb, dm);
        float2 e = make_float2(0.f, 0.f), em = e;
        if constexpr (NOISE) {
            e = eta[ky * N + kx];
            em = eta[mirror_index<N>(ky, kx)];
        }
        sa = mode(c, u, um, e, em, d);
        sb = mode(c, um, u, em, e, dm);
    }
    __device__ __forceinline__ float2 single(unsigned ky, unsigned kx, float2 z, float2 zm) const {
        const float np = nP[ky * N + kx];
        const Filt c = ky == 0 && kx == 0 ? prior_filt<N>(np, r) : filt<N>(np, r, T);
        const float2 d = ks<N>(ky, kx);
        const bool flip = (ky == (unsigned)(N / 2)) != (kx == (unsigned)(N / 2));
        float2 e = make_float2(0.f, 0.f), em = e;
        if constexpr (NOISE) {
            e = eta[ky * N + kx];
            em = eta[mirror_index<N>(ky, kx)];
        }
        return mode(c, mulc(z, d), mulc(zm, make_float2(d.x, flip ? -d.y : d.y)), e, em, d);
    }
};

// Every thread must call it.  One mode's coefficients (two reciprocals, two
// square roots) and D serve the mode and its mirror; the draws go through LDS,
// since a Philox call's two modes sit in neighbouring lanes.  VALU-bound: about
// 3,400 instructions per wave and sweep at 128^2 (4,900 with Z and eta exchanged
// for the mirror and the coefficients evaluated three times), 88% of the issue
// rate; 512 chains x 80 sweeps 5.23 -> 4.06 ms.
template <int N>
__device__ __forceinline__ void harmonic_shear(float2 (&v)[16], float2* lds, float2* sz, const ShearArgs& a, const ProbDev& pr,
                                               float T, uint32_t sweep, int chain, unsigned tid, bool times_d) {
    using S = typename SquareShape<N>::type;
    const DPair dp = d_pair<S>(tid);
    mirror_put<S>(v, dp, sz);
    const float* nP = a.nP + pr.pix_off;
    if (a.stochastic) {
        __syncthreads();  // other threads may still read the forward transform's last exchange
        const unsigned jx = tid % (N / 2), k1 = tid / (N / 2);
#pragma unroll
        for (int k2 = 0; k2 < 8; ++k2) {
            __builtin_amdgcn_sched_barrier(0);
            const unsigned ky = k1 + S::RC * k2;
            const uint32_t e2 = (uint32_t)(ky * (N / 2) + jx);
            const Polar2 z = pair_polar(e2, sweep, (uint32_t)pr.pid, kStageHarmonic, (uint32_t)chain, a.key0, a.key1);
            st2(lds, ky * N + 2 * jx, make_float2(z.a.r * z.a.c, z.a.r * z.a.s), make_float2(z.b.r * z.b.c, z.b.r * z.b.s));
        }
        __syncthreads();
        if (times_d) mirror_step<S>(v, dp, tid, sz, ShearStep<N, true, true>(nP, lds, a.b_ratio, T, dp));
        else mirror_step<S>(v, dp, tid, sz, ShearStep<N, true, false>(nP, lds, a.b_ratio, T, dp));
    } else {
        __syncthreads();
        if (times_d) mirror_step<S>(v, dp, tid, sz, ShearStep<N, false, true>(nP, nullptr, a.b_ratio, T, dp));
        else mirror_step<S>(v, dp, tid, sz, ShearStep<N, false, false>(nP, nullptr, a.b_ratio, T, dp));
    }
    __syncthreads();
    mirror_get<S>(v, dp, sz);
}

template <int N>
__global__ __launch_bounds__(SquareShape<N>::type::NT, 4) void resident_shear_kernel(ShearArgs a) {
    using S = typename SquareShape<N>::type;
    constexpr int P = S::RB;
    __shared__ __align__(16) float2 lds[S::LDS];
    __shared__ float2 twl[S::TWS];  // twiddle tables of the four passes
    __shared__ float2 sz[8 * S::RD];
    const unsigned tid = threadIdx.x;
    rect_twiddles<S>(twl, a.tw, a.tw, 1, tid);
    __syncthreads();
    const ItemDev it = a.items[blockIdx.x];
    const ProbDev pr = a.probs[it.prob];
    const unsigned y = tid / (P / 2), j = tid % (P / 2);
    const int64_t nn = (int64_t)N * N;

    float2 v[16];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int64_t o = it.field_off + (int64_t)y * N + 2 * j + P * m;
        v[m] = a.state_in ? a.state_in[o] : make_float2(0.f, 0.f);
        v[8 + m] = a.state_in ? a.state_in[o + 1] : make_float2(0.f, 0.f);
    }

    int64_t k = 0;
    for (int lv = 0; lv < a.lv.n; ++lv) {
        const float T = (float)(a.lv.lambda[lv] * (double)pr.tau);
        const float sdT = kBoxMuller * __builtin_amdgcn_sqrtf(T);  // apart from sqrt(1 - a): T (1 - a) may be subnormal
        for (int s = 0; s < a.lv.sweeps[lv]; ++s, ++k) {
            const uint32_t sweep = a.sweep0 + (uint32_t)k;
            const float2* tw = twl + per_sweep_zero();
            unsigned t = tid;
            asm volatile("" : "+v"(t));
            {
                // pixel step in shear space
                const unsigned yy = t / (P / 2), jj = t % (P / 2);
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    __builtin_amdgcn_sched_barrier(0);
                    const uint32_t e2 = (uint32_t)(yy * (N / 2) + jj + (P / 2) * m);
                    const int64_t px = pr.pix_off + 2 * (int64_t)e2;
                    const float2 nb = *reinterpret_cast<const float2*>(a.nbar + px);
                    const float4 g = *reinterpret_cast<const float4*>(a.gamma + px);
                    const float a0 = T * __builtin_amdgcn_rcpf(T + nb.x), a1 = T * __builtin_amdgcn_rcpf(T + nb.y);
                    const float2 g0 = a0 > 0.f ? make_float2(a0 * g.x, a0 * g.y) : make_float2(0.f, 0.f);
                    const float2 g1 = a1 > 0.f ? make_float2(a1 * g.z, a1 * g.w) : make_float2(0.f, 0.f);
                    float2& s0 = v[m];
                    float2& s1 = v[8 + m];
                    s0 = make_float2(fmaf(1.f - a0, s0.x, g0.x), fmaf(1.f - a0, s0.y, g0.y));
                    s1 = make_float2(fmaf(1.f - a1, s1.x, g1.x), fmaf(1.f - a1, s1.y, g1.y));
                    if (a.stochastic) {
                        const Polar2 z = pair_polar(e2, sweep, (uint32_t)pr.pid, kStagePixel, (uint32_t)it.pair,
                                                    a.key0, a.key1);
                        const float r0 = z.a.r * (sdT * __builtin_amdgcn_sqrtf(fmaxf(1.f - a0, 0.f)));
                        const float r1 = z.b.r * (sdT * __builtin_amdgcn_sqrtf(fmaxf(1.f - a1, 0.f)));
                        s0 = make_float2(fmaf(r0, z.a.c, s0.x), fmaf(r0, z.a.s, s0.y));
                        s1 = make_float2(fmaf(r1, z.b.c, s1.x), fmaf(r1, z.b.s, s1.y));
                    }
                }
            }
            rect_forward<S>(v, lds, tw, t, d_pair<S>(t));
            unsigned t2 = tid;
            asm volatile("" : "+v"(t2));
            const bool last = lv == a.lv.n - 1 && s == a.lv.sweeps[lv] - 1;
            const bool emit = a.samples && k >= a.burn_in && ((k - a.burn_in + 1) % a.thin) == 0;
            const bool write = emit || (last && a.kappa_out);
            harmonic_shear<N>(v, lds, sz, a, pr, T, sweep, it.pair, t2, !write);
            if (write) {
                // kappa = F^-1 kappa^, written out, then transformed back
                unsigned t3 = tid;
                asm volatile("" : "+v"(t3));
                const float2* tw3 = twl + per_sweep_zero();
                rect_inverse<S>(v, lds, tw3, t3, d_pair<S>(t3));
                float2* o;
                if (emit) {
                    const int64_t slot = (k - a.burn_in + 1) / a.thin - 1;
                    o = a.samples + (int64_t)a.chains * a.n_samples * pr.pix_off +
                        ((int64_t)it.pair * a.n_samples + slot) * nn;
                } else {
                    o = a.kappa_out + pr.pix_off;
                }
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const int64_t px = (int64_t)y * N + 2 * j + P * m;
                    o[px] = v[m];
                    o[px + 1] = v[8 + m];
                }
                unsigned t4 = tid;
                asm volatile("" : "+v"(t4));
                const DPair dp = d_pair<S>(t4);
                rect_forward<S>(v, lds, tw3, t4, dp);
                // the unnormalised forward transform returned n kappa^
                constexpr float back = 1.0f / (float)(N * N);
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const unsigned ky = (e < 8 ? dp.k1a : dp.k1b) + S::RC * (e % 8), kx = e < 8 ? dp.kxa : dp.kxb;
                    v[e] = cmul(v[e], cscale(ks<N>(ky, kx), back));
                }
            }
            // next state: F^-1 (D kappa^)
            unsigned t5 = tid;
            asm volatile("" : "+v"(t5));
            const float2* tw5 = twl + per_sweep_zero();
            rect_inverse<S>(v, lds, tw5, t5, d_pair<S>(t5));
        }
    }
    if (a.state_out) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int64_t o = it.field_off + (int64_t)y * N + 2 * j + P * m;
            a.state_out[o] = v[m];
            a.state_out[o + 1] = v[8 + m];
        }
    }
}

}  // namespace

hipError_t launch_resident_shear(int N, const ShearArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.n_items);
    switch (N) {
        case 32: hipLaunchKernelGGL(resident_shear_kernel<32>, grid, dim3(SquareShape<32>::type::NT), 0, s, a); break;
        case 64: hipLaunchKernelGGL(resident_shear_kernel<64>, grid, dim3(SquareShape<64>::type::NT), 0, s, a); break;
        case 128: hipLaunchKernelGGL(resident_shear_kernel<128>, grid, dim3(SquareShape<128>::type::NT), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mf

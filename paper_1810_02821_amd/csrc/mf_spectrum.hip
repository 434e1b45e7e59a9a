// Hierarchical sampler (Sec. 5): Algorithm 1 for the signal, alternated with a
// draw of the band amplitudes theta_b of the power spectrum given the signal.
// One workgroup owns one chain pair of an N x N band-spectrum problem and runs
// every iteration on chip, like the persistent sampler.
//
// Each chain of the pair has its own amplitudes, so the Fourier-space step can
// no longer apply one real filter to the complex pair field Z = Z_A + i Z_B.
// With f_+- = (f_A +- f_B)/2 and w_+- = (w_A +- w_B)/2 (real and even in k),
//     S(k) = f_+ Z(k) + f_- conj(Z(-k)) + w_+ eta(k) + w_- conj(eta(-k))
// gives chain A (real part of the inverse transform) the update f_A Z_A + w_A
// noise and chain B (imaginary part) f_B Z_B + w_B noise, exactly.  The
// transform leaves k and -k in one thread (mf_resident_fft.hpp); eta goes through
// LDS, since a Philox call's two modes sit in neighbouring lanes.
//
// The amplitudes given the signal are inverse-gamma: theta_b = (2 beta_0 +
// sigma_b / n^2) / x_b, with sigma_b the band power of the chain's signal and
// x_b a chi-square variate of m_b + nu_0 degrees of freedom, the sum of squared
// normals from stage 3 of the stream (flat index over the bands' degrees of
// freedom, counter word 1 = the global iteration).
#include "mf_device.hpp"
#include "mf_resident.hpp"
#include "mf_resident_fft.hpp"
#include "mf_spectrum.hpp"

namespace mf {

namespace {

constexpr uint32_t kStageSpectrum = 3;
constexpr int kNB = kMaxBandsPerProblem;

struct SpecShared {
    float4 coef[kNB];      // (f_A/n, w_A/n, f_B/n, w_B/n) per band
    double theta[2][kNB];  // current amplitudes, chains A and B
    double sum[2][2][kNB]; // [0]: band powers of the last signal, in units of n^2; [1]: chi-square sums
    int32_t dof[kNB];      // degrees of freedom per band
    int32_t pre[kNB + 1];  // their prefix sums (flat index of each band's first variate)
};

template <int N>
__device__ __forceinline__ unsigned mirror(unsigned ky, unsigned kx) {
    return ((N - ky) & (N - 1)) * N + ((N - kx) & (N - 1));
}

// f/n and w/n of both chains for band b, from the current amplitudes.
__device__ __forceinline__ void refresh_coef(SpecShared& sh, int b, double T, double n) {
    float c[4];
#pragma unroll
    for (int ch = 0; ch < 2; ++ch) {
        const double nP = n * sh.theta[ch][b];
        const double f = nP / (nP + T);
        const double w = sqrt(n * nP * T / (nP + T));
        c[2 * ch] = (float)(f / n);
        c[2 * ch + 1] = (float)(w / n);
    }
    sh.coef[b] = make_float4(c[0], c[1], c[2], c[3]);
}

// The Fourier step S(k)/n of a mode and its mirror (one band, one set of coefficients).
template <int N>
struct SpecStep {
    const float4* coef;
    const int16_t* band;
    const float2* eta;
    __device__ __forceinline__ float2 mode(float fp, float fm, float wp, float wm, float2 z, float2 zm, float2 e,
                                           float2 em) const {
        float2 s = make_float2(fmaf(fp, z.x, fm * zm.x), fmaf(fp, z.y, -fm * zm.y));
        s = make_float2(fmaf(wp, e.x, s.x), fmaf(wp, e.y, s.y));
        return make_float2(fmaf(wm, em.x, s.x), fmaf(-wm, em.y, s.y));
    }
    __device__ __forceinline__ void pair(int, unsigned ky, unsigned kx, float2 za, float2 zb, float2& sa,
                                         float2& sb) const {
        const float4 c = coef[band[ky * N + kx]];
        const float fp = 0.5f * (c.x + c.z), fm = 0.5f * (c.x - c.z);
        const float wp = 0.5f * (c.y + c.w), wm = 0.5f * (c.y - c.w);
        const float2 e = eta[ky * N + kx], em = eta[mirror<N>(ky, kx)];
        sa = mode(fp, fm, wp, wm, za, zb, e, em);
        sb = mode(fp, fm, wp, wm, zb, za, em, e);
    }
    __device__ __forceinline__ float2 single(unsigned ky, unsigned kx, float2 z, float2 zm) const {
        float2 sa, sb;
        pair(0, ky, kx, z, zm, sa, sb);
        return sa;
    }
};

// Fourier-space step on layout D; on return v holds S(k)/n.  Every thread must call it.
template <int N>
__device__ __forceinline__ void harmonic_pair(float2 (&v)[16], float2* lds, float2* sz, const SpectrumArgs& a,
                                              const ProbDev& pr, const SpecShared& sh, uint32_t sweep,
                                              int pair, unsigned tid) {
    using S = typename SquareShape<N>::type;
    const DPair dp = d_pair<S>(tid);
    mirror_put<S>(v, dp, sz);
    __syncthreads();  // other threads may still read the forward transform's last exchange
    const unsigned jx = tid % (N / 2), k1 = tid / (N / 2);
#pragma unroll
    for (int k2 = 0; k2 < 8; ++k2) {
        __builtin_amdgcn_sched_barrier(0);
        const unsigned ky = k1 + S::RC * k2;
        const uint32_t e2 = (uint32_t)(ky * (N / 2) + jx);
        const Normals2 z = pair_normals(e2, sweep, (uint32_t)pr.pid, kStageHarmonic, (uint32_t)pair, a.key0, a.key1);
        st2(lds, ky * N + 2 * jx, z.a, z.b);
    }
    __syncthreads();
    mirror_step<S>(v, dp, tid, sz, SpecStep<N>{sh.coef, a.band + pr.pix_off, lds});
    __syncthreads();
    mirror_get<S>(v, dp, sz);
}

// FP64 sums by band in LDS.  Each sum is kept in R copies, one for every R-th
// lane: the modes of a wave (and the variates of a thread's run) mostly share a
// band, and the atomics of lanes that meet in one address run one after the
// other.  The copies take the exchange buffer, which is free between the
// Fourier step and the inverse transform.
template <int N>
struct BandSums {
    using S = typename SquareShape<N>::type;
    static constexpr int R = N == 128 ? 32 : N == 64 ? 16 : 4;
    static_assert(4 * kNB * R * 8 <= S::LDS * 8, "the copies fit in the exchange buffer");
    double* acc;  // [kind][chain][band][copy]
    int nb;
    unsigned copy;
    __device__ __forceinline__ BandSums(float2* lds, int nb_, unsigned tid)
        : acc(reinterpret_cast<double*>(lds)), nb(nb_), copy(tid % R) {}
    __device__ __forceinline__ void clear(unsigned tid) const {
        for (int i = (int)tid; i < 4 * nb * R; i += S::NT) acc[i] = 0.0;
    }
    __device__ __forceinline__ void add(int kind, int b, double pa, double pb) const {
        atomicAdd(&acc[((kind * 2 + 0) * nb + b) * R + copy], pa);
        atomicAdd(&acc[((kind * 2 + 1) * nb + b) * R + copy], pb);
    }
    __device__ __forceinline__ void collect(SpecShared& sh, unsigned tid) const {
        constexpr int G = R < 8 ? R : 8;  // lanes per sum
        for (int o = (int)tid / G; o < 4 * nb; o += S::NT / G) {
            double x = 0.0;
#pragma unroll
            for (int i = 0; i < R / G; ++i) x += acc[o * R + tid % G + i * G];
#pragma unroll
            for (int i = G / 2; i > 0; i >>= 1) x += __shfl_xor(x, i);
            if (tid % G == 0) sh.sum[o / (2 * nb)][(o / nb) % 2][o % nb] = x;
        }
    }
};

// Band powers of both chains of the signal S/n held on layout D (sz: the modes
// that mirror themselves): X_A = (S(k) + conj S(-k))/2, X_B = (S(k) - conj
// S(-k))/(2i).  A mode and its mirror have the same powers.
__device__ __forceinline__ void mode_powers(float2 s, float2 m, double& pa, double& pb) {
    const double ar = 0.5 * ((double)s.x + m.x), ai = 0.5 * ((double)s.y - m.y);
    const double br = 0.5 * ((double)s.y + m.y), bi = 0.5 * ((double)s.x - m.x);
    pa = ar * ar + ai * ai;
    pb = br * br + bi * bi;
}
template <int N>
__device__ __forceinline__ void band_powers(const float2 (&v)[16], const float2* sz, const SpectrumArgs& a,
                                            const ProbDev& pr, const BandSums<N>& bs, unsigned tid) {
    using S = typename SquareShape<N>::type;
    constexpr int RC = S::RC, RD = S::RD;
    const DPair dp = d_pair<S>(tid);
    const int16_t* band = a.band + pr.pix_off;
    double pa, pb;
    if (!dp.self) {
#pragma unroll
        for (int k2 = 0; k2 < RD; ++k2) {
            __builtin_amdgcn_sched_barrier(0);
            mode_powers(v[k2], pick(dp.zero, v[RD + (RD - k2) % RD], v[2 * RD - 1 - k2]), pa, pb);
            bs.add(0, band[(dp.k1a + RC * k2) * N + dp.kxa], 2.0 * pa, 2.0 * pb);
        }
    }
    if (tid < 4 * RD) {
        const unsigned k2 = tid % RD, task = tid / RD, m = task < 2 ? (RD - k2) % RD : RD - 1 - k2;
        mode_powers(sz[4 * RD + tid], sz[4 * RD + tid - k2 + m], pa, pb);
        bs.add(0, band[((task < 2 ? 0 : RC / 2) + RC * k2) * N + (task % 2 ? N / 2 : 0)], pa, pb);
    }
}

// Chi-square sums: thread tid owns a contiguous run of the flat variate index,
// which starts in band b0.
template <int N>
__device__ __forceinline__ int chi_run(int total) {
    constexpr int NT = SquareShape<N>::type::NT;
    return 2 * ((total + 2 * NT - 1) / (2 * NT));
}
template <int N>
__device__ __forceinline__ void chi_square(const SpectrumArgs& a, const ProbDev& pr, const SpecShared& sh, int nb,
                                           int b0, uint32_t iteration, int pair, const BandSums<N>& bs, unsigned tid) {
    const int total = sh.pre[nb];
    const int run = chi_run<N>(total);
    const int e0 = (int)tid * run;
    if (e0 >= total) return;
    const int e1 = min(total, e0 + run);
    int b = b0, next = sh.pre[b0 + 1];
    double accA = 0.0, accB = 0.0;
    for (int e = e0; e < e1; e += 2) {
        const Normals2 z = pair_normals((uint32_t)(e >> 1), iteration, (uint32_t)pr.pid, kStageSpectrum,
                                        (uint32_t)pair, a.key0, a.key1);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ee = e + h;
            if (ee >= e1) break;
            if (ee >= next) {
                bs.add(1, b, accA, accB);
                accA = accB = 0.0;
                do next = sh.pre[++b + 1];
                while (next <= ee);
            }
            const float2 zz = h ? z.b : z.a;
            accA += (double)zz.x * zz.x;
            accB += (double)zz.y * zz.y;
        }
    }
    bs.add(1, b, accA, accB);
}

template <int N>
__global__ __launch_bounds__(SquareShape<N>::type::NT, N == 128 ? 4 : N == 64 ? 3 : 2) void resident_spectrum_kernel(SpectrumArgs a) {
    using S = typename SquareShape<N>::type;
    constexpr int P = S::RB, NT = S::NT;
    __shared__ __align__(16) float2 lds[S::LDS];
    __shared__ SpecShared sh;
    __shared__ float2 twl[S::TWS];  // twiddle tables of the four passes
    __shared__ float2 sz[8 * S::RD];
    const unsigned tid = threadIdx.x;
    rect_twiddles<S>(twl, a.tw, a.tw, 1, tid);
    __syncthreads();
    const ItemDev it = a.items[blockIdx.x];
    const ProbDev pr = a.probs[it.prob];
    const unsigned y = tid / (P / 2), j = tid % (P / 2);
    const int nb = a.band_count[it.prob];
    const int bbase = a.band_base[it.prob];
    const double n = (double)N * N;
    const double T = pr.tau;
    const int c0 = 2 * it.pair, c1 = 2 * it.pair + 1;

    // amplitudes, degrees of freedom, coefficient table
    for (int t = tid; t < 2 * nb; t += NT) {
        const int ch = t / nb, b = t % nb;
        const int c = ch ? c1 : c0;
        sh.theta[ch][b] = a.theta_in ? a.theta_in[(int64_t)a.chains_pad * bbase + (int64_t)c * nb + b]
                                     : a.theta0[bbase + b];
    }
    if (tid == 0) {
        int acc = 0;
        for (int b = 0; b < nb; ++b) {
            sh.dof[b] = a.dof[bbase + b];
            sh.pre[b] = acc;
            acc += sh.dof[b];
        }
        sh.pre[nb] = acc;
    }
    __syncthreads();
    for (int b = tid; b < nb; b += NT) refresh_coef(sh, b, T, n);
    int b0 = 0;  // band of this thread's first chi-square variate
    for (const int e0 = (int)tid * chi_run<N>(sh.pre[nb]); b0 < nb - 1 && sh.pre[b0 + 1] <= e0;) ++b0;

    float2 v[16];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int x = 2 * j + P * m;
        if (a.state_in) {
            v[m] = a.state_in[it.field_off + (int64_t)y * N + x];
            v[8 + m] = a.state_in[it.field_off + (int64_t)y * N + x + 1];
        } else if (a.init_scale > 0.f) {
            const uint32_t e2 = (uint32_t)((y * N + x) >> 1);
            const Normals2 z = pair_normals(e2, 0u, (uint32_t)pr.pid, kStageInit, (uint32_t)it.pair, a.key0, a.key1);
            v[m] = cscale(z.a, a.init_scale);
            v[8 + m] = cscale(z.b, a.init_scale);
        } else {
            v[m] = v[8 + m] = make_float2(0.f, 0.f);
        }
    }
    __syncthreads();

    const int64_t iters = (int64_t)a.burn_in + (int64_t)a.n_samples * a.thin;
    for (int64_t i = 0; i < iters; ++i) {
        const uint32_t g = a.iter0 + (uint32_t)i;
        for (int k = 0; k < a.sweeps; ++k) {
            const uint32_t sweep = g * (uint32_t)a.sweeps + (uint32_t)k;
            const float4* pcoef = per_sweep(a.pcoef);
            const float2* psrc = per_sweep(a.psrc);
            const float2* tw = twl + per_sweep_zero();
            unsigned t = tid;
            asm volatile("" : "+v"(t));
            {
                // pixel step t = (1-a) s + a d + sqrt(T(1-a)) xi (spectrum-independent tables)
                const unsigned yy = t / (P / 2), jj = t % (P / 2);
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    __builtin_amdgcn_sched_barrier(0);
                    const uint32_t e2 = (uint32_t)(yy * (N / 2) + jj + (P / 2) * m);
                    const int64_t pp = pr.pix_off / 2 + e2;
                    const float4 c = pcoef[pp];
                    const float2 src = psrc[pp];
                    const Normals2 z =
                        pair_normals(e2, sweep, (uint32_t)pr.pid, kStagePixel, (uint32_t)it.pair, a.key0, a.key1);
                    float2& s0 = v[m];
                    float2& s1 = v[8 + m];
                    s0.x = fmaf(c.x, s0.x, fmaf(c.y, z.a.x, src.x));
                    s0.y = fmaf(c.x, s0.y, fmaf(c.y, z.a.y, src.x));
                    s1.x = fmaf(c.z, s1.x, fmaf(c.w, z.b.x, src.y));
                    s1.y = fmaf(c.z, s1.y, fmaf(c.w, z.b.y, src.y));
                }
            }
            rect_forward<S>(v, lds, tw, t, d_pair<S>(t));
            unsigned t2 = tid;
            asm volatile("" : "+v"(t2));
            harmonic_pair<N>(v, lds, sz, a, pr, sh, sweep, it.pair, t2);
            if (k == a.sweeps - 1) {
                // spectrum draw from this signal: band powers, chi-square sums, new amplitudes
                const BandSums<N> bs(lds, nb, tid);
                bs.clear(tid);
                __syncthreads();
                band_powers<N>(v, sz, a, pr, bs, t2);
                chi_square<N>(a, pr, sh, nb, b0, g, it.pair, bs, tid);
                __syncthreads();
                bs.collect(sh, tid);
                __syncthreads();
                const bool emit = i >= a.burn_in && ((i - a.burn_in + 1) % a.thin) == 0;
                const int64_t slot = emit ? (i - a.burn_in + 1) / a.thin - 1 : 0;
                for (int b = tid; b < nb; b += NT) {
#pragma unroll
                    for (int ch = 0; ch < 2; ++ch) {
                        const double x = sh.sum[1][ch][b];
                        if (sh.dof[b] > 0 && x > 0.0) sh.theta[ch][b] = (2.0 * a.prior_beta + sh.sum[0][ch][b]) / x;
                        const int c = ch ? c1 : c0;
                        if (emit && a.theta_samples && c < a.chains)
                            a.theta_samples[(int64_t)a.chains * a.n_samples * bbase +
                                            ((int64_t)c * a.n_samples + slot) * nb + b] = sh.theta[ch][b];
                    }
                    refresh_coef(sh, b, T, n);
                }
            }
            unsigned t3 = tid;
            asm volatile("" : "+v"(t3));
            rect_inverse<S>(v, lds, tw, t3, d_pair<S>(t3));
        }
        if (a.samples && i >= a.burn_in && ((i - a.burn_in + 1) % a.thin) == 0) {
            const int64_t slot = (i - a.burn_in + 1) / a.thin - 1;
            const int64_t nn = (int64_t)N * N;
            const int64_t base = (int64_t)a.chains * a.n_samples * pr.pix_off;
            float* o0 = a.samples + base + ((int64_t)c0 * a.n_samples + slot) * nn + (int64_t)y * N;
            float* o1 = a.samples + base + ((int64_t)c1 * a.n_samples + slot) * nn + (int64_t)y * N;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int x = 2 * j + P * m;
                *reinterpret_cast<float2*>(o0 + x) = make_float2(v[m].x, v[8 + m].x);
                if (c1 < a.chains) *reinterpret_cast<float2*>(o1 + x) = make_float2(v[m].y, v[8 + m].y);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int64_t o = it.field_off + (int64_t)y * N + 2 * j + P * m;
        a.field[o] = v[m];
        a.field[o + 1] = v[8 + m];
    }
    if (a.theta_out)
        for (int u = tid; u < 2 * nb; u += NT) {
            const int ch = u / nb, b = u % nb;
            const int c = ch ? c1 : c0;
            a.theta_out[(int64_t)a.chains_pad * bbase + (int64_t)c * nb + b] = sh.theta[ch][b];
        }
}

}  // namespace

hipError_t launch_resident_spectrum(int N, const SpectrumArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)a.n_items);
    switch (N) {
        case 32: hipLaunchKernelGGL(resident_spectrum_kernel<32>, grid, dim3(SquareShape<32>::type::NT), 0, s, a); break;
        case 64: hipLaunchKernelGGL(resident_spectrum_kernel<64>, grid, dim3(SquareShape<64>::type::NT), 0, s, a); break;
        case 128: hipLaunchKernelGGL(resident_spectrum_kernel<128>, grid, dim3(SquareShape<128>::type::NT), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mf

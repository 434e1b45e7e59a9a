// Persistent LDS-resident sampler: one workgroup owns one chain pair of an
// N x N image and runs every sweep of Algorithm 1 without leaving the chip;
// only emitted samples and the final state reach HBM.  The field stays in
// registers between the passes of the 2D FFT (mf_resident_fft.hpp).  VALU-bound:
// about 2,390 instructions per wave and sweep at 128^2 in a 512-item launch,
// most of them the transforms' arithmetic (1,550) and the random stream (16
// Philox calls and 32 Box-Muller pairs per thread).
#include "mf_device.hpp"
#include "mf_resident.hpp"
#include "mf_resident_fft.hpp"

namespace mf {

namespace {

// --------------------------------------------------------------- updates --
// The normals of one element pair (two neighbouring pixels, or modes) in units
// of sqrt(2 ln 2), which the tables' standard deviations carry: sd r c feeds the
// pair's first chain (or the real part), sd r s the second.
template <uint32_t STAGE>
__device__ __forceinline__ Polar2 draw(const ResidentArgs& a, const ProbDev& pr, int pair, uint32_t sweep, uint32_t e2) {
    return pair_polar(e2, sweep, (uint32_t)pr.pid, STAGE, (uint32_t)pair, a.key0, a.key1);
}
__device__ __forceinline__ void pixel_draw(float2& s, float2 c, float src, const Polar& z) {
    const float r = c.y * z.r;
    s.x = fmaf(c.x, s.x, fmaf(r, z.c, src));
    s.y = fmaf(c.x, s.y, fmaf(r, z.s, src));
}
__device__ __forceinline__ void mode_draw(float2& s, float2 c, const Polar& z) {
    const float r = c.y * z.r;
    s.x = fmaf(c.x, s.x, r * z.c);
    s.y = fmaf(c.x, s.y, r * z.s);
}

// Draws of a thread that holds one element of each pair (8 values per thread;
// the pair's other element is in the neighbouring lane): each lane draws half of
// its pairs, the even one elements m < R/2, the odd one the others, and passes
// the neighbour its half.  f(m, z) takes element m's normals; pair(m) is its
// pair's stream index.
template <int R, uint32_t STAGE, typename Pair, typename F>
__device__ __forceinline__ void shared_draws(const ResidentArgs& a, const ProbDev& pr, int pair, uint32_t sweep,
                                             bool odd, Pair&& index, F&& f) {
#pragma unroll
    for (int h = 0; h < R / 2; ++h) {
        __builtin_amdgcn_sched_barrier(0);
        const Polar2 z = draw<STAGE>(a, pr, pair, sweep, odd ? index(h + R / 2) : index(h));
        const Polar own = odd ? Polar{z.b.r, z.b.c, z.b.s} : Polar{z.a.r, z.a.c, z.a.s};
        const Polar out = odd ? Polar{z.a.r, z.a.c, z.a.s} : Polar{z.b.r, z.b.c, z.b.s};
        const Polar in{swap_lanes(out.r), swap_lanes(out.c), swap_lanes(out.s)};
        f(h, Polar{odd ? in.r : own.r, odd ? in.c : own.c, odd ? in.s : own.s});
        f(h + R / 2, Polar{odd ? own.r : in.r, odd ? own.c : in.c, odd ? own.s : in.s});
    }
}

// Pixel-space messenger draw on layout A: t = (1-a) s + a d + sqrt(T(1-a)) xi,
// with (1-a, sqrt(T(1-a))) and a d read from per-call tables.
template <typename S>
__device__ __forceinline__ void pixel_update(float2 (&v)[S::V], const ResidentArgs& a, const ProbDev& pr, int pair,
                                             uint32_t sweep, unsigned tid) {
    constexpr int W = S::W, RA = S::RA, RB = S::RB;
    const unsigned y = tid / (RB / S::TA), j = tid % (RB / S::TA);
    if constexpr (S::TA == 2) {
#pragma unroll
        for (int m = 0; m < RA; ++m) {
            // keep the Philox chains from being interleaved (register pressure)
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t e2 = (uint32_t)(y * (W / 2) + j + (RB / 2) * m);  // pixel pair index in the image
            const int64_t pp = pr.pix_off / 2 + e2;
            const float4 c = a.pcoef[pp];   // (1-a, sigma) of pixels x, x+1
            const float2 src = a.psrc[pp];  // a d of pixels x, x+1
            const Polar2 z = draw<kStagePixel>(a, pr, pair, sweep, e2);
            pixel_draw(v[m], make_float2(c.x, c.y), src.x, z.a);
            pixel_draw(v[RA + m], make_float2(c.z, c.w), src.y, z.b);
        }
    } else {
        const uint32_t e0 = y * (W / 2) + (j >> 1);
        const float2* pcoef = reinterpret_cast<const float2*>(a.pcoef) + pr.pix_off + y * W + j;
        const float* psrc = reinterpret_cast<const float*>(a.psrc) + pr.pix_off + y * W + j;
        shared_draws<RA, kStagePixel>(
            a, pr, pair, sweep, j & 1, [&](int m) { return e0 + (RB / 2) * m; },
            [&](int m, const Polar& z) { pixel_draw(v[m], pcoef[RB * m], psrc[RB * m], z); });
    }
}

// Fourier-space draw on layout D: S = (f T + w eta) / n, (f/n, w/n) from a table.
template <typename S>
__device__ __forceinline__ void harmonic_update(float2 (&v)[S::V], const ResidentArgs& a, const ProbDev& pr, int pair,
                                                uint32_t sweep, const DNat<S>& dp) {
    constexpr int W = S::W, RC = S::RC, RD = S::RD;
    if constexpr (S::TD == 2) {
#pragma unroll
        for (int k2 = 0; k2 < RD; ++k2) {
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t e2 = (uint32_t)((dp.k + RC * k2) * (W / 2) + dp.j);  // mode pair index
            const float4 c = a.mcoef[pr.pix_off / 2 + e2];                     // (f, w) of modes kx, kx+1
            const Polar2 z = draw<kStageHarmonic>(a, pr, pair, sweep, e2);
            mode_draw(v[k2], make_float2(c.x, c.y), z.a);
            mode_draw(v[RD + k2], make_float2(c.z, c.w), z.b);
        }
    } else {
        const uint32_t e0 = dp.k * (W / 2) + (dp.j >> 1);
        const float2* mcoef = reinterpret_cast<const float2*>(a.mcoef) + pr.pix_off + dp.k * W + dp.j;
        shared_draws<RD, kStageHarmonic>(
            a, pr, pair, sweep, dp.j & 1, [&](int k2) { return e0 + RC * (W / 2) * k2; },
            [&](int k2, const Polar& z) { mode_draw(v[k2], mcoef[RC * W * k2], z); });
    }
}

// A small call is bound by its launches: the kernel finds its work items and
// checks its final states itself, so that a call is the tables' kernel, this
// one and a synchronisation (2 chains at 32^2, 10 sweeps: 72 -> 58 us).
// Shapes: 16 values per thread, or 8 at 32^2 and, for launches with few items,
// at 64^2 (launch_resident_sample).
template <int N, int V> struct SampleShape { using type = typename SquareShape<N>::type; };
template <> struct SampleShape<32, 8> { using type = Rect<32, 32, 8, 8, 4, 4, 8>; };
template <> struct SampleShape<64, 8> { using type = Rect<64, 64, 8, 8, 8, 8, 8>; };

template <int N, int V>
__global__ __launch_bounds__((SampleShape<N, V>::type::NT), 4) void resident_sample_kernel(ResidentArgs a) {
    using S = typename SampleShape<N, V>::type;
    constexpr int RA = S::RA, RB = S::RB, TA = S::TA;
    __shared__ __align__(16) float2 lds[S::LDS];
    __shared__ float2 twl[S::TWS];  // twiddle tables of the four passes
    const unsigned tid = threadIdx.x;
    rect_twiddles<S>(twl, a.tw, a.tw, 1, tid);
    __syncthreads();  // the first forward pass reads twiddles before any exchange barrier
    // the work item, from the class's problems (no list to build beforehand)
    struct {
        int prob, pair;
        int64_t field_off;
    } it;
    it.prob = a.pids[blockIdx.x / (unsigned)a.pairs];
    it.pair = (int)(blockIdx.x % (unsigned)a.pairs);
    const ProbDev pr = a.probs[it.prob];
    it.field_off = a.pairs * pr.pix_off + (int64_t)it.pair * N * N;
    const unsigned y = tid / (RB / TA), j = tid % (RB / TA);
    auto column = [&](int e) { return TA * j + e / RA + RB * (e % RA); };  // of v[e] in layout A

    // initial state in layout A
    float2 v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const unsigned x = column(e);
        if (a.state_in) {
            v[e] = a.state_in[it.field_off + (int64_t)y * N + x];
        } else if (a.init_scale > 0.f) {
            const Normals2 z = pair_normals((y * N + x) >> 1, 0u, (uint32_t)pr.pid, kStageInit, (uint32_t)it.pair,
                                            a.key0, a.key1);
            v[e] = cscale(make_float2(x & 1 ? z.b.x : z.a.x, x & 1 ? z.b.y : z.a.y), a.init_scale);
        } else {
            v[e] = make_float2(0.f, 0.f);
        }
    }

    const int64_t n = (int64_t)N * N;
    const int64_t K = (int64_t)a.burn_in + (int64_t)a.n_samples * a.thin;
    const int c0 = 2 * it.pair, c1 = 2 * it.pair + 1;
    for (int64_t k = 0; k < K; ++k) {
        const uint32_t sweep = a.sweep0 + (uint32_t)k;
        ResidentArgs ak = a;
        ak.pcoef = per_sweep(a.pcoef);
        ak.psrc = per_sweep(a.psrc);
        ak.mcoef = per_sweep(a.mcoef);
        const float2* tw = twl + per_sweep_zero();
        // The first half of the sweep (pixel draw, forward FFT) keeps what it
        // indexes by the thread id (LDS bases, counter words) live across
        // sweeps; the second half recomputes its own from an opaque copy of
        // the id each sweep, since keeping both halves' live spills registers
        // (16 complex values per thread, 4 waves per SIMD).
        pixel_update<S>(v, ak, pr, it.pair, sweep, tid);
        rect_forward<S>(v, lds, tw, tid, DNat<S>(tid));
        unsigned t2 = tid;
        asm volatile("" : "+v"(t2));
        const DNat<S> dp(t2);
        harmonic_update<S>(v, ak, pr, it.pair, sweep, dp);
        rect_inverse<S>(v, lds, tw, t2, dp);
        if (a.samples && k >= a.burn_in && ((k - a.burn_in + 1) % a.thin) == 0) {
            const int64_t slot = (k - a.burn_in + 1) / a.thin - 1;
            const int64_t base = (int64_t)a.chains * a.n_samples * pr.pix_off;
            float* o0 = a.samples + base + ((int64_t)c0 * a.n_samples + slot) * n + (int64_t)y * N;
            float* o1 = a.samples + base + ((int64_t)c1 * a.n_samples + slot) * n + (int64_t)y * N;
#pragma unroll
            for (int m = 0; m < RA; ++m) {
                const unsigned x = column(m);
                if constexpr (TA == 2) {
                    *reinterpret_cast<float2*>(o0 + x) = make_float2(v[m].x, v[RA + m].x);
                    if (c1 < a.chains) *reinterpret_cast<float2*>(o1 + x) = make_float2(v[m].y, v[RA + m].y);
                } else {
                    o0[x] = v[m].x;
                    if (c1 < a.chains) o1[x] = v[m].y;
                }
            }
        }
    }
    bool bad = false;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        a.field[it.field_off + (int64_t)y * N + column(e)] = v[e];
        bad |= !isfinite(v[e].x) || !isfinite(v[e].y);
    }
    // a NaN or an infinity anywhere in a chain's history reaches its final state
    if (a.flag.call != 0 && __ballot(bad) != 0 && tid % 64 == 0) report_non_finite(a.flag, it.prob);
}

// Per-call coefficient tables of the sampler at lambda = 1 (pairs of elements):
//   pcoef = (1 - a, sqrt(T (1 - a))) for pixels 2e, 2e+1;  psrc = a d
//   mcoef = (f / n, w / n) for modes 2e, 2e+1 with f = nP/(nP+T), w = sqrt(n nP T/(nP+T))
// with the standard deviations times sd_scale.
__global__ void sampler_coef_kernel(const ProbDev* probs, const float* d, const float* nbar, const float* nP,
                                    float4* pcoef, float2* psrc, float4* mcoef, double sd_scale) {
    const ProbDev pr = probs[blockIdx.y];
    const int64_t n = (int64_t)pr.H * pr.W;
    const double T = pr.tau;
    const double inv_n = 1.0 / (double)n;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n / 2; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t g = pr.pix_off + 2 * e;
        float oma[2], sig[2], src[2], f[2], w[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const double nb = nbar[g + q];
            const double aa = isinf(nb) ? 0.0 : T / (T + nb);
            oma[q] = (float)(1.0 - aa);
            sig[q] = (float)(sd_scale * sqrt(T * (1.0 - aa)));
            src[q] = aa > 0.0 ? (float)(aa * (double)d[g + q]) : 0.f;
            const double P = nP[g + q];
            f[q] = (float)(P / (P + T) * inv_n);
            w[q] = (float)(sd_scale * sqrt(P * T / (P + T) * inv_n));
        }
        pcoef[g / 2] = make_float4(oma[0], sig[0], oma[1], sig[1]);
        psrc[g / 2] = make_float2(src[0], src[1]);
        mcoef[g / 2] = make_float4(f[0], w[0], f[1], w[1]);
    }
}

}  // namespace

bool resident_supported(int H, int W) { return H == W && (H == 32 || H == 64 || H == 128); }

hipError_t launch_sampler_coefs(const ProbDev* probs, int n_problems, const float* d, const float* nbar,
                                const float* nP, float4* pcoef, float2* psrc, float4* mcoef, bool polar, hipStream_t s) {
    hipLaunchKernelGGL(sampler_coef_kernel, dim3(32, n_problems), dim3(256), 0, s, probs, d, nbar, nP, pcoef, psrc,
                       mcoef, polar ? 1.1774100225154747 : 1.0);
    return hipGetLastError();
}

template <int N, int V>
static void launch_sample(const ResidentArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((resident_sample_kernel<N, V>), dim3((unsigned)a.n_items), dim3((SampleShape<N, V>::type::NT)), 0,
                       s, a);
}

hipError_t launch_resident_sample(int N, const ResidentArgs& a, hipStream_t s) {
    // 64^2: 8 values per thread (512 threads) while the launch leaves a CU two
    // items or fewer, so that its SIMDs hold up to four waves; beyond that 16
    // values (256 threads) fill the SIMDs too, with fewer exchanges in flight
    // (per sweep, 8 against 16 values: 1-256 items 5.4 against 6.9 us, 512
    // 8.3 against 8.8, 768 12.3 against 11.5, 4096 59 against 53).  32^2 takes 8
    // values throughout (1 item 3.4 against 5.3 us, 1024 4.7 against 5.8, 4096
    // 14.7 against 16.0).  Both shapes round alike, bit for bit.
    constexpr int kTwoPerCu = 2 * kFillBlocks;
    switch (N) {
        case 32: launch_sample<32, 8>(a, s); break;
        case 64: a.n_items <= kTwoPerCu ? launch_sample<64, 8>(a, s) : launch_sample<64, 16>(a, s); break;
        case 128: launch_sample<128, 16>(a, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mf

// Persistent deterministic solve (Wiener filter or adjoint): one workgroup
// owns one problem of N x N pixels and runs every cooling level and the
// convergence phase of the messenger iteration with the variates set to zero
// (Sec. 2.2).  The residual test of the convergence phase is reduced in FP64
// through LDS on the device, so no sweep waits for the host.
//
// The field is real, so it runs as an M x N complex field (M = N/2),
// z(y, x) = t(2y, x) + i t(2y+1, x), which halves the transform.  With E, O the
// transforms of the even and odd rows, Z = E + i O, T(k) = E + W O and T(k + M)
// = E - W O (W = exp(-i th), th = 2 pi ky / N, k + M short for (ky + M, kx)).
// The real, even filter f on T(k) and T(k + M) becomes, with f_+- = (f(k) +-
// f(k + M))/2,
//     E' = f_+ E + f_- W O,   O' = f_- conj(W) E + f_+ O,
// and, since E = (Z(k) + conj Z(-k))/2 and O = (Z(k) - conj Z(-k))/2i,
//     S(k) = E' + i O' = (f_+ - f_- sin th) Z(k) + i f_- cos th conj Z(-k).
// k and -k sit in one thread (mf_resident_fft.hpp), so the step takes no exchange.
//
// 16 complex values per thread at 128^2 (512 threads: two waves per SIMD with
// 256 VGPRs), 8 at 64^2 and 32^2 (256 and 64 threads).  The registers hold the
// pixel coefficients 1 - a and a d and the filter's two coefficients per mode;
// they change only between cooling levels, so a sweep reads no global memory.
// Per sweep, against the full complex field of 16 values per thread with its
// coefficients re-read every sweep: one problem 128^2 11.4 -> 6.6 us, 64^2
// 5.0 -> 3.1, 32^2 3.4 -> 2.4; 256 problems of 128^2 to a residual of 1e-5
// 21.0 -> 11.2 ms.  With 16 values per thread 32^2 and 64^2 took 4.2 us (half
// a wave and two waves, one after the other's latencies).  At 128^2 the VALU
// issues 1,440 instructions per wave and sweep, 72% of the time at two waves
// per SIMD; the rest is latency (LDS exchanges behind block barriers).  A batch
// lasts as long as its slowest image (those 256: 860 to 1,620 sweeps, mean 1,089),
// so over its whole run the VALU issues 51% of the time.
#include "mf_device.hpp"
#include "mf_resident.hpp"
#include "mf_resident_fft.hpp"

namespace mf {

namespace {

// 1 - a and the source of one pixel: a d (Wiener filter) or T g (adjoint).
__device__ __forceinline__ void pixel_coef(float nbar, float sv, float T, int32_t kind, float& oma, float& src) {
    const float aa = T * __builtin_amdgcn_rcpf(T + nbar);  // Nbar = inf: 0
    oma = 1.0f - aa;
    src = kind == kSrcData ? (aa > 0.f ? aa * sv : 0.f) : T * sv;
}

// Sum a double over the workgroup; every thread gets the total.
template <int NT>
__device__ __forceinline__ double block_sum(double x, double* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    if constexpr (NT <= 64) return x;
    const unsigned w = threadIdx.x / 64;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = x;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) s += red[i];
    return s;
}

// The field of an N x N problem.
template <int N> struct SolveShape;
template <> struct SolveShape<32> { using type = Rect<16, 32, 8, 8, 4, 4, 4>; };
template <> struct SolveShape<64> { using type = Rect<32, 64, 8, 8, 8, 8, 4>; };
template <> struct SolveShape<128> { using type = Rect<64, 128, 16, 8, 16, 8, 8>; };

template <int N>
__global__ __launch_bounds__(SolveShape<N>::type::NT, N == 128 ? 2 : 4) void resident_solve_kernel(SolveArgs a) {
    using S = typename SolveShape<N>::type;
    constexpr int M = N / 2, V = S::V, NT = S::NT, RA = S::RA, RD = S::RD;
    __shared__ __align__(16) float2 lds[S::LDS];
    __shared__ float2 tprev[N * M];  // the messenger field of the sweep before a test (each thread's own values)
    __shared__ double red[(NT + 63) / 64];
    __shared__ float2 twl[S::TWS];  // twiddle tables of the four passes
    const unsigned tid = threadIdx.x;
    rect_twiddles<S>(twl, a.tw, a.tw, 2, tid);
    __syncthreads();
    const ItemDev it = a.items[blockIdx.x];
    const ProbDev pr = a.probs[it.prob];
    // v[RA q + m] holds pixels (2y, x) and (2y+1, x), x = TA j + q + RB m
    const int64_t pix0 = pr.pix_off + (int64_t)(tid / (S::RB / S::TA)) * (2 * N) + S::TA * (tid % (S::RB / S::TA));
    auto pixel = [&](int e) { return pix0 + e / RA + S::RB * (e % RA); };

    float2 v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int64_t px = pixel(e);
        v[e] = a.s_init ? make_float2(a.s_init[px], a.s_init[px + N]) : make_float2(0.f, 0.f);
    }

    float2 oma[V], src[V];  // 1 - a and the source of both pixels
    float fa[V], fb[V];     // the filter's coefficients of Z(k) and i conj Z(-k), 1/(N M) folded in
    auto level = [&](float lam) __attribute__((always_inline)) {
        const float T = lam * pr.tau;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const int64_t px = pixel(e);
            pixel_coef(a.nbar[px], a.src[px], T, a.src_kind, oma[e].x, src[e].x);
            pixel_coef(a.nbar[px + N], a.src[px + N], T, a.src_kind, oma[e].y, src[e].y);
        }
        const DPair dp = d_pair<S>(tid);
        constexpr float scale = 0.5f / (float)(N * M);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const unsigned kx = e < RD ? dp.kxa : dp.kxb;
            const unsigned ky = (e < RD ? dp.k1a : dp.k1b) + S::RC * (e % RD);
            const float2 w = a.th[ky];  // (cos th, -sin th)
            const float* np = a.nP + pr.pix_off + (int64_t)ky * N + kx;
            const RealFilter f = real_filter(np[0], np[M * N], T, w, scale);
            fa[e] = f.a;
            fb[e] = f.b;
        }
    };

    auto sweep = [&](bool save, bool check) __attribute__((always_inline)) -> double {
        double acc = 0.0;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            v[e] = make_float2(fmaf(oma[e].x, v[e].x, src[e].x), fmaf(oma[e].y, v[e].y, src[e].y));
            if (check) {
                const float2 tp = tprev[e * NT + tid];
                const double dx = (double)v[e].x - (double)tp.x, dy = (double)v[e].y - (double)tp.y;
                acc += dx * dx + dy * dy;
            }
            if (save) tprev[e * NT + tid] = v[e];
        }
        // thread coordinates from opaque copies of the id, per transform: kept
        // live across sweeps, the LDS addresses of both would spill
        unsigned t = tid;
        asm volatile("" : "+v"(t));
        const DPair dp = d_pair<S>(t);
        rect_forward<S>(v, lds, twl, t, dp);
        // Z(-k) of both tasks: the other task's values (its own if it mirrors itself), in mirrored order
        float2 z[V];
#pragma unroll
        for (int k2 = 0; k2 < RD; ++k2) {
            const float2 ma = pick(dp.zero, v[(RD - k2) % RD], v[RD - 1 - k2]);
            const float2 mb = pick(dp.zero, v[RD + (RD - k2) % RD], v[2 * RD - 1 - k2]);
            z[k2] = pick(dp.self, ma, mb);
            z[RD + k2] = pick(dp.self, mb, ma);
        }
#pragma unroll
        for (int e = 0; e < V; ++e)
            v[e] = make_float2(fmaf(fa[e], v[e].x, fb[e] * z[e].y), fmaf(fa[e], v[e].y, fb[e] * z[e].x));
        unsigned t2 = tid;
        asm volatile("" : "+v"(t2));
        rect_inverse<S>(v, lds, twl, t2, d_pair<S>(t2));
        return check ? block_sum<NT>(acc, red) : 0.0;
    };

    // the cooling levels, then (phase n) the convergence phase at the last one
    int total = a.total0;
    double residual = __builtin_nan("");
    int converged = a.tol > 0 ? 0 : 1;
    for (int ph = 0; ph < a.lv.n + (a.tol > 0 ? 1 : 0); ++ph) {
        const bool conv = ph == a.lv.n;
        const double lam = a.lv.lambda[conv ? ph - 1 : ph];
        const int end = conv ? a.max_sweeps : total + a.lv.sweeps[ph];
        if (!conv && end <= total) continue;
        level((float)lam);
        const double T = lam * (double)pr.tau;
        double bnorm = 0.0;
        if (conv) {
            // ||b||^2 with b = N_eff^-1 d (data) or g (gradient) at the final level
            double bb = 0.0;
            for (int64_t px = pr.pix_off + tid; px < pr.pix_off + N * N; px += NT) {
                const double nb = a.nbar[px];
                const double b = a.src_kind == kSrcData ? (isinf(nb) ? 0.0 : (double)a.src[px] / (nb + T))
                                                        : (double)a.src[px];
                bb += b * b;
            }
            bnorm = sqrt(block_sum<NT>(bb, red));
        }
        const int before = total;
        while (total < end) {
            const int c = total + 1;
            const bool check = conv && (c % a.check_every == 0) && (c - 1 >= before + 1);
            const bool save = conv && ((c + 1) % a.check_every == 0);
            const double acc = sweep(save, check);
            ++total;
            if (check) {
                residual = bnorm == 0.0 ? 0.0 : sqrt(acc) / (T * bnorm);  // NaN stays NaN
                if (residual <= a.tol) {
                    converged = 1;
                    break;
                }
                if (!isfinite(residual)) {  // NaN or Inf in the inputs or the iterate: stop
                    converged = -1;
                    break;
                }
            }
        }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int64_t px = pixel(e);
        a.s_out[px] = v[e].x;
        a.s_out[px + N] = v[e].y;
    }
    if (tid == 0 && a.info) {
        a.info[3 * blockIdx.x + 0] = (double)total;
        a.info[3 * blockIdx.x + 1] = (double)converged;
        a.info[3 * blockIdx.x + 2] = residual;
    }
}

template <int N>
void launch_solve(const SolveArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(resident_solve_kernel<N>, dim3((unsigned)a.n_items), dim3(SolveShape<N>::type::NT), 0, s, a);
}

}  // namespace

hipError_t launch_resident_solve(int N, const SolveArgs& a, hipStream_t s) {
    switch (N) {
        case 32: launch_solve<32>(a, s); break;
        case 64: launch_solve<64>(a, s); break;
        case 128: launch_solve<128>(a, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace mf

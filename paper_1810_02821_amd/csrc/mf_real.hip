// Streamed deterministic solve of real fields: the Wiener filter and the
// adjoint with the variates set to zero (Sec. 2.2), for power-of-two sides from
// 256.  The field is real, so it runs as an H x M complex field (M = W/2),
// z(y, x) = t(y, 2x) + i t(y, 2x+1), which is the image itself in memory.  As in
// the persistent solve (mf_solve.hip, there along y), with th = 2 pi kx / W,
// f_+- = (f(k) +- f(k + M))/2 and k + M short for (ky, kx + M),
//     S(k) = (f_+ - f_- sin th) Z(k) + i f_- cos th conj Z(-k).
// Against the complex field whose imaginary part was zero, that halves the
// bytes and the transforms of both kernels.
//
// row kernel: inverse row FFT, pixel step t = (1 - a) s + src, forward row FFT.
// column kernel: forward column FFT, Fourier step, inverse column FFT on pairs
//   of mirrored columns (c and M - c; 0 and M/2 together); Z(-k) comes through
//   LDS, in natural order.
// The usual launch is one image (a filter or its gradient), far too small to
// fill the GPU, so what counts is the length of a wave's own chain:
//   - four elements per lane (radix-4 passes at both ends, one or two larger
//     ones between): a quarter of the instructions per wave that 16 take (256^2,
//     16 per lane: 14 us a sweep, 4 per lane: 9.7);
//   - the field in 4 x 4 tiles (one 128-byte line each), so that a wave's column
//     access touches 16 lines instead of 64 and its row access 8 or 16;
//   - rows and columns that fit in a wave exchange without block barriers.
// Batches take the same shapes (us a sweep, complex fields / these): 1 of 256^2
// 12.2 / 8.4, 64 of 256^2 41.1 / 24.0, 16 of 512^2 42.7 / 26.4, 16 of 1024^2 193
// / 93, 4 of 2048^2 244 / 138.
#pragma clang fp contract(on)
#include "mf_device.hpp"
#include "mf_kernels.hpp"
#include "mf_real.hpp"
#include "mf_streamed_fft.hpp"

namespace mf {

namespace {

// Radices of a transform of length L: 4, M1, M2, M3 (1: none), 4.
template <int L> struct RealPlan;
template <> struct RealPlan<128> { static constexpr int M1 = 4, M2 = 2, M3 = 1; };
template <> struct RealPlan<256> { static constexpr int M1 = 4, M2 = 4, M3 = 1; };
template <> struct RealPlan<512> { static constexpr int M1 = 4, M2 = 4, M3 = 2; };
template <> struct RealPlan<1024> { static constexpr int M1 = 4, M2 = 4, M3 = 4; };
template <> struct RealPlan<2048> { static constexpr int M1 = 8, M2 = 4, M3 = 4; };

// LDS layouts of a transform's exchanges: the first pass writes A0, the middle
// passes A1 to A3 (the last pass reads AL).  The same for both directions.
template <int L>
struct RealLayout {
    static constexpr int M1 = RealPlan<L>::M1, M2 = RealPlan<L>::M2, M3 = RealPlan<L>::M3;
    static_assert(16 * M1 * M2 * M3 == L, "radix plan");
    static constexpr int A0 = pad_of(L, 4, 1), A1 = pad_of(L, M1, 4), A2 = pad_of(L, M2, 4 * M1);
    static constexpr int A3 = M3 > 1 ? pad_of(L, M3, 4 * M1 * M2) : A2;
    static constexpr int AL = A3;
    static constexpr int LEN = pad_len(L, std::max({A0, A1, A2, A3}));
};
// Synchronise the threads of one transform: a wave's LDS operations take effect
// in order, so inside a wave only the compiler has to keep them so.
template <bool WAVE>
__device__ __forceinline__ void sync_group() {
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    } else {
        __syncthreads();
    }
}
// A middle pass of radix R after NS points: forward as stockham_pass, from layout
// AI to AO; inverse its adjoint, from AO back to AI (inverse butterfly, then the
// conjugate twiddle).  With every pass of the inverse transform the adjoint of
// one of the forward transform's, their twiddles' errors in angle cancel.
template <int L, int R, int NS, int TPG, bool INV, int AI, int AO>
__device__ __forceinline__ void real_pass(float2* buf, unsigned lane, const float2* tw) {
    constexpr bool WAVE = TPG <= 64;
    constexpr int NT = L / R, TPT = (NT + TPG - 1) / TPG;
    float2 v[TPT][R];
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const unsigned j = lane + t * TPG;
        if (NT % TPG == 0 || j < (unsigned)NT) {
            const unsigned k = j % NS, o = (j / NS) * NS * R + k;
#pragma unroll
            for (int r = 0; r < R; ++r) v[t][r] = buf[INV ? lpos_write<AO, R, NS>(o, r) : lpos_step<AI, NT>(j, r)];
            if constexpr (INV) dft<R, true>(v[t]);
#pragma unroll
            for (int r = 1; r < R; ++r) {
                const float2 w = tw[(r * k) * (L / (NS * R))];
                v[t][r] = INV ? cmulc(v[t][r], w) : cmul(v[t][r], w);
            }
            if constexpr (!INV) dft<R, false>(v[t]);
        }
    }
    sync_group<WAVE>();
#pragma unroll
    for (int t = 0; t < TPT; ++t) {
        const unsigned j = lane + t * TPG;
        if (NT % TPG == 0 || j < (unsigned)NT) {
            const unsigned o = (j / NS) * NS * R + j % NS;
#pragma unroll
            for (int r = 0; r < R; ++r) buf[INV ? lpos_step<AI, NT>(j, r) : lpos_write<AO, R, NS>(o, r)] = v[t][r];
        }
    }
    sync_group<WAVE>();
}
// The transform of a row or column, element (mode) j + r L/4 at v[r] on both
// sides; `buf` in LDS.
template <int L, int TPG, bool INV>
__device__ __forceinline__ void real_fft(float2 (&v)[4], float2* buf, unsigned j, const float2* tw) {
    using Y = RealLayout<L>;
    constexpr bool WAVE = TPG <= 64;
    constexpr int Q = L / 4, N1 = 4, N2 = 4 * Y::M1, N3 = 4 * Y::M1 * Y::M2;
    if constexpr (!INV) {
        dft4<false>(v[0], v[1], v[2], v[3]);
#pragma unroll
        for (int r = 0; r < 4; ++r) buf[lpos_run<Y::A0, 4>(j, r)] = v[r];
        sync_group<WAVE>();
        real_pass<L, Y::M1, N1, TPG, false, Y::A0, Y::A1>(buf, j, tw);
        real_pass<L, Y::M2, N2, TPG, false, Y::A1, Y::A2>(buf, j, tw);
        if constexpr (Y::M3 > 1) real_pass<L, Y::M3, N3, TPG, false, Y::A2, Y::A3>(buf, j, tw);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = buf[lpos_step<Y::AL, Q>(j, r)];
#pragma unroll
        for (int r = 1; r < 4; ++r) v[r] = cmul(v[r], tw[r * j]);
        dft4<false>(v[0], v[1], v[2], v[3]);
    } else {
        dft4<true>(v[0], v[1], v[2], v[3]);
#pragma unroll
        for (int r = 1; r < 4; ++r) v[r] = cmulc(v[r], tw[r * j]);
#pragma unroll
        for (int r = 0; r < 4; ++r) buf[lpos_step<Y::AL, Q>(j, r)] = v[r];
        sync_group<WAVE>();
        if constexpr (Y::M3 > 1) real_pass<L, Y::M3, N3, TPG, true, Y::A2, Y::A3>(buf, j, tw);
        real_pass<L, Y::M2, N2, TPG, true, Y::A1, Y::A2>(buf, j, tw);
        real_pass<L, Y::M1, N1, TPG, true, Y::A0, Y::A1>(buf, j, tw);
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = buf[lpos_run<Y::A0, 4>(j, r)];
        dft4<true>(v[0], v[1], v[2], v[3]);
    }
}

// Offset of row y (column c) of a field in 4 x 4 tiles of M columns; element
// (y, c) is at their sum.
__device__ __forceinline__ unsigned tile_y(unsigned y, unsigned M) { return (y >> 2) * 4 * M + (y & 3) * 4; }
__device__ __forceinline__ unsigned tile_c(unsigned c) { return (c >> 2) * 16 + (c & 3); }

// Rows of a block: four elements per lane, at least a wave.
template <int L>
struct RealRow {
    static constexpr int TPR = L / 4;                 // threads per row
    static constexpr int ROWS = TPR < 64 ? 64 / TPR : 1;
    static constexpr int NTH = ROWS * TPR;
};

template <int L, int MODE>
__global__ __launch_bounds__(RealRow<L>::NTH) void real_row_kernel(RealArgs a) {
    using Y = RealLayout<L>;
    constexpr int W = 2 * L, Q = L / 4, ROWS = RealRow<L>::ROWS, NTH = RealRow<L>::NTH;
    constexpr bool WAVE = Q <= 64;
    __shared__ float2 lds[ROWS * Y::LEN];
    __shared__ float2 twl[L];  // W_L^r
    __shared__ double red[NTH / 64];
    const unsigned tid = threadIdx.x, rid = tid / Q, lane = tid % Q;
    const unsigned g0 = xcd_block(blockIdx.x, gridDim.x) * ROWS;  // ROWS divides H
    const int item = (int)(g0 >> a.log_h), y = (int)((g0 & ((1u << a.log_h) - 1)) + rid);
    const ItemDev it = a.items[item];
    const int64_t prow = it.pix_off + (int64_t)y * W;  // pixels of the row
    const int64_t frow = it.pix_off / 2 + tile_y((unsigned)y, L) + tile_c(lane);  // + 4 Q r: element lane + r Q
    float2* fld = a.field + frow;
    float2* row = lds + rid * Y::LEN;
    const float2* tw = a.tw_w;

    float2 v[4];
    if constexpr (MODE & kRowInv) {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fld[4 * Q * r];
    }
    // the pixel tables go out beside the field
    float2 nb[4], sr[4];
    if constexpr (MODE & kRowFwd) {
        const float* src = a.src + prow + 2 * lane;
        const float* nbar = a.nbar + prow + 2 * lane;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            nb[r] = *reinterpret_cast<const float2*>(nbar + 2 * r * Q);
            sr[r] = make_float2(src[2 * r * Q], src[2 * r * Q + 1]);
        }
    }
#pragma unroll
    for (int i = 0; i < L / NTH; ++i) twl[tid + i * NTH] = tw[2 * (tid + i * NTH)];
    __syncthreads();  // the twiddles
    if constexpr (MODE & kRowInv) {
        real_fft<L, Q, true>(v, row, lane, twl);
        // v[r] is the state at pixels 2x, 2x + 1, x = lane + r L/4
        if constexpr (!(MODE & kRowFwd)) {
            float* o = a.s_out + prow + 2 * lane;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[2 * r * Q] = v[r].x;
                o[2 * r * Q + 1] = v[r].y;
            }
            return;
        }
    } else {
        const float* s0 = a.s_init;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t px = prow + 2 * (lane + r * Q);
            v[r] = s0 ? make_float2(s0[px], s0[px + 1]) : make_float2(0.f, 0.f);
        }
    }
    if constexpr (MODE & kRowFwd) {
        // ---- pixel step t = (1 - a) s + src
        const float T = a.lambda * it.tau;
        const int32_t kind = a.src_kind;
        auto step = [&](float s, float nbar, float sv) {
            const float aa = T * __builtin_amdgcn_rcpf(T + nbar);  // Nbar = inf: 0
            return fmaf(1.0f - aa, s, kind == kSrcData ? (aa > 0.f ? aa * sv : 0.f) : T * sv);
        };
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = make_float2(step(v[r].x, nb[r].x, sr[r].x), step(v[r].y, nb[r].y, sr[r].y));
        if (a.check_t | a.save_t) {
            float2* ts = a.t_save + frow;
            if (a.check_t) {
                double acc = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float2 p = ts[4 * Q * r];
                    const double dx = (double)v[r].x - p.x, dy = (double)v[r].y - p.y;
                    acc += dx * dx + dy * dy;
                }
                constexpr int G = Q < 64 ? Q : 64;  // lanes of one row in a wave
#pragma unroll
                for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
                if constexpr (Q > 64) {
                    if (tid % 64 == 0) red[tid / 64] = acc;
                    __syncthreads();
                    acc = 0.0;
#pragma unroll
                    for (int i = 0; i < NTH / 64; ++i) acc += red[i];
                }
                if (lane == 0) a.partials[(int64_t)y * a.n_items + item] = acc;
            }
            if (a.save_t) {
#pragma unroll
                for (int r = 0; r < 4; ++r) ts[4 * Q * r] = v[r];
            }
        }
        sync_group<WAVE>();  // the row's last reads are done
        real_fft<L, Q, false>(v, row, lane, twl);
#pragma unroll
        for (int r = 0; r < 4; ++r) fld[4 * Q * r] = v[r];
    }
}

// A pair of mirrored columns per block, L/4 threads per column: slot 0 of pair P
// is column P, slot 1 its mirror M - P; pair 0 is columns 0 and M/2, which mirror
// themselves.  (Two pairs per block took 14% longer at one 256^2 image, as long
// at 8 of 512^2 and 9% less at 64 of 256^2.)
template <int L>
__global__ __launch_bounds__(L / 2) void real_col_kernel(RealArgs a) {
    using Y = RealLayout<L>;
    constexpr int Q = L / 4, NTH = 2 * Q;
    constexpr bool WAVE = Q <= 64;
    constexpr int AN = pad_of(L, 4, Q);  // the modes in natural order
    constexpr int SEG = std::max(Y::LEN, pad_len(L, AN)) | 1;
    __shared__ float2 lds[2 * SEG];
    __shared__ float2 twl[L];
    const unsigned tid = threadIdx.x, slot = tid / Q, j = tid % Q;
    const unsigned log_m = a.log_w - 1, M = 1u << log_m;
    const unsigned t = xcd_block(blockIdx.x, gridDim.x);
    const int item = (int)(t >> (log_m - 1));
    const unsigned P = t & (M / 2 - 1);
    const unsigned c = slot == 0 ? P : P == 0 ? M / 2 : M - P;  // this thread's column
    const ItemDev it = a.items[item];
    float2* fld = a.field + it.pix_off / 2 + tile_c(c) + tile_y(j, M);  // + Q M r: row j + r Q
    float2 v[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = fld[Q * M * r];
    // n P at modes (j + r Q, c) and (j + r Q, c + M)
    const float2* np = a.nPt + it.pix_off / 2 + ((int64_t)(c >> 1) * L) + j;
    float2 q0[4], q1[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        q0[r] = np[r * Q];
        q1[r] = np[r * Q + (int64_t)(M >> 1) * L];
    }
    const float2 th = a.th[c];  // (cos th, -sin th)
#pragma unroll
    for (int i = 0; i < (L + NTH - 1) / NTH; ++i)
        if (L % NTH == 0 || tid + i * NTH < (unsigned)L) twl[tid + i * NTH] = a.tw_h[tid + i * NTH];
    float2* col = lds + slot * SEG;
    __syncthreads();  // the twiddles
    real_fft<L, Q, false>(v, col, j, twl);
    sync_group<WAVE>();
#pragma unroll
    for (int r = 0; r < 4; ++r) col[lpos_step<AN, Q>(j, r)] = v[r];
    __syncthreads();

    // ---- Fourier step: v[r] is mode ky = j + r Q
    {
        const float T = a.lambda * it.tau;
        const float scale = 0.5f / ((float)L * (float)M);
        const float2* other = P == 0 ? col : lds + (slot ^ 1) * SEG;
        const bool odd = c & 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float2 zm = other[lpos<AN>((L - j - r * Q) % L)];
            const float2 p0 = q0[r], p1 = q1[r];
            const float px0 = p0.x, py0 = p0.y, px1 = p1.x, py1 = p1.y;
            const RealFilter f = real_filter(odd ? py0 : px0, odd ? py1 : px1, T, th, scale);
            v[r] = make_float2(fmaf(f.a, v[r].x, f.b * zm.y), fmaf(f.a, v[r].y, f.b * zm.x));
        }
    }
    __syncthreads();  // the other column has read its mirrors
    real_fft<L, Q, true>(v, col, j, twl);
#pragma unroll
    for (int r = 0; r < 4; ++r) fld[Q * M * r] = v[r];
}

template <int L, int MODE>
hipError_t row_launch(const RealArgs& a, hipStream_t s) {
    using R = RealRow<L>;
    hipLaunchKernelGGL((real_row_kernel<L, MODE>), dim3((unsigned)((int64_t)a.n_items * (1 << a.log_h) / R::ROWS)), dim3(R::NTH), 0, s,
                       a);
    return hipGetLastError();
}
template <int MODE>
hipError_t row_mode(const RealArgs& a, hipStream_t s) {
    switch (1 << a.log_w) {
        case 256: return row_launch<128, MODE>(a, s);
        case 512: return row_launch<256, MODE>(a, s);
        case 1024: return row_launch<512, MODE>(a, s);
        case 2048: return row_launch<1024, MODE>(a, s);
        default: return hipErrorInvalidValue;
    }
}
template <int L>
hipError_t col_launch(const RealArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(real_col_kernel<L>, dim3((unsigned)((int64_t)a.n_items << (a.log_w - 2))), dim3(L / 2), 0, s, a);
    return hipGetLastError();
}

}  // namespace

bool real_solve_supported(int H, int W) {
    auto ok = [](int v) { return v == 256 || v == 512 || v == 1024 || v == 2048; };
    return ok(H) && ok(W);
}
hipError_t launch_real_row(int mode, const RealArgs& a, hipStream_t s) {
    switch (mode) {
        case kRowInv: return row_mode<kRowInv>(a, s);
        case kRowFwd: return row_mode<kRowFwd>(a, s);
        case kRowInvFwd: return row_mode<kRowInvFwd>(a, s);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_real_col(const RealArgs& a, hipStream_t s) {
    switch (1 << a.log_h) {
        case 256: return col_launch<256>(a, s);
        case 512: return col_launch<512>(a, s);
        case 1024: return col_launch<1024>(a, s);
        case 2048: return col_launch<2048>(a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mf

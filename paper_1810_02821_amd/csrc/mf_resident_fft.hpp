// Register/LDS 2D FFT of one workgroup over an H x W complex field (H = RC RD,
// W = RA RB), V values per thread.  A 2D FFT is four passes, two along each
// dimension:
//   rows    x = x0 + RB m,  kx = k1 + RA k2  (pass A: radix-RA over m, pass B: radix-RB over x0)
//   columns y = y0 + RD m,  ky = k1 + RC k2  (pass C: radix-RC over m, pass D: radix-RD over y0)
// with twiddles W_W^(x0 k1) after A and W_H^(y0 k1) after C.  The forward
// transform runs A, B, C, D (decimation in frequency); the inverse runs the
// transposed passes D', C', B', A' (decimation in time), so the Fourier-space
// update happens in pass D's registers and the pixel-space update in pass A's,
// and LDS is touched only for the three exchanges between passes.
//
// LDS exchanges place each row at a base of its own and keep the column in
// order, so that the elements one thread moves in an exchange lie at constant
// offsets from one base (the immediate offsets of ds_read/ds_write, no address
// arithmetic per element), while every 16- or 32-lane phase of an LDS
// instruction still touches distinct banks:
//   E1  row y starts at y W + 2 s(y) + 32 (y / R1), R1 = 32/RB, s(y) = (RB/2)(y % R1) + (y / R1) % (RB/2):
//       the R1 rows of one phase of pass A's accesses fall on disjoint parts
//       of the banks, and 16 consecutive rows (pass B's lanes) on 16 distinct
//       16-byte bank groups;
//   E2  pitch W + 1 (pass B's lanes walk rows, pass C's walk columns);
//   E3  pitch W + 1 as well (both sides' lanes walk columns).
// In the exchanges C -> C (E2 read, E3 written, and back), D -> D and A -> A
// each thread writes exactly the addresses it has just read (E2 and E3 share a
// layout), and a wave's LDS operations take effect in order, so no block
// barrier is needed there: 8 a sweep.  A caller that writes the buffer between
// two transforms synchronises the block first.
// Twiddles W^(a b) sit in LDS in one small table per pass, row a (the thread's
// own index: x0 in A, k1 in B and D, y0 in C) by column b (the register's), so
// that a thread's twiddles too lie at constant offsets from one base.
//
// A pass-D task (kx, k1) is one radix-RD butterfly and holds the modes (k1 +
// RC k2, kx), k2 < RD.  Two assignments of tasks to threads: DNat, neighbouring
// columns (a Philox call's two modes in one thread or in neighbouring lanes);
// and DPair (V = 2 RD), a task and its mirror (-kx, -k1), which holds the modes
// -k of the first, so that a Fourier step that combines Z(k) with Z(-k) needs
// no exchange.  Four tasks (kx in {0, W/2}, k1 in {0, RC/2}) are their own
// mirrors; two threads take two of them each.
#pragma once
#include "mf_device.hpp"

namespace mf {

namespace {

__device__ __forceinline__ void st2(float2* lds, unsigned i, float2 a, float2 b) {
    *reinterpret_cast<float4*>(lds + i) = make_float4(a.x, a.y, b.x, b.y);
}
__device__ __forceinline__ void ld2(const float2* lds, unsigned i, float2& a, float2& b) {
    const float4 q = *reinterpret_cast<const float4*>(lds + i);
    a = make_float2(q.x, q.y);
    b = make_float2(q.z, q.w);
}

template <int R, bool INV>
__device__ __forceinline__ void dft_slice(float2* v) {
    float2 t[R];
#pragma unroll
    for (int i = 0; i < R; ++i) t[i] = v[i];
    dft<R, INV>(t);
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = t[i];
}

// Hide a pointer from loop-invariant code motion: tables are re-read (from
// cache) every sweep instead of being held in registers across sweeps.
// An opaque zero, to offset an LDS table per sweep without losing its address space.
__device__ __forceinline__ unsigned per_sweep_zero() {
    unsigned z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

template <typename T>
__device__ __forceinline__ const T* per_sweep(const T* p) {
    // an opaque zero offset (not the pointer itself), so that the pointer
    // keeps its global address space: flat loads would also count against
    // the LDS wait counter
    unsigned z = 0;
    asm volatile("" : "+s"(z));
    return p + z;
}

template <bool INV>
__device__ __forceinline__ float2 twiddle(float2 v, const float2* __restrict__ row, int col) {
    const float2 w = row[col];
    return INV ? cmulc(v, w) : cmul(v, w);
}

template <int H_, int W_, int V_, int RA_, int RB_, int RC_, int RD_>
struct Rect {
    static constexpr int H = H_, W = W_, V = V_, RA = RA_, RB = RB_, RC = RC_, RD = RD_;
    static_assert(H == RC * RD && W == RA * RB, "Rect shape");
    static constexpr int NT = H * W / V;    // threads per workgroup
    static constexpr int TA = V / RA;       // tasks per thread in passes A and D (1 or 2), B and C
    static constexpr int TD = V / RD;
    static constexpr int TB = V / RB;
    static constexpr int TC = V / RC;
    static constexpr int R1 = 32 / RB;
    static constexpr int YC = H / V;        // step of pass C's y0 between a thread's tasks
    static_assert(TA <= 2 && TD <= 2 && TB >= 1 && TC >= 1 && NT % W == 0, "Rect shape");
    static constexpr int e1_base(int r) { return r * W + 2 * ((RB / 2) * (r % R1) + (r / R1) % (RB / 2)) + 32 * (r / R1); }
    static constexpr int extent() {
        int m = H * (W + 1);
        for (int r = 0; r < H; ++r) m = e1_base(r) + W > m ? e1_base(r) + W : m;
        return m;
    }
    static constexpr int LDS = extent();    // float2 elements of the exchange buffer
    // twiddle tables: A [x0 < RB][k1 < RA] pitch RA + 1, B [k1 < RA][x0 < RB],
    // C [y0 < RD][k1 < RC], D [k1 < RC][y0 < RD] pitch RD + 1
    static constexpr int TWA = 0, TWB = TWA + (RA + 1) * RB, TWC = TWB + RA * RB, TWD = TWC + RD * RC;
    static constexpr int TWS = TWD + (RD + 1) * RC;
};

// The tasks of a thread in pass D: task q's column kx(q) and k1(q).
struct DPair {
    unsigned kxa, k1a, kxb, k1b;
    bool self;  // each task is its own mirror (else each is the other's)
    bool zero;  // k1a = 0: mode k2 mirrors (RD - k2) mod RD, else RD - 1 - k2
    __device__ __forceinline__ unsigned kx(int q) const { return q ? kxb : kxa; }
    __device__ __forceinline__ unsigned k1(int q) const { return q ? k1b : k1a; }
};
template <typename S>
struct DNat {
    unsigned j, k;  // columns TD j + q, k1
    __device__ __forceinline__ explicit DNat(unsigned tid) : j(tid % (S::W / S::TD)), k(tid / (S::W / S::TD)) {}
    __device__ __forceinline__ unsigned kx(int q) const { return S::TD * j + q; }
    __device__ __forceinline__ unsigned k1(int) const { return k; }
};
template <typename S>
__device__ __forceinline__ DPair d_pair(unsigned tid) {
    static_assert(S::TD == 2, "a task and its mirror per thread");
    constexpr unsigned W = S::W, RC = S::RC;
    const unsigned kx = tid % (W / 2), k1 = tid / (W / 2);
    DPair p;
    p.self = kx == 0 && (k1 == 0 || k1 == RC / 2);
    p.zero = k1 == 0;
    p.kxa = kx == 0 && k1 > RC / 2 ? W / 2 : kx;
    p.k1a = k1;
    p.kxb = p.self ? W / 2 : (W - p.kxa) % W;
    p.k1b = p.self ? k1 : (RC - k1) % RC;
    return p;
}

// Fill the twiddle tables from twr[r] = W_W^r and twc[r * sc] = W_H^r.
template <typename S>
__device__ __forceinline__ void rect_twiddles(float2* t, const float2* __restrict__ twr,
                                              const float2* __restrict__ twc, int sc, unsigned tid) {
    for (unsigned e = tid; e < (unsigned)S::TWS; e += S::NT) {
        if (e < (unsigned)S::TWB) {
            const unsigned a = e / (S::RA + 1), b = e % (S::RA + 1);
            t[e] = twr[b < (unsigned)S::RA ? a * b : 0];
        } else if (e < (unsigned)S::TWC) {
            const unsigned q = e - S::TWB;
            t[e] = twr[(q / S::RB) * (q % S::RB)];
        } else if (e < (unsigned)S::TWD) {
            const unsigned q = e - S::TWC;
            t[e] = twc[(q / S::RC) * (q % S::RC) * sc];
        } else {
            const unsigned q = e - S::TWD, a = q / (S::RD + 1), b = q % (S::RD + 1);
            t[e] = twc[b < (unsigned)S::RD ? a * b * sc : 0];
        }
    }
}

template <typename S>
__device__ __forceinline__ unsigned rect_e1(unsigned r, unsigned c) {
    return r * S::W + 2 * ((S::RB / 2) * (r % S::R1) + (r / S::R1) % (S::RB / 2)) + 32 * (r / S::R1) + c;
}
template <typename S>
__device__ __forceinline__ unsigned rect_e2(unsigned r, unsigned c) {
    return r * (S::W + 1) + c;
}

// Thread coordinates in each layout (tid in [0, NT)):
//   A: y = tid / (RB/TA), j = tid % (RB/TA); holds x = TA j + q + RB m  at v[RA q + m]
//   B: t = tid + i NT (i < TB): y = t % H, k1 = t / H; holds x0         at v[RB i + x0]
//   C: kx = tid % W, y0 = tid / W + i YC (i < TC); holds m              at v[RC i + m]
//   D: task q's modes (k1 + RC k2, kx) at v[RD q + k2]
template <typename S>
__device__ __forceinline__ void store_e1_a(float2* lds, const float2 (&v)[S::V], unsigned y, unsigned j) {
#pragma unroll
    for (int k = 0; k < S::RA; ++k) {
        if constexpr (S::TA == 2) st2(lds, rect_e1<S>(y, k * S::RB + 2 * j), v[k], v[S::RA + k]);
        else lds[rect_e1<S>(y, k * S::RB + j)] = v[k];
    }
}
template <typename S>
__device__ __forceinline__ void load_e1_a(const float2* lds, float2 (&v)[S::V], unsigned y, unsigned j) {
#pragma unroll
    for (int k = 0; k < S::RA; ++k) {
        if constexpr (S::TA == 2) ld2(lds, rect_e1<S>(y, k * S::RB + 2 * j), v[k], v[S::RA + k]);
        else v[k] = lds[rect_e1<S>(y, k * S::RB + j)];
    }
}

template <typename S, typename D>
__device__ __forceinline__ void rect_forward(float2 (&v)[S::V], float2* lds, const float2* __restrict__ tw,
                                             unsigned tid, const D& dp) {
    constexpr int RA = S::RA, RB = S::RB, RC = S::RC, RD = S::RD, H = S::H;
    const unsigned ya = tid / (RB / S::TA), j = tid % (RB / S::TA);
    // A
#pragma unroll
    for (int q = 0; q < S::TA; ++q) {
        dft_slice<RA, false>(v + RA * q);
        const float2* row = tw + S::TWA + (RA + 1) * (S::TA * j + q);
#pragma unroll
        for (int k = 1; k < RA; ++k) v[RA * q + k] = twiddle<false>(v[RA * q + k], row, k);
    }
    store_e1_a<S>(lds, v, ya, j);
    __syncthreads();
    // B
#pragma unroll
    for (int i = 0; i < S::TB; ++i) {
        const unsigned t = tid + i * S::NT, y = t % H, k1 = t / H;
#pragma unroll
        for (int x = 0; x < RB; x += 2) ld2(lds, rect_e1<S>(y, k1 * RB + x), v[RB * i + x], v[RB * i + x + 1]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::TB; ++i) dft_slice<RB, false>(v + RB * i);
#pragma unroll
    for (int i = 0; i < S::TB; ++i) {
        const unsigned t = tid + i * S::NT, y = t % H, k1 = t / H;
#pragma unroll
        for (int k = 0; k < RB; ++k) lds[rect_e2<S>(y, k1 + RA * k)] = v[RB * i + k];
    }
    __syncthreads();
    // C
    const unsigned kx = tid % S::W, yc = tid / S::W;
#pragma unroll
    for (int i = 0; i < S::TC; ++i)
#pragma unroll
        for (int m = 0; m < RC; ++m) v[RC * i + m] = lds[rect_e2<S>(yc + i * S::YC + RD * m, kx)];
#pragma unroll
    for (int i = 0; i < S::TC; ++i) {
        dft_slice<RC, false>(v + RC * i);
        const float2* row = tw + S::TWC + RC * (yc + i * S::YC);
#pragma unroll
        for (int k = 1; k < RC; ++k) v[RC * i + k] = twiddle<false>(v[RC * i + k], row, k);
#pragma unroll
        for (int k = 0; k < RC; ++k) lds[rect_e2<S>(RD * k + yc + i * S::YC, kx)] = v[RC * i + k];
    }
    __syncthreads();
    // D
#pragma unroll
    for (int y = 0; y < RD; ++y)
#pragma unroll
        for (int q = 0; q < S::TD; ++q) v[RD * q + y] = lds[rect_e2<S>(RD * dp.k1(q) + y, dp.kx(q))];
#pragma unroll
    for (int q = 0; q < S::TD; ++q) dft_slice<RD, false>(v + RD * q);
}

template <typename S, typename D>
__device__ __forceinline__ void rect_inverse(float2 (&v)[S::V], float2* lds, const float2* __restrict__ tw,
                                             unsigned tid, const D& dp) {
    constexpr int RA = S::RA, RB = S::RB, RC = S::RC, RD = S::RD, H = S::H;
    // D
#pragma unroll
    for (int q = 0; q < S::TD; ++q) {
        dft_slice<RD, true>(v + RD * q);
        const float2* row = tw + S::TWD + (RD + 1) * dp.k1(q);
#pragma unroll
        for (int y = 1; y < RD; ++y) v[RD * q + y] = twiddle<true>(v[RD * q + y], row, y);
    }
#pragma unroll
    for (int y = 0; y < RD; ++y)
#pragma unroll
        for (int q = 0; q < S::TD; ++q) lds[rect_e2<S>(RD * dp.k1(q) + y, dp.kx(q))] = v[RD * q + y];
    __syncthreads();
    // C
    const unsigned kx = tid % S::W, yc = tid / S::W;
#pragma unroll
    for (int i = 0; i < S::TC; ++i)
#pragma unroll
        for (int k = 0; k < RC; ++k) v[RC * i + k] = lds[rect_e2<S>(RD * k + yc + i * S::YC, kx)];
#pragma unroll
    for (int i = 0; i < S::TC; ++i) {
        dft_slice<RC, true>(v + RC * i);
#pragma unroll
        for (int m = 0; m < RC; ++m) lds[rect_e2<S>(yc + i * S::YC + RD * m, kx)] = v[RC * i + m];
    }
    __syncthreads();
    // B
#pragma unroll
    for (int i = 0; i < S::TB; ++i) {
        const unsigned t = tid + i * S::NT, y = t % H, k1 = t / H;
#pragma unroll
        for (int k = 0; k < RB; ++k) v[RB * i + k] = lds[rect_e2<S>(y, k1 + RA * k)];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < S::TB; ++i) {
        const unsigned t = tid + i * S::NT, y = t % H, k1 = t / H;
        dft_slice<RB, true>(v + RB * i);
        const float2* row = tw + S::TWB + RB * k1;
#pragma unroll
        for (int x = 1; x < RB; ++x) v[RB * i + x] = twiddle<true>(v[RB * i + x], row, x);
#pragma unroll
        for (int x = 0; x < RB; x += 2) st2(lds, rect_e1<S>(y, k1 * RB + x), v[RB * i + x], v[RB * i + x + 1]);
    }
    __syncthreads();
    // A
    load_e1_a<S>(lds, v, tid / (RB / S::TA), tid % (RB / S::TA));
#pragma unroll
    for (int q = 0; q < S::TA; ++q) dft_slice<RA, true>(v + RA * q);
}

// A Fourier step on layout D that combines every mode with its mirror:
//   mirror_put, barrier, mirror_step, barrier, mirror_get
// with `sz` 8 RD elements of LDS.  f.pair(k2, ky, kx, za, zb, sa, sb) takes
// Z(k) and Z(-k) of task a's mode k = (ky, kx), ky = k1a + RC k2, and gives both
// new values.  The modes of the tasks that mirror themselves go through sz to
// 4 RD threads, one mode each (left to the two threads that hold them, they
// would be 2 RD modes one after the other while every other wave waits at the
// barrier: 2 us of a 128^2 mass-mapping sweep); f.single(ky, kx, z, zm) gives the
// new value of one of them.
template <typename S>
__device__ __forceinline__ void mirror_put(const float2 (&v)[S::V], const DPair& dp, float2* sz) {
    if (dp.self) {
        float2* o = sz + (dp.zero ? 0 : 2 * S::RD);  // tasks (0, 0), (W/2, 0), (0, RC/2), (W/2, RC/2)
#pragma unroll
        for (int e = 0; e < S::V; ++e) o[e] = v[e];
    }
}
template <typename S>
__device__ __forceinline__ void mirror_get(float2 (&v)[S::V], const DPair& dp, const float2* sz) {
    if (dp.self) {
        const float2* o = sz + 4 * S::RD + (dp.zero ? 0 : 2 * S::RD);
#pragma unroll
        for (int e = 0; e < S::V; ++e) v[e] = o[e];
    }
}
template <typename S, typename F>
__device__ __forceinline__ void mirror_step(float2 (&v)[S::V], const DPair& dp, unsigned tid, float2* sz, F&& f) {
    constexpr int RC = S::RC, RD = S::RD;
    static_assert(S::NT >= 4 * RD, "one thread per self-mirrored mode");
    float2 om[RD];
#pragma unroll
    for (int k2 = 0; k2 < RD; ++k2) {
        __builtin_amdgcn_sched_barrier(0);
        const float2 zb = pick(dp.zero, v[RD + (RD - k2) % RD], v[2 * RD - 1 - k2]);
        float2 sa;
        f.pair(k2, dp.k1a + RC * k2, dp.kxa, v[k2], zb, sa, om[k2]);
        v[k2] = sa;
    }
#pragma unroll
    for (int k2 = 0; k2 < RD; ++k2) v[RD + k2] = pick(dp.zero, om[(RD - k2) % RD], om[RD - 1 - k2]);
    if (tid < 4 * RD) {
        __builtin_amdgcn_sched_barrier(0);
        const unsigned k2 = tid % RD, task = tid / RD;
        const unsigned m = task < 2 ? (RD - k2) % RD : RD - 1 - k2;
        sz[4 * RD + tid] = f.single((task < 2 ? 0 : RC / 2) + RC * k2, task % 2 ? S::W / 2 : 0, sz[tid],
                                    sz[tid - k2 + m]);
    }
}

// Square fields with 16 values per thread.
template <int N> struct SquareShape;
template <> struct SquareShape<32> { using type = Rect<32, 32, 16, 8, 4, 4, 8>; };
template <> struct SquareShape<64> { using type = Rect<64, 64, 16, 8, 8, 8, 8>; };
template <> struct SquareShape<128> { using type = Rect<128, 128, 16, 8, 16, 16, 8>; };

}  // namespace

}  // namespace mf

// Streamed deterministic solve (Wiener filter and adjoint) of real fields with
// power-of-two sides from 256: host launchers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mf_kernels.hpp"

namespace mf {

// One sweep is a row kernel and a column kernel over an H x W/2 complex field,
// z(y, x) = t(y, 2x) + i t(y, 2x+1); an item's field is the float2 elements from
// its pix_off / 2 (half of its pixels).
//
struct RealArgs {
    const ItemDev* items;     // one per problem
    int32_t n_items;
    int32_t log_h, log_w;     // sides 2^log_h x 2^log_w
    int32_t src_kind;
    float2* field;            // fields between the kernels
    const float* src;         // concatenated data d or adjoint rhs g
    const float* nbar;        // concatenated Nbar (+inf missing)
    const float2* nPt;        // column-pair table of n P(|k|): [pix_off/2 + (kx/2) H + ky] = (kx, kx + 1)
    const float2* th;         // W_W^r, r < W, to the nearest (the fold's angles)
    const float2* tw_w;       // W_W^r and W_H^r of modulus 1 (the transforms' twiddles)
    const float2* tw_h;
    const float* s_init;      // kRowFwd: concatenated start, or null for zero
    float* s_out;             // kRowInv: concatenated result
    float2* t_save;           // messenger snapshot (field layout), or null
    double* partials;         // |t - t_save|^2 per row, [y][item]
    float lambda;             // cooling level: T = lambda * tau
    int32_t save_t, check_t;  // write the snapshot; sum the squared distance from it
};

bool real_solve_supported(int H, int W);
// kRowFwd: start from s_init; kRowInvFwd: a middle sweep; kRowInv: write s_out.
hipError_t launch_real_row(int row_mode, const RealArgs& a, hipStream_t s);
hipError_t launch_real_col(const RealArgs& a, hipStream_t s);

}  // namespace mf

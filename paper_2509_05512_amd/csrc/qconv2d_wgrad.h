// Shared by the weight-gradient kernels.
#pragma once

#include "quan_launch.h"

namespace quan {

// Bit 4*p + q is set when entry (p, q) of the Hamilton matrix (eq. 6) is
// negative.  Row r: + - - -, row i: + + - +, row j: + + + -, row k: + - + +.
constexpr unsigned kWgradNeg = (1u << 1) | (1u << 2) | (1u << 3) | (1u << 6) | (1u << 11) | (1u << 13);
// Bit 4*p + q is set when the separable form (eq. 7) subtracts W_q (*) x_q
// from output component p: S[p][q] = -1.  Row r: + - - -, row i: + + + -,
// row j: + - + +, row k: + + - +.
constexpr unsigned kWgradSepNeg = (1u << 1) | (1u << 2) | (1u << 3) | (1u << 7) | (1u << 9) | (1u << 14);

// The row kernel (several taps of a kernel row per work-group): whether it
// takes the layer, and how it splits it.  It writes splits * segs slices of
// partial sums, [slice][taps][4][c_out][c_in] in fp64 with `fold`, else the
// product of all component pairs [slice][taps][4 c_out][4 c_in] in fp32.
struct WgradRows {
    bool takes, fold;
    int wo, wc, kw;  // blocks of 32 per tile, taps of a work-group
    int segs, u4;    // column segments of u4 pixels
    int rh, ksteps;  // rows and MFMA K steps of a chunk
    int x_pos, step; // window positions of a row, from one pixel to the next
    int chunks, per_split, splits;
    int most_splits;  // of this layer with this many images or fewer
    int kx_groups, o_tiles, c_tiles;
};
WgradRows qconv2d_wgrad_rows_plan(const ConvGeom &g, DType dt);
hipError_t qconv2d_wgrad_rows_run(const WgradRows &p, const ConvGeom &g, DType dt, const void *x, const void *dy,
                                  float *part, hipStream_t stream, bool sep);

}  // namespace quan

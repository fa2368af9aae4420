// The search through row spectra as the other entry points use it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "reduce.h"
#include "register_plan.h"

namespace rd {

// Workspace for the spectra and partials of the frames of one round: what a call that asks
// for the spectral search takes, and the smaller one of a plain search that takes it by
// itself (a search of 1024x1024 frames still holds fifty of them per round).
constexpr size_t SPEC_ROUND_BYTES = size_t(2) << 30;
constexpr size_t SPEC_ROUND_BYTES_PLAIN = size_t(512) << 20;

// Whether a full-window search (radius_max = radius, interior template, no centres, no score
// planes asked for) of N frames goes through row spectra.
bool spectra_pay(int32_t W, int32_t H, int32_t N, int32_t R);

// Sizes, launch plans and workspace offsets of one search.  The plans come from the tuner's
// table, which another thread may change at any time, so a call makes its layout once, checks
// its workspace against it and searches with it.
struct FftLayout {
    int32_t P, N2, log2n2, PS, D, Dg, n_grp, M, n_blk, bpb, n_band, n_kt, F;
    RegPlan refine, full;
    int32_t Ffull;
    size_t tw, mean_parts, mean, Bt, rowsq_b, A, rowsq_a, Zp, S_fft, cen, info, fb;
    size_t part_r, part_f, sc_f, total;
};

// The layout of a search of N frames (false: not for these sizes).
bool fft_layout(int32_t W, int32_t H, int32_t N, int32_t R, size_t round_bytes, FftLayout *L);

// N frames k + (k >= skip), k < N, of `frames` against ref; out and info are indexed by frame,
// scores by k.  L as fft_layout made it for these sizes, ws of L.total bytes.
int spectral_search(const FftLayout &L, const float *ref, const float *frames, int32_t W, int32_t H, int32_t N,
                    int32_t R, int32_t skip, reduce_offset_t *out, double *scores, int32_t *info, void *ws,
                    hipStream_t s);

}  // namespace rd

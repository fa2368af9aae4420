// The search through row spectra as the other entry points use it.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <hip/hip_runtime.h>

#include "reduce.h"

namespace rd {

// Workspace for the spectra and partials of the frames of one round: what a call that asks
// for the spectral search takes, and the smaller one of a plain search that takes it by
// itself (a search of 1024x1024 frames still holds fifty of them per round).
constexpr size_t SPEC_ROUND_BYTES = size_t(2) << 30;
constexpr size_t SPEC_ROUND_BYTES_PLAIN = size_t(512) << 20;

// Whether a full-window search (radius_max = radius, interior template, no centres, no score
// planes asked for) of N frames goes through row spectra.
bool spectra_pay(int32_t W, int32_t H, int32_t N, int32_t R);

// Workspace bytes of spectral_search (0: not for these sizes).
size_t spectral_ws(int32_t W, int32_t H, int32_t N, int32_t R, size_t round_bytes);

// N frames k + (k >= skip), k < N, of `frames` against ref; out and info are indexed by frame,
// scores by k.  Sizes as spectral_ws accepts them, ws of that many bytes.
int spectral_search(const float *ref, const float *frames, int32_t W, int32_t H, int32_t N, int32_t R, int32_t skip,
                    reduce_offset_t *out, double *scores, int32_t *info, void *ws, size_t round_bytes, hipStream_t s);

}  // namespace rd

// Convolution part of FULL far sets (FftGrid in plan.hpp): launchers.
#pragma once

#include <hip/hip_runtime_api.h>

#include "kernels.hpp"
#include "plan.hpp"

namespace ubf {

// Fill the spectra of the plan's lattices (p.d_fft_spec), with the scratch
// p.d_fft. Runs when the plan is bound.
int launch_fft_spectra(const Plan& p, hipStream_t s);

// The convolution of every lattice and right-hand side: box vectors P (in
// the plan's form) to each box's first partial row. `start` and `stop`
// (events or NULL) mark the first kernel's start and the last one's end.
int launch_fft(const Plan& p, const float* P, float* part, int nrhs, hipStream_t s,
               hipEvent_t start, hipEvent_t stop);

}  // namespace ubf

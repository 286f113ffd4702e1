// Kernel arguments and launch helpers of the harmonic analysis (sht_kernel.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pisco {

constexpr int SHT_MAX_NSIDE = 1024;        // ring FFT buffers (2 x 4N complex) fit one CU's LDS

constexpr int SHT_STEP_BYTES = 48;

struct ShtArgs {
    int nside, lmax, mmax, nfields;        // nfields: 1 (T) or 3 (T, Q, U)
    const double *map[3];                  // RING order, 12 nside^2 each
    double2 *F;                            // [nfields signals][mmax + 1][2 nside ring pairs][P, M]: ring Fourier sums
    double *alm[3];                        // complex interleaved, m-major: T, E, B
    int add;                               // analysis: add to alm instead of replacing it
    int wx_m, wx_parts;                    // analysis: m < wx_m in wx_parts workgroups each (filled in by launch_alm)
    void *steps;                           // recurrence steps, SHT_STEP_BYTES per a_lm (launch_steps)
    double *partial;                       // analysis: [part][alm size][6] sums of the first m
    const double *alm_in[3];               // synthesis input (complex interleaved)
    double *map_out[3];                    // synthesis output (RING order)
    int residual;                          // synthesis: map less the synthesised map
};

struct ClArgs {
    int lmax;
    bool teb;                              // x = a^T, a^E, a^B: spectra TT, EE, BB, TE, EB, TB; else of x[0] and y[0]
    const double *x[3], *y[1];             // complex interleaved
    double *cl;                            // [6 or 1][lmax + 1]
};

hipError_t launch_steps(const ShtArgs &a, hipStream_t s);            // before any launch_alm or launch_alm2map of its lmax
hipError_t launch_ring_fourier(const ShtArgs &a, hipStream_t s);
hipError_t launch_alm(const ShtArgs &a, hipStream_t s);
hipError_t launch_alm2map(const ShtArgs &a, hipStream_t s);          // alm_in -> F (as G) -> map_out
hipError_t launch_alm2cl(const ClArgs &a, hipStream_t s);

}  // namespace pisco

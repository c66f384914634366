// me_launch.h -- host-side process table shared by the C ABI and the kernels.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "me_host.h"
#include "me_process.h"

#define ME_BLOCK 64

// lg: 2^lg lanes per event, each summing every 2^lg-th helicity (0 <= lg <= 6).
typedef hipError_t (*me_launch_fn)(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                   const me_params& prm, double* qhel, int lg, hipStream_t stream);

// Indexed variant: evaluate events idx[0..*count) only (count on the device);
// where there is no launch_sum.
typedef hipError_t (*me_launch_idx_fn)(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                       const me_params& prm, const int* idx, const int* count,
                                       hipStream_t stream);

// Mixed-precision form: float32 amplitudes, float16 hi/lo MFMA colour sum,
// per-event error estimate; flagged events appended to flag_idx.  part: room for
// two floats per helicity and event, for blocks with a few helicities each, or null.
typedef hipError_t (*me_launch_mixed_fn)(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                         const me_params& prm, float tol, float cest, int* flag_count,
                                         int* flag_idx, float* err_out, unsigned char* flag_out,
                                         float2* part, hipStream_t stream);

// Multi-channel form: |M|^2 and the single-diagram weight of each event's channel.
typedef hipError_t (*me_launch_mc_fn)(const double* mom, int64_t nevt, double* out, const int* hels, int nh,
                                      const me_params& prm, const int* chan, double* alpha, hipStream_t stream);

// Blocks of a grid whose blocks stride over the events, one event per block at a time.
#define ME_WAVE_BLOCKS 8192

// Blocks of the kernel with one event per workgroup and CU.
#define ME_GROUP_BLOCKS 1024

// Events that such a block sets up together: two, which fills the lanes of
// the setup phases, once there are enough events to keep every CU's eight waves
// busy that way; below that one, since a call then takes as long as one block.
static inline int me_wave_events(int64_t nevt) { return nevt > 4096 ? 2 : 1; }

// Spin sum with one event per wave: |M|^2 only, no single helicities.  spins:
// bit s3 + 2 s4 for each spin pair of t and tbar to sum; idx, count as in the
// indexed variant or null; mfma: colour sum on the matrix cores.
typedef hipError_t (*me_launch_sum_fn)(const double* mom, int64_t nevt, double* out, unsigned spins,
                                       const me_params& prm, const int* idx, const int* count, bool mfma,
                                       hipStream_t stream);

// Multi-channel form with shared wavefunctions: sums over all helicities.
typedef hipError_t (*me_launch_chan_fn)(const double* mom, int64_t nevt, double* out, const me_params& prm,
                                        const int* chan, double* alpha, hipStream_t stream);

enum { ME_KIND_EE = 0, ME_KIND_GG = 1, ME_KIND_QEW = 2 };

struct me_process_desc {
    const char* name;
    int kind;
    int npart, ndiag, ncol, nhel;
    double flops_amp, flops_colour;  // per helicity, algorithmic
    double flops_executed;           // per helicity, as the kernel executes it (recomputation included)
    me_launch_fn launch_f64;
    me_launch_idx_fn launch_f64_idx;
    me_launch_mixed_fn launch_mixed;  // nullptr: the process has no mixed form
    double mixed_cest;                // calibration of the amplitude error estimate
    me_launch_fn launch_f64_cm;       // float64 with the colour sum on the matrix cores (nullptr: none)
    me_launch_mc_fn launch_mc;        // multi-channel form (nullptr: none)
    int nchan;                        // its channels
    const char* const* chan_desc;     // their descriptors
    me_launch_sum_fn launch_sum;      // spin sum with one event per wave (nullptr: none)
    me_launch_chan_fn launch_chan;    // multi-channel form with shared wavefunctions (nullptr: none)
    bool mixed_part;                  // launch_mixed makes use of `part`
    int hel_turn;                     // lanes of launch_f64 that the chip runs at full rate: a wave per SIMD, or a
                                      // workgroup per CU (0: single helicities take one lane per event)
};

const me_process_desc* me_find_process(const char* name);

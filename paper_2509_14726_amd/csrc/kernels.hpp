// Launch entry points of the device code (internal to the library).
#pragma once

#include <hip/hip_runtime.h>

#include "device.hpp"

namespace mppi {

// Convert the problem tables of a context to the device layout.
hipError_t launch_setup(const KArgs &a, bool fp64, hipStream_t st);

// Write a request record, passed as a kernel argument, to device memory.
hipError_t launch_request(const double *values, double *d_req, hipStream_t st);

// Enqueue one MPPI step: sample (with the head), rollout, average (+ tail).
// acc64 selects binary64 accumulation of the weighted average.
// When ev is non-null, ev[0..3] are recorded before the sample, rollout and
// average kernels and after the average kernel.  *ran becomes the MPPI_RAN_*
// bits of the rollout that was launched.
hipError_t launch_solve(const KArgs &a, bool fp64, bool acc64, hipStream_t st, hipEvent_t *ev, int32_t *ran);

// Device address of the fixed solve workspace (kScratchBytes, 256-byte
// aligned) on the current device.  The first call on a device resolves it
// (with that device current) and later calls return the cached address.
hipError_t scratch_address(void **ptr);

// Waves per SIMD of the batched one-wave rollouts that draw (binary32): few,
// where the pipeline's arithmetic or the rate input needs the registers.
constexpr int draw_waves(bool few) { return few ? 2 : 3; }

// Launch shape of one batch group.
struct BatchLaunch {
    int objective;
    bool fp64, acc64;
    int rollout_waves;    // 1..4 (see mppi_batch_cfg)
    int ring_steps;       // rings of the pipeline (binary32): 8 steps, one workgroup per CU; 4, two
    bool draw;            // one-wave rollouts that draw their samples (binary32); with rollout_waves 4
                          // in the pipeline's arithmetic
    bool rate, thrust;    // the group has contexts of the rate input, of the thrust input
    int rollout_groups;   // persistent rollout workgroups
    int draw_groups;      // the same for the drawing one-wave rollouts
    int sample_groups;    // grid-stride workgroups of the sample kernel
    int final_groups;     // grid-stride workgroups of the weighted-average kernel
    bool regen;           // it draws the samples again
    bool single;          // its units are single horizon steps, else final_steps() of them
    int ctrl_groups;      // grid-stride workgroups of the control-cost kernel (0: no item has the term)
};

// Enqueue one batched MPPI step over the items described in device memory;
// the MPPI_RAN_* bits of its rollout are added to *ran.
hipError_t launch_batch(const BArgs &b, const BatchLaunch &L, hipStream_t st, int32_t *ran);

}  // namespace mppi

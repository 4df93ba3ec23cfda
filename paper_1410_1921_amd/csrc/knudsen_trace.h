// The traced Knudsen solve, an internal entry point of liblbm.so for the tests.
#pragma once

#include "lbm_internal.h"

namespace lbm {

// What a Knudsen solve's resident sweeps did, and how the tests make one give up:
// lbm_knudsen_solve_traced is lbm_knudsen_solve with this as one more argument.
struct KnTrace {
    // longest wait for a packet, in ticks of the 100 MHz clock
    int64_t wait_ticks = 50000;
    int32_t give_up_at = 0;      // in this launch (1, 2, ..) one workgroup sends no packets,
    int32_t refuse_at = 0;       // this one counts as refused by the runtime
    int64_t resident_steps = 0;  // steps taken by resident sweeps
    int32_t launches = 0;        // their launches,
    int32_t gave_up = 0;         // those that gave up a wait (plain sweeps then took their steps),
    int32_t refused = 0;         // and those the runtime refused
    int32_t lists = 0;           // times their send lists were formed
    int32_t min_steps = 0;       // > 0: the fewest steps of a launch, instead of the rule's
    int32_t pad = 0;
};

}  // namespace lbm

extern "C" lbm_status lbm_knudsen_solve_traced(const int32_t n[3], const uint8_t *fluid,
                                               const double *pore_diam, const lbm_knudsen_params *p,
                                               lbm_knudsen_result *r, float *c_field,
                                               const float *c_init, double *plane_flux_h,
                                               void *workspace, size_t ws_bytes, void *stream,
                                               lbm::KnTrace *trace_h);

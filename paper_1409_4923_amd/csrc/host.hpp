// host.hpp -- host-side helpers shared by the ensemble and scan entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <vector>

#include "bmotor.h"
#include "common.hpp"

namespace bm {
namespace host {

int fail(int code, const char *fmt, ...);           // set the thread's message, return code
int ok();                                           // clear the message, return BM_OK
int hip_fail(hipError_t e, const char *what);       // BM_ERR_DEVICE with HIP's message
const char *last_error_text();

int validate(const bm_model *m, const bm_run *r);   // argument checks of one (model, run)
double step_of(const bm_model *m, const bm_run *r); // dt
size_t table_entries(const bm_run *r);              // forcing table length (period + 16)
void forcing_table(const bm_model *m, const bm_run *r, std::vector<double> &tab);
PointConst point_const(const bm_model *m, const bm_run *r, const void *d_tab);
int check_device(int *dev_out);                     // a gfx950 device is current

// Launch shapes for calls without a bm_tune: the one installed for the model (by
// bm_tune_set_default, bm_scan_autotune or bm_tune_load), else a built-in one.
// ensemble_tune is what ensembles run; default_tune is what bm_tune_get_default and
// bm_tune_lookup report, which for FP32 inertial models without jumps is the shape that
// ensembles used to run (programs may rely on the answer).
bm_tune default_tune(uint32_t dyn, uint32_t pot, uint32_t noise, uint32_t prec);
bm_tune ensemble_tune(uint32_t dyn, uint32_t pot, uint32_t noise, uint32_t prec);
size_t queue_lds_bytes(uint32_t noise, uint32_t prec, uint32_t ppl, uint32_t block);
int check_tune(const bm_tune *t, uint32_t noise, uint32_t prec);

} // namespace host
} // namespace bm

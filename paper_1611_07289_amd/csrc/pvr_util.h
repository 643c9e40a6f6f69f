// Host-side error handling and allocation helpers of the PVR library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>

#include <exception>

#include "pvr_internal.h"

namespace pvr {

pvr_status fail(pvr_status st, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();
void plan_free(pvr_plan *p);
pvr_status plan_build_index(pvr_plan *p, hipStream_t stream);
pvr_status launch_bp_prep(const pvr_plan *p, const float *e, const float *pp, hipStream_t stream);
// The registration with all patches in step (pvr_register.hip), for at most
// REG_STEP_MAX trial steps and, with the exact gradient, at least
// REG_STEP_MIN_EXACT forward chunks.  A step that patches take is 2 to 10 times
// faster in step; one after every patch has ended still costs its launches, where one
// workgroup per patch has stopped.  Central differences, 216 patches of 16 x 16 / 64
// of 64 x 64: 200 steps 9.6 / 13.7 ms in step, 15.3 / 133 ms per patch; 40 steps that
// no patch takes 0.50 ms against 0.07 (12 us a step), with 1 152 patches of 64 x 64 1.1
// against 0.3, with 8 064 6.1 against 1.3 (130 us a step).  At REG_STEP_MAX such steps
// lose at most 3 to 31 ms, far less than steps that are taken gain.
constexpr int REG_STEP_MAX = 256, REG_STEP_MIN_EXACT = 1024;
pvr_status register_in_step(const pvr_plan *p, const float *X, const float *XT, const float *y,
                            float *theta, float *ncc, const uint8_t *reg, const pvr_reg_params &prm,
                            hipStream_t stream);
size_t reg_state_bytes(const pvr_plan *p, size_t off[5]);
void launch_fill_i32(int *dst, int v, long long n, hipStream_t stream);
void launch_fill_f32(float *dst, float v, long long n, hipStream_t stream);
void launch_fill_f64(double *dst, double v, long long n, hipStream_t stream);
// The id of the capture that `stream` records into a graph, 0 outside one: what
// a captured call leaves behind exists for the calls of the same capture only.
unsigned long long capture_id(hipStream_t stream);
// The event pair to record around the next launch of kernel k, or nullptr
// when the plan is not timing (or the kernel's slots are full).
hipEvent_t *timing_slot(const pvr_plan *p, int k);

struct PlanGuard {
  pvr_plan *p;
  explicit PlanGuard(pvr_plan *q) : p(q) {}
  ~PlanGuard() { if (p) plan_free(p); }
  void release() { p = nullptr; }
};

}  // namespace pvr

#define PVR_API_BEGIN() \
  pvr::clear_error();   \
  try {
#define PVR_API_END()                                                          \
  }                                                                            \
  catch (const std::exception &e) {                                            \
    return pvr::fail(PVR_EINVAL, "internal error: %s", e.what());              \
  }                                                                            \
  catch (...) {                                                                \
    return pvr::fail(PVR_EINVAL, "internal error");                            \
  }

// Return a non-OK status of a library call from the enclosing entry point.
#define PVR_TRY_STATUS(expr)                                                   \
  do {                                                                         \
    const pvr_status st_try_ = (expr);                                         \
    if (st_try_ != PVR_OK) return st_try_;                                     \
  } while (0)

#define HIP_TRY(expr)                                                          \
  do {                                                                         \
    hipError_t e_ = (expr);                                                    \
    if (e_ != hipSuccess)                                                      \
      return pvr::fail(PVR_EHIP, "%s failed: %s (%s:%d)", #expr,               \
                       hipGetErrorString(e_), __FILE__, __LINE__);             \
  } while (0)

// Device arrays must be aligned to the width the kernels read them with; a
// NULL pointer passes (whether it may be NULL is checked separately).
#define PVR_ALIGNED(fn, ptr, a)                                                \
  do {                                                                         \
    if ((reinterpret_cast<uintptr_t>(ptr) & ((uintptr_t)(a) - 1)) != 0)        \
      return pvr::fail(PVR_EINVAL, "%s: %s is not %d-byte aligned", fn, #ptr,  \
                       (int)(a));                                              \
  } while (0)

// Places `count` elements of T at the next 256-byte boundary of a workspace
// and advances the cursor.  With a NULL base it only measures: the same
// sequence of calls sizes a workspace and then carves it.
struct WsCursor {
  char *base;
  size_t off;
};
template <typename T>
inline T *ws_take(WsCursor &c, long long count) {
  c.off = (c.off + 255) & ~(size_t)255;
  T *r = c.base ? reinterpret_cast<T *>(c.base + c.off) : nullptr;
  c.off += (size_t)(count > 0 ? count : 1) * sizeof(T);
  return r;
}

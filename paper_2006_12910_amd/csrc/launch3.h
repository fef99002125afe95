// launch3.h -- host-side entry points into the 3D sweeps (internal to the
// library).
#pragma once

#include "sweep3_impl.h"

namespace lbk3 {

// one step: `blocks` workgroups, step kstep after the device's counter;
// wide: 64-bit byte offsets
void sweep3_f64(const Dom3 &h, const Dom3 *dd, int q, bool wide, unsigned blocks, int kstep, hipStream_t s);
void sweep3_f32(const Dom3 &h, const Dom3 *dd, int q, bool wide, unsigned blocks, int kstep, hipStream_t s);
void sweep3_f16(const Dom3 &h, const Dom3 *dd, int q, bool wide, unsigned blocks, int kstep, hipStream_t s);
void sweep3_bf16(const Dom3 &h, const Dom3 *dd, int q, bool wide, unsigned blocks, int kstep, hipStream_t s);

// two steps per launch, FP32 and FP64 without noise: segments of `planes` planes
// (split3)
void launch_sweep3x2(const Dom3 &h, int q, int planes, int kstep, int which, hipStream_t s);

}  // namespace lbk3

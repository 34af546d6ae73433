// fp32 prefill kernel (internal to the library).
#pragma once
#include "attn_common.h"
#include "device_map.h"

namespace bs {

// Workgroups that fit a CU side by side (LDS).
inline int32_t f32_wgs_per_cu(int32_t head_dim) { return head_dim == 64 ? 2 : 1; }
// Bytes of partial results of these shares.
size_t f32_workspace(const ShareSet &shares, int32_t head_dim);
void launch_f32(const KernelArgs &a, const DeviceMap *d, const ShareSet &shares, void *workspace, int32_t head_dim, hipStream_t st);
// Raises the kernels' dynamic-LDS limits on the current device.
hipError_t f32_device_setup();

}  // namespace bs

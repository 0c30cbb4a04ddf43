// Kernels that take more dynamic LDS than a launch gets unasked.
#pragma once
#include <hip/hip_runtime.h>

namespace f3d {

// The most dynamic LDS a launch may ask for is a property of the kernel, not of the call. Set to what a call itself needs, it could be
// lowered by a smaller call of another thread between this one's setting and its launch. So `most` is what the kernel can ever
// need, the same in every call.
inline hipError_t allow_lds(const void* kernel, size_t most)
{
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
}

}  // namespace f3d

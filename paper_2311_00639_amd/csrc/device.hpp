// Device helpers shared by the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace syk {

// A factor known in 64 bits, applied to a T with one rounding of the product: for float its high and
// low parts, as a factor rounded to 32 bits would multiply a whole vector by 1 + 2^-24 at worst.
template <typename T>
struct Scale {
    T hi = 0, lo = 0;
    Scale() = default;
    __device__ __forceinline__ explicit Scale(double s) : hi(static_cast<T>(s)), lo(static_cast<T>(s - hi)) {}
    __device__ __forceinline__ T operator()(T v) const {
        if constexpr (sizeof(T) == 8)
            return hi * v;
        else
            return fmaf(hi, v, lo * v);
    }
};

}  // namespace syk

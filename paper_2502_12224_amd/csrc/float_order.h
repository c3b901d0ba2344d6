// Integer keys in the order of floats.  No device code: the CPU tests compile this header by itself.
#pragma once

namespace fate {

#ifdef __HIPCC__
#define FATE_ORDER_FN __host__ __device__ inline
#else
#define FATE_ORDER_FN inline
#endif

// An integer in the order of the float (both zeros alike), above the least one.
FATE_ORDER_FN int float_order(float v) {
    const int b = __builtin_bit_cast(int, v + 0.0f);
    return b ^ ((b >> 31) & 0x7fffffff);
}

}  // namespace fate

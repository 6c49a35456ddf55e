// Loop over registers that is unrolled whatever its body.
#ifndef CL_STATIC_FOR_H
#define CL_STATIC_FOR_H

#include <hip/hip_runtime.h>
#include <type_traits>

namespace cl {

// f(integral_constant<int, 0>) .. f(integral_constant<int, E - 1>)
template <int E, int B = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<E, B + 1>(f);
    }
}

}  // namespace cl

#endif  // CL_STATIC_FOR_H

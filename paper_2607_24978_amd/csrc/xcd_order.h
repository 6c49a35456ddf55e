// Order of workgroups over the eight XCDs.
#ifndef CL_XCD_ORDER_H
#define CL_XCD_ORDER_H

#include <hip/hip_runtime.h>

namespace cl {

// XCD-aware order: consecutive workgroup ids land on different XCDs (round
// robin over 8), so give XCD k a contiguous range of tiles; its co-resident
// workgroups then share halos in their L2.
__device__ __forceinline__ int xcd_order(int bid, int nblocks) {
    const int per = nblocks / 8, rem = nblocks % 8;
    const int xcd = bid % 8, slot = bid / 8;
    if (per == 0) return bid;
    return (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + slot;
}

}  // namespace cl

#endif  // CL_XCD_ORDER_H

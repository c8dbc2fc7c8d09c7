// The bound that keeps every write of the outlier selection inside idx[0 .. f), in a file without HIP so that the host
// can check it too.
#pragma once
#include <stdint.h>

// True for the ranks that have a slot in idx.  The rank shares its scratch word with a column sum; where calls overlap on one
// scratch array (which aser_smooth_outliers_noalloc documents as a race) any bit pattern may be found there, so a
// negative rank has no slot either.
static inline
#ifdef __HIPCC__
    __host__ __device__
#endif
    bool rank_has_slot(int32_t rank, int32_t f) {
    return (uint32_t)rank < (uint32_t)f;
}

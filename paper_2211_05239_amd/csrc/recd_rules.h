// Sizes and bounds that host code and kernels share.  Plain C++, so that they can be built and checked
// without a GPU.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define RECD_RULE __host__ __device__ inline
#else
#define RECD_RULE inline
#endif

// Unique lists that the backward's workspace has room for (rows of g_u).  U_cap bounds their number; a
// plain IKJT has at most one empty list per feature and so at most M + F, but a grouped one stores an empty
// list for every slot of the group, so U_cap cannot be replaced by M_cap + F.
RECD_RULE int64_t recd_lists_held(int64_t F, int64_t B, int64_t U_cap, int64_t M_cap)
{
    const int64_t most = U_cap > M_cap + F ? U_cap : M_cap + F;
    return most < F * B ? most : F * B;
}

// What the two search files share: the search of few queries (xc_mine_few.hip), called by xc_mine.hip.
#pragma once

#include "xc_common.h"

namespace xc {

struct FewPlan {
    int ks;                  // 64-byte steps of a row
    int nb;                  // blocks of 16 queries per workgroup
    int n_qb;                // groups of nb blocks
    int gshift;              // labels of a group: 16 << gshift
    int64_t n_groups;
    int n_split;             // workgroups per query in the second kernel
    size_t lds;              // bytes of the query block in LDS
};

// Whether the search of few queries takes this shape, and how.  `scratch`: bytes for the group maxima
// and the candidates of shared queries.
bool plan_few(int64_t Zq, int64_t L, int64_t row_bytes, int k, xc_dtype t, size_t scratch, FewPlan* p);

int run_mine_few(const FewPlan& p, const void* Z, const void* W, int64_t Zq, int64_t L, int64_t row_bytes, int k,
                 xc_dtype t, unsigned char* scratch, uint32_t* tau_g, int32_t* flag /* null: leave alone */, int n_flag,
                 int32_t* shortlist, float* scores, hipStream_t st);

}  // namespace xc

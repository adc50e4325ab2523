// bed_kernels.hip -- launches of the n <= 64 solver: dispatch by storage type and
// the binary32 instantiations.
#include "bed_kernels.hpp"

namespace bed {

BED_KERNELS_OF(extern, double)

bool team_supported(bed_dtype dt, TeamShape ts)
{
    (void)dt;
    if (!leaf_supported(ts.leaf)) return false;
#define X(NM, NTT) if (ts.nmax == NM && ts.nt == NTT) return true;
    BED_SHAPES(X)
#undef X
    return false;
}

hipError_t launch_tri(TeamShape ts, const float *tri, int n, int64_t batch, float *lam, float *Q,
                      int32_t *info, float *ends, const int32_t *skip, int64_t skip_count,
                      hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    if (!leaf_supported(ts.leaf) || batch > 2 * skip_count) return hipErrorInvalidValue;
#define X(NM, NTT)                                                                          \
    if (ts.nmax == NM && ts.nt == NTT) {                                                    \
        hipLaunchKernelGGL((k_syevd_tri<float, NM, NTT>), dim3((unsigned)batch), dim3(NTT), \
                           0, s, tri, n, batch, lam, Q, info, ends, skip, skip_count,       \
                           ts.leaf);                                                        \
        return hipGetLastError();                                                           \
    }
    X(32, 128)
    X(32, 256)
    X(64, 256)
#undef X
    return hipErrorInvalidValue;
}

hipError_t launch_uniform(bed_dtype dt, TeamShape ts, const void *A, int n, int64_t batch,
                          void *lam, void *Q, int32_t *info, hipStream_t s)
{
    if (batch <= 0) return hipSuccess;
    if (n <= SMALL_MAX && ts.leaf == 0) return launch_small(dt, A, n, batch, lam, Q, info, s);
    return dt == BED_F32 ? uniform_t<float>(ts, A, n, batch, lam, Q, info, s)
                         : uniform_t<double>(ts, A, n, batch, lam, Q, info, s);
}

hipError_t launch_list(bed_dtype dt, TeamShape ts, const void *A, void *lam, void *Q,
                       int32_t *info, const WorkItem *items, int count, int *counter, int grid,
                       hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    return dt == BED_F32 ? list_t<float>(ts, A, lam, Q, info, items, count, counter, grid, s)
                         : list_t<double>(ts, A, lam, Q, info, items, count, counter, grid, s);
}

hipError_t launch_ptrlist(bed_dtype dt, TeamShape ts, const PtrItem *items, int count,
                          hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    return dt == BED_F32 ? ptrlist_t<float>(ts, items, count, s)
                         : ptrlist_t<double>(ts, items, count, s);
}

int blocks_per_cu(bed_dtype dt, TeamShape ts)
{
    return dt == BED_F32 ? bpc_t<float>(ts) : bpc_t<double>(ts);
}

}  // namespace bed

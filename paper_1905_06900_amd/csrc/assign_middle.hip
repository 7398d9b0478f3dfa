// The filters of assign.hip for sub-vectors of 17 to 32 components.
#define DCPQ_ASSIGN_KERNELS_ONLY
#include "assign.hip"

namespace dcpq {

int launch_assign_middle(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                         void *labels, int label_bytes, float *dist, hipStream_t st)
{
    const int ks = (3 * dp + 15) / 16;
    if (ks <= 4) return launch_assign_ks<4>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 5) return launch_assign_ks<5>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return launch_assign_ks<6>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
}

}  // namespace dcpq

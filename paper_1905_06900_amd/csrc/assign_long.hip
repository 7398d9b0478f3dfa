// The filters of assign.hip for sub-vectors of 33 to 128 components.
#define DCPQ_ASSIGN_KERNELS_ONLY
#include "assign.hip"

namespace dcpq {

int launch_assign_long(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                       void *labels, int label_bytes, float *dist, hipStream_t st)
{
    const int ks = (3 * dp + 15) / 16;
    if (ks <= 8) return launch_assign_ks<8>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 10) return launch_assign_ks<10>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 12) return launch_assign_ks<12>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 16) return launch_assign_ks<16>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 20) return launch_assign_ks<20>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return launch_assign_ks<24>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
}

}  // namespace dcpq

// Training of the quantizers and encoding (Sec. 3.2, Alg. 2 build_quantizers; the encoding rule of the
// last paragraph of Sec. 3.2).
//
//   step 1  kmeans                 temporary codebook of 2^b centroids per sub-quantizer
//   step 2  kmeans_same_size       the temporary centroids partitioned into 2^bbar groups of equal size
//   step 3  build_final_codebook   the temporary centroids reordered so that the low bbar bits of a
//                                  centroid's index name its group (property P1)
//   encode                         sub-code j of a vector = index of the centroid of C_j nearest to its
//                                  j-th sub-vector
//
// The paper leaves the insides of steps 1 and 2 to standard algorithms; what is computed here:
//   - nearest centroid: smallest (distance, index), distances in double precision (assign.hip: a filter on the bf16
//     matrix cores with a proven error bound, double precision for what it leaves);
//   - a k-means iteration assigns every point and replaces each centroid by the mean of its members
//     (double-precision sums, one division, rounded to fp32); a centroid without members keeps its value;
//     initial centroids are an input; after the last iteration the points are assigned once more;
//   - same-size k-means: an iteration makes a balanced assignment (groups of exactly n / kbar points) and
//     takes the means; the labels returned are those of the last assignment, whose means the returned
//     centroids are;
//   - balanced assignment, in rounds: every point without a group proposes to the group with the smallest
//     (distance, index) among those with room; every group takes, among its proposers, those with the
//     smallest (distance, point) up to its room; until no point is left.  Distances are fp32 table entries
//     (the distance-table kernel of tables_full.hip).
#include "common.h"
#include "device_util.h"
#include "assign.h"

namespace dcpq {

// sums[label][t] += point[t] (double), counts[label] += 1.  One thread per (point, component).  For m sub-quantizers at once
// (points of m d components, labels [n][m], sums [m][k][d], counts [m][k]); m = 1: points and labels as they are.
__global__ __launch_bounds__(256) void accumulate_kernel(const float *__restrict__ points, uint64_t n, int ld, int d,
                                                         const uint32_t *__restrict__ labels, int m, int k, double *__restrict__ sums,
                                                         uint32_t *__restrict__ counts)
{
    const uint64_t e = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= n * static_cast<uint64_t>(m * d)) return;
    const uint64_t i = e / (m * d);
    const int at = static_cast<int>(e % (m * d)), j = at / d, t = at - j * d;
    const size_t c = static_cast<size_t>(j) * k + labels[i * m + j];
    unsafeAtomicAdd(&sums[c * d + t], static_cast<double>(points[i * ld + at]));
    if (t == 0) atomicAdd(&counts[c], 1u);
}

__global__ __launch_bounds__(256) void means_kernel(const double *__restrict__ sums, const uint32_t *__restrict__ counts,
                                                    size_t n, int d, float *__restrict__ centroids)
{
    const size_t e = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const uint32_t c = counts[e / d];
    if (c) centroids[e] = static_cast<float>(sums[e] / static_cast<double>(c));    // no members: keeps its value
}

__global__ __launch_bounds__(256) void clear_kernel(uint32_t *p, size_t nwords)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < nwords) p[i] = 0u;
}

constexpr uint32_t kAcceptKeys = 4096;        // proposers of a group that are sorted in LDS

// ---- balanced assignment ----------------------------------------------------------------------------
// state: labels[n] (0xFFFFFFFF = no group yet), room[kbar], left[0] = points without a group; count[kbar]: proposers of a round
__global__ __launch_bounds__(256) void balanced_init_kernel(uint32_t *labels, int n, uint32_t *room, uint32_t *count, int kbar, uint32_t *left)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) labels[i] = 0xFFFFFFFFu;
    if (i < kbar) { room[i] = static_cast<uint32_t>(n / kbar); count[i] = 0; }
    if (i == 0) left[0] = static_cast<uint32_t>(n);
}

// The room that an assignment which was left after some rounds leaves the groups, from its labels.  One workgroup.
__global__ __launch_bounds__(1024) void balanced_resume_kernel(const uint32_t *__restrict__ labels, int n, uint32_t *__restrict__ room, uint32_t *__restrict__ count,
                                                               int kbar)
{
    __shared__ uint32_t have[256];
    const int tid = threadIdx.x;
    if (tid < 256) have[tid] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += 1024) {
        const uint32_t l = labels[i];
        if (l < static_cast<uint32_t>(kbar)) atomicAdd(&have[l], 1u);
    }
    __syncthreads();
    if (tid < kbar) { room[tid] = static_cast<uint32_t>(n / kbar) - have[tid]; count[tid] = 0; }
}

// Every point without a group goes into the list of the group with room that is nearest to it (smallest (distance, index)), as a
// key (distance, point).  A wavefront takes 4 points, a row of distances at a time: 256 bytes to a load.  (With a thread per row
// that leaves its proposal in an array, and every group looking through that: 56 us for a round and its acceptances, 65536 points and
// 256 groups; so 33.)  The 64 points of a workgroup take their places in a list with one atomic: with one per point, 13 ns each on a
// group's counter, an iteration over 65536 points and 16 groups took 1.93 ms, and so 0.98; with 256 groups 0.49 and 0.43.
// list: np2 keys per group (np2 = n rounded up to a power of two).
constexpr int kProposePoints = 4, kProposeWaves = 16, kProposeBlock = kProposePoints * kProposeWaves;
static_assert(kProposeBlock == 64, "a proposal per lane of a wavefront");
__global__ __launch_bounds__(64 * kProposeWaves) void propose_kernel(const float *__restrict__ T, int n, int kbar,
                                                      const uint32_t *__restrict__ labels, const uint32_t *__restrict__ room,
                                                      const uint32_t *__restrict__ left, uint32_t *__restrict__ count,
                                                      uint64_t *__restrict__ list, uint32_t np2)
{
    if (*left == 0) return;                                      // uniform: a round too many
    __shared__ uint64_t proposal[kProposeBlock];                 // of every point: (distance, group), ~0 for a point that makes none
    __shared__ uint32_t mine[256], place[256];                   // the workgroup's proposals to a group, and where they go in its list
    const int tid = threadIdx.x, lane = tid & 63, p0 = (tid >> 6) * kProposePoints;
    const int i0 = static_cast<int>(blockIdx.x) * kProposeBlock + p0;
    uint64_t todo = __builtin_amdgcn_ballot_w64(lane < kProposePoints && i0 + lane < n && labels[min(i0 + lane, n - 1)] == 0xFFFFFFFFu);
    if (tid < kProposeBlock) proposal[tid] = ~0ull;
    if (tid < 256) mine[tid] = 0;
    if (!__syncthreads_or(todo != 0)) return;                    // uniform
    bool open[4];
    int first = 256;                                             // first group with room
#pragma unroll
    for (int z = 3; z >= 0; --z) {
        const int l = 64 * z + lane;
        open[z] = l < kbar && room[l] > 0;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(open[z]);
        if (mask) first = 64 * z + __builtin_ctzll(mask);
    }
    while (todo) {                                               // uniform
        const int i = i0 + __builtin_ctzll(todo);
        todo &= todo - 1;
        const float *row = T + static_cast<size_t>(i) * kbar;
        // distances are >= +0: they order like their bits, NaN behind all (unless the first group with room has it: that one is kept)
        uint64_t best = ~0ull;
        bool nan = false;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int l = 64 * z + lane;
            if (!open[z]) continue;
            const float v = row[l];
            if (l == first && v != v) nan = true;
            const uint64_t key = make_key(__float_as_uint(v), static_cast<uint32_t>(l));
            best = key < best ? key : best;
        }
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint64_t o = __shfl_xor(best, off);
            best = o < best ? o : best;
        }
        if (__builtin_amdgcn_ballot_w64(nan)) best = make_key(__float_as_uint(row[first]), static_cast<uint32_t>(first));
        if (lane == 0) proposal[p0 + (i - i0)] = best;
    }
    __syncthreads();
    const uint64_t best = tid < kProposeBlock ? proposal[tid] : ~0ull;
    const uint32_t l = static_cast<uint32_t>(best);
    uint32_t rank = 0;
    if (best != ~0ull) rank = atomicAdd(&mine[l], 1u);
    __syncthreads();
    if (tid < kbar && mine[tid]) place[tid] = atomicAdd(&count[tid], mine[tid]);
    __syncthreads();
    if (best != ~0ull)
        list[static_cast<size_t>(l) * np2 + place[l] + rank] =
            make_key(static_cast<uint32_t>(best >> 32), blockIdx.x * static_cast<uint32_t>(kProposeBlock) + static_cast<uint32_t>(tid));
}

// One workgroup per group: its proposers ordered by (distance, point), the first `room` of them accepted.
__global__ __launch_bounds__(1024) void accept_kernel(uint32_t *__restrict__ labels, uint32_t *__restrict__ room, uint32_t *__restrict__ count,
                                                      uint32_t *__restrict__ left, uint64_t *__restrict__ list, uint32_t np2)
{
    __shared__ uint64_t keys[kAcceptKeys];
    __shared__ uint32_t s_count, s_room;
    const int l = blockIdx.x, tid = threadIdx.x;
    // (read by the thread that overwrites them at the end: another wavefront might start after that)
    if (tid == 0) { s_count = count[l]; s_room = room[l]; }
    __syncthreads();
    const uint32_t p = s_count, have = s_room;
    if (p == 0) return;                                          // uniform
    uint64_t *a = list + static_cast<size_t>(l) * np2;
    uint32_t take = p;
    if (p > have) {                                              // uniform: more proposers than room, keep the closest
        uint32_t s2 = 1;
        while (s2 < p) s2 <<= 1;
        if (s2 <= kAcceptKeys) {
            for (uint32_t t = tid; t < s2; t += 1024) keys[t] = t < p ? a[t] : ~0ull;
            a = keys;
        } else {
            for (uint32_t t = p + tid; t < s2; t += 1024) a[t] = ~0ull;
        }
        __syncthreads();
        bitonic_sort(a, s2);
        take = have;
    }
    for (uint32_t t = tid; t < take; t += 1024) labels[static_cast<uint32_t>(a[t])] = static_cast<uint32_t>(l);
    if (tid == 0) { room[l] = have - take; count[l] = 0; atomicSub(left, take); }
}

// Step 3: one workgroup per group l walks the labels in index order; the i-th member met gets the final
// index (i << bbar) | l.  A wavefront has a stretch of the labels: it counts its members, then places them; the rows are copied
// together at the end (a walk by the whole workgroup, three barriers for 1024 labels, copying as it goes: 167 us at k = 65536, 256 groups; so 22).
__global__ __launch_bounds__(1024) void final_codebook_kernel(const float *__restrict__ temp, int k, int d,
                                                              const uint32_t *__restrict__ labels, int bbar,
                                                              float *__restrict__ final_cb, uint32_t *perm)
{
    __shared__ uint32_t wsum[16];
    const uint32_t l = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = ((k + 15) / 16 + 63) / 64 * 64, lo = min(k, wave * per), hi = min(k, lo + per);
    uint32_t mine = 0;
#pragma unroll 8
    for (int i = lo + lane; i < hi; i += 64) mine += labels[i] == l ? 1u : 0u;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) mine += __shfl_xor(mine, off);
    if (lane == 0) wsum[wave] = mine;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) before += wsum[w];
        total += wsum[w];
    }
#pragma unroll 8
    for (int i = lo + lane; i - lane < hi; i += 64) {            // uniform trip count
        const bool is = i < hi && labels[min(i, k - 1)] == l;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(is);
        if (is) {
            const uint32_t f = ((before + __popcll(mask & ((1ull << lane) - 1ull))) << bbar) | l;
            if (f < static_cast<uint32_t>(k)) perm[f] = static_cast<uint32_t>(i);      // labels with unequal groups would point past the end
        }
        before += __popcll(mask);
    }
    __syncthreads();
    const uint32_t fits = (static_cast<uint32_t>(k) - l + (1u << bbar) - 1u) >> bbar, members = min(total, fits);       // (final indices below k)
    for (uint32_t e = tid; e < members * d; e += 1024) {
        const uint32_t f = (e / d) << bbar | l, t = e % d;
        final_cb[static_cast<size_t>(f) * d + t] = temp[static_cast<size_t>(perm[f]) * d + t];
    }
}

// ---- host side --------------------------------------------------------------------------------------

static size_t means_bytes(size_t k, int d) { return align_up(sizeof(double) * k * d + sizeof(uint32_t) * k, 256); }

// centroids[j][c] = mean of the sub-vectors j labelled c, j < m (ws: means_bytes(m k, d))
static int launch_means(const float *points, uint64_t n, int ld, int m, int d, const uint32_t *labels, int k, float *centroids,
                        void *ws, hipStream_t st)
{
    double *sums = static_cast<double *>(ws);
    const size_t mk = static_cast<size_t>(m) * k;
    uint32_t *counts = reinterpret_cast<uint32_t *>(sums + mk * d);
    const size_t nwords = (sizeof(double) * mk * d + sizeof(uint32_t) * mk) / 4;
    DCPQ_LAUNCH(kStageTrain, st, clear_kernel, dim3(static_cast<unsigned>((nwords + 255) / 256)), dim3(256), 0,
                reinterpret_cast<uint32_t *>(ws), nwords);
    DCPQ_CHECK_LAUNCH("clear_kernel");
    const uint64_t e = n * static_cast<uint64_t>(m * d);
    DCPQ_LAUNCH(kStageTrain, st, accumulate_kernel, dim3(static_cast<unsigned>((e + 255) / 256)), dim3(256), 0, points, n, ld, d,
                labels, m, k, sums, counts);
    DCPQ_CHECK_LAUNCH("accumulate_kernel");
    DCPQ_LAUNCH(kStageTrain, st, means_kernel, dim3(static_cast<unsigned>((mk * d + 255) / 256)), dim3(256), 0, sums, counts, mk * d, d, centroids);
    DCPQ_CHECK_LAUNCH("means_kernel");
    return DCPQ_OK;
}

// k-means iterations of m sub-quantizers at once: sub-vectors j of the points, centroids [m][k][d], labels [n][m] (those the
// centroids are the means of)
static int launch_kmeans(const float *points, uint64_t n, int ld, int m, int d, int k, int iters, float *centroids, uint32_t *labels,
                         void *ws, hipStream_t st)
{
    for (int it = 0; it < iters; ++it) {
        int rc = launch_assign(points, n, ld, centroids, m, d, k, labels, 4, nullptr, st);
        if (rc) return rc;
        rc = launch_means(points, n, ld, m, d, labels, k, centroids, ws, st);
        if (rc) return rc;
    }
    return DCPQ_OK;
}

static uint32_t pow2_at_least(uint32_t x)
{
    uint32_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

constexpr int kRoundsAhead = 12;             // of a balanced assignment, before it is looked at with others
constexpr int kMostLeft = 64;                // words for points without a group
struct SameSizePlan { size_t off_T, off_count, off_room, off_left, off_list, off_means, total; uint32_t np2; };

static SameSizePlan plan_same_size(int n, int d, int kbar)
{
    SameSizePlan p{};
    p.np2 = pow2_at_least(static_cast<uint32_t>(n));
    size_t off = 0;
    p.off_T = off;     off = align_up(off + sizeof(float) * static_cast<size_t>(n) * kbar, 256);
    p.off_count = off; off = align_up(off + sizeof(uint32_t) * static_cast<size_t>(n), 256);     // (kbar <= n counters; as much as there always was here)
    p.off_room = off;  off = align_up(off + sizeof(uint32_t) * kbar, 256);
    p.off_left = off;  off = align_up(off + sizeof(uint32_t) * kMostLeft, 256);
    p.off_list = off;  off = align_up(off + sizeof(uint64_t) * static_cast<size_t>(kbar) * p.np2, 256);
    p.off_means = off; off = align_up(off + means_bytes(kbar, d), 256);
    p.total = off;
    return p;
}

// A balanced assignment of n points in a workspace of the plan, in parts: distances and empty groups (begin) or, for one that was left after some rounds, distances
// and the room there still is (resume); rounds.  left: points without a group, one word.
struct Balanced {
    const float *points;
    int n, d, kbar;
    const float *centroids;
    uint32_t *labels, *left;
    uint8_t *base;
    const SameSizePlan &p;
    hipStream_t st;

    uint32_t *count() const { return reinterpret_cast<uint32_t *>(base + p.off_count); }
    uint32_t *room() const { return reinterpret_cast<uint32_t *>(base + p.off_room); }

    int distances() const { return launch_distance_tables(points, n, centroids, 1, d, kbar, reinterpret_cast<float *>(base + p.off_T), kStageTrain, st); }

    int begin() const
    {
        const int rc = distances(), nb = n > kbar ? n : kbar;
        if (rc) return rc;
        DCPQ_LAUNCH(kStageTrain, st, balanced_init_kernel, dim3((nb + 255) / 256), dim3(256), 0, labels, n, room(), count(), kbar, left);
        DCPQ_CHECK_LAUNCH("balanced_init_kernel");
        return DCPQ_OK;
    }

    int resume() const
    {
        const int rc = distances();
        if (rc) return rc;
        DCPQ_LAUNCH(kStageTrain, st, balanced_resume_kernel, dim3(1), dim3(1024), 0, labels, n, room(), count(), kbar);
        DCPQ_CHECK_LAUNCH("balanced_resume_kernel");
        return DCPQ_OK;
    }

    int rounds(int how_many) const
    {
        uint64_t *list = reinterpret_cast<uint64_t *>(base + p.off_list);
        for (int round = 0; round < how_many; ++round) {
            DCPQ_LAUNCH(kStageTrain, st, propose_kernel, dim3((n + kProposeBlock - 1) / kProposeBlock), dim3(64 * kProposeWaves), 0,
                        reinterpret_cast<const float *>(base + p.off_T), n, kbar, labels, room(), left, count(), list, p.np2);
            DCPQ_CHECK_LAUNCH("propose_kernel");
            DCPQ_LAUNCH(kStageTrain, st, accept_kernel, dim3(kbar), dim3(1024), 0, labels, room(), count(), left, list, p.np2);
            DCPQ_CHECK_LAUNCH("accept_kernel");
        }
        return DCPQ_OK;
    }

    // Rounds until every point has a group, `ahead` at first; every round gives at least one point a group.  The count is read back after
    // these and after every four more: a round too many returns at once.  (A round that
    // leaves points without a group has filled one that turned them away: kbar rounds are enough.)
    int finish(int ahead) const
    {
        uint32_t h_left = static_cast<uint32_t>(n);
        for (int round = 0; h_left > 0; ahead = 4) {
            if (round > kbar) return fail(DCPQ_EHIP, "kmeans_same_size: balanced assignment did not finish");
            const int rc = rounds(ahead);
            if (rc) return rc;
            round += ahead;
            DCPQ_CHECK_HIP(hipMemcpyAsync(&h_left, left, sizeof(uint32_t), hipMemcpyDeviceToHost, st));
            DCPQ_CHECK_HIP(hipStreamSynchronize(st));
        }
        return DCPQ_OK;
    }

    int means(float *to) const { return launch_means(points, static_cast<uint64_t>(n), d, 1, d, labels, kbar, to, base + p.off_means, st); }
};

static int launch_final_codebook(const float *temp, int k, int d, const uint32_t *labels, int bbar, float *final_cb, uint32_t *perm, hipStream_t st)
{
    DCPQ_LAUNCH(kStageTrain, st, final_codebook_kernel, dim3(1 << bbar), dim3(1024), 0, temp, k, d, labels, bbar, final_cb, perm);
    DCPQ_CHECK_LAUNCH("final_codebook_kernel");
    return DCPQ_OK;
}

}  // namespace dcpq

using namespace dcpq;

extern "C" int dcpq_assign(const float *points, uint64_t n, int ld, const float *codebooks, int m, int dsub, int n_entries,
                           void *labels, int label_bytes, float *dist, void *stream)
{
    clear_error();
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "assign: m=%d dsub=%d not supported", m, dsub);
    DCPQ_REQUIRE(n < (1ull << 37), "assign: n out of range");
    DCPQ_REQUIRE(ld >= m * dsub, "assign: row stride %d below m * dsub = %d", ld, m * dsub);
    DCPQ_REQUIRE(label_bytes == 1 || label_bytes == 2 || label_bytes == 4, "assign: label_bytes=%d (1, 2 or 4)", label_bytes);
    DCPQ_REQUIRE(n_entries >= 1 && (label_bytes == 4 || n_entries <= (1 << (8 * label_bytes))),
                 "assign: %d centroids do not fit labels of %d byte(s)", n_entries, label_bytes);
    if (n == 0) return DCPQ_OK;
    DCPQ_REQUIRE(points && codebooks && labels, "assign: null pointer");
    return launch_assign(points, n, ld, codebooks, m, dsub, n_entries, labels, label_bytes, dist, as_stream(stream));
}

extern "C" int dcpq_encode(const float *vectors, uint64_t n, const float *codebooks, int m, int dsub, int b, void *codes,
                           void *stream)
{
    if (!dcpq_bits_supported(b, 1)) {
        clear_error();
        return fail(DCPQ_EUNSUPPORTED, "encode: b=%d not supported", b);
    }
    return dcpq_assign(vectors, n, m * dsub, codebooks, m, dsub, 1 << b, codes, b / 8, nullptr, stream);
}

extern "C" size_t dcpq_kmeans_workspace_bytes(int k, int d)
{
    if (k <= 0 || d <= 0) return 0;
    return means_bytes(k, d);
}

extern "C" int dcpq_kmeans(const float *points, uint64_t n, int ld, int d, int k, int iters, float *centroids,
                           uint32_t *labels, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    if (!dcpq_shape_supported(1, d)) return fail(DCPQ_EUNSUPPORTED, "kmeans: d=%d not supported", d);
    DCPQ_REQUIRE(n >= 1 && n < (1ull << 32), "kmeans: n out of range");
    DCPQ_REQUIRE(k >= 1 && iters >= 0 && ld >= d, "kmeans: k=%d iters=%d ld=%d", k, iters, ld);
    DCPQ_REQUIRE(points && centroids && labels && workspace, "kmeans: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "kmeans: workspace must be 256-byte aligned");
    if (workspace_bytes < means_bytes(k, d))
        return fail(DCPQ_EWORKSPACE, "kmeans: workspace %zu < %zu bytes", workspace_bytes, means_bytes(k, d));
    const int rc = launch_kmeans(points, n, ld, 1, d, k, iters, centroids, labels, workspace, as_stream(stream));
    if (rc) return rc;
    return launch_assign(points, n, ld, centroids, 1, d, k, labels, 4, nullptr, as_stream(stream));
}

extern "C" size_t dcpq_kmeans_same_size_workspace_bytes(int n, int d, int kbar)
{
    if (n <= 0 || d <= 0 || kbar <= 0 || kbar > 256) return 0;
    return plan_same_size(n, d, kbar).total;
}

extern "C" int dcpq_kmeans_same_size(const float *points, int n, int d, int kbar, int iters, float *centroids,
                                     uint32_t *labels, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    if (!dcpq_shape_supported(1, d)) return fail(DCPQ_EUNSUPPORTED, "kmeans_same_size: d=%d not supported", d);
    DCPQ_REQUIRE(kbar >= 1 && kbar <= 256, "kmeans_same_size: kbar=%d (1..256)", kbar);
    DCPQ_REQUIRE(n >= kbar && n % kbar == 0 && n <= (1 << 20), "kmeans_same_size: n=%d must be a multiple of kbar=%d, at most 2^20", n, kbar);
    DCPQ_REQUIRE(iters >= 1, "kmeans_same_size: iters=%d", iters);
    DCPQ_REQUIRE(points && centroids && labels && workspace, "kmeans_same_size: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "kmeans_same_size: workspace must be 256-byte aligned");
    const SameSizePlan p = plan_same_size(n, d, kbar);
    if (workspace_bytes < p.total) return fail(DCPQ_EWORKSPACE, "kmeans_same_size: workspace %zu < %zu bytes", workspace_bytes, p.total);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    const Balanced a{points, n, d, kbar, centroids, labels, reinterpret_cast<uint32_t *>(base + p.off_left), base, p, as_stream(stream)};
    for (int it = 0; it < iters; ++it) {
        int rc = a.begin();
        if (rc) return rc;
        rc = a.finish(kbar < 8 ? kbar : 8);                      // (eight rounds are what it takes as a rule)
        if (rc) return rc;
        rc = a.means(centroids);
        if (rc) return rc;
    }
    return DCPQ_OK;
}

extern "C" int dcpq_build_final_codebook(const float *temp_codebook, int k, int d, const uint32_t *labels, int bbar,
                                         float *final_codebook, uint32_t *perm, void *stream)
{
    clear_error();
    DCPQ_REQUIRE(k >= 1 && d >= 1 && bbar >= 0 && bbar <= 8 && k % (1 << bbar) == 0, "build_final_codebook: k=%d d=%d bbar=%d", k, d, bbar);
    DCPQ_REQUIRE(temp_codebook && labels && final_codebook && perm, "build_final_codebook: null pointer");
    DCPQ_REQUIRE(temp_codebook != final_codebook, "build_final_codebook: in place is not supported");
    return launch_final_codebook(temp_codebook, k, d, labels, bbar, final_codebook, perm, as_stream(stream));
}

// Alg. 2 for all m sub-quantizers.  Workspace: labels of the training points, labels and groups' centroids of a codebook, a copy
// and the order of one, and the larger of the two k-means workspaces.
struct BuildPlan { size_t off_clabels, clabels_bytes, group_bytes, off_temp, off_perm, off_ws, ws_bytes, total; };

static BuildPlan plan_build(uint64_t n, int dsub, int b, int bbar)
{
    BuildPlan p{};
    const int k = 1 << b, kbar = 1 << bbar;
    p.clabels_bytes = align_up(sizeof(uint32_t) * k, 256);
    p.group_bytes = align_up(sizeof(float) * static_cast<size_t>(kbar) * dsub, 256);
    size_t off = align_up(sizeof(uint32_t) * n, 256);
    p.off_clabels = off; off += p.clabels_bytes + p.group_bytes;
    p.off_temp = off;    off = align_up(off + sizeof(float) * static_cast<size_t>(k) * dsub, 256);
    p.off_perm = off;    off = align_up(off + sizeof(uint32_t) * k, 256);
    const size_t a = means_bytes(k, dsub), c = plan_same_size(k, dsub, kbar).total;
    p.ws_bytes = a > c ? a : c;
    p.off_ws = off;      off = align_up(off + p.ws_bytes, 256);
    p.total = off;
    return p;
}

extern "C" size_t dcpq_build_quantizers_workspace_bytes(uint64_t n_train, int dsub, int b, int bbar)
{
    if (n_train == 0 || dsub <= 0 || !dcpq_bits_supported(b, bbar)) return 0;
    return plan_build(n_train, dsub, b, bbar).total;
}

extern "C" int dcpq_build_quantizers(const float *train, uint64_t n_train, int m, int dsub, int b, int bbar, int iters,
                                     int iters_same_size, float *codebooks, float *derived, void *workspace,
                                     size_t workspace_bytes, void *stream)
{
    clear_error();
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "build_quantizers: m=%d dsub=%d not supported", m, dsub);
    if (!dcpq_bits_supported(b, bbar)) return fail(DCPQ_EUNSUPPORTED, "build_quantizers: b=%d bbar=%d not supported", b, bbar);
    DCPQ_REQUIRE(n_train >= 1 && n_train < (1ull << 32), "build_quantizers: n_train out of range");
    DCPQ_REQUIRE(iters >= 0 && iters_same_size >= 1, "build_quantizers: iters=%d iters_same_size=%d", iters, iters_same_size);
    DCPQ_REQUIRE(train && codebooks && derived && workspace, "build_quantizers: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "build_quantizers: workspace must be 256-byte aligned");
    const BuildPlan p = plan_build(n_train, dsub, b, bbar);
    if (workspace_bytes < p.total) return fail(DCPQ_EWORKSPACE, "build_quantizers: workspace %zu < %zu bytes", workspace_bytes, p.total);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    const int k = 1 << b, kbar = 1 << bbar, D = m * dsub;
    hipStream_t st = as_stream(stream);
    // step 1: k-means of the centroids the caller left in `codebooks`, in place (the points' labels after the last iteration are no
    // result of the training and are not taken), of as many sub-quantizers at once as the room
    // for same-size k-means (256 rows of all centroids) holds labels and sums for.  One at a time leaves half of the chip idle
    // (131072 points, 65536 centroids of 16 components: an assignment for 8 sub-quantizers 6.5 ms one by one, 4.5 together).
    int together = 0;
    while (together < m && align_up(sizeof(uint32_t) * n_train * (together + 1), 256) + means_bytes(static_cast<size_t>(together + 1) * k, dsub) <= p.ws_bytes) ++together;
    for (int j = 0; j < m; j += together ? together : 1) {
        const int mj = !together ? 1 : m - j < together ? m - j : together;
        uint32_t *labels = reinterpret_cast<uint32_t *>(together ? base + p.off_ws : base);
        void *sums = together ? base + p.off_ws + align_up(sizeof(uint32_t) * n_train * mj, 256) : base + p.off_ws;
        const int rc = launch_kmeans(train + static_cast<size_t>(j) * dsub, n_train, D, mj, dsub, k, iters, codebooks + static_cast<size_t>(j) * k * dsub,
                                     labels, sums, st);
        if (rc) return rc;
    }
    // Steps 2 and 3.  An iteration's balanced assignments of several sub-quantizers are enqueued one after the other, each with the rounds that it takes as a rule and
    // some more, and looked at together, which saves a wait for each (131072 x 8 x 16: 9.45 ms with every assignment waited for, 9.0 so).  One
    // that was not done (crowded centroids: as many rounds as there are groups) goes on from the labels it has reached; only its distances are
    // computed again.  So labels and centroids of every sub-quantizer of a batch are kept: in the place of the training points' labels, and of the
    // codebook's copy too where the lists of proposers, which nobody reads once the assignments are done, are long enough to take copy and order.
    const SameSizePlan sp = plan_same_size(k, dsub, kbar);
    const size_t copy_bytes = align_up(sizeof(float) * static_cast<size_t>(k) * dsub, 256);
    const bool in_lists = copy_bytes + sizeof(uint32_t) * k <= sizeof(uint64_t) * static_cast<size_t>(kbar) * sp.np2;
    float *temp = reinterpret_cast<float *>(base + (in_lists ? p.off_ws + sp.off_list : p.off_temp));
    uint32_t *perm = reinterpret_cast<uint32_t *>(in_lists ? base + p.off_ws + sp.off_list + copy_bytes : base + p.off_perm);
    const size_t per = p.clabels_bytes + p.group_bytes, places = (in_lists ? p.off_ws : p.off_temp) / per;        // (one at least)
    const int batch = places < static_cast<size_t>(m) ? static_cast<int>(places) : m, ahead = kbar < kRoundsAhead ? kbar : kRoundsAhead;
    uint32_t *left = reinterpret_cast<uint32_t *>(base + p.off_ws + sp.off_left);         // a word per sub-quantizer of a batch
    for (int j0 = 0; j0 < m; j0 += batch) {
        const int mj = m - j0 < batch ? m - j0 : batch;
        auto codebook = [&](int i) { return codebooks + static_cast<size_t>(j0 + i) * k * dsub; };
        auto labels = [&](int i) { return reinterpret_cast<uint32_t *>(base + per * i); };
        auto groups = [&](int i) { return reinterpret_cast<float *>(base + per * i + p.clabels_bytes); };
        for (int it = 0; it < iters_same_size; ++it) {
            // (groups are started from the first 2^bbar temporary centroids)
            auto assignment = [&](int i) { return Balanced{codebook(i), k, dsub, kbar, it ? groups(i) : codebook(i), labels(i), left + i, base + p.off_ws, sp, st}; };
            for (int i = 0; i < mj; ++i) {
                const Balanced a = assignment(i);
                int rc = a.begin();
                if (rc) return rc;
                rc = a.rounds(ahead);
                if (rc) return rc;
            }
            uint32_t h_left[kMostLeft];
            DCPQ_CHECK_HIP(hipMemcpyAsync(h_left, left, sizeof(uint32_t) * mj, hipMemcpyDeviceToHost, st));
            DCPQ_CHECK_HIP(hipStreamSynchronize(st));
            for (int i = 0; i < mj; ++i) {
                const Balanced a = assignment(i);
                int rc = DCPQ_OK;
                if (h_left[i]) {
                    rc = a.resume();
                    if (rc) return rc;
                    rc = a.finish(4);
                    if (rc) return rc;
                }
                if (it + 1 < iters_same_size) rc = a.means(groups(i));       // (nobody reads those of the last assignment)
                if (rc) return rc;
            }
        }
        for (int i = 0; i < mj; ++i) {
            // step 3: final order; it reads the temporary codebook while it writes the final one.  The derived codebook is the mean of every low-bits group of it
            DCPQ_CHECK_HIP(hipMemcpyAsync(temp, codebook(i), sizeof(float) * static_cast<size_t>(k) * dsub, hipMemcpyDeviceToDevice, st));
            const int rc = launch_final_codebook(temp, k, dsub, labels(i), bbar, codebook(i), perm, st);
            if (rc) return rc;
        }
    }
    return launch_derive(codebooks, m, dsub, b, bbar, derived, st);
}

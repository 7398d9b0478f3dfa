// Alg. 3 with an inverted index and residual encoding (Sec. 2.2; Sec. 2.3: every step after the
// Index step is done once per probed list; Sec. 3.3).  List l holds the codes at positions offsets[l] .. offsets[l+1]-1 of the
// code array (a vector's id is its position); codes quantize the residual x - c_l.
//
//   Index   ivf_probe           the nprobe closest cell centres per query (all distances on the matrix cores in fp64; for many
//                               queries only of the centres that an fp16 estimate leaves, ivf_probe.hip)
//   Tables  ivf_small_tables    per (query, probed list): small tables of the residual query
//                               rho = y - c_l on the derived codebooks; ONE (qmin, qmax) pair per
//                               query -- qmin over all its lists' tables, qmax over the first
//                               min(r, total) codes met walking its lists in probe order -- so that
//                               integer distances from different lists are comparable
//   Scan    ivf_scan            the r smallest (qd, id) over the union of the probed lists: one streaming
//                               pass with a running bucket bound and an exact selection (as in
//                               scan_fast.hip), a workgroup per "part" (a run of codes of one list, for
//                               one query) with that (query, list)'s 8-bit tables in LDS; for the queries
//                               it flags the three-pass selection of scan.hip, a wavefront per "unit"
//                               (runs of codes inside one list, in increasing id order)
//   Refine  ivf_refine_topk     Eq. 3 on the residual of each candidate's own list, directly from
//                               the full codebooks in double precision (per-list 2^16-entry tables
//                               would cost nprobe table builds per query), then the k best
#include <type_traits>

#include "common.h"
#include "ivf_select.h"
#include "redo_wait.h"
#include "scan_internal.h"

namespace dcpq {

constexpr int kIvfUnitsPerQuery = 1024;   // upper bound of scan units per query (unit size adapts)
constexpr uint32_t kIvfSampleStep = 32;   // the first 1 / kIvfSampleStep of every probed list (at most) is the sample that gives the scan its starting bounds
constexpr uint32_t kIvfBins = 65536;      // bins of list ids that the scan's work is ordered by, at most
constexpr uint32_t kIvfMinPart = 512;     // codes a workgroup of the single-pass scan takes at least (large batches: twice as many)
constexpr uint32_t kIvfNotes = 1024;      // candidates it can note until it has walked its part

struct IvfUnit {
    uint64_t begin;    // first code of the unit (global position)
    uint32_t count;    // codes in the unit
    uint32_t p;        // index of the list in the query's probe order (selects the tables); in the single-pass
                       // scan's list of parts q * nprobe + p
};

// ------------------------------------------------------------------------------------------------
// Index step: nprobe smallest coarse distances per query, ordered by (distance, list id).
// dist: [nq][nlist] fp32 squared distances.  One workgroup per query; redo: only for those that have a negative number in the place of their first list.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void ivf_select_probe_kernel(const float *__restrict__ dist, int nlist, int nprobe,
                                                               int32_t *__restrict__ probe, int redo)
{
    if (redo && probe[static_cast<size_t>(blockIdx.x) * nprobe] >= 0) return;      // uniform
    select_probe_of_row(dist + static_cast<size_t>(blockIdx.x) * nlist, nlist, nprobe, probe + static_cast<size_t>(blockIdx.x) * nprobe);
}

// ------------------------------------------------------------------------------------------------
// Tables step.  All arithmetic fp32, one rounding per operation, fixed order (feeds integers).
// ------------------------------------------------------------------------------------------------

// MODE 0: the entries to `keep` [nq][nprobe][m][256], the smallest of a workgroup to the first bytes of its part of qtab; or,
// without `keep`, the smallest entry of the (query, list) tables only -> atomic min into qmin_bits[q].
// MODE 1: quantize with the query's bounds -> qtab[q][p][m][256].
// grid (ceil(nprobe / kIvfTabProbes), nq), 256 threads; thread i owns entry i of every table of
// kIvfTabProbes probed lists of the query, of the sub-quantizers blockIdx.z * per_z on (all of them where the batch fills the
// chip; a query or two are spread out).  The derived centroid is read once per component and used for
// all of those lists' residuals (the kernel is bound by these reads, which all come from the L2); every
// entry is still the sum over t, in ascending t, of the individually rounded squares.
constexpr int kIvfTabProbes = 8;

template <int MODE>
__global__ __launch_bounds__(256) void ivf_tables_kernel(const float *__restrict__ queries, const float *__restrict__ coarse,
                                                        const int32_t *__restrict__ probe, int nprobe,
                                                        const float *__restrict__ derived, int m, int dsub,
                                                        uint32_t *__restrict__ qmin_bits, const float *__restrict__ bounds,
                                                        uint8_t *__restrict__ qtab, float *__restrict__ keep, int per_z)
{
    extern __shared__ __align__(16) float lds[];         // rho [kIvfTabProbes][m*dsub]
    __shared__ float red[4];
    const int p0 = blockIdx.x * kIvfTabProbes, q = blockIdx.y, tid = threadIdx.x;
    const int np = min(kIvfTabProbes, nprobe - p0);
    const int D = m * dsub, j0 = blockIdx.z * per_z, j1 = min(m, j0 + per_z);
    for (int pp = 0; pp < np; ++pp) {
        const int l = probe[static_cast<size_t>(q) * nprobe + p0 + pp];
        for (int t = j0 * dsub + tid; t < j1 * dsub; t += 256)
            lds[pp * D + t] = __fsub_rn(queries[static_cast<size_t>(q) * D + t], coarse[static_cast<size_t>(l) * D + t]);
    }
    __syncthreads();
    float qmin = 0.0f, qmax = 0.0f;
    if (MODE == 1) {
        qmin = bounds[2 * q];
        qmax = bounds[2 * q + 1];
    }
    float lo = INFINITY;
    for (int j = j0; j < j1; ++j) {
        const float *c = derived + (static_cast<size_t>(j) * kSmallSize + tid) * dsub;
        float acc[kIvfTabProbes];
#pragma unroll
        for (int pp = 0; pp < kIvfTabProbes; ++pp) acc[pp] = 0.0f;
        if ((dsub & 3) == 0) {
            // four components per step: one 16-byte load of the centroid, one 16-byte (broadcast) LDS read per
            // list; the squares are still added one by one in ascending t
            for (int t = 0; t < dsub; t += 4) {
                const float4 c4 = *reinterpret_cast<const float4 *>(c + t);
#pragma unroll
                for (int pp = 0; pp < kIvfTabProbes; ++pp) {
                    if (pp < np) {                                // uniform
                        const float4 r4 = *reinterpret_cast<const float4 *>(lds + pp * D + j * dsub + t);
                        float diff = __fsub_rn(r4.x, c4.x);
                        acc[pp] = __fadd_rn(acc[pp], __fmul_rn(diff, diff));
                        diff = __fsub_rn(r4.y, c4.y);
                        acc[pp] = __fadd_rn(acc[pp], __fmul_rn(diff, diff));
                        diff = __fsub_rn(r4.z, c4.z);
                        acc[pp] = __fadd_rn(acc[pp], __fmul_rn(diff, diff));
                        diff = __fsub_rn(r4.w, c4.w);
                        acc[pp] = __fadd_rn(acc[pp], __fmul_rn(diff, diff));
                    }
                }
            }
        } else {
            for (int t = 0; t < dsub; ++t) {
                const float ct = c[t];
#pragma unroll
                for (int pp = 0; pp < kIvfTabProbes; ++pp) {
                    if (pp < np) {                                // uniform
                        const float diff = __fsub_rn(lds[pp * D + j * dsub + t], ct);
                        acc[pp] = __fadd_rn(acc[pp], __fmul_rn(diff, diff));
                    }
                }
            }
        }
#pragma unroll
        for (int pp = 0; pp < kIvfTabProbes; ++pp) {
            if (pp >= np) continue;                               // uniform
            if (MODE == 0) {
                lo = fminf(lo, acc[pp]);
                if (keep) keep[((static_cast<size_t>(q) * nprobe + p0 + pp) * m + j) * kSmallSize + tid] = acc[pp];
            } else {
                qtab[((static_cast<size_t>(q) * nprobe + p0 + pp) * m + j) * kSmallSize + tid] =
                    quantize_entry(acc[pp], qmin, qmax);
            }
        }
    }
    if (MODE == 0) {
        lo = block_reduce(lo, false, red);
        if (tid == 0) {
            if (keep) *reinterpret_cast<float *>(qtab + ((static_cast<size_t>(q) * nprobe + p0) * m + j0) * kSmallSize) = lo;
            else atomicMin(&qmin_bits[q], __float_as_uint(lo));         // entries are >= +0
        }
    }
}

// The quantization of entries kept by the first pass: qtab[e] = quantizer(keep[e]) with the bounds of the
// entry's query (per_query = nprobe * m * 256 entries each).
__global__ __launch_bounds__(256) void ivf_quantize_kept_kernel(const float *__restrict__ keep, size_t n, size_t per_query,
                                                               const float *__restrict__ bounds, uint8_t *__restrict__ qtab)
{
    const size_t e = (static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4;
    if (e >= n) return;                                         // n is a multiple of 256
    const size_t q = e / per_query;
    const float qmin = bounds[2 * q], qmax = bounds[2 * q + 1];
    const float4 v = *reinterpret_cast<const float4 *>(keep + e);
    uchar4 o;
    o.x = quantize_entry(v.x, qmin, qmax); o.y = quantize_entry(v.y, qmin, qmax);
    o.z = quantize_entry(v.z, qmin, qmax); o.w = quantize_entry(v.w, qmin, qmax);
    *reinterpret_cast<uchar4 *>(qtab + e) = o;
}

// The bounds from kept entries: qmin from the minima that the workgroups of the first pass left in qtab, qmax by looking the
// entries of the first min(r, total) codes up, in probe order.  One workgroup per query.  (With the entries worked out again from
// the centroids, 256 threads and the prefix of the list sizes taken by one of them from memory: 69 us for 1024
// queries, r = 1000, and 22 for one; so 17 and 5.)
__global__ __launch_bounds__(1024) void ivf_bounds_kept_kernel(const float *__restrict__ keep, const uint8_t *__restrict__ qtab,
                                                               const int32_t *__restrict__ probe, int nprobe, int m, int per_z,
                                                               const uint16_t *__restrict__ codes, const int64_t *__restrict__ offsets,
                                                               uint32_t r, float *__restrict__ bounds)
{
    __shared__ uint64_t first[kIvfMaxProbe];       // first code of a probed list
    __shared__ uint32_t start[kIvfMaxProbe + 1];   // codes before it in probe order, r at most
    __shared__ float red[2][16];
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
    const int32_t *pq = probe + static_cast<size_t>(q) * nprobe;
    // (list sizes of 64 lists at a time, by the first wavefront)
    if (wave == 0) {
        uint64_t before = 0;
        for (int p0 = 0; p0 < nprobe; p0 += 64) {
            const int p = p0 + lane;
            uint64_t at = 0, n = 0;
            if (p < nprobe) {
                const int l = pq[p];
                at = static_cast<uint64_t>(offsets[l]);
                n = static_cast<uint64_t>(offsets[l + 1]) - at;
            }
            uint64_t incl = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint64_t o = __shfl(incl, lane >= d ? lane - d : lane);
                if (lane >= d) incl += o;
            }
            const uint64_t b = before + incl - n;
            if (p < nprobe) {
                first[p] = at;
                start[p] = static_cast<uint32_t>(b < r ? b : r);
            }
            before += __shfl(incl, 63);
        }
        if (lane == 0) start[nprobe] = static_cast<uint32_t>(before < r ? before : r);
    }
    float lo = INFINITY, hi = -INFINITY;
    const int nz = (m + per_z - 1) / per_z, nmin = (nprobe + kIvfTabProbes - 1) / kIvfTabProbes * nz;
    for (int t = tid; t < nmin; t += blockDim.x)
        lo = fminf(lo, *reinterpret_cast<const float *>(qtab + ((static_cast<size_t>(q) * nprobe + t / nz * kIvfTabProbes) * m + t % nz * per_z) * kSmallSize));
    __syncthreads();
    const uint32_t n_first = start[nprobe];
    const bool vec = (m & 7) == 0 && (reinterpret_cast<uintptr_t>(codes) & 15) == 0;       // uniform
    for (uint32_t i = tid; i < n_first; i += blockDim.x) {
        int a = 0, b = nprobe;                     // the list that holds it: start[a] <= i < start[a + 1] (empty ones are passed over)
        while (b - a > 1) {
            const int mid = (a + b) >> 1;
            if (start[mid] <= i) a = mid; else b = mid;
        }
        const uint16_t *c = codes + (first[a] + (i - start[a])) * m;
        const float *tab = keep + (static_cast<size_t>(q) * nprobe + a) * m * kSmallSize;
        float d = 0.0f;
        if (vec) {
            for (int j = 0; j < m; j += 8) {
                uint32_t low[8];
                load_low_bytes<8>(c + j, 0, low);
                float e[8];
#pragma unroll
                for (int z = 0; z < 8; ++z) e[z] = tab[(j + z) * kSmallSize + low[z]];
#pragma unroll
                for (int z = 0; z < 8; ++z) d = j + z == 0 ? e[z] : __fadd_rn(d, e[z]);
            }
        } else {
            for (int j = 0; j < m; ++j) {
                const float e = tab[j * kSmallSize + (c[j] & 255)];
                d = j == 0 ? e : __fadd_rn(d, e);
            }
        }
        hi = fmaxf(hi, d);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        lo = fminf(lo, __shfl_xor(lo, o));
        hi = fmaxf(hi, __shfl_xor(hi, o));
    }
    if (lane == 0) { red[0][wave] = lo; red[1][wave] = hi; }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < nw; ++w) { lo = fminf(lo, red[0][w]); hi = fmaxf(hi, red[1][w]); }
        bounds[2 * q] = n_first ? lo : 0.0f;       // (0, 0) when the probed lists are empty
        bounds[2 * q + 1] = n_first ? hi : 0.0f;
    }
}

// qmax: largest small-table distance over the first min(r, total) codes met walking the probed
// lists in probe order (each code against its own list's residual).  One workgroup per query.
// Also finishes the bounds: (qmin, qmax), or (0, 0) when the probed lists are empty.
__global__ __launch_bounds__(256) void ivf_qmax_kernel(const float *__restrict__ queries, const float *__restrict__ coarse,
                                                      const int32_t *__restrict__ probe, int nprobe,
                                                      const float *__restrict__ derived, int m, int dsub,
                                                      const uint16_t *__restrict__ codes, const int64_t *__restrict__ offsets,
                                                      uint32_t r, const uint32_t *__restrict__ qmin_bits,
                                                      float *__restrict__ bounds)
{
    extern __shared__ __align__(16) float rho[];   // D floats: the query minus the centroid of the list being walked
    __shared__ uint64_t start[kIvfMaxProbe + 1];   // exclusive prefix of the list sizes in probe order
    __shared__ int lst[kIvfMaxProbe];
    __shared__ float red[4];
    const int q = blockIdx.x, tid = threadIdx.x;
    const int D = m * dsub;
    for (int p = tid; p < nprobe; p += 256) lst[p] = probe[static_cast<size_t>(q) * nprobe + p];
    __syncthreads();
    if (tid == 0) {
        uint64_t s = 0;
        for (int p = 0; p < nprobe; ++p) { start[p] = s; s += static_cast<uint64_t>(offsets[lst[p] + 1] - offsets[lst[p]]); }
        start[nprobe] = s;
    }
    __syncthreads();
    const uint64_t total = start[nprobe];
    const uint32_t n_first = static_cast<uint32_t>(total < r ? total : r);
    const float *y = queries + static_cast<size_t>(q) * D;
    const bool vec4 = (dsub & 3) == 0;               // centroid rows of whole 16-byte vectors (derived is 16-byte aligned)
    float hi = -INFINITY;
    // The walk takes the lists in probe order; the codes of one list share the residual of the query against
    // that list's centroid, which the workgroup works out once per list (the walk seldom leaves the first one).
    for (int p = 0; p < nprobe && start[p] < n_first; ++p) {              // uniform
        const uint32_t lo = static_cast<uint32_t>(start[p]);
        const uint32_t up = static_cast<uint32_t>(start[p + 1] < n_first ? start[p + 1] : n_first);
        if (up == lo) continue;                                           // an empty list (uniform)
        const int l = lst[p];
        const float *cl = coarse + static_cast<size_t>(l) * D;
        __syncthreads();                                                  // the previous list's residual is no longer read
        for (int t = tid; t < D; t += 256) rho[t] = __fsub_rn(y[t], cl[t]);
        __syncthreads();
        for (uint32_t i = lo + tid; i < up; i += 256) {
            const uint16_t *c = codes + (static_cast<size_t>(offsets[l]) + (i - lo)) * m;
            float d = 0.0f;
            for (int j = 0; j < m; ++j) {
                const float *cen = derived + (static_cast<size_t>(j) * kSmallSize + (c[j] & 255)) * dsub;
                const float *rj = rho + j * dsub;
                float acc = 0.0f;
                if (vec4) {
                    for (int t = 0; t < dsub; t += 4) {
                        const float4 cv = *reinterpret_cast<const float4 *>(cen + t);
                        const float d0 = __fsub_rn(rj[t], cv.x), d1 = __fsub_rn(rj[t + 1], cv.y);
                        const float d2 = __fsub_rn(rj[t + 2], cv.z), d3 = __fsub_rn(rj[t + 3], cv.w);
                        acc = __fadd_rn(acc, __fmul_rn(d0, d0)); acc = __fadd_rn(acc, __fmul_rn(d1, d1));
                        acc = __fadd_rn(acc, __fmul_rn(d2, d2)); acc = __fadd_rn(acc, __fmul_rn(d3, d3));
                    }
                } else {
                    for (int t = 0; t < dsub; ++t) {
                        const float diff = __fsub_rn(rj[t], cen[t]);
                        acc = __fadd_rn(acc, __fmul_rn(diff, diff));
                    }
                }
                d = j == 0 ? acc : __fadd_rn(d, acc);
            }
            hi = fmaxf(hi, d);
        }
    }
    hi = block_reduce(hi, true, red);
    if (tid == 0) {
        if (total == 0) { bounds[2 * q] = 0.0f; bounds[2 * q + 1] = 0.0f; }
        else { bounds[2 * q] = __uint_as_float(qmin_bits[q]); bounds[2 * q + 1] = hi; }
    }
}

// ------------------------------------------------------------------------------------------------
// Scan step: per-query unit lists.
// ------------------------------------------------------------------------------------------------
// One workgroup per query: probed lists sorted by list id (so that units follow increasing vector
// id), a unit size that keeps the query within kIvfUnitsPerQuery units, and the unit records; and the query's
// share of the single-pass scan's work, cut into about `parts` parts of equal length (no part spans two lists).
// The parts of all queries lie in one list that `cursor` fills.  Without `bins` a query's parts are written here, one
// behind the other; with them only their places are drawn (`rank`, within the bin of the list), ivf_bin_base_kernel
// and ivf_parts_kernel do the rest.
// (Everything after the sort is done by all threads at once, two lists each: one thread's walk over 64 lists, with a
// 64-bit division each, and a round of loads per list took 57 us for 1024 queries.)
__device__ inline uint32_t ivf_bin_of(uint32_t list, uint32_t nlist, uint32_t nbins)
{
    return nlist <= nbins ? list : static_cast<uint32_t>(static_cast<uint64_t>(list) * nbins / nlist);
}

__global__ __launch_bounds__(256) void ivf_plan_kernel(const int32_t *__restrict__ probe, int nprobe,
                                                      const int64_t *__restrict__ offsets, uint32_t nlist, uint32_t r,
                                                      uint32_t parts, uint32_t min_part, IvfUnit *__restrict__ units,
                                                      uint32_t *__restrict__ nunits, uint32_t *__restrict__ count,
                                                      uint32_t *__restrict__ probed, uint32_t *__restrict__ part_of,
                                                      uint32_t *__restrict__ bins, uint32_t nbins, uint32_t *__restrict__ rank,
                                                      uint32_t *__restrict__ cursor, IvfUnit *__restrict__ items)
{
    __shared__ uint64_t key[kIvfMaxProbe];         // (list id << 32) | probe position
    __shared__ uint32_t ubase[kIvfMaxProbe + 1];   // first unit of the s-th probed list (lists in id order)
    __shared__ uint32_t pbase[kIvfMaxProbe + 1];   // first part
    __shared__ uint64_t lbeg[kIvfMaxProbe];        // position and number of its codes
    __shared__ uint64_t lsize[kIvfMaxProbe];
    __shared__ unsigned long long s_total;
    __shared__ uint32_t wsum[2][4], s_base;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) s_total = 0;
    uint32_t np2 = 1;
    while (np2 < static_cast<uint32_t>(nprobe)) np2 <<= 1;
    for (uint32_t p = tid; p < np2; p += 256)
        key[p] = p < static_cast<uint32_t>(nprobe)
                     ? make_key(static_cast<uint32_t>(probe[static_cast<size_t>(q) * nprobe + p]), p) : ~0ull;
    bitonic_sort(key, np2);
    for (int s = tid; s < nprobe; s += 256) {
        const int l = static_cast<int>(key[s] >> 32);
        lbeg[s] = static_cast<uint64_t>(offsets[l]);
        lsize[s] = static_cast<uint64_t>(offsets[l + 1]) - lbeg[s];
        atomicAdd(&s_total, static_cast<unsigned long long>(lsize[s]));
    }
    __syncthreads();
    const uint64_t total = s_total;
    // three units per probed list on average, and at least 512 less one per list in all (measured: fewer,
    // longer units leave the chip unevenly loaded, more of them pay the latency of a wavefront's first
    // loads too often); never more than the unit table holds
    uint64_t want = 4ull * nprobe < 512 ? 512 : 4ull * nprobe;
    if (want > static_cast<uint64_t>(kIvfUnitsPerQuery)) want = kIvfUnitsPerQuery;
    uint64_t unit = (total + (want - nprobe) - 1) / (want - nprobe);
    unit = (unit + 63) / 64 * 64;
    if (unit < 256) unit = 256;
    uint64_t part = (total + parts - 1) / parts;
    part = (part + 255) / 256 * 256;
    if (part < min_part) part = min_part;
    // exclusive prefix sums of the units and parts per list, two lists per thread
    uint32_t nu[2], ni[2], incl[2];
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        const int s = 2 * tid + z;
        nu[z] = s < nprobe ? static_cast<uint32_t>((lsize[s] + unit - 1) / unit) : 0u;
        ni[z] = s < nprobe ? static_cast<uint32_t>((lsize[s] + part - 1) / part) : 0u;
    }
    incl[0] = nu[0] + nu[1];
    incl[1] = ni[0] + ni[1];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t a = __shfl(incl[0], lane >= o ? lane - o : lane), b = __shfl(incl[1], lane >= o ? lane - o : lane);
        if (lane >= o) { incl[0] += a; incl[1] += b; }
    }
    if (lane == 63) { wsum[0][wave] = incl[0]; wsum[1][wave] = incl[1]; }
    __syncthreads();
    for (int w = 0; w < wave; ++w) { incl[0] += wsum[0][w]; incl[1] += wsum[1][w]; }
#pragma unroll
    for (int z = 1; z >= 0; --z) {
        incl[0] -= nu[z];
        incl[1] -= ni[z];
        if (2 * tid + z < nprobe) { ubase[2 * tid + z] = incl[0]; pbase[2 * tid + z] = incl[1]; }
    }
    const uint32_t all_units = wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3];
    const uint32_t all_parts = wsum[1][0] + wsum[1][1] + wsum[1][2] + wsum[1][3];
    if (tid == 0) {
        ubase[nprobe] = all_units;
        pbase[nprobe] = all_parts;
        nunits[q] = all_units;
        part_of[q] = static_cast<uint32_t>(part);
        count[q] = static_cast<uint32_t>(total < r ? total : r);
        probed[q] = static_cast<uint32_t>(total < 0xFFFFFFFFull ? total : 0xFFFFFFFFull);     // codes in the probed lists
        if (!bins) s_base = atomicAdd(cursor, all_parts);
    }
    __syncthreads();
    // the list that holds entry x of a prefix array: the last s with base[s] <= x
    auto list_of = [&](const uint32_t *base, uint32_t x) {
        uint32_t lo = 0, hi = static_cast<uint32_t>(nprobe);
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (base[mid] <= x) lo = mid; else hi = mid;
        }
        return lo;
    };
    for (uint32_t x = tid; x < all_units; x += 256) {
        const uint32_t s = list_of(ubase, x);
        const uint64_t first = static_cast<uint64_t>(x - ubase[s]) * unit;
        units[static_cast<size_t>(q) * kIvfUnitsPerQuery + x] =
            IvfUnit{lbeg[s] + first, static_cast<uint32_t>(min(unit, lsize[s] - first)), static_cast<uint32_t>(key[s])};
    }
    if (bins) {
        for (uint32_t s = tid; s < static_cast<uint32_t>(nprobe); s += 256) {
            const uint32_t n = pbase[s + 1] - pbase[s];
            if (n) rank[static_cast<size_t>(q) * nprobe + static_cast<uint32_t>(key[s])] =
                atomicAdd(&bins[ivf_bin_of(static_cast<uint32_t>(key[s] >> 32), nlist, nbins)], n);
        }
    } else {
        for (uint32_t x = tid; x < all_parts; x += 256) {
            const uint32_t s = list_of(pbase, x);
            const uint64_t first = static_cast<uint64_t>(x - pbase[s]) * part;
            items[s_base + x] = IvfUnit{lbeg[s] + first, static_cast<uint32_t>(min(part, lsize[s] - first)),
                                        static_cast<uint32_t>(q) * nprobe + static_cast<uint32_t>(key[s])};
        }
    }
}

// bins[b]: number of parts in bin b -> place of its first part (in any order of 256-bin blocks).
__global__ __launch_bounds__(256) void ivf_bin_base_kernel(uint32_t *__restrict__ bins, uint32_t nbins, uint32_t *__restrict__ cursor)
{
    __shared__ uint32_t wsum[4], s_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t b = blockIdx.x * 256 + tid;
    const uint32_t c = b < nbins ? bins[b] : 0u;
    uint32_t incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t other = __shfl(incl, lane >= o ? lane - o : lane);
        if (lane >= o) incl += other;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    if (tid == 0) s_base = atomicAdd(cursor, wsum[0] + wsum[1] + wsum[2] + wsum[3]);
    for (int w = 0; w < wave; ++w) incl += wsum[w];
    __syncthreads();
    if (b < nbins) bins[b] = s_base + incl - c;
}

// The parts of (query, probed list) pair e, at the places drawn for them; a thread per pair.
__global__ __launch_bounds__(256) void ivf_parts_kernel(const int32_t *__restrict__ probe, uint32_t npairs, uint32_t nprobe,
                                                       const int64_t *__restrict__ offsets, uint32_t nlist,
                                                       const uint32_t *__restrict__ bins, uint32_t nbins, const uint32_t *__restrict__ rank,
                                                       const uint32_t *__restrict__ part_of, IvfUnit *__restrict__ items)
{
    const uint32_t e = blockIdx.x * 256 + threadIdx.x;
    if (e >= npairs) return;
    const uint32_t l = static_cast<uint32_t>(probe[e]), part = part_of[e / nprobe];
    const uint64_t lo = static_cast<uint64_t>(offsets[l]), size = static_cast<uint64_t>(offsets[l + 1]) - lo;
    if (size == 0) return;
    IvfUnit *out = items + bins[ivf_bin_of(l, nlist, nbins)] + rank[e];
    for (uint64_t first = 0; first < size; first += part)
        *out++ = IvfUnit{lo + first, static_cast<uint32_t>(min(static_cast<uint64_t>(part), size - first)), e};
}

enum IvfMode { kIvfHist = 0, kIvfTieCount = 1, kIvfCollect = 2 };
constexpr int ivf_ahead(int m) { return m <= 16 ? 4 : 2; }      // 64-code groups whose codes a wavefront loads together (four of m = 32 do not fit the registers)

constexpr int kIvfRedoLine = 32;             // words from one count of the redo to the next
constexpr int kIvfRedoWaves = 16;

// One (query, unit) by one wavefront, which keeps the
// 8-bit tables of its (query, list) in its own LDS slot and walks the unit 64 codes at a time; nothing in it waits for another wavefront.
// CodeT: uint16_t (the codes as stored) or uint8_t (their low-byte plane).  What a pass leaves for the next, in the same launch, goes through
// device-scope atomics, stores and loads.
template <int M, int MODE, typename CodeT>
__device__ inline void ivf_scan_unit(int q, uint32_t u, const CodeT *__restrict__ codes, const IvfUnit *__restrict__ units,
                                     const uint32_t *__restrict__ nunits, const uint8_t *__restrict__ qtab,
                                     int nprobe, uint32_t r,
                                     const uint32_t *__restrict__ thr, uint32_t *__restrict__ tie,
                                     uint32_t *__restrict__ counter, uint64_t *__restrict__ keys)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint8_t *tab = smem + wave * (M * 256);                                      // [M][256]
    uint32_t *lhist = reinterpret_cast<uint32_t *>(smem + kIvfRedoWaves * M * 256);   // kIvfHist: the workgroup's
    const bool active = u < nunits[q];
    IvfUnit un{0, 0, 0};
    if (active) un = units[static_cast<size_t>(q) * kIvfUnitsPerQuery + u];
    if (active) {
        const uint4 *src = reinterpret_cast<const uint4 *>(qtab + (static_cast<size_t>(q) * nprobe + un.p) * M * 256);
        uint4 *dst = reinterpret_cast<uint4 *>(tab);
        for (int v = lane; v < M * 256 / 16; v += 64) dst[v] = src[v];
    }
    // the tables are this wavefront's own: its lanes run in lockstep, the fences order the LDS accesses
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (!active) return;

    uint32_t T = 0, aux = 0;
    if (MODE != kIvfHist) {
        T = __hip_atomic_load(&thr[2 * q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (MODE == kIvfCollect) aux = __hip_atomic_load(&tie[static_cast<size_t>(q) * kIvfUnitsPerQuery + u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // The unit is walked 64 codes at a time, in id order; the codes of AHEAD such groups are loaded
    // together, so that one memory latency covers all of them.
    constexpr int AHEAD = ivf_ahead(M);
    for (uint32_t base0 = 0; base0 < un.count; base0 += 64 * AHEAD) {
        uint32_t low[AHEAD][M];
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) {
            const uint32_t k = base0 + g * 64 + lane;
            if (k < un.count) {
                load_low_bytes<M>(codes, un.begin + k, low[g]);
            } else {
#pragma unroll
                for (int j = 0; j < M; ++j) low[g][j] = 0;
            }
        }
#pragma unroll
      for (int g = 0; g < AHEAD; ++g) {
        const uint32_t base = base0 + g * 64;
        if (base >= un.count) break;                                  // uniform
        const uint32_t k = base + lane;
        const bool live = k < un.count;
        const uint64_t id = un.begin + k;
        uint32_t s = 0;
#pragma unroll
        for (int j = 0; j < M; ++j) s += tab[j * 256 + low[g][j]];
        const uint32_t qd = min(s, 255u);
        if (MODE == kIvfHist) {
            if (live) atomicAdd(&lhist[qd], 1u);
        } else if (MODE == kIvfTieCount) {
            aux += __popcll(__ballot(live && qd == T));
        } else {
            const bool below = live && qd < T;
            const bool tied = live && qd == T;
            const uint64_t tied_mask = __ballot(tied);
            bool take = below;
            if (tied_mask) {
                const uint32_t rank = __popcll(tied_mask & ((1ull << lane) - 1ull));
                take = below || (tied && rank < aux);
                const uint32_t n_tied = __popcll(tied_mask);
                aux = aux > n_tied ? aux - n_tied : 0u;
            }
            const uint64_t take_mask = __ballot(take);
            if (take_mask) {
                uint32_t slot0 = 0;
                if (lane == 0) slot0 = atomicAdd(&counter[q], static_cast<uint32_t>(__popcll(take_mask)));
                slot0 = __shfl(slot0, 0, kWave);
                if (take) {
                    const uint32_t slot = slot0 + __popcll(take_mask & ((1ull << lane) - 1ull));
                    if (slot < r)
                        __hip_atomic_store(&keys[static_cast<size_t>(q) * r + slot], make_key(qd, static_cast<uint32_t>(id)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
      }
    }
    if (MODE == kIvfTieCount) {
        if (lane == 0) __hip_atomic_store(&tie[static_cast<size_t>(q) * kIvfUnitsPerQuery + u], aux, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The three passes and the sort for the flagged queries qlist[0 .. *nflag), in one launch, as for the flat scan (scan_redo_kernel, where the
// waits are explained): the items of a pass are parts of a query's units, handed out in order by one counter.  A query has as many parts, units
// that far apart, as bring a pass to 512 items, and at most 256 (of 1024 units four wavefronts of a workgroup have one then, and every CU has
// work): the counter's atomics follow each other at 15 ns, and with 11 queries over 31M codes (800 000 a query) and few of them flagged 64
// parts and 512 cost 20 and 30 us more than 256.
// What the items of the next pass wait for is a word away from the count that the workgroups of this one add to: their loads of that line
// queued the adds (106 -> 100 us there).  A workgroup adds its counts to the query's histogram once, from its own in LDS.
// done: [3][nq] items that are done, of each pass, a memory line apart (side by side their returning atomics queue for one line), and beside
// the last pass's count the two words that the first two passes set; ticket: the counter; all at zero on entry.  (Not this call's own: given up,
// redo_wait.h; queries that were not finished get no candidates then.)

template <int M, typename CodeT>
__global__ __launch_bounds__(64 * kIvfRedoWaves) void ivf_redo_kernel(const CodeT *__restrict__ codes, const IvfUnit *__restrict__ units,
                                                      const uint32_t *__restrict__ nunits, const uint8_t *__restrict__ qtab, int nprobe, int nq, uint32_t r,
                                                      const uint32_t *__restrict__ nflag, const int *__restrict__ qlist, uint32_t *hist, uint32_t *thr, uint32_t *tie,
                                                      uint32_t *counter, uint64_t *keys, uint32_t *done, unsigned long long *ticket, uint32_t n_pow2, int use_lds,
                                                      uint64_t *__restrict__ spill, uint32_t *__restrict__ cand_id, uint8_t *__restrict__ cand_qd)
{
    const uint32_t nf = *nflag;
    if (nf == 0) return;
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ unsigned long long s_item;
    __shared__ uint32_t s_last, s_there;
    uint32_t *lhist = reinterpret_cast<uint32_t *>(smem + kIvfRedoWaves * M * 256);
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t parts = min(256u, max(1u, 512u / nf));             // ... of a query
    const uint64_t per = static_cast<uint64_t>(nf) * parts, all = 3 * per + nf;
    auto count_of = [&](uint32_t pass, uint32_t f) { return done + (static_cast<size_t>(pass) * nq + f) * kIvfRedoLine; };
    auto word_of = [&](uint32_t pass, uint32_t f) { return count_of(2, f) + 1 + pass; };
    auto wait_for = [&](const uint32_t *count, uint32_t n) {
        if (tid == 0) {
            s_there = wait_until([count] { return __hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                                 [] { __builtin_amdgcn_s_sleep(16); }, n, kRedoPatience);
            if (!s_there) atomicOr(ticket, kRedoGivenUp);
        }
        __syncthreads();
        return s_there != 0;
    };
    auto finished = [&](uint32_t *count) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(count, 1u) == parts - 1;
        __syncthreads();
        return s_last != 0;
    };
    auto ready = [&](uint32_t *word) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) atomicAdd(word, 1u);
    };
    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(ticket, 1ull);
        __syncthreads();
        const uint64_t item = s_item & ~kRedoGivenUp;
        const bool given_up = s_item != item;
        if (item >= all) return;                                      // uniform
        if (item < 3 * per) {
            if (given_up) continue;                                   // uniform
            const uint32_t pass = static_cast<uint32_t>(item / per), in_pass = static_cast<uint32_t>(item % per), f = in_pass / parts, part = in_pass % parts;
            const int q = qlist[f];
            auto walk = [&](auto mode) {
                const uint32_t n = nunits[q];
                for (uint32_t u = part + wave * parts; u < n; u += kIvfRedoWaves * parts) {
                    ivf_scan_unit<M, decltype(mode)::value, CodeT>(q, u, codes, units, nunits, qtab, nprobe, r, thr, tie, counter, keys);
                    // the next unit's tables overwrite this one's: every lane is done with them
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                }
            };
            if (pass == 0) {
                if (tid < 256) lhist[tid] = 0;
                __syncthreads();
                walk(std::integral_constant<int, kIvfHist>{});
                __syncthreads();
                if (tid < 256 && lhist[tid]) atomicAdd(&hist[static_cast<size_t>(q) * 256 + tid], lhist[tid]);
                if (finished(count_of(0, f))) {                       // uniform
                    if (wave == 0) exact_threshold(hist + static_cast<size_t>(q) * 256, r, thr + 2 * q);
                    ready(word_of(0, f));
                }
            } else if (pass == 1) {
                if (!wait_for(word_of(0, f), 1)) continue;            // uniform
                walk(std::integral_constant<int, kIvfTieCount>{});
                if (finished(count_of(1, f))) {                       // uniform
                    if (wave == 0)
                        tie_quotas(tie + static_cast<size_t>(q) * kIvfUnitsPerQuery, nunits[q],
                                   __hip_atomic_load(&thr[2 * q + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    ready(word_of(1, f));
                }
            } else {
                if (!wait_for(word_of(1, f), 1)) continue;            // uniform
                walk(std::integral_constant<int, kIvfCollect>{});
                finished(count_of(2, f));
            }
            continue;
        }
        const uint32_t f = static_cast<uint32_t>(item - 3 * per);
        const size_t q = qlist[f];
        if (given_up || !wait_for(count_of(2, f), parts)) {           // uniform
            for (uint32_t t = tid; t < r; t += 64 * kIvfRedoWaves) { cand_id[q * r + t] = 0xFFFFFFFFu; cand_qd[q * r + t] = 255; }
            continue;
        }
        uint64_t *a = use_lds ? reinterpret_cast<uint64_t *>(smem) : spill + q * n_pow2;
        for (uint32_t t = tid; t < n_pow2; t += 64 * kIvfRedoWaves)
            a[t] = t < r ? __hip_atomic_load(&keys[q * r + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : ~0ull;
        bitonic_sort(a, n_pow2);
        for (uint32_t t = tid; t < r; t += 64 * kIvfRedoWaves) {
            cand_id[q * r + t] = static_cast<uint32_t>(a[t]);
            cand_qd[q * r + t] = static_cast<uint8_t>(a[t] >> 32);
        }
    }
}

// The same scan in ONE pass over the probed lists (each pass reads every probed code from memory, so passes are what
// the scan costs).  As in the flat single pass, a query has
// a running bucket bound, initialised from the histogram of a sample (the first 1 / kIvfSampleStep of every list) and
// lowered as exact per-bucket counts of appended candidates accumulate; pairs at or below the bound are
// appended to the query's sliced buffer, the exact r are selected afterwards, and a query whose buffer
// overflows (or whose lists hold fewer than r codes) is redone by the three passes above.
//
// One workgroup per part (a run of codes of one list, for one query): the tables are read once per part, and the
// wavefronts walk it together, one set of codes after the other.  The parts are ordered by list, and consecutive ones
// go to the same XCD (workgroup i runs on XCD i mod 8), so that the queries that probe the same list read
// it at about the same time through one second-level cache, while the parts of one query are spread over the whole
// launch.
//
// Candidates are noted in LDS and appended together when the part is done: one returning atomic on the query's cursor
// and one addition per bucket that occurs, instead of one per candidate on the few counters that all of a query's
// candidates share (they serialize in the L2 at 13 to 20 ns each).
// The bound is lowered at these points only; it starts where a few r candidates are expected.
//
// The kernel is bound by the stream of codes, so a wavefront is built around keeping that
// stream in flight: the codes stay in registers as loaded (their low bytes are picked out when they
// are looked up), in two sets of kIvfRawWords words per lane; while one set is processed the loads
// of the next are under way, the first of them issued together with the load of the part's tables.
constexpr int kIvfRawWords = 16;         // registers per lane and set that hold codes in flight

// The bytes of code i as stored, in RW words (a narrower code is zero-extended).
template <int M, typename CodeT, int RW>
__device__ inline void load_raw_code(const CodeT *__restrict__ codes, uint64_t i, uint32_t (&w)[RW])
{
    constexpr int BPC = M * static_cast<int>(sizeof(CodeT));
    const uint8_t *p = reinterpret_cast<const uint8_t *>(codes) + i * BPC;
    if constexpr (BPC >= 16) {
#pragma unroll
        for (int v = 0; v < BPC / 16; ++v) {
            const uint4 x = reinterpret_cast<const uint4 *>(p)[v];
            w[4 * v] = x.x; w[4 * v + 1] = x.y; w[4 * v + 2] = x.z; w[4 * v + 3] = x.w;
        }
    } else if constexpr (BPC == 8) {
        const uint2 x = *reinterpret_cast<const uint2 *>(p);
        w[0] = x.x; w[1] = x.y;
    } else if constexpr (BPC == 4) {
        w[0] = *reinterpret_cast<const uint32_t *>(p);
    } else if constexpr (BPC == 2) {
        w[0] = *reinterpret_cast<const uint16_t *>(p);
    } else {
        w[0] = *p;
    }
}

// Low byte of sub-code j of a code held as loaded (property P1: the derived index is the low 8 bits).
template <typename CodeT, int RW>
__device__ inline uint32_t low_byte_of(const uint32_t (&w)[RW], int j)
{
    if constexpr (sizeof(CodeT) == 2) return (w[j >> 1] >> (16 * (j & 1))) & 255u;
    else return (w[j >> 2] >> (8 * (j & 3))) & 255u;
}

// Codes of one set of a wavefront, from `p` codes behind `begin`; past the end (`hi` codes behind it) the last code is
// read again (a valid address), to be masked by the caller.
template <int M, typename CodeT, int GPB, int RW>
__device__ inline void load_raw_set(const CodeT *__restrict__ codes, uint64_t begin, uint32_t base0, uint32_t hi, uint32_t (&w)[GPB][RW])
{
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int g = 0; g < GPB; ++g) {
        const uint32_t k = base0 + g * 64 + lane;
        load_raw_code<M, CodeT, RW>(codes, begin + (k < hi ? k : hi - 1), w[g]);
    }
}

template <int M, typename CodeT>
struct IvfRaw {
    static constexpr int BPC = M * static_cast<int>(sizeof(CodeT));
    static constexpr int RW = BPC >= 4 ? BPC / 4 : 1;                // words per code
    static constexpr int GPB = RW >= kIvfRawWords ? 1 : kIvfRawWords / RW;   // 64-code groups per set
    static constexpr uint32_t SET = 64 * GPB;
};

template <int M, typename CodeT>
__global__ __launch_bounds__(256) void ivf_scan_parts_kernel(const CodeT *__restrict__ codes, const IvfUnit *__restrict__ items,
                                                            const uint32_t *__restrict__ nitems,
                                                            const uint8_t *__restrict__ qtab, uint32_t nprobe, uint32_t r,
                                                            uint32_t cap, uint32_t upd, Bound *bound,
                                                            uint32_t *count, uint32_t *chist, uint64_t *__restrict__ keys)
{
    constexpr int RW = IvfRaw<M, CodeT>::RW, GPB = IvfRaw<M, CodeT>::GPB;
    constexpr uint32_t SET = IvfRaw<M, CodeT>::SET;
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // consecutive parts on one XCD: each of the eight takes an eighth of the list
    const uint32_t n_all = *nitems, per = (n_all + 7) / 8;
    const uint64_t idx = static_cast<uint64_t>(blockIdx.y) * gridDim.x + blockIdx.x;      // gridDim.x is a multiple of 8
    const uint64_t at = (idx & 7) * per + (idx >> 3);
    if ((idx >> 3) >= per || at >= n_all) return;                // uniform
    const IvfUnit un = items[at];
    const int q = static_cast<int>(un.p / nprobe);
    uint8_t *tab = smem;                                                              // [M][256]
    uint64_t *notes = reinterpret_cast<uint64_t *>(smem + M * 256);                   // [kIvfNotes]
    __shared__ uint32_t s_n, s_first, bhist[256];

    // The wavefronts take the part's sets of codes in turn; a part that has less than a set for each is cut evenly.
    const bool turns = un.count >= 4 * SET;
    const uint32_t strip = turns ? SET : (un.count + 255) / 256 * 64;
    const uint32_t lo = wave * strip, hi = turns ? un.count : min(un.count, lo + strip);
    auto load_bound = [&]() {
        const int t = __hip_atomic_load(&bound[q].t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return t >= 255 ? 0x7fffffff : t;
    };
    // The part's first codes and its tables travel together: the code loads are issued first, the table words
    // follow them and go from their registers straight to LDS.
    uint32_t wa[GPB][RW], wb[GPB][RW];
    if (lo < hi) load_raw_set<M, CodeT, GPB, RW>(codes, un.begin, lo, hi, wa);       // uniform per wavefront
    int T = load_bound();
    {
        constexpr int NTW = M * 256 / 16;                                // 16-byte words of the tables
        const uint4 *src = reinterpret_cast<const uint4 *>(qtab + static_cast<size_t>(un.p) * M * 256);
        uint4 *dst = reinterpret_cast<uint4 *>(tab);
#pragma unroll
        for (int v = 0; v < (NTW + 255) / 256; ++v)
            if (NTW % 256 == 0 || tid + 256 * v < NTW) dst[tid + 256 * v] = src[tid + 256 * v];
    }
    bhist[tid] = 0;
    if (tid == 0) s_n = 0;
    __syncthreads();

    const size_t cell = static_cast<size_t>(q) * kFastSlices + static_cast<uint32_t>(at) % kFastSlices;
    // n keys, the wavefront's lane l holding key l of them, straight to the query's buffer
    auto append = [&](uint64_t key, bool mine, uint32_t rank, uint32_t n) {
        uint32_t first = 0;
        if (lane == 0) first = atomicAdd(&count[cell], n);
        first = __builtin_amdgcn_readfirstlane(first);
        if (mine) {
            if (first + rank < cap) keys[cell * cap + first + rank] = key;
            else atomicMin(&bound[q].t, -1);               // slice full: stop appending, the query is redone
            atomicAdd(&chist[static_cast<size_t>(q) * 256 + static_cast<uint32_t>(key >> 32)], 1u);
        }
        if (first / upd != (first + n) / upd) lower_bound_of(q, r, bound, chist);   // uniform
    };
    auto process = [&](uint32_t base0, const uint32_t (&w)[GPB][RW], int bound) {
#pragma unroll
        for (int g = 0; g < GPB; ++g) {
            const uint32_t base = base0 + g * 64;
            if (base >= hi) break;                                    // uniform
            const uint32_t k = base + lane;
            uint32_t s = 0;
#pragma unroll
            for (int j = 0; j < M; ++j) s += tab[j * 256 + low_byte_of<CodeT, RW>(w[g], j)];
            const uint32_t qd = min(s, 255u);
            const bool h = k < hi && static_cast<int>(qd) <= bound;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(h);
            if (!mask) continue;                                      // uniform
            const uint32_t cnt = __popcll(mask);
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                            __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
            const uint64_t key = make_key(qd, static_cast<uint32_t>(un.begin + k));
            uint32_t pos = 0;
            // (a full buffer's counter is not counted on, so that it cannot wrap)
            if (lane == 0) pos = *static_cast<volatile uint32_t *>(&s_n) < kIvfNotes ? atomicAdd(&s_n, cnt) : kIvfNotes;
            pos = __builtin_amdgcn_readfirstlane(pos);
            const bool noted = pos + rank < kIvfNotes;
            if (h && noted) notes[pos + rank] = key;
            if (pos + cnt > kIvfNotes) {                               // uniform
                const uint32_t fit = pos < kIvfNotes ? kIvfNotes - pos : 0u;
                append(key, h && !noted, rank - fit, cnt - fit);
            }
        }
    };

    // (64-bit positions: a part may be close to 2^32 codes long)
    constexpr uint64_t STEP = 4 * SET;
    for (uint64_t base0 = lo; base0 < hi && T >= 0; base0 += 2 * STEP) {
        int Tn = T;
        if (base0 + STEP < hi) { load_raw_set<M, CodeT, GPB, RW>(codes, un.begin, static_cast<uint32_t>(base0 + STEP), hi, wb); Tn = load_bound(); }
        process(static_cast<uint32_t>(base0), wa, T);
        if (base0 + STEP >= hi) break;
        T = Tn;
        if (base0 + 2 * STEP < hi) { load_raw_set<M, CodeT, GPB, RW>(codes, un.begin, static_cast<uint32_t>(base0 + 2 * STEP), hi, wa); Tn = load_bound(); }
        process(static_cast<uint32_t>(base0 + STEP), wb, T);
        T = Tn;
    }
    __syncthreads();
    const uint32_t n = s_n < kIvfNotes ? s_n : kIvfNotes;
    if (n == 0) return;                                               // uniform
    if (tid == 0) s_first = atomicAdd(&count[cell], n);
    __syncthreads();
    const uint32_t first = s_first;
    if (first + n > cap && tid == 0) atomicMin(&bound[q].t, -1);      // slice full: stop appending, the query is redone
    for (uint32_t x = tid; x < n; x += 256) {
        const uint64_t key = notes[x];
        if (first + x < cap) keys[cell * cap + first + x] = key;
        atomicAdd(&bhist[static_cast<uint32_t>(key >> 32)], 1u);
    }
    __syncthreads();
    if (bhist[tid]) atomicAdd(&chist[static_cast<size_t>(q) * 256 + tid], bhist[tid]);
    if (first / upd != (first + n) / upd) {                           // uniform
        // (the additions of the other wavefronts may still be under way: any snapshot of the counts gives a valid bound)
        if (wave == 0) lower_bound_of(q, r, bound, chist);
    }
}

// The starting bounds: a histogram of the integer distances of the first 1 / step of every probed list, and
// from it the bucket that r of the query's probed codes would reach (starting_bound), by the workgroup that ends the
// query last.  step is kIvfSampleStep, and more where that would be a sample of over 32 K codes, as long as 16 of the r are
// expected in it, and less where it would be one of under 1 K (every list gives one code at least: of short lists of unequal
// length the short ones would give too many, and too low a bound sends the query to the three passes: 1416 queries, 8
// lists of 225 codes: 450 us, now 348).  Grid (nq, rows): the sample is cut into sets of codes, of which every wavefront of the query's takes
// as many (lists differ in length by orders of magnitude: with a wavefront per list the longest one's took 1.7 ms).
// Bound by the latency of fetching a 2 KB table and a few hundred codes per list; a
// workgroup counts in LDS and adds up once.  (As a wavefront per list with a histogram of its own the additions to
// global memory alone were 6 million for 1024 queries x 64 lists: 309 us.)
template <int M>
struct IvfSampleCfg { static constexpr int WAVES = M <= 8 ? 16 : M == 16 ? 8 : 4; };   // tables of at most 32 KB in LDS

template <int M, typename CodeT>
__global__ __launch_bounds__(64 * IvfSampleCfg<M>::WAVES) void ivf_sample_kernel(const CodeT *__restrict__ codes,
                                                            const int64_t *__restrict__ offsets,
                                                            const int32_t *__restrict__ probe, int nprobe,
                                                            const uint8_t *__restrict__ qtab, uint32_t r,
                                                            const uint32_t *__restrict__ probed, uint32_t *__restrict__ shist,
                                                            uint32_t *__restrict__ done, uint32_t cap, Bound *bound)
{
    constexpr int NW = IvfSampleCfg<M>::WAVES, COPIES = 4;
    constexpr int RW = IvfRaw<M, CodeT>::RW, GPB = IvfRaw<M, CodeT>::GPB;
    constexpr uint32_t SET = IvfRaw<M, CodeT>::SET;
    __shared__ __align__(16) uint8_t tabs[NW][M * 256];
    __shared__ uint32_t lhist[COPIES][256];
    __shared__ uint64_t lbeg[kIvfMaxProbe];
    __shared__ uint32_t lpart[kIvfMaxProbe], sbase[kIvfMaxProbe + 1];      // codes of a list in the sample; its first set
    __shared__ uint32_t s_last;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6), np = static_cast<uint32_t>(nprobe);
    for (int v = tid; v < COPIES * 256; v += 64 * NW) (&lhist[0][0])[v] = 0;
    uint32_t step = kIvfSampleStep;
    while (probed[q] / step > 32768 && r / step >= 32) step *= 2;
    while (probed[q] / step < 1024 && step > 1) step /= 2;
    for (uint32_t p = tid; p < np; p += 64 * NW) {
        const int l = probe[static_cast<size_t>(q) * np + p];
        lbeg[p] = static_cast<uint64_t>(offsets[l]);
        lpart[p] = static_cast<uint32_t>((static_cast<uint64_t>(offsets[l + 1]) - lbeg[p] + step - 1) / step);
    }
    __syncthreads();
    if (wave == 0) {                                           // exclusive prefix sums of the sets per list
        uint32_t run = 0;
        for (uint32_t p0 = 0; p0 < np; p0 += 64) {
            const uint32_t n = p0 + lane < np ? (lpart[p0 + lane] + SET - 1) / SET : 0u;
            uint32_t incl = n;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t other = __shfl(incl, lane >= o ? lane - o : lane);
                if (lane >= o) incl += other;
            }
            if (p0 + lane < np) sbase[p0 + lane] = run + incl - n;
            run += __shfl(incl, 63);
        }
        if (lane == 0) sbase[np] = run;
    }
    __syncthreads();
    const uint32_t nsets = sbase[np], w = blockIdx.y * NW + wave, all = gridDim.y * NW;
    uint32_t x = static_cast<uint32_t>(static_cast<uint64_t>(nsets) * w / all);             // this wavefront's sets: [x, end)
    const uint32_t end = static_cast<uint32_t>(static_cast<uint64_t>(nsets) * (w + 1) / all);
    uint8_t *tab = tabs[wave];
    uint32_t *hist = lhist[wave % COPIES];
    if (x < end) {                                                     // uniform per wavefront
        uint32_t p = 0;
        for (uint32_t hi = np; hi - p > 1;) {                          // the last list whose first set is at or before x
            const uint32_t mid = (p + hi) >> 1;
            if (sbase[mid] <= x) p = mid; else hi = mid;
        }
        bool fresh = true;
        uint32_t wa[GPB][RW];
        for (; x < end; ++x) {
            while (sbase[p + 1] <= x) { ++p; fresh = true; }           // (lists without a set are passed over)
            const uint32_t base0 = (x - sbase[p]) * SET, hi = lpart[p];
            load_raw_set<M, CodeT, GPB, RW>(codes, lbeg[p], base0, hi, wa);
            if (fresh) {
                fresh = false;
                constexpr int NTW = M * 256 / 16;                                // 16-byte words of the tables
                const uint4 *src = reinterpret_cast<const uint4 *>(qtab + (static_cast<size_t>(q) * np + p) * M * 256);
                uint4 *dst = reinterpret_cast<uint4 *>(tab);
                // the wavefront's own tables: its lanes are done with the previous list's, the fences order the accesses
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
                for (int v = 0; v < (NTW + 63) / 64; ++v)
                    if (NTW % 64 == 0 || lane + 64 * v < NTW) dst[lane + 64 * v] = src[lane + 64 * v];
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            }
#pragma unroll
            for (int g = 0; g < GPB; ++g) {
                uint32_t s = 0;
#pragma unroll
                for (int j = 0; j < M; ++j) s += tab[j * 256 + low_byte_of<CodeT, RW>(wa[g], j)];
                if (base0 + g * 64 + lane < hi) atomicAdd(&hist[min(s, 255u)], 1u);
            }
        }
    }
    __syncthreads();
    for (int v = tid; v < 256; v += 64 * NW) {
        uint32_t c = 0;
#pragma unroll
        for (int z = 0; z < COPIES; ++z) c += lhist[z][v];
        if (c) atomicAdd(&shist[static_cast<size_t>(q) * 256 + v], c);
    }
    // every addition is in place before this workgroup's count is (device-scope atomics: their completion is all there
    // is to wait for)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(&done[q], 1u) == gridDim.y - 1;
    __syncthreads();
    // A query with so many ties at the starting bucket that they would overflow its buffer is left to the three passes, at
    // seven eighths of the buffer (the slices do not fill evenly).  The buffer is the measure, not r: below r = 512 it holds more
    // than 32 r (255 queries, r = 3, two lists of 1400 codes: 168 us, 250 with every query left to the three passes).
    if (s_last && wave == 0) starting_bound<false>(shist + static_cast<size_t>(q) * 256, r, probed[q], kCrowdedSkip, bound + q, 0.875f * kFastSlices * static_cast<float>(cap));
}

// ------------------------------------------------------------------------------------------------
// Refine step: Eq. 3 on residuals, double precision, then top-k.  One workgroup per query.
// ------------------------------------------------------------------------------------------------
template <int M>
__global__ __launch_bounds__(1024) void ivf_refine_kernel(const float *__restrict__ queries, const float *__restrict__ coarse,
                                                         const float *__restrict__ cb, int dsub,
                                                         const uint16_t *__restrict__ codes, const int64_t *__restrict__ offsets,
                                                         const int32_t *__restrict__ probe, int nprobe,
                                                         const uint32_t *__restrict__ cand_id, uint32_t r, uint32_t k,
                                                         uint32_t n_pow2, int use_lds, uint64_t *__restrict__ spill,
                                                         uint32_t *__restrict__ ids, float *__restrict__ dist)
{
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ uint32_t lbeg[kIvfMaxProbe], lend[kIvfMaxProbe];   // ids are 32-bit, so are list bounds
    __shared__ int lst[kIvfMaxProbe];
    const int q = blockIdx.x;
    const int D = M * dsub;
    for (int p = threadIdx.x; p < nprobe; p += blockDim.x) {
        const int l = probe[static_cast<size_t>(q) * nprobe + p];
        lst[p] = l;
        lbeg[p] = static_cast<uint32_t>(offsets[l]);
        lend[p] = static_cast<uint32_t>(offsets[l + 1]);
    }
    __syncthreads();
    uint64_t *a = use_lds ? reinterpret_cast<uint64_t *>(smem) : spill + static_cast<size_t>(q) * n_pow2;
    const float *y = queries + static_cast<size_t>(q) * D;
    // One lane per (candidate, sub-quantizer): the M lanes of a candidate are neighbours in a wavefront.  They
    // share the search for the candidate's list, each computes the squared distance of its own sub-vector
    // (components in ascending order), and the sums are added in ascending j, as a single thread would.
    {
        const uint32_t lane = threadIdx.x & 63u;
        const int j = static_cast<int>(threadIdx.x % M);
        const bool vec4 = (dsub & 3) == 0;
        for (uint32_t base = 0; base < n_pow2; base += blockDim.x / M) {      // uniform trip count
            const uint32_t t = base + threadIdx.x / M;
            uint32_t id = 0xFFFFFFFFu;
            if (t < r) id = cand_id[static_cast<size_t>(q) * r + t];
            int p = -1;                                                      // pad slots (id 0xFFFFFFFF) belong to no probed list
            for (int z = j; z < nprobe; z += M)
                if (id >= lbeg[z] && id < lend[z]) p = z;                    // the lists are disjoint: at most one
#pragma unroll
            for (int off = 1; off < M; off <<= 1) p = max(p, __shfl_xor(p, off));
            double dj = 0.0;
            if (p >= 0) {
                const float *cl = coarse + static_cast<size_t>(lst[p]) * D + j * dsub;
                const float *yj = y + j * dsub;
                const float *cen = cb + (static_cast<size_t>(j) * kFullSize + codes[static_cast<size_t>(id) * M + j]) * dsub;
                if (vec4) {
                    for (int tt = 0; tt < dsub; tt += 4) {
                        const float4 yv = *reinterpret_cast<const float4 *>(yj + tt);
                        const float4 lv = *reinterpret_cast<const float4 *>(cl + tt);
                        const float4 cv = *reinterpret_cast<const float4 *>(cen + tt);
                        double diff = (static_cast<double>(yv.x) - static_cast<double>(lv.x)) - static_cast<double>(cv.x);
                        dj += diff * diff;
                        diff = (static_cast<double>(yv.y) - static_cast<double>(lv.y)) - static_cast<double>(cv.y);
                        dj += diff * diff;
                        diff = (static_cast<double>(yv.z) - static_cast<double>(lv.z)) - static_cast<double>(cv.z);
                        dj += diff * diff;
                        diff = (static_cast<double>(yv.w) - static_cast<double>(lv.w)) - static_cast<double>(cv.w);
                        dj += diff * diff;
                    }
                } else {
                    for (int tt = 0; tt < dsub; ++tt) {
                        const double diff = (static_cast<double>(yj[tt]) - static_cast<double>(cl[tt])) - static_cast<double>(cen[tt]);
                        dj += diff * diff;
                    }
                }
            }
            double d = __shfl(dj, static_cast<int>(lane - j));
#pragma unroll
            for (int jj = 1; jj < M; ++jj) d += __shfl(dj, static_cast<int>(lane - j + jj));
            if (j == 0 && t < n_pow2) a[t] = p >= 0 ? make_key(__float_as_uint(static_cast<float>(d)), id) : ~0ull;
        }
    }
    bitonic_sort(a, n_pow2);
    for (uint32_t t = threadIdx.x; t < k; t += blockDim.x) {
        const uint64_t key = a[t];
        ids[static_cast<size_t>(q) * k + t] = static_cast<uint32_t>(key);
        dist[static_cast<size_t>(q) * k + t] = (key == ~0ull) ? INFINITY : __uint_as_float(static_cast<uint32_t>(key >> 32));
    }
}

// The same distances as keys in memory, by 256 lanes to a workgroup and one (candidate, sub-quantizer) to a lane: for batches that
// leave most of the chip idle with a workgroup per query.  The selection is a kernel of its own.  A chain of loads (id, code,
// row): 4 us for one query with r = 1000 and 9 for the selection, where a workgroup that also sorts took 41.
template <int M>
__global__ __launch_bounds__(256) void ivf_refine_keys_kernel(const float *__restrict__ queries, const float *__restrict__ coarse,
                                                              const float *__restrict__ cb, int dsub, const uint16_t *__restrict__ codes,
                                                              const int64_t *__restrict__ offsets, const int32_t *__restrict__ probe,
                                                              int nprobe, const uint32_t *__restrict__ cand_id, uint32_t r,
                                                              uint64_t *__restrict__ keys)
{
    __shared__ uint32_t lbeg[kIvfMaxProbe], lend[kIvfMaxProbe];   // ids are 32-bit, so are list bounds
    __shared__ int lst[kIvfMaxProbe];
    const int q = blockIdx.y;
    const int D = M * dsub;
    const uint32_t lane = threadIdx.x & 63u;
    const int j = static_cast<int>(threadIdx.x % M);
    const uint32_t t = blockIdx.x * (256 / M) + threadIdx.x / M;
    const uint32_t id = t < r ? cand_id[static_cast<size_t>(q) * r + t] : 0xFFFFFFFFu;
    for (int p = threadIdx.x; p < nprobe; p += 256) {
        const int l = probe[static_cast<size_t>(q) * nprobe + p];
        lst[p] = l;
        lbeg[p] = static_cast<uint32_t>(offsets[l]);
        lend[p] = static_cast<uint32_t>(offsets[l + 1]);
    }
    __syncthreads();
    int p = -1;                                                   // pad slots (id 0xFFFFFFFF) belong to no probed list
    for (int z = j; z < nprobe; z += M)
        if (id >= lbeg[z] && id < lend[z]) p = z;                 // the lists are disjoint: at most one
#pragma unroll
    for (int off = 1; off < M; off <<= 1) p = max(p, __shfl_xor(p, off));
    double dj = 0.0;
    if (p >= 0) {
        const float *yj = queries + static_cast<size_t>(q) * D + j * dsub;
        const float *cl = coarse + static_cast<size_t>(lst[p]) * D + j * dsub;
        const float *cen = cb + (static_cast<size_t>(j) * kFullSize + codes[static_cast<size_t>(id) * M + j]) * dsub;
        auto add = [&](float y, float l, float c) {
            const double diff = (static_cast<double>(y) - static_cast<double>(l)) - static_cast<double>(c);
            dj += diff * diff;
        };
        if ((dsub & 3) == 0) {
#pragma unroll 4
            for (int tt = 0; tt < dsub; tt += 4) {
                const float4 yv = *reinterpret_cast<const float4 *>(yj + tt);
                const float4 lv = *reinterpret_cast<const float4 *>(cl + tt);
                const float4 cv = *reinterpret_cast<const float4 *>(cen + tt);
                add(yv.x, lv.x, cv.x);
                add(yv.y, lv.y, cv.y);
                add(yv.z, lv.z, cv.z);
                add(yv.w, lv.w, cv.w);
            }
        } else {
            for (int tt = 0; tt < dsub; ++tt) add(yj[tt], cl[tt], cen[tt]);
        }
    }
    double d = __shfl(dj, static_cast<int>(lane - j));
#pragma unroll
    for (int jj = 1; jj < M; ++jj) d += __shfl(dj, static_cast<int>(lane - j + jj));
    if (j == 0 && t < r) keys[static_cast<size_t>(q) * r + t] = p >= 0 ? make_key(__float_as_uint(static_cast<float>(d)), id) : ~0ull;
}

// ------------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------------
struct IvfScanPlan {
    size_t off_hist, off_thr, off_counter, off_nunits, zero_bytes, off_tie, off_units, off_keys, off_spill, total;
    // single pass: sample histogram, cursors, appended histogram (cleared with the rest); bounds, flags, buffers
    size_t off_shist, off_fcount, off_chist, off_bound, off_flags, off_fkeys, off_fsort, off_probed;
    // its parts: bins of list ids, cursor, finished sample workgroups (cleared with the rest); places, lengths, records
    size_t off_bins, off_cursor, off_done, off_redo, off_rank, off_part, off_items, off_qlist;
    bool order;              // parts ordered by list ...
    uint32_t nbins;          // ... in so many bins
    uint32_t parts;          // parts per query, about (and one more per probed list at most) ...
    uint32_t min_part;       // ... of no fewer codes than this
    uint32_t cap, upd, sortcap;
};

static IvfScanPlan plan_ivf_scan(int nq, uint32_t r)
{
    IvfScanPlan p{};
    const size_t Q = static_cast<size_t>(nq);
    size_t off = 0;
    p.off_hist = off;    off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
    p.off_thr = off;     off = align_up(off + sizeof(uint32_t) * 2 * Q, 256);
    p.off_counter = off; off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_nunits = off;  off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_tie = off;     off = align_up(off + sizeof(uint32_t) * Q * kIvfUnitsPerQuery, 256);
    p.off_shist = off;   off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
    p.off_fcount = off;  off = align_up(off + sizeof(uint32_t) * Q * kFastSlices, 256);
    p.off_chist = off;   off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
    // Parts: at least 128 per query, and 4096 in all, for 2048 resident workgroups.  They are ordered by list (two short launches more) where
    // there are queries enough to share lists or to crowd one another's cursors.
    p.parts = nq >= 32 ? 128u : 4096u / static_cast<uint32_t>(nq < 2 ? 2 : nq);
    // (a part reads tables of 256 bytes per sub-quantizer; where queries are many enough parts are left with longer ones:
    // 1040 queries, 5 lists of 11000 codes of 16: 463 us with parts of 512 codes, 418 with 1024)
    p.min_part = nq >= 256 ? 2 * kIvfMinPart : kIvfMinPart;
    p.order = nq > 4;
    p.nbins = Q * 4096 < kIvfBins ? static_cast<uint32_t>(Q) * 4096 : kIvfBins;
    p.off_cursor = off;  off = align_up(off + sizeof(uint32_t), 256);             // (two words on: the uint64 counter that hands out the redo's items)
    p.off_done = off;    off = align_up(off + sizeof(uint32_t) * (Q + 1), 256);
    const size_t redo_bytes = align_up(sizeof(uint32_t) * 3 * kIvfRedoLine * Q, 256);
    p.off_redo = off;    off += redo_bytes;
    p.off_bins = off;    off = align_up(off + (p.order ? sizeof(uint32_t) * p.nbins : 0), 256);
    p.zero_bytes = off;  // everything above is cleared together
    p.off_rank = off;    off = align_up(off + (p.order ? sizeof(uint32_t) * Q * kIvfMaxProbe : 0), 256);
    p.off_part = off;    off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_qlist = off;   off = align_up(off + sizeof(int) * Q, 256);
    p.off_items = off;   off = align_up(off + sizeof(IvfUnit) * Q * (p.parts + kIvfMaxProbe), 256);
    p.off_units = off;   off = align_up(off + sizeof(IvfUnit) * Q * kIvfUnitsPerQuery, 256);
    p.off_keys = off;    off = align_up(off + sizeof(uint64_t) * Q * r, 256);
    p.off_spill = off;
    if (next_pow2(r) > kSortLdsKeys) off = align_up(off + sizeof(uint64_t) * Q * next_pow2(r), 256);
    // Per slice: 32 r entries per query in all (16384 where r is smaller), less what the parts' arrays and the redo's counters take, which came later
    // and make the workspace no larger than it was
    p.cap = 2 * r < 1024 ? 1024 : 2 * r;
    {
        const size_t parts_bytes = redo_bytes + (p.order ? sizeof(uint32_t) * (p.nbins + Q * kIvfMaxProbe) : 0) + sizeof(IvfUnit) * Q * (p.parts + kIvfMaxProbe);
        const size_t slices_bytes = sizeof(uint64_t) * Q * kFastSlices;
        p.cap -= static_cast<uint32_t>((parts_bytes + slices_bytes - 1) / slices_bytes);     // (at most 325 of 1024 and more)
    }
    p.upd = r / 16 < 16 ? 16 : r / 16;                   // appends to one slice between bound updates
    p.sortcap = next_pow2(2 * r) < kSortLdsKeys ? kSortLdsKeys : next_pow2(2 * r);
    p.off_bound = off;    off = align_up(off + sizeof(Bound) * Q, 256);
    p.off_flags = off;   off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_probed = off;  off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_fkeys = off;   off = align_up(off + sizeof(uint64_t) * Q * kFastSlices * p.cap, 256);
    p.off_fsort = off;
    if (p.sortcap > kSortLdsKeys) off = align_up(off + sizeof(uint64_t) * Q * p.sortcap, 256);
    p.total = off;
    return p;
}

template <int M, typename CodeT>
static int ivf_scan_m(const CodeT *codes, const int64_t *offsets, int nlist, const int32_t *probe, int nprobe,
                      const uint8_t *qtab, int nq, uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, uint32_t *count,
                      uint8_t *base, hipStream_t st)
{
    const IvfScanPlan p = plan_ivf_scan(nq, r);
    uint32_t *hist = reinterpret_cast<uint32_t *>(base + p.off_hist);
    uint32_t *thr = reinterpret_cast<uint32_t *>(base + p.off_thr);
    uint32_t *counter = reinterpret_cast<uint32_t *>(base + p.off_counter);
    uint32_t *nunits = reinterpret_cast<uint32_t *>(base + p.off_nunits);
    uint32_t *tie = reinterpret_cast<uint32_t *>(base + p.off_tie);
    IvfUnit *units = reinterpret_cast<IvfUnit *>(base + p.off_units);
    uint64_t *keys = reinterpret_cast<uint64_t *>(base + p.off_keys);
    uint64_t *spill = reinterpret_cast<uint64_t *>(base + p.off_spill);
    // counters to zero; unused slots of the keys read as padding
    int rc = launch_zero_and_fill(reinterpret_cast<uint64_t *>(base), p.zero_bytes / 8, keys, static_cast<size_t>(nq) * r, ~0ull, st);
    if (rc) return rc;
    uint32_t *probed = reinterpret_cast<uint32_t *>(base + p.off_probed);
    uint32_t *bins = p.order ? reinterpret_cast<uint32_t *>(base + p.off_bins) : nullptr;
    uint32_t *cursor = reinterpret_cast<uint32_t *>(base + p.off_cursor);
    uint32_t *done = reinterpret_cast<uint32_t *>(base + p.off_done);      // [nq], and behind them the number of flagged queries
    uint32_t *rank = reinterpret_cast<uint32_t *>(base + p.off_rank);
    uint32_t *part_of = reinterpret_cast<uint32_t *>(base + p.off_part);
    IvfUnit *items = reinterpret_cast<IvfUnit *>(base + p.off_items);
    DCPQ_LAUNCH(kStageIvf, st, ivf_plan_kernel, dim3(nq), dim3(256), 0, probe, nprobe, offsets, static_cast<uint32_t>(nlist), r,
                p.parts, p.min_part, units, nunits, count, probed, part_of, bins, p.nbins, rank, cursor, items);
    DCPQ_CHECK_LAUNCH("ivf_plan_kernel");
    if (p.order) {
        const uint32_t nbins = static_cast<uint32_t>(nlist) < p.nbins ? static_cast<uint32_t>(nlist) : p.nbins;
        const uint32_t npairs = static_cast<uint32_t>(nq) * static_cast<uint32_t>(nprobe);
        DCPQ_LAUNCH(kStageIvf, st, ivf_bin_base_kernel, dim3((nbins + 255) / 256), dim3(256), 0, bins, nbins, cursor);
        DCPQ_CHECK_LAUNCH("ivf_bin_base_kernel");
        DCPQ_LAUNCH(kStageIvf, st, ivf_parts_kernel, dim3((npairs + 255) / 256), dim3(256), 0, probe, npairs,
                    static_cast<uint32_t>(nprobe), offsets, static_cast<uint32_t>(nlist), bins, p.nbins, rank, part_of, items);
        DCPQ_CHECK_LAUNCH("ivf_parts_kernel");
    }
    uint32_t *shist = reinterpret_cast<uint32_t *>(base + p.off_shist);
    uint32_t *fcount = reinterpret_cast<uint32_t *>(base + p.off_fcount);
    uint32_t *chist = reinterpret_cast<uint32_t *>(base + p.off_chist);
    Bound *bound = reinterpret_cast<Bound *>(base + p.off_bound);
    uint32_t *flags = reinterpret_cast<uint32_t *>(base + p.off_flags);
    uint64_t *fkeys = reinterpret_cast<uint64_t *>(base + p.off_fkeys);
    uint64_t *fsort = reinterpret_cast<uint64_t *>(base + p.off_fsort);
    // single pass: bounds from a sample of the probed lists, one pass over all their units, exact selection
    // As in the flat scan, the bound starts at the bucket where the sample's count reaches what r codes of all the
    // query's probed codes would leave in a sample of that size, plus slack; a query whose bucket holds fewer than
    // r codes after all is flagged by the selection and redone below.
    {
        // two workgroups per query, or as many as bring the launch to 1024, up to four wavefronts per list
        constexpr int NW = IvfSampleCfg<M>::WAVES;
        const int most = (4 * nprobe + NW - 1) / NW;
        int rows = nq >= 512 ? 2 : 1024 / nq;
        if (rows > most) rows = most;
        DCPQ_LAUNCH(kStageIvf, st, (ivf_sample_kernel<M, CodeT>), dim3(nq, rows), dim3(64 * NW), 0, codes, offsets, probe, nprobe,
                    qtab, r, probed, shist, done, p.cap, bound);
        DCPQ_CHECK_LAUNCH("ivf_sample_kernel");
    }
    {
        const uint64_t most = static_cast<uint64_t>(nq) * (p.parts + nprobe);     // workgroups behind the last part leave at once
        const uint64_t gx = most < (1u << 20) ? (most + 7) / 8 * 8 : (1u << 20);
        DCPQ_LAUNCH(kStageIvfScan, st, (ivf_scan_parts_kernel<M, CodeT>), dim3(static_cast<unsigned>(gx), static_cast<unsigned>((most + gx - 1) / gx)),
                    dim3(256), M * 256 + kIvfNotes * 8, codes, items, cursor, qtab, static_cast<uint32_t>(nprobe), r, p.cap, p.upd,
                    bound, fcount, chist, fkeys);
        DCPQ_CHECK_LAUNCH("ivf_scan_parts_kernel");
    }
    uint32_t *nflag = done + nq;
    rc = launch_fast_select(fkeys, fcount, chist, nq, r, kFastSlices, p.cap, p.sortcap, 0, fsort, cand_id, cand_qd, flags, st,
                            reinterpret_cast<int *>(base + p.off_qlist), nflag);
    if (rc) return rc;
    // the queries it flagged (a full slice, or fewer than r codes in the probed lists): three passes
    const uint32_t np2 = next_pow2(r);
    const bool use_lds = np2 <= kSortLdsKeys;
    size_t lds = kIvfRedoWaves * M * 256 + 256 * 4;
    if (use_lds && sizeof(uint64_t) * np2 > lds) lds = sizeof(uint64_t) * np2;
    rc = allow_dynamic_lds(reinterpret_cast<const void *>(&ivf_redo_kernel<M, CodeT>), static_cast<int>(lds));
    if (rc) return rc;
    DCPQ_LAUNCH(kStageIvf, st, (ivf_redo_kernel<M, CodeT>), dim3(512), dim3(64 * kIvfRedoWaves), lds, codes, units, nunits, qtab, nprobe, nq, r,
                nflag, reinterpret_cast<const int *>(base + p.off_qlist), hist, thr, tie, counter, keys, reinterpret_cast<uint32_t *>(base + p.off_redo),
                reinterpret_cast<unsigned long long *>(cursor + 2), np2, use_lds ? 1 : 0, spill, cand_id, cand_qd);
    DCPQ_CHECK_LAUNCH("ivf_redo_kernel");
    return DCPQ_OK;
}

static int ivf_check_common(const char *what, int nq, int m, int dsub, int nlist, int nprobe)
{
    DCPQ_REQUIRE(nq >= 0, "%s: nq=%d", what, nq);
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "%s: m=%d dsub=%d not supported", what, m, dsub);
    DCPQ_REQUIRE(nlist >= 1 && nprobe >= 1 && nprobe <= nlist, "%s: needs 1 <= nprobe <= nlist (nprobe=%d nlist=%d)", what, nprobe, nlist);
    if (nprobe > kIvfMaxProbe) return fail(DCPQ_EUNSUPPORTED, "%s: nprobe=%d above the supported %d", what, nprobe, kIvfMaxProbe);
    return DCPQ_OK;
}

}  // namespace dcpq

using namespace dcpq;

extern "C" size_t dcpq_ivf_probe_workspace_bytes(int nq, int nlist)
{
    if (nq <= 0 || nlist <= 0) return 0;
    return align_up(sizeof(float) * static_cast<size_t>(nq) * nlist, 256);
}

extern "C" int dcpq_ivf_probe(const float *queries, int nq, int D, const float *coarse, int nlist, int nprobe,
                              int32_t *probe, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    DCPQ_REQUIRE(nq >= 0 && D >= 1, "ivf_probe: nq=%d D=%d", nq, D);
    DCPQ_REQUIRE(nlist >= 1 && nprobe >= 1 && nprobe <= nlist, "ivf_probe: needs 1 <= nprobe <= nlist");
    if (nprobe > kIvfMaxProbe) return fail(DCPQ_EUNSUPPORTED, "ivf_probe: nprobe=%d above the supported %d", nprobe, kIvfMaxProbe);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && coarse && probe && workspace, "ivf_probe: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "ivf_probe: workspace must be 256-byte aligned");
    const size_t need = dcpq_ivf_probe_workspace_bytes(nq, nlist);
    if (workspace_bytes < need) return fail(DCPQ_EWORKSPACE, "ivf_probe: workspace %zu < %zu bytes", workspace_bytes, need);
    hipStream_t st = as_stream(stream);
    float *dist = static_cast<float *>(workspace);
    const bool filter = probe_filter_serves(queries, nq, D, coarse, nlist, nprobe);
    // (the filter's: of the queries that it has left)
    const int rc = filter ? launch_probe_filter(queries, nq, D, coarse, nlist, nprobe, workspace, probe, st)
                          : launch_distance_tables(queries, nq, coarse, 1, D, nlist, dist, kStageIvfProbe, st);
    if (rc) return rc;
    DCPQ_LAUNCH(kStageIvfProbe, st, ivf_select_probe_kernel, dim3(nq), dim3(1024), 0, dist, nlist, nprobe, probe, filter ? 1 : 0);
    DCPQ_CHECK_LAUNCH("ivf_select_probe_kernel");
    return DCPQ_OK;
}

extern "C" size_t dcpq_ivf_tables_workspace_bytes(int nq) { return nq > 0 ? align_up(sizeof(uint32_t) * static_cast<size_t>(nq), 256) : 0; }

// With this much workspace (or more) dcpq_ivf_build_small_tables keeps the entries of its first pass and
// quantizes them from memory instead of computing them twice.
extern "C" size_t dcpq_ivf_tables_workspace_bytes_fast(int nq, int nprobe, int m)
{
    if (nq <= 0 || nprobe <= 0 || !m_supported(m)) return 0;
    return dcpq_ivf_tables_workspace_bytes(nq) + align_up(sizeof(float) * static_cast<size_t>(nq) * nprobe * m * kSmallSize, 256);
}

extern "C" int dcpq_ivf_build_small_tables(const float *queries, int nq, const float *coarse, int nlist,
                                           const int32_t *probe, int nprobe, const float *derived, int m, int dsub,
                                           const uint16_t *codes, const int64_t *offsets, uint32_t r, uint8_t *qtab,
                                           float *bounds, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    int rc = ivf_check_common("ivf_build_small_tables", nq, m, dsub, nlist, nprobe);
    if (rc) return rc;
    DCPQ_REQUIRE(r >= 1, "ivf_build_small_tables: r=%u", r);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && coarse && probe && derived && codes && offsets && qtab && bounds && workspace,
                 "ivf_build_small_tables: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(derived) & 15) == 0, "ivf_build_small_tables: derived must be 16-byte aligned");
    if (workspace_bytes < dcpq_ivf_tables_workspace_bytes(nq))
        return fail(DCPQ_EWORKSPACE, "ivf_build_small_tables: workspace too small");
    hipStream_t st = as_stream(stream);
    uint32_t *qmin_bits = static_cast<uint32_t *>(workspace);
    const size_t lds = sizeof(float) * static_cast<size_t>(kIvfTabProbes) * m * dsub;
    dim3 tgrid((nprobe + kIvfTabProbes - 1) / kIvfTabProbes, nq);
    if (lds > 64 * 1024) {                  // LDS above 64 KiB must be requested per kernel (at most 128 KiB here)
        const int most = static_cast<int>(sizeof(float) * kIvfTabProbes * 32 * 128);
        rc = allow_dynamic_lds(reinterpret_cast<const void *>(&ivf_tables_kernel<0>), most);
        if (rc) return rc;
        rc = allow_dynamic_lds(reinterpret_cast<const void *>(&ivf_tables_kernel<1>), most);
        if (rc) return rc;
    }
    // with room for them, the entries are kept by the first pass and quantized from memory
    const size_t n_entries = static_cast<size_t>(nq) * nprobe * m * kSmallSize;
    float *keep = nullptr;
    if (workspace_bytes >= dcpq_ivf_tables_workspace_bytes_fast(nq, nprobe, m))
        keep = reinterpret_cast<float *>(static_cast<uint8_t *>(workspace) + dcpq_ivf_tables_workspace_bytes(nq));
    // (the minima of the first pass lie in qtab as floats)
    if (keep && (reinterpret_cast<uintptr_t>(qtab) & 3) == 0) {
        // one sub-quantizer per workgroup where all of them would not give every CU one
        const int per_z = tgrid.x * tgrid.y < 256 ? 1 : m;
        tgrid.z = m / per_z;
        DCPQ_LAUNCH(kStageIvfTables, st, ivf_tables_kernel<0>, tgrid, dim3(256), lds, queries, coarse, probe, nprobe,
                    derived, m, dsub, qmin_bits, bounds, qtab, keep, per_z);
        DCPQ_CHECK_LAUNCH("ivf_tables_kernel<keep>");
        DCPQ_LAUNCH(kStageIvfTables, st, ivf_bounds_kept_kernel, dim3(nq), dim3(nq <= 256 ? 1024 : 256), 0, keep, qtab, probe, nprobe, m, per_z,
                    codes, offsets, r, bounds);
        DCPQ_CHECK_LAUNCH("ivf_bounds_kept_kernel");
        DCPQ_LAUNCH(kStageIvfTables, st, ivf_quantize_kept_kernel, dim3(static_cast<unsigned>((n_entries / 4 + 255) / 256)), dim3(256),
                    0, keep, n_entries, static_cast<size_t>(nprobe) * m * kSmallSize, bounds, qtab);
        DCPQ_CHECK_LAUNCH("ivf_quantize_kept_kernel");
        return DCPQ_OK;
    }
    // +inf as the starting minimum
    rc = launch_fill_u64(reinterpret_cast<uint64_t *>(qmin_bits), (static_cast<size_t>(nq) + 1) / 2, 0x7f8000007f800000ull, st);
    if (rc) return rc;
    DCPQ_LAUNCH(kStageIvfTables, st, ivf_tables_kernel<0>, tgrid, dim3(256), lds, queries, coarse, probe, nprobe,
                derived, m, dsub, qmin_bits, bounds, qtab, nullptr, m);
    DCPQ_CHECK_LAUNCH("ivf_tables_kernel<min>");
    DCPQ_LAUNCH(kStageIvfTables, st, ivf_qmax_kernel, dim3(nq), dim3(256), sizeof(float) * m * dsub, queries, coarse, probe, nprobe, derived, m, dsub,
                codes, offsets, r, qmin_bits, bounds);
    DCPQ_CHECK_LAUNCH("ivf_qmax_kernel");
    DCPQ_LAUNCH(kStageIvfTables, st, ivf_tables_kernel<1>, tgrid, dim3(256), lds, queries, coarse, probe, nprobe,
                derived, m, dsub, qmin_bits, bounds, qtab, nullptr, m);
    DCPQ_CHECK_LAUNCH("ivf_tables_kernel<quantize>");
    return DCPQ_OK;
}

extern "C" size_t dcpq_ivf_scan_workspace_bytes(int nq, uint32_t r)
{
    if (nq <= 0 || r == 0) return 0;
    return plan_ivf_scan(nq, r).total;
}

template <typename CodeT>
static int ivf_scan_checked(const char *what, const CodeT *codes, const int64_t *offsets, int nlist, int m,
                            const int32_t *probe, int nprobe, const uint8_t *qtab, int nq, uint32_t r,
                            uint32_t *cand_id, uint8_t *cand_qd, uint32_t *count, void *workspace,
                            size_t workspace_bytes, void *stream)
{
    clear_error();
    int rc = ivf_check_common(what, nq, m, 1, nlist, nprobe);
    if (rc) return rc;
    DCPQ_REQUIRE(r >= 1 && r <= (1u << 26), "%s: r=%u out of range", what, r);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(codes && offsets && probe && qtab && cand_id && cand_qd && count && workspace, "%s: null pointer", what);
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "%s: workspace must be 256-byte aligned", what);
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(qtab) & 15) == 0 && (reinterpret_cast<uintptr_t>(codes) & 15) == 0,
                 "%s: codes and qtab must be 16-byte aligned", what);
    if (workspace_bytes < dcpq_ivf_scan_workspace_bytes(nq, r))
        return fail(DCPQ_EWORKSPACE, "%s: workspace %zu < %zu bytes", what, workspace_bytes, dcpq_ivf_scan_workspace_bytes(nq, r));
    hipStream_t st = as_stream(stream);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    switch (m) {
        case 1: return ivf_scan_m<1>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        case 2: return ivf_scan_m<2>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        case 4: return ivf_scan_m<4>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        case 8: return ivf_scan_m<8>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        case 16: return ivf_scan_m<16>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        case 32: return ivf_scan_m<32>(codes, offsets, nlist, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, base, st);
        default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
    }
}

extern "C" int dcpq_ivf_scan_candidates(const uint16_t *codes, const int64_t *offsets, int nlist, int m,
                                        const int32_t *probe, int nprobe, const uint8_t *qtab, int nq, uint32_t r,
                                        uint32_t *cand_id, uint8_t *cand_qd, uint32_t *count, void *workspace,
                                        size_t workspace_bytes, void *stream)
{
    return ivf_scan_checked("ivf_scan_candidates", codes, offsets, nlist, m, probe, nprobe, qtab, nq, r, cand_id, cand_qd,
                            count, workspace, workspace_bytes, stream);
}

extern "C" int dcpq_ivf_scan_candidates_packed(const uint8_t *plane, const int64_t *offsets, int nlist, int m,
                                               const int32_t *probe, int nprobe, const uint8_t *qtab, int nq,
                                               uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, uint32_t *count,
                                               void *workspace, size_t workspace_bytes, void *stream)
{
    return ivf_scan_checked("ivf_scan_candidates_packed", plane, offsets, nlist, m, probe, nprobe, qtab, nq, r, cand_id,
                            cand_qd, count, workspace, workspace_bytes, stream);
}

namespace dcpq {
// plane[i][j] = codes[i][j] & 255, eight sub-codes per thread
__global__ __launch_bounds__(256) void pack_low_bytes_kernel(const uint16_t *__restrict__ codes, uint64_t nsub,
                                                            uint8_t *__restrict__ plane)
{
    const uint64_t t = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x;     // 8 sub-codes per thread
    const uint64_t i = t * 8;
    if (i + 8 <= nsub) {
        const uint4 x = *reinterpret_cast<const uint4 *>(codes + i);
        uint2 o;
        o.x = (x.x & 255u) | ((x.x >> 8) & 0xff00u) | ((x.y & 255u) << 16) | ((x.y << 8) & 0xff000000u);
        o.y = (x.z & 255u) | ((x.z >> 8) & 0xff00u) | ((x.w & 255u) << 16) | ((x.w << 8) & 0xff000000u);
        *reinterpret_cast<uint2 *>(plane + i) = o;
    } else {
        for (uint64_t k = i; k < nsub; ++k) plane[k] = static_cast<uint8_t>(codes[k] & 255u);
    }
}
}  // namespace dcpq

extern "C" int dcpq_pack_low_bytes(const uint16_t *codes, uint64_t n_codes, int m, uint8_t *plane, void *stream)
{
    clear_error();
    DCPQ_REQUIRE(m >= 1 && m <= 64, "pack_low_bytes: m=%d", m);
    if (n_codes == 0) return DCPQ_OK;
    DCPQ_REQUIRE(codes && plane, "pack_low_bytes: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(codes) & 15) == 0 && (reinterpret_cast<uintptr_t>(plane) & 15) == 0,
                 "pack_low_bytes: codes and plane must be 16-byte aligned");
    const uint64_t nsub = n_codes * static_cast<uint64_t>(m);
    const uint64_t nthreads = (nsub + 7) / 8;
    hipStream_t st = as_stream(stream);
    DCPQ_LAUNCH(kStageMisc, st, pack_low_bytes_kernel, dim3(static_cast<unsigned>((nthreads + 255) / 256)), dim3(256), 0,
                codes, nsub, plane);
    DCPQ_CHECK_LAUNCH("pack_low_bytes_kernel");
    return DCPQ_OK;
}

extern "C" size_t dcpq_ivf_refine_workspace_bytes(int nq, uint32_t r)
{
    if (nq <= 0 || r == 0) return 0;
    const uint32_t np2 = next_pow2(r);
    return np2 <= kSortLdsKeys ? 0 : sizeof(uint64_t) * static_cast<size_t>(nq) * np2;
}

extern "C" int dcpq_ivf_refine_topk(const float *queries, const float *coarse, int nlist, const float *codebooks, int m,
                                    int dsub, const uint16_t *codes, const int64_t *offsets, const int32_t *probe,
                                    int nprobe, const uint32_t *cand_id, int nq, uint32_t r, uint32_t k, uint32_t *ids,
                                    float *dist, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    int rc = ivf_check_common("ivf_refine_topk", nq, m, dsub, nlist, nprobe);
    if (rc) return rc;
    DCPQ_REQUIRE(k >= 1 && k <= r, "ivf_refine_topk: needs 1 <= k <= r (k=%u r=%u)", k, r);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && coarse && codebooks && codes && offsets && probe && cand_id && ids && dist, "ivf_refine_topk: null pointer");
    DCPQ_REQUIRE(((reinterpret_cast<uintptr_t>(queries) | reinterpret_cast<uintptr_t>(coarse) | reinterpret_cast<uintptr_t>(codebooks)) & 15) == 0,
                 "ivf_refine_topk: queries, coarse and codebooks must be 16-byte aligned");
    const size_t need = dcpq_ivf_refine_workspace_bytes(nq, r);
    if (need && (!workspace || workspace_bytes < need)) return fail(DCPQ_EWORKSPACE, "ivf_refine_topk: workspace too small");
    hipStream_t st = as_stream(stream);
    // With room for the keys: distances by as many workgroups as it takes, then the selection of the flat search.  Whole searches
    // against a workgroup per query that sorts as well, in us (20 M codes in 8192 lists, 32 probed): r = 1000, 1 query 88 and 119,
    // 64 queries 174 and 209, 1024 queries 820 and 900; r = 4000: 117 and 323, 262 and 440, 1726 and 2184.  Not where the workgroup has few
    // keys to sort: the refinement alone, m = 8, r = 100: 12.5 and 10.8 (1 query), 46.7 and 43.7 (1024); r = 50: 33 and 27 (1024); r = 200: 12.9
    // and 15.2, but with m = 4 and 2000 queries 147 and 126; r = 400: 13 and 23, 208 and 236.
    const size_t key_bytes = align_up(sizeof(uint64_t) * static_cast<size_t>(nq) * r, 256);
    // (within the limits of a grid: 65535 queries along y, 2^32 threads along x)
    const bool fits = nq <= 65535 && static_cast<uint64_t>(r) * m <= 0xFFFFF000ull;
    const bool spread = r > 256 || (r > 128 && nq <= 64);
    if (fits && spread && workspace && workspace_bytes >= key_bytes + dcpq_refine_workspace_bytes(nq, r) && (reinterpret_cast<uintptr_t>(workspace) & 7) == 0) {
        uint64_t *keys = static_cast<uint64_t *>(workspace);
        switch (m) {
#define DCPQ_IVF_KEYS(MV)                                                                                                     \
    case MV:                                                                                                                  \
        DCPQ_LAUNCH(kStageIvfRefine, st, ivf_refine_keys_kernel<MV>, dim3((r + 256 / MV - 1) / (256 / MV), nq), dim3(256), 0, queries, \
                    coarse, codebooks, dsub, codes, offsets, probe, nprobe, cand_id, r, keys);                                \
        break;
            DCPQ_IVF_KEYS(1) DCPQ_IVF_KEYS(2) DCPQ_IVF_KEYS(4) DCPQ_IVF_KEYS(8) DCPQ_IVF_KEYS(16) DCPQ_IVF_KEYS(32)
#undef DCPQ_IVF_KEYS
            default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
        }
        DCPQ_CHECK_LAUNCH("ivf_refine_keys_kernel");
        return launch_topk_of_keys(keys, nq, r, k, ids, dist, static_cast<uint8_t *>(workspace) + key_bytes, st);
    }
    const uint32_t np2 = next_pow2(r);
    const int use_lds = np2 <= kSortLdsKeys;
    const size_t lds = use_lds ? sizeof(uint64_t) * np2 : 0;
    uint64_t *spill = static_cast<uint64_t *>(workspace);
#define DCPQ_LAUNCH_IVF_REFINE(MV)                                                                                   \
    case MV:                                                                                                         \
        DCPQ_CHECK_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&ivf_refine_kernel<MV>),                  \
                                           hipFuncAttributeMaxDynamicSharedMemorySize,                              \
                                           static_cast<int>(sizeof(uint64_t) * kSortLdsKeys)));                      \
        DCPQ_LAUNCH(kStageIvfRefine, st, ivf_refine_kernel<MV>, dim3(nq), dim3(1024), lds, queries, coarse, codebooks, dsub, \
                    codes, offsets, probe, nprobe, cand_id, r, k, np2, use_lds, spill, ids, dist);                   \
        break;
    switch (m) {
        DCPQ_LAUNCH_IVF_REFINE(1) DCPQ_LAUNCH_IVF_REFINE(2) DCPQ_LAUNCH_IVF_REFINE(4) DCPQ_LAUNCH_IVF_REFINE(8)
        DCPQ_LAUNCH_IVF_REFINE(16) DCPQ_LAUNCH_IVF_REFINE(32)
        default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
    }
#undef DCPQ_LAUNCH_IVF_REFINE
    DCPQ_CHECK_LAUNCH("ivf_refine_kernel");
    return DCPQ_OK;
}

// ---- the whole inverted-index search in one call ------------------------------------------------
namespace {
struct IvfSearchPlan {
    size_t off_probe, off_qtab, off_bounds, off_cand_id, off_cand_qd, off_count, off_sub, sub_bytes, total;
};
IvfSearchPlan plan_ivf_search(int nq, int nlist, int nprobe, int m, uint32_t r)
{
    IvfSearchPlan p{};
    const size_t Q = static_cast<size_t>(nq);
    size_t off = 0;
    p.off_probe = off;   off = align_up(off + sizeof(int32_t) * Q * nprobe, 256);
    p.off_qtab = off;    off = align_up(off + Q * nprobe * m * kSmallSize, 256);
    p.off_bounds = off;  off = align_up(off + sizeof(float) * 2 * Q, 256);
    p.off_cand_id = off; off = align_up(off + sizeof(uint32_t) * Q * r, 256);
    p.off_cand_qd = off; off = align_up(off + Q * r, 256);
    p.off_count = off;   off = align_up(off + sizeof(uint32_t) * Q, 256);
    // the four steps run one after the other on the stream and share one scratch region
    size_t sub = dcpq_ivf_probe_workspace_bytes(nq, nlist);
    // (the small-table entries are kept between the two table passes when that takes no more than 2 GiB)
    const size_t keep_tables = dcpq_ivf_tables_workspace_bytes_fast(nq, nprobe, m);
    const size_t others[] = {keep_tables <= (static_cast<size_t>(2) << 30) ? keep_tables : dcpq_ivf_tables_workspace_bytes(nq),
                             dcpq_ivf_scan_workspace_bytes(nq, r),
                             dcpq_ivf_refine_workspace_bytes(nq, r)};
    for (size_t o : others) sub = o > sub ? o : sub;
    p.off_sub = off;     p.sub_bytes = align_up(sub, 256); off += p.sub_bytes;
    p.total = off;
    return p;
}
}  // namespace

extern "C" size_t dcpq_ivf_search_workspace_bytes(int nq, int nlist, int nprobe, int m, uint32_t r)
{
    if (nq <= 0 || nlist <= 0 || nprobe <= 0 || nprobe > nlist || !m_supported(m) || r == 0 || r > (1u << 26)) return 0;
    return plan_ivf_search(nq, nlist, nprobe, m, r).total;
}

extern "C" int dcpq_ivf_search(const float *queries, int nq, const float *coarse, int nlist, int nprobe,
                               const float *codebooks, const float *derived, int m, int dsub, const uint16_t *codes,
                               const uint8_t *plane, const int64_t *offsets, uint32_t r, uint32_t k, uint32_t *ids,
                               float *dist, void *workspace, size_t workspace_bytes, void *stream)
{
    clear_error();
    int rc = ivf_check_common("ivf_search", nq, m, dsub, nlist, nprobe);
    if (rc) return rc;
    DCPQ_REQUIRE(r >= 1 && r <= (1u << 26) && k >= 1 && k <= r, "ivf_search: needs 1 <= k <= r <= 2^26 (k=%u r=%u)", k, r);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && coarse && codebooks && derived && codes && offsets && ids && dist && workspace,
                 "ivf_search: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "ivf_search: workspace must be 256-byte aligned");
    const IvfSearchPlan p = plan_ivf_search(nq, nlist, nprobe, m, r);
    if (workspace_bytes < p.total) return fail(DCPQ_EWORKSPACE, "ivf_search: workspace %zu < %zu bytes", workspace_bytes, p.total);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    int32_t *probe = reinterpret_cast<int32_t *>(base + p.off_probe);
    uint8_t *qtab = base + p.off_qtab;
    float *bounds = reinterpret_cast<float *>(base + p.off_bounds);
    uint32_t *cand_id = reinterpret_cast<uint32_t *>(base + p.off_cand_id);
    uint8_t *cand_qd = base + p.off_cand_qd;
    uint32_t *count = reinterpret_cast<uint32_t *>(base + p.off_count);
    void *sub = base + p.off_sub;
    rc = dcpq_ivf_probe(queries, nq, m * dsub, coarse, nlist, nprobe, probe, sub, p.sub_bytes, stream);
    if (rc) return rc;
    rc = dcpq_ivf_build_small_tables(queries, nq, coarse, nlist, probe, nprobe, derived, m, dsub, codes, offsets, r, qtab,
                                     bounds, sub, p.sub_bytes, stream);
    if (rc) return rc;
    rc = plane ? dcpq_ivf_scan_candidates_packed(plane, offsets, nlist, m, probe, nprobe, qtab, nq, r, cand_id, cand_qd,
                                                 count, sub, p.sub_bytes, stream)
               : dcpq_ivf_scan_candidates(codes, offsets, nlist, m, probe, nprobe, qtab, nq, r, cand_id, cand_qd, count, sub,
                                          p.sub_bytes, stream);
    if (rc) return rc;
    return dcpq_ivf_refine_topk(queries, coarse, nlist, codebooks, m, dsub, codes, offsets, probe, nprobe, cand_id, nq, r,
                                k, ids, dist, sub, p.sub_bytes, stream);
}

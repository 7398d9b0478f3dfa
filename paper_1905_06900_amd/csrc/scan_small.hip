// Alg. 3 for small problems (few queries over a short array): pass one and the distances of pass two in two kernels.
//
// On a large array the scan keeps a running bound so that nearly all codes are rejected by a sign test; that takes a
// sample, a selection of what was appended and a redo path, ten launches in all, and on a stream of short kernels
// every launch costs 4 to 5 us.  With few (query, code) pairs it is cheaper to look at all of them twice:
//   small_hist_kernel      qd of every pair (one byte each, kept), histograms of 32 stretches of the codes
//   small_collect_kernel   from the histograms of all stretches: the bucket T of the r-th candidate, how many ids of T
//                          are taken before this stretch and in it; then the stretch's candidates -- exactly the r smallest
//                          by (qd, id) over all stretches -- and at once their re-ranking distances (Eq. 1 entries
//                          computed on demand in double precision, rounded once, added in fp32, j increasing)
// followed by the selection of the k smallest (refine.hip).  The result does not depend on the order in which the
// candidates are stored, so they need no sorting.
#include <cmath>

#include "common.h"
#include "scan_internal.h"
#include "refine_entry.h"

namespace dcpq {

constexpr int kSmallThreads = 1024;
constexpr int kSmallStep = 4096;            // codes a workgroup takes at a time: 16 wavefronts x 64 lanes x 4 codes
constexpr uint32_t kSmallMostBlocks = 256;  // workgroups along the codes that compute qd ...
// Stretches with a histogram of their own.  Every collector reads the histograms of all of them (with 128 stretches that was
// half of the time for 16 queries over 1 M codes: 114 us, 76 with 32) and walks the qd bytes of its own (3 M codes, 8
// queries: 147 us with 32 stretches, 107 with 128): their number grows with the root of codes per query.  Below that root
// no more of them than give two collectors per CU: 550 queries over 60000 codes took 212 us with a collector for every
// 4096 codes.
static uint32_t small_stretches(uint64_t n_codes, int nq)
{
    const double s = sqrt(static_cast<double>(n_codes) / (80.0 * nq));
    const uint32_t fill = 512u / static_cast<uint32_t>(nq < 512 ? nq : 512), least = fill < 16u ? fill : 16u;
    return s < least ? least : s > 128.0 ? 128u : static_cast<uint32_t>(s);
}
constexpr int small_qt(int m) { return m <= 8 ? 8 : 64 / m; }      // queries whose tables share a workgroup (<= 16 KiB)

struct SmallPlan {
    uint32_t unit, nblocks;                 // codes per workgroup of the first kernel, its workgroups
    uint32_t per, nstretch;                 // workgroups per stretch, stretches
    size_t npad;                            // bytes of qd per query
    size_t off_qd, off_hist, off_keys, total;
};

static SmallPlan plan_small(uint64_t n_codes, int nq, uint32_t r)
{
    SmallPlan p{};
    uint64_t nb = (n_codes + kSmallStep - 1) / kSmallStep;
    if (nb > kSmallMostBlocks) nb = kSmallMostBlocks;
    const uint64_t unit = ((n_codes + nb - 1) / nb + kSmallStep - 1) / kSmallStep * kSmallStep;
    p.unit = static_cast<uint32_t>(unit);
    p.nblocks = static_cast<uint32_t>((n_codes + unit - 1) / unit);
    const uint32_t want = small_stretches(n_codes, nq);
    if (want >= 100 && p.nblocks > 128) {               // one workgroup per stretch: no adding up, nothing to clear
        const uint64_t u = ((n_codes + 127) / 128 + kSmallStep - 1) / kSmallStep * kSmallStep;
        p.unit = static_cast<uint32_t>(u);
        p.nblocks = static_cast<uint32_t>((n_codes + u - 1) / u);
    }
    p.per = (p.nblocks + want - 1) / want;
    p.nstretch = (p.nblocks + p.per - 1) / p.per;
    p.npad = static_cast<size_t>(p.nblocks) * p.unit;
    size_t off = 0;
    p.off_hist = off; off = align_up(off + sizeof(uint32_t) * 256 * static_cast<size_t>(p.nstretch) * nq, 256);
    p.off_qd = off;   off = align_up(off + p.npad * nq, 256);
    p.off_keys = off; off = align_up(off + sizeof(uint64_t) * static_cast<size_t>(nq) * r, 256);
    p.total = off;
    return p;
}

// The byte gathers of the two-kernel form run at about 0.3e12 pairs/s (m = 8) against 20e12 in the row-lookup kernel, so it is
// taken while that costs no more than the launches it saves (both sides measured: 1 M codes of 4 sub-codes, one
// query 95 -> 32 us, 16 queries 183 -> 72; 3 M codes, 8 queries 310 -> 92; 1 M codes of 8, 16 queries 120 -> 78, and 32 queries,
// twice beyond the line, 127 -> 190 had the line been there).
bool small_search_pays(uint64_t n_codes, int m, int nq)
{
    return n_codes * static_cast<uint64_t>(nq) * static_cast<uint64_t>(m < 4 ? 4 : m) <= (1ull << 27);
}

size_t small_search_bytes(uint64_t n_codes, int nq, uint32_t r) { return plan_small(n_codes, nq, r).total; }

// words at the start of its workspace that must be zero: the histograms
size_t small_search_clear_words(uint64_t n_codes, int nq, uint32_t r)
{
    const SmallPlan p = plan_small(n_codes, nq, r);
    return p.per == 1 ? 0 : 256 * static_cast<size_t>(p.nstretch) * nq;
}

// Four consecutive codes of one lane: low bytes of all sub-codes.
template <int M, typename CodeT>
__global__ __launch_bounds__(kSmallThreads) void small_hist_kernel(const CodeT *__restrict__ codes, uint32_t n_codes, uint32_t unit,
                                                                  uint32_t per, uint32_t nstretch, const uint8_t *__restrict__ qtab, int nq,
                                                                  size_t npad, uint8_t *__restrict__ qdbuf, uint32_t *__restrict__ bhist)
{
    constexpr int QT = small_qt(M);
    extern __shared__ __align__(16) uint8_t smem[];
    uint8_t *ltab = smem;                                                     // [QT][M][256]
    uint32_t *lhist = reinterpret_cast<uint32_t *>(smem + QT * M * 256);      // [4][QT][256]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q0 = blockIdx.x * QT, nqt = min(QT, nq - q0);
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(qtab + static_cast<size_t>(q0) * M * 256);
        for (int v = tid; v < nqt * M * 16; v += kSmallThreads) reinterpret_cast<uint4 *>(ltab)[v] = src[v];
        for (int v = tid; v < 4 * QT * 256; v += kSmallThreads) lhist[v] = 0;
    }
    __syncthreads();
    const uint32_t begin = blockIdx.y * unit, end = min(n_codes, begin + unit);
    for (uint32_t base = begin; base < end; base += kSmallStep) {             // uniform
        const uint32_t i0 = base + wave * 256 + lane * 4;
        if (i0 >= end) continue;
        uint32_t low[4][M];
#pragma unroll
        for (int c = 0; c < 4; ++c) load_low_bytes<M>(codes, min(i0 + c, n_codes - 1), low[c]);
        for (int q = 0; q < nqt; ++q) {                                       // uniform
            const uint8_t *t = ltab + q * (M * 256);
            uint32_t s[4] = {0, 0, 0, 0};
#pragma unroll
            for (int j = 0; j < M; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) s[c] += t[j * 256 + low[c][j]];
            uint32_t w = 0;
            uint32_t *h = lhist + ((wave & 3) * QT + q) * 256;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t qd = min(s[c], 255u);
                w |= qd << (8 * c);
                if (i0 + c < end) atomicAdd(&h[qd], 1u);
            }
            *reinterpret_cast<uint32_t *>(qdbuf + static_cast<size_t>(q0 + q) * npad + i0) = w;
        }
    }
    __syncthreads();
    for (int v = tid; v < nqt * 256; v += kSmallThreads) {
        const uint32_t c = lhist[v] + lhist[QT * 256 + v] + lhist[2 * QT * 256 + v] + lhist[3 * QT * 256 + v];
        uint32_t *h = &bhist[(static_cast<size_t>(q0 + (v >> 8)) * nstretch + blockIdx.y / per) * 256 + (v & 255)];
        if (per == 1) *h = c;
        else if (c) atomicAdd(h, c);
    }
}

template <int M, typename CodeT>
__global__ __launch_bounds__(kSmallThreads) void small_collect_kernel(
    const CodeT *__restrict__ codes, uint32_t n_codes, uint32_t unit, uint32_t nblocks, const uint8_t *__restrict__ qdbuf, size_t npad,
    const uint32_t *__restrict__ bhist, uint32_t r, const float *__restrict__ queries, const float *__restrict__ cb, int dsub,
    uint32_t table_size, uint64_t *__restrict__ keys)
{
    constexpr int kList = M >= 8 ? 256 : 2048 / M;       // candidates whose distances are worked out together
    __shared__ uint32_t all[4][256], bef[4][256];
    __shared__ uint32_t s_T, s_need, s_base, s_quota;
    __shared__ uint32_t wlt[16], weq[16];
    __shared__ uint32_t list[kList];
    __shared__ float ent[kList * M];
    extern __shared__ __align__(16) float ly[];          // the query
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int q = blockIdx.x, D = M * dsub;
    const uint32_t blk = blockIdx.y;
    for (int t = tid; t < D; t += kSmallThreads) ly[t] = queries[static_cast<size_t>(q) * D + t];
    {
        const int bucket = tid & 255, part = tid >> 8;
        const uint32_t *h = bhist + static_cast<size_t>(q) * nblocks * 256 + bucket;
        uint32_t a = 0, b = 0;
#pragma unroll 8
        for (uint32_t x = part; x < nblocks; x += 4) {
            const uint32_t c = h[static_cast<size_t>(x) * 256];
            a += c;
            b += x < blk ? c : 0u;
        }
        all[part][bucket] = a;
        bef[part][bucket] = b;
    }
    __syncthreads();
    if (wave == 0) {                                     // bucket of the r-th, ids still wanted from it, what lies before this stretch
        uint32_t c[4], b[4], mine = 0, minb = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const int x = 4 * lane + z;
            c[z] = all[0][x] + all[1][x] + all[2][x] + all[3][x];
            b[z] = bef[0][x] + bef[1][x] + bef[2][x] + bef[3][x];
            mine += c[z]; minb += b[z];
        }
        uint32_t incl = mine, inclb = minb;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t o = __shfl(incl, lane >= d ? lane - d : lane), ob = __shfl(inclb, lane >= d ? lane - d : lane);
            if (lane >= d) { incl += o; inclb += ob; }
        }
        uint32_t cum = incl - mine, cumb = inclb - minb;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            if (cum < r && cum + c[z] >= r) {            // one lane, one bucket (r <= n_codes)
                const uint32_t need = r - cum, tb = min(b[z], need);
                s_T = 4 * lane + z;
                s_need = need;
                s_base = cumb + tb;                      // candidates in the stretches before this one
                s_quota = need - tb;                     // ids of bucket T that this stretch may still take
            }
            cum += c[z]; cumb += b[z];
        }
    }
    __syncthreads();
    const uint32_t T = s_T, quota = s_quota;
    // this wavefront's part of the stretch: contiguous, so that ids come in order
    const uint32_t begin = blk * unit, end = min(n_codes, begin + unit), wpart = unit / 16;
    const uint32_t wb = begin + wave * wpart, we = min(end, wb + wpart);
    const uint8_t *qd = qdbuf + static_cast<size_t>(q) * npad;
    // 16 codes per lane: counts of qd below T and equal to T
    auto load16 = [&](uint32_t i0) { return i0 < we ? *reinterpret_cast<const uint4 *>(qd + i0) : make_uint4(~0u, ~0u, ~0u, ~0u); };
    auto classify = [&](const uint4 &x, uint32_t i0, int c, bool &below, bool &tied) {
        const uint32_t w = (c >> 2) == 0 ? x.x : (c >> 2) == 1 ? x.y : (c >> 2) == 2 ? x.z : x.w;
        const uint32_t v = (w >> (8 * (c & 3))) & 255u;
        const bool live = i0 + c < we;
        below = live && v < T;
        tied = live && v == T;
    };
    uint32_t lt = 0, eq = 0;
#pragma unroll 4
    for (uint32_t base = wb; base < we; base += 1024) {  // uniform over the wavefront
        const uint32_t i0 = base + lane * 16;
        const uint4 x = load16(i0);
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            bool below, tied;
            classify(x, i0, c, below, tied);
            lt += below ? 1u : 0u;
            eq += tied ? 1u : 0u;
        }
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { lt += __shfl_xor(lt, d); eq += __shfl_xor(eq, d); }
    if (lane == 0) { wlt[wave] = lt; weq[wave] = eq; }
    __syncthreads();
    uint32_t before_lt = 0, before_eq = 0, total_lt = 0, total_eq = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) { before_lt += wlt[w]; before_eq += weq[w]; }
        total_lt += wlt[w]; total_eq += weq[w];
    }
    const uint32_t total = total_lt + min(total_eq, quota);                   // candidates of this stretch
    const bool vec4 = (dsub & 3) == 0;
    // The candidates' ids, in order: to the list, or, where there are more than it holds, to the places of their keys, from
    // which they are then taken a list at a time.  (Ties go to the smallest ids: with many of them in the bucket of the r-th
    // candidate, nearly all candidates of a query can lie in one stretch.  Walked once per list 15000 candidates in a
    // stretch of 125000 codes took 1.6 ms.)
    uint64_t *out = keys + static_cast<size_t>(q) * r + s_base;
    const bool listed = total <= kList;                                       // uniform
    {
        uint32_t nlt = before_lt, neq = before_eq;                            // walked past so far, in id order
        for (uint32_t base = wb; base < we; base += 1024) {
            const uint32_t i0 = base + lane * 16;
            const uint4 x = load16(i0);
            uint32_t my_lt = 0, my_eq = 0;
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                bool below, tied;
                classify(x, i0, c, below, tied);
                my_lt += below ? 1u : 0u;
                my_eq += tied ? 1u : 0u;
            }
            if (!__ballot(my_lt + my_eq != 0)) continue;                      // uniform
            uint32_t pre = my_lt | my_eq << 16;                               // (at most 1024 each)
            const uint32_t own = pre;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t o = __shfl(pre, lane >= d ? lane - d : lane);
                if (lane >= d) pre += o;
            }
            const uint32_t sum = __shfl(pre, 63);
            uint32_t plt = nlt + ((pre - own) & 0xFFFFu), peq = neq + ((pre - own) >> 16);
#pragma unroll
            for (int c = 0; c < 16; ++c) {
                bool below, tied;
                classify(x, i0, c, below, tied);
                if (below || (tied && peq < quota)) {
                    const uint32_t pos = plt + min(peq, quota);               // position among the candidates of this stretch
                    if (listed) list[pos] = i0 + c;
                    else out[pos] = i0 + c;
                }
                plt += below ? 1u : 0u;
                peq += tied ? 1u : 0u;
            }
            nlt += sum & 0xFFFFu;
            neq += sum >> 16;
        }
    }
    __syncthreads();
    for (uint32_t first = 0; first < total; first += kList) {                 // uniform; nearly always one round
        const uint32_t n_here = min(static_cast<uint32_t>(kList), total - first);
        if (!listed) {
            for (uint32_t x = tid; x < n_here; x += kSmallThreads) list[x] = static_cast<uint32_t>(out[first + x]);
            __syncthreads();
        }
        for (uint32_t x = tid; x < n_here * M; x += kSmallThreads) {
            const uint32_t j = x % M, id = list[x / M];
            const uint32_t cj = codes[static_cast<size_t>(id) * M + j];
            ent[x] = entry_on_demand(ly + j * dsub, cb + (static_cast<size_t>(j) * table_size + cj) * dsub, dsub, vec4);
        }
        __syncthreads();
        for (uint32_t x = tid; x < n_here; x += kSmallThreads) {
            float d = ent[x * M];
#pragma unroll
            for (int j = 1; j < M; ++j) d = __fadd_rn(d, ent[x * M + j]);
            out[first + x] = make_key(__float_as_uint(d), list[x]);
        }
        __syncthreads();
    }
}

template <int M, typename CodeT>
static int launch_small_m(const float *queries, int nq, const float *codebooks, int dsub, uint32_t table_size, const CodeT *codes,
                          uint64_t n_codes, const uint8_t *qtab, uint32_t r, uint8_t *base, const SmallPlan &p, hipStream_t st)
{
    constexpr int QT = small_qt(M);
    uint8_t *qd = base + p.off_qd;
    uint32_t *hist = reinterpret_cast<uint32_t *>(base + p.off_hist);
    uint64_t *keys = reinterpret_cast<uint64_t *>(base + p.off_keys);
    const size_t lds = static_cast<size_t>(QT) * M * 256 + 4 * QT * 256 * sizeof(uint32_t);
    // (queries along x: a batch over a few hundred 8-bit codes can have more of them than the 65535 that y is sure to take)
    DCPQ_LAUNCH(kStageScanHist, st, (small_hist_kernel<M, CodeT>), dim3((nq + QT - 1) / QT, p.nblocks), dim3(kSmallThreads), lds, codes,
                static_cast<uint32_t>(n_codes), p.unit, p.per, p.nstretch, qtab, nq, p.npad, qd, hist);
    DCPQ_CHECK_LAUNCH("small_hist_kernel");
    DCPQ_LAUNCH(kStageScanCollect, st, (small_collect_kernel<M, CodeT>), dim3(nq, p.nstretch), dim3(kSmallThreads),
                sizeof(float) * M * dsub, codes, static_cast<uint32_t>(n_codes), p.unit * p.per, p.nstretch, qd, p.npad, hist, r, queries,
                codebooks, dsub, table_size, keys);
    DCPQ_CHECK_LAUNCH("small_collect_kernel");
    return DCPQ_OK;
}

template <typename CodeT>
static int launch_small_t(const float *queries, int nq, const float *codebooks, int m, int dsub, uint32_t table_size, const CodeT *codes,
                          uint64_t n_codes, const uint8_t *qtab, uint32_t r, uint8_t *base, const SmallPlan &p, hipStream_t st)
{
#define DCPQ_LAUNCH_SMALL_SEARCH(MV) \
    case MV: return launch_small_m<MV, CodeT>(queries, nq, codebooks, dsub, table_size, codes, n_codes, qtab, r, base, p, st);
    switch (m) {
        DCPQ_LAUNCH_SMALL_SEARCH(1) DCPQ_LAUNCH_SMALL_SEARCH(2) DCPQ_LAUNCH_SMALL_SEARCH(4) DCPQ_LAUNCH_SMALL_SEARCH(8)
        DCPQ_LAUNCH_SMALL_SEARCH(16) DCPQ_LAUNCH_SMALL_SEARCH(32)
        default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
    }
#undef DCPQ_LAUNCH_SMALL_SEARCH
}

// Candidates and their distances: *keys = uint64 [nq][r], (fp32 bits of the distance, id), in ws (small_search_bytes).
int launch_small_search(const float *queries, int nq, const float *codebooks, int m, int dsub, uint32_t table_size, const void *codes,
                        int code_bytes, uint64_t n_codes, const uint8_t *qtab, uint32_t r, void *ws, const uint64_t **keys, hipStream_t st)
{
    const SmallPlan p = plan_small(n_codes, nq, r);
    uint8_t *base = static_cast<uint8_t *>(ws);
    *keys = reinterpret_cast<const uint64_t *>(base + p.off_keys);
    if (code_bytes == 1)
        return launch_small_t(queries, nq, codebooks, m, dsub, table_size, static_cast<const uint8_t *>(codes), n_codes, qtab, r, base, p, st);
    return launch_small_t(queries, nq, codebooks, m, dsub, table_size, static_cast<const uint16_t *>(codes), n_codes, qtab, r, base, p, st);
}

}  // namespace dcpq

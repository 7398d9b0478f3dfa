// Shared between the two translation units of the scan stage (not part of the ABI).
#pragma once

#include "common.h"

namespace dcpq {

constexpr uint32_t kSortLdsKeys = 8192;   // keys a workgroup sorts in LDS (64 KiB)

inline uint32_t next_pow2(uint32_t x)
{
    uint32_t p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Sizes and workspace layout of one scan_candidates call (offsets in bytes from a 256-byte
// aligned base).  The three-pass path can always run; the single-pass path exists for m >= 4.
// Each query's candidate buffer and append cursor are split into slices, one per residue of the
// workgroup's position along the codes: workgroups that run at the same time append to different
// cursors, which keeps same-address atomics (they serialize in the L2) off the critical path.
constexpr int kFastSlices = 16;      // at most; fewer when there are fewer workgroups along the codes

constexpr uint32_t kPilotEvery = 16;
constexpr int kNoteWaves = 16;       // wavefronts per workgroup of the single-pass kernel, at most

// Running bucket bound of a query in the single-pass scans (one 16-byte record per query).
struct __attribute__((aligned(16))) Bound {
    int t;              // codes above this bucket are not wanted (only ever lowered, by atomicMin)
    uint32_t t0, last;  // of the starting bucket t0 only the ids up to `last` are wanted (256: no bucket is limited)
    int guess;          // t, or a lower bucket that is more likely than not to do (see starting_bound)
};

// What becomes of a query whose starting bucket holds many more codes than are wanted, or is about to
// have its codes counted one by one (see starting_bound).
enum Crowded { kCrowdedLimit, kCrowdedSkip, kCountBelow };

struct ScanPlan {
    // three-pass path
    uint32_t unit;        // codes scanned by one wavefront
    uint32_t nunits;      // ceil(n_codes / unit)
    uint32_t qt;          // queries per workgroup tile
    size_t off_hist;      // uint32 [nq][256]
    size_t off_thr;       // uint32 [nq][2]   (threshold bucket, ids still needed from it)
    size_t off_counter;   // uint32 [nq]
    size_t off_done;      // uint32 [3][ceil(nq / qt)]  finished workgroups of a query tile of the sample, and again zero; from the second row on finished items of a tile of the redo (at least half as many queries)
    size_t zero_bytes;    // everything that a call expects at zero lies together from offset 0: the four arrays
                          // above and, for the single-pass path, fcount, chist, shist and nflag
    size_t off_tie;       // uint32 [nq][nunits]
    size_t off_keys;      // uint64 [nq][r]
    size_t off_spill;     // uint64 [nq][next_pow2(r)], only when r keys do not fit the LDS sort
    // single-pass path
    bool fast;
    uint32_t fqt;             // queries per tile
    uint32_t ntiles;
    uint32_t fblocks;         // workgroups along the code axis
    uint32_t codes_per_block;
    uint32_t slices;          // slices per query: min(kFastSlices, fblocks)
    uint32_t cap;             // candidate-buffer entries per query and slice
    uint32_t upd;             // appended candidates between two bound updates
    uint32_t wcap;            // candidates a wavefront can note until its workgroup ends
    uint32_t sortcap;         // keys the final selection can sort (power of two)
    uint32_t s_unit, s_nunits;    // sample: s_nunits runs of s_unit codes ...
    uint64_t s_stride;            // ... starting every s_stride codes
    // pilot pass (large arrays): the histogram pass reads only every kPilotEvery-th run of the sample, and the
    // sample itself goes through the single-pass kernel, counting only
    bool pilot;
    uint32_t s1_nunits;           // runs the histogram pass reads
    uint64_t s_count;             // codes in the sample
    uint32_t pilot_r;             // rank wanted within the sample: what r codes of the array leave in it, plus slack
    uint32_t pilot_blocks;        // workgroups per tile of the pilot pass ...
    uint32_t pilot_runs;          // ... and sample runs per workgroup
    size_t off_fzero, fzero_bytes;   // fcount, chist, shist: cleared once more after a pilot pass
    size_t off_fcount;    // uint32 [nq][slices]
    size_t off_chist;     // uint32 [nq][256]
    size_t off_shist;     // uint32 [nq][256]
    size_t off_nflag;     // uint32 [1], two words on the uint64 counter that hands out the redo's items
    size_t off_bound;     // Bound [nq], in the place of tie, keys and spill: only the redo uses those, and it never reads a bound
    size_t off_flags;     // uint32 [nq]
    size_t off_qlist;     // int32 [nq]
    size_t off_qsw;       // uint8 [ntiles][fast_table_bytes(m, fqt)]
    size_t off_fkeys;     // uint64 [nq][slices][cap]
    size_t off_fsort;     // uint64 [nq][sortcap], only when sortcap exceeds the LDS sort
    size_t off_notes;     // uint64 [ntiles * max(fblocks, pilot_blocks)][kNoteWaves][wcap]
    size_t total;
};
// mode: DCPQ_SCAN_AUTO picks the single-pass query tile from the batch size; DCPQ_SCAN_TILE16/32/64 force it
// room: bytes of the workspace; the notes (the last array, a matter of speed only) shrink to what is left of it
ScanPlan plan_scan(uint64_t n_codes, int m, int nq, uint32_t r, int mode = 0, size_t room = ~static_cast<size_t>(0));

int fast_query_tile(int m, int nq, int mode);   // 0 when the single-pass path does not exist for this m (and tile)
size_t fast_table_bytes(int m, int qt);
// CodeT: uint16_t (the codes as stored) or uint8_t (their low-byte plane); both are instantiated.
template <typename CodeT>
int launch_sample_hist(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq,
                       uint32_t r, uint32_t *shist, const ScanPlan &p, uint32_t want_r, uint64_t want_n, Crowded crowded,
                       bool guess, Bound *bound, uint32_t *done, hipStream_t st);
template <typename CodeT>
int launch_scan_fast(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq,
                     uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, uint8_t *base, const ScanPlan &p, const CellsArea *cells,
                     hipStream_t st);
// The scan over cells, between the starting bounds and the selection; *used: the device flag that says whether it served the batch
template <typename CodeT>
int launch_scan_cells(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r, const CellsArea &area, const Bound *bound,
                      uint32_t nslices, uint32_t cap, uint32_t *fcount, uint32_t *chist, uint64_t *keys, const uint32_t **used, hipStream_t st);

// The selection from what the single-pass scans have appended, for the inverted lists too.
// n_ids: the ids are below this (0 = unknown); qlist, nflag (optional): the flagged queries, in any order, and their number
int launch_fast_select(const uint64_t *keys, const uint32_t *count, const uint32_t *chist, int nq, uint32_t r,
                       uint32_t nslices, uint32_t cap, uint32_t sortcap, uint64_t n_ids, uint64_t *spill, uint32_t *cand_id,
                       uint8_t *cand_qd, uint32_t *flags, hipStream_t st, int *qlist = nullptr, uint32_t *nflag = nullptr);

// Small shared steps of the three-pass selection, reused by the inverted-list variant.
int launch_zero_words(uint32_t *p, size_t nwords, hipStream_t st);
int launch_fill_u64(uint64_t *p, size_t n, uint64_t v, hipStream_t st);
int launch_zero_and_fill(uint64_t *z, size_t nz, uint64_t *p, size_t n, uint64_t v, hipStream_t st);      // z to zero, p to v
int launch_threshold(const uint32_t *hist, int nq, uint32_t r, uint32_t *thr, hipStream_t st);
int launch_tie_quota(uint32_t *tie, uint32_t nunits, int nq, const uint32_t *thr, hipStream_t st);
int launch_sort_candidates(const uint64_t *keys, int nq, uint32_t r, uint64_t *spill, uint32_t *cand_id, uint8_t *cand_qd, hipStream_t st);

#ifdef __HIPCC__
}  // namespace dcpq
#include "device_util.h"
namespace dcpq {
// Low bytes of the m sub-codes of code i (property P1: the derived index is the low 8 bits).
template <int M>
__device__ inline void load_low_bytes(const uint16_t *__restrict__ codes, uint64_t i, uint32_t (&low)[M])
{
    if constexpr (M % 8 == 0) {
        const uint4 *p = reinterpret_cast<const uint4 *>(codes + i * M);
#pragma unroll
        for (int v = 0; v < M / 8; ++v) {
            const uint4 x = p[v];
            low[8 * v + 0] = x.x & 255u; low[8 * v + 1] = (x.x >> 16) & 255u;
            low[8 * v + 2] = x.y & 255u; low[8 * v + 3] = (x.y >> 16) & 255u;
            low[8 * v + 4] = x.z & 255u; low[8 * v + 5] = (x.z >> 16) & 255u;
            low[8 * v + 6] = x.w & 255u; low[8 * v + 7] = (x.w >> 16) & 255u;
        }
    } else if constexpr (M == 4) {
        const uint2 x = *reinterpret_cast<const uint2 *>(codes + i * 4);
        low[0] = x.x & 255u; low[1] = (x.x >> 16) & 255u;
        low[2] = x.y & 255u; low[3] = (x.y >> 16) & 255u;
    } else if constexpr (M == 2) {
        const uint32_t x = *reinterpret_cast<const uint32_t *>(codes + i * 2);
        low[0] = x & 255u; low[1] = (x >> 16) & 255u;
    } else {
        low[0] = codes[i] & 255u;
    }
}

// Inclusive prefix sums of 256 bucket counts over a wavefront, lane l owning buckets 4l .. 4l + 3: c becomes
// the counts, cum the inclusive prefixes.  The counts may just have been added by other workgroups' atomics.
__device__ inline void wave_prefix_of_buckets(const uint32_t *hist, uint32_t (&c)[4], uint32_t (&cum)[4], int more_in = -1, uint32_t more = 0)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int z = 0; z < 4; ++z) c[z] = __hip_atomic_load(&hist[4 * lane + z], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int z = 0; z < 4; ++z)
        if (4 * lane + z == more_in) c[z] += more;
    const uint32_t mine = c[0] + c[1] + c[2] + c[3];
    uint32_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t other = __shfl(incl, lane >= d ? lane - d : lane);
        if (lane >= d) incl += other;
    }
    uint32_t run = incl - mine;
#pragma unroll
    for (int z = 0; z < 4; ++z) { run += c[z]; cum[z] = run; }
}

// put(T, need): T = bucket holding the r-th smallest qd; need = ids still to take from bucket T (called by one lane of a wavefront).
template <typename Put>
__device__ inline void exact_threshold(const uint32_t *hist, uint32_t r, Put put)
{
    uint32_t c[4], cum[4];
    wave_prefix_of_buckets(hist, c, cum);
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int z = 0; z < 4; ++z)
        if (cum[z] - c[z] < r && cum[z] >= r) put(static_cast<uint32_t>(4 * lane + z), r - (cum[z] - c[z]));
    // fewer than r codes in all (inverted lists only): bucket "256" takes everything
    if (lane == 63 && cum[3] < r) put(256u, 0u);
}

// The same into thr[0 .. 1].  (Device-scope stores: workgroups of the same launch may read them.)
__device__ inline void exact_threshold(const uint32_t *hist, uint32_t r, uint32_t *thr)
{
    exact_threshold(hist, r, [thr](uint32_t t, uint32_t need) {
        __hip_atomic_store(&thr[0], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&thr[1], need, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
}

// Turns per-unit counts of bucket T into per-unit quotas: units are in id order, so unit u may
// take min(count_u, need - sum of counts before u) ids (its smallest ones).  One wavefront; a lane takes 8
// neighbouring units, and the counts of the next 512 are on their way while these are added up.  (The counts may
// just have been stored by other workgroups.)
__device__ inline void tie_quotas(uint32_t *row, uint32_t nunits, uint32_t need)
{
    constexpr uint32_t PER = 8, STEP = 64 * PER;
    const uint32_t lane = threadIdx.x & 63;
    uint32_t next[PER];
    auto load = [&](uint32_t base) {
#pragma unroll
        for (uint32_t z = 0; z < PER; ++z) {
            const uint32_t u = base + lane * PER + z;
            next[z] = u < nunits ? __hip_atomic_load(&row[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
        }
    };
    load(0);
    uint32_t carry = 0;                                        // ids of the bucket in the units before these
    for (uint32_t base = 0; base < nunits; base += STEP) {     // uniform
        uint32_t c[PER], mine = 0;
#pragma unroll
        for (uint32_t z = 0; z < PER; ++z) { c[z] = next[z]; mine += c[z]; }
        if (base + STEP < nunits && carry < need) load(base + STEP);      // (no ids left to take: the rest is all zeros)
        uint32_t incl = mine;
#pragma unroll
        for (uint32_t d = 1; d < 64; d <<= 1) {
            const uint32_t other = __shfl(incl, lane >= d ? lane - d : lane);
            if (lane >= d) incl += other;
        }
        uint32_t before = carry + incl - mine;                 // exclusive prefix in id order
#pragma unroll
        for (uint32_t z = 0; z < PER; ++z) {
            const uint32_t u = base + lane * PER + z;
            if (u < nunits) __hip_atomic_store(&row[u], before >= need ? 0u : min(c[z], need - before), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            before += c[z];
        }
        carry += __shfl(incl, 63);
    }
}

// Starting bucket bound of a query from the histogram of a sample of S of the n codes, by one wavefront.
// The bucket of the sample's r-th smallest qd is a bound that cannot fail (the sample is part of the
// array), but it lets r / S of all codes through.  The array's r-th smallest qd is about the sample's
// (r S / n)-th smallest, so the bound starts at the bucket where the sample's cumulative count reaches
// e + 5 sqrt(e) + 5 with e = r S / n (five standard deviations of the count above its mean: a query in
// ten million starts too low), or r if that is smaller.  Should that bucket hold fewer than r codes of the whole array after all, the
// selection sees fewer than r appended candidates and has the query redone by the three-pass path.
// Where so many codes tie in that bucket that more than 16 r would be appended, only the codes with ids up to
// twice the share of the bucket that is wanted are (kCrowdedLimit; ties are broken by id, and the sample's runs are spread
// over the array).  Where no order of the ids is known and more than `room` would be (kCrowdedSkip), the bound starts one
// bucket lower if that is likely to do (a standard deviation above the mean instead of five), and otherwise below all
// buckets, which flags the query.
// Before a pilot pass, which counts what is within its bound one by one, the bound is the bucket below (kCountBelow), and t0 the crowded
// bucket: that one is known to do, and how many codes it holds the histogram says well enough.
// (n = 0, with exact counts of a sample, and `more` in bucket more_in: r is its rank already; `all` codes, `scale` times the sample,
// of which all_r are wanted.)
// bound->guess: the same with two standard deviations (of rank guess_r where that is given), for a scan that can look again
// at the queries for which it is too low.
template <bool GUESS = true>
__device__ inline void starting_bound(const uint32_t *shist, uint32_t r, uint64_t n, Crowded crowded, Bound *bound, float room = 0.0f, uint32_t guess_r = 0,
                                      uint64_t all = 0, float scale = 0.0f, uint32_t all_r = 0, int more_in = -1, uint32_t more = 0)
{
    const int lane = threadIdx.x & 63;
    uint32_t c[4], cum[4];
    wave_prefix_of_buckets(shist, c, cum, more_in, more);
    const uint32_t total = __shfl(cum[3], 63);
    uint32_t rs = r;
    float e = 0.0f;
    if (n) {                                                  // 0: the sample's own r-th smallest
        all = n;
        scale = static_cast<float>(n) / static_cast<float>(total);
        all_r = r;
        e = static_cast<float>(r) * static_cast<float>(total) / static_cast<float>(n);
        const float want = e + 5.0f * sqrtf(e) + 5.0f;
        if (want < static_cast<float>(r)) rs = static_cast<uint32_t>(want) + 1u;
        guess_r = static_cast<uint32_t>(e + 2.0f * sqrtf(e)) + 2u;
    }
    int guess = 255;
    if constexpr (GUESS) {
        if (guess_r == 0 || guess_r > rs) guess_r = rs;
        int mine = -1;
#pragma unroll
        for (int z = 0; z < 4; ++z)
            if (cum[z] - c[z] < guess_r && cum[z] >= guess_r) mine = 4 * lane + z;
        const uint64_t where = __builtin_amdgcn_ballot_w64(mine >= 0);
        if (where) guess = __shfl(mine, __builtin_ctzll(where));
    }
#pragma unroll
    for (int z = 0; z < 4; ++z) {
        const uint32_t before = cum[z] - c[z];
        if (before < rs && cum[z] >= rs) {                    // one lane, one bucket
            uint32_t last = 0xFFFFFFFFu;
            const float expect = static_cast<float>(cum[z]) * scale;
            int t = 4 * lane + z;
            if (crowded == kCrowdedSkip && n && expect > room) t = static_cast<float>(before) >= e + sqrtf(e) ? t - 1 : -1;
            if (crowded == kCrowdedLimit && expect > 16.0f * static_cast<float>(all_r)) {
                const float upto = 2.0f * static_cast<float>(all) * static_cast<float>(rs - before) / static_cast<float>(c[z]);
                if (upto < 4294967040.0f) last = static_cast<uint32_t>(upto);
            }
            if (crowded == kCountBelow && expect > 16.0f * static_cast<float>(all_r)) *bound = Bound{t - 1, static_cast<uint32_t>(t), last, guess};
            else *bound = Bound{t, last == 0xFFFFFFFFu ? 256u : static_cast<uint32_t>(4 * lane + z), last, guess};
        }
    }
    if (lane == 63 && total < rs) *bound = Bound{255, 256u, 0xFFFFFFFFu, 255};
}

// Lowers query q's bucket bound to the bucket that holds its r-th best appended candidate (nothing
// happens while fewer than r are appended).  Called by
// a whole wavefront: lane l reads the counts of buckets 4l .. 4l+3, a wavefront prefix sum locates the
// bucket.  The counts only grow, so any snapshot of them gives a bound that is still valid later.
static __device__ __noinline__ void lower_bound_of(int q, uint32_t r, Bound *bound, const uint32_t *chist)
{
    const int lane = threadIdx.x & 63;
    uint32_t c[4];
#pragma unroll
    for (int z = 0; z < 4; ++z)
        c[z] = __hip_atomic_load(&chist[static_cast<size_t>(q) * 256 + 4 * lane + z], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t mine = c[0] + c[1] + c[2] + c[3];
    uint32_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t other = __shfl(incl, lane >= d ? lane - d : lane);
        if (lane >= d) incl += other;
    }
    uint32_t cum = incl - mine;                          // appended candidates in buckets below 4 * lane
    if (cum < r && incl >= r) {                          // at most one lane
        int tn = 4 * lane;
#pragma unroll
        for (int z = 0; z < 3; ++z) {
            cum += c[z];
            if (cum < r) tn = 4 * lane + z + 1;
        }
        atomicMin(&bound[q].t, tn);
    }
}

// The same from the low-byte plane of the codes (uint8 [n][m], the bytes pass one consumes).
template <int M>
__device__ inline void load_low_bytes(const uint8_t *__restrict__ plane, uint64_t i, uint32_t (&low)[M])
{
    if constexpr (M % 8 == 0) {
        const uint2 *p = reinterpret_cast<const uint2 *>(plane + i * M);
#pragma unroll
        for (int v = 0; v < M / 8; ++v) {
            const uint2 x = p[v];
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                low[8 * v + z] = (x.x >> (8 * z)) & 255u;
                low[8 * v + 4 + z] = (x.y >> (8 * z)) & 255u;
            }
        }
    } else if constexpr (M == 4) {
        const uint32_t x = *reinterpret_cast<const uint32_t *>(plane + i * 4);
#pragma unroll
        for (int z = 0; z < 4; ++z) low[z] = (x >> (8 * z)) & 255u;
    } else if constexpr (M == 2) {
        const uint32_t x = *reinterpret_cast<const uint16_t *>(plane + i * 2);
        low[0] = x & 255u; low[1] = (x >> 8) & 255u;
    } else {
        low[0] = plane[i];
    }
}
#endif

}  // namespace dcpq

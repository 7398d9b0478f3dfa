// Pass one of Alg. 3 (Sec. 3.3, "Scan step"): adc_low_bits over the whole code array with the
// 8-bit quantized small tables, and the candidate set of exactly the r smallest by (qd, id).
//
// The paper's capped buckets (one bucket per integer distance 0..254, ids appended in list
// order, read out by increasing bucket) have an order-independent meaning: a 256-bin histogram
// of qd fixes the threshold bucket T that holds the r-th candidate; every id with qd < T is a
// candidate and bucket T contributes its smallest ids.
//
// This file holds (a) the THREE-PASS path, which computes exactly that for any input in three
// streaming passes over the codes:
//   pass A  histogram of qd per query                       -> T and the number still needed from T
//   pass B  per (query, scan unit) count of qd == T         -> quota of bucket T per unit (prefix in id order)
//   pass C  collect ids with qd < T, and the first `quota` ids of bucket T in each unit
// followed by a per-query sort of the r keys (qd, id); and (b) the driver that runs the
// single-pass kernel of scan_fast.hip first and sends only the queries it flags through (a).
//
// Three-pass work layout: a wavefront owns one "unit" of consecutive codes and walks it 64 codes
// at a time (lane = code, fully coalesced 2m-byte loads), so id order inside a unit is
// (iteration, lane).  A workgroup is 4 wavefronts (the sample's 4, 8 or 16, the redo's 16) and serves a tile of QT queries whose u8 tables
// (QT * m * 256 bytes) sit in LDS; each lane gathers its m table bytes per query from LDS.
// Over a whole batch the passes are launches of their own; for the few flagged queries (as a rule none, their number is known on the
// device only) all of them and the sort are one launch (scan_redo_kernel).
#include <cmath>
#include <type_traits>

#include "common.h"
#include "redo_wait.h"
#include <mutex>

#include "scan_internal.h"

namespace dcpq {

constexpr int kScanThreads = 256;
constexpr int kScanWaves = kScanThreads / kWave;

enum ScanMode { kHist = 0, kTieCount = 1, kCollect = 2 };

// Queries are addressed by their position p in the active list: query id = qlist ? qlist[p] : p.
// Workspace arrays (hist, thr, tie, counter, keys) are indexed by p; qtab by the query id.
// CodeT: uint16_t (the codes as stored) or uint8_t (their low-byte plane).
struct ScanArrays {
    const uint8_t *qtab;
    const int *qlist;       // NULL: all queries
    uint32_t r;
    uint32_t *hist;         // [nq][256]     (kHist: accumulated)
    uint32_t *thr;          // [nq][2]       (kTieCount, kCollect: read)
    uint32_t *tie;          // [nq][nunits]  (kTieCount: counts out; kCollect: quotas in)
    uint32_t *counter;      // [nq]          (kCollect)
    uint64_t *keys;         // [nq][r]       (kCollect)
};

// The starting bounds are taken by the workgroup that finishes a query tile of the sample's histogram last, which saves a launch (4.5 us on
// a stream of short kernels).
struct TileEnd {
    uint32_t *done;         // a counter per tile, at zero on entry and again at the end; NULL: nothing follows
    Bound *bound;
    uint32_t want_r;        // of starting_bound
    uint64_t want_n;
    Crowded crowded;
    bool guess;             // a guess below the bound is asked for too
};

template <typename T>
__device__ inline T agent_load(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ inline void agent_store(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// One item of a pass: a unit for each of the WAVES wavefronts of a workgroup (u: this wavefront's, past the last: none), for the queries at positions q0 .. q0 + QT - 1.
template <int M, int QT, int MODE, typename CodeT, int WAVES>
__device__ __forceinline__ void scan_item(const CodeT *__restrict__ codes, uint64_t n_codes, uint32_t unit, uint32_t nunits, uint64_t unit_stride, int q0, int nqt,
                                          uint32_t u, const ScanArrays &w, uint8_t *smem)
{
    uint8_t *ltab = smem;                                                   // [QT][M][256]
    uint32_t *lhist = reinterpret_cast<uint32_t *>(smem + QT * M * 256);    // [QT][256] (kHist)
    const int tid = threadIdx.x, lane = tid & 63;

    __syncthreads();                           // previous item's LDS is no longer in use
    for (int q = 0; q < nqt; ++q) {            // stage the tile's tables (rows of absent queries are never read)
        const int qid = w.qlist ? w.qlist[q0 + q] : q0 + q;
        const uint4 *src = reinterpret_cast<const uint4 *>(w.qtab + static_cast<size_t>(qid) * M * 256);
        uint4 *dst = reinterpret_cast<uint4 *>(ltab + q * M * 256);
        for (int v = tid; v < M * 256 / 16; v += 64 * WAVES) dst[v] = src[v];
    }
    if (MODE == kHist)
        for (int v = tid; v < QT * 256; v += 64 * WAVES) lhist[v] = 0;
    __syncthreads();

    const uint64_t begin = static_cast<uint64_t>(u) * unit_stride;
    const uint64_t end = (u < nunits) ? min(n_codes, begin + unit) : begin;

    uint32_t T[QT], aux[QT];   // threshold bucket; kTieCount: running count, kCollect: quota left
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        T[q] = 0; aux[q] = 0;
        if (MODE != kHist && q < nqt) {
            T[q] = w.thr[2 * (q0 + q)];
            if (MODE == kCollect && u < nunits) aux[q] = w.tie[static_cast<size_t>(q0 + q) * nunits + u];
        }
    }

    for (uint64_t base = begin; base < end; base += kWave) {
        const uint64_t i = base + lane;
        const bool live = i < end;
        uint32_t low[M];
        if (live) {
            load_low_bytes<M>(codes, i, low);
        } else {
#pragma unroll
            for (int j = 0; j < M; ++j) low[j] = 0;
        }
#pragma unroll
        for (int q = 0; q < QT; ++q) {
            if (q >= nqt) continue;                               // uniform
            const uint8_t *t = ltab + q * (M * 256);
            uint32_t s = 0;
#pragma unroll
            for (int j = 0; j < M; ++j) s += t[j * 256 + low[j]];
            const uint32_t qd = min(s, 255u);                     // saturate: 255 = beyond qmax
            if (MODE == kHist) {
                if (live) atomicAdd(&lhist[q * 256 + qd], 1u);
            } else if (MODE == kTieCount) {
                aux[q] += __popcll(__ballot(live && qd == T[q]));
            } else {
                const bool below = live && qd < T[q];
                const bool tied = live && qd == T[q];
                const uint64_t tied_mask = __ballot(tied);
                bool take = below;
                if (tied_mask) {                                  // uniform
                    const uint32_t rank = __popcll(tied_mask & ((1ull << lane) - 1ull));
                    take = below || (tied && rank < aux[q]);
                    const uint32_t n_tied = __popcll(tied_mask);
                    aux[q] = aux[q] > n_tied ? aux[q] - n_tied : 0u;
                }
                const uint64_t take_mask = __ballot(take);
                if (take_mask) {                                  // uniform, rare
                    const uint32_t n_take = __popcll(take_mask);
                    uint32_t slot0 = 0;
                    if (lane == 0) slot0 = atomicAdd(&w.counter[q0 + q], n_take);
                    slot0 = __shfl(slot0, 0, kWave);
                    if (take) {
                        const uint32_t slot = slot0 + __popcll(take_mask & ((1ull << lane) - 1ull));
                        if (slot < w.r)   // exactly r ids are taken over the whole scan; guard anyway
                            w.keys[static_cast<size_t>(q0 + q) * w.r + slot] = make_key(qd, static_cast<uint32_t>(i));
                    }
                }
            }
        }
    }

    if (MODE == kHist) {
        __syncthreads();
        for (int v = tid; v < nqt * 256; v += 64 * WAVES) {
            const uint32_t c = lhist[v];
            if (c) atomicAdd(&w.hist[static_cast<size_t>(q0) * 256 + v], c);
        }
    } else if (MODE == kTieCount) {
        if (u < nunits && lane == 0) {
#pragma unroll
            for (int q = 0; q < QT; ++q)
                if (q < nqt) agent_store(&w.tie[static_cast<size_t>(q0 + q) * nunits + u], aux[q]);
        }
    }
}

// WAVES: wavefronts, and units of codes, per workgroup.
template <int M, int QT, int MODE, typename CodeT, int WAVES = kScanWaves>
__global__ __launch_bounds__(64 * WAVES) void scan_kernel(const CodeT *__restrict__ codes, uint64_t n_codes, uint32_t unit, uint32_t nunits,
                                                          uint64_t unit_stride, int nq, const ScanArrays w, const TileEnd end_of)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, wave = tid >> 6;
    const uint32_t nxb = (nunits + WAVES - 1) / WAVES;
    const uint64_t nitems = static_cast<uint64_t>((nq + QT - 1) / QT) * nxb;

    for (uint64_t item = blockIdx.x; item < nitems; item += gridDim.x) {
        const int q0 = static_cast<int>(item / nxb) * QT;
        const int nqt = min(QT, nq - q0);
        // (of the sample a workgroup takes units that lie far apart: neighbouring ones may hold the same code all over, whose counts queue for one word of LDS)
        const uint32_t xb = static_cast<uint32_t>(item % nxb), u = MODE == kHist && end_of.done ? xb + wave * nxb : xb * WAVES + wave;
        scan_item<M, QT, MODE, CodeT, WAVES>(codes, n_codes, unit, nunits, unit_stride, q0, nqt, u, w, smem);
        if (MODE == kHist && end_of.done) {
            // Everything this workgroup has added is in place before its count is.  (Histograms are only added to by
            // device-scope atomics, whose completion is all there is to wait
            // for; a release fence would write back the second-level cache once per workgroup: 100 us for the sample of 251
            // queries.)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            uint32_t *last = reinterpret_cast<uint32_t *>(smem);
            if (tid == 0) *last = atomicAdd(&end_of.done[q0 / QT], 1u) == nxb - 1;
            __syncthreads();
            const bool mine = *last != 0;
            __syncthreads();
            if (mine) {                                               // uniform
                if (tid == 0) agent_store(&end_of.done[q0 / QT], 0u);
                for (int q = wave; q < nqt; q += WAVES) {
                    const uint32_t *h = w.hist + static_cast<size_t>(q0 + q) * 256;
                    if (end_of.guess) starting_bound<true>(h, end_of.want_r, end_of.want_n, end_of.crowded, end_of.bound + q0 + q);
                    else starting_bound<false>(h, end_of.want_r, end_of.want_n, end_of.crowded, end_of.bound + q0 + q);
                }
            }
        }
    }
}

// ---- the flagged queries ------------------------------------------------------------------------------
constexpr int kRedoWaves = 16, kRedoThreads = 64 * kRedoWaves;
constexpr int redo_qt(int m) { return m <= 8 ? 8 : 64 / m; }              // queries of a tile
constexpr int redo_ahead(int m) { return m <= 8 ? 4 : 2; }                             // groups of 64 codes that a wavefront loads together
constexpr int redo_per_cu(int m) { return m <= 8 ? 2 : 1; }                // workgroups that a CU has the registers for
// In the threshold of a query, bucket | ids still needed from it << 32: it is there; the quotas of its units are there.
constexpr uint64_t kThresholdThere = 1ull << 31, kQuotasThere = 1ull << 30, kThresholdBucket = 511;

// A pass over one unit of codes by a wavefront, for a tile of nqt queries whose tables and thresholds are in LDS.  What it leaves for the next pass goes through
// device-scope atomics and stores; it waits for nothing.
template <int M, int QT, int MODE, typename CodeT>
__device__ __forceinline__ void redo_unit(const CodeT *__restrict__ codes, uint64_t n_codes, uint32_t unit, uint32_t nunits, uint32_t u, int q0, int nqt,
                                          const ScanArrays &w, const uint8_t *ltab, uint32_t *lhist, const uint64_t *s_thr)
{
    constexpr int AHEAD = redo_ahead(M), W = sizeof(CodeT), WORDS = M * W / 4, PIECE = WORDS < 4 ? WORDS : 4;       // dwords of a code; of a load
    struct __attribute__((aligned(4 * PIECE))) Piece { uint32_t v[PIECE]; };
    const int lane = threadIdx.x & 63;
    const uint64_t begin = static_cast<uint64_t>(u) * unit, end = min(n_codes, begin + unit);
    uint32_t T[QT], aux[QT];                                          // threshold bucket; kTieCount: running count, kCollect: quota left
#pragma unroll
    for (int q = 0; q < QT; ++q) {
        const int p = min(q, nqt - 1);
        T[q] = MODE == kHist ? 0u : static_cast<uint32_t>(s_thr[p] & kThresholdBucket);
        aux[q] = MODE == kCollect ? agent_load(&w.tie[static_cast<size_t>(q0 + p) * nunits + u]) : 0u;
    }
#pragma unroll
    for (int q = 0; q < QT; ++q) {                                    // (the same in all lanes)
        T[q] = __builtin_amdgcn_readfirstlane(T[q]);
        aux[q] = __builtin_amdgcn_readfirstlane(aux[q]);
    }
    for (uint64_t base0 = begin; base0 < end; base0 += 64 * AHEAD) {  // uniform
        uint32_t raw[AHEAD][WORDS];
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) {
            const Piece *from = reinterpret_cast<const Piece *>(codes + min(base0 + 64 * g + lane, end - 1) * M);
#pragma unroll
            for (int v = 0; v < WORDS / PIECE; ++v) {
                const Piece x = from[v];
#pragma unroll
                for (int z = 0; z < PIECE; ++z) raw[g][PIECE * v + z] = x.v[z];
            }
        }
#pragma unroll
        for (int g = 0; g < AHEAD; ++g) {
            const uint64_t i = base0 + 64 * g + lane;
            if (base0 + 64 * g >= end) break;                         // uniform
            const bool live = i < end;
            uint32_t low[M];
#pragma unroll
            for (int j = 0; j < M; ++j) low[j] = raw[g][j * W / 4] >> (j * W % 4 * 8) & 255u;
#pragma unroll
            for (int q = 0; q < QT; ++q) {
                if (q >= nqt) break;                                  // uniform
                const uint8_t *t = ltab + q * (M * 256);
                uint32_t s = 0;
#pragma unroll
                for (int j = 0; j < M; ++j) s += t[j * 256 + low[j]];
                const uint32_t qd = min(s, 255u);
                if (MODE == kHist) {
                    if (live) atomicAdd(&lhist[q * 256 + qd], 1u);
                } else if (MODE == kTieCount) {
                    aux[q] += __popcll(__ballot(live && qd == T[q]));
                } else {
                    const bool tied = live && qd == T[q];
                    const uint64_t tied_mask = __ballot(tied);
                    bool take = live && qd < T[q];
                    if (tied_mask) {                                  // uniform
                        take = take || (tied && static_cast<uint32_t>(__popcll(tied_mask & ((1ull << lane) - 1ull))) < aux[q]);
                        const uint32_t n_tied = __popcll(tied_mask);
                        aux[q] = aux[q] > n_tied ? aux[q] - n_tied : 0u;
                    }
                    const uint64_t take_mask = __ballot(take);
                    if (take_mask) {                                  // uniform, rare
                        uint32_t slot = 0;
                        if (lane == 0) slot = atomicAdd(&w.counter[q0 + q], static_cast<uint32_t>(__popcll(take_mask)));
                        slot = __shfl(slot, 0, kWave) + __popcll(take_mask & ((1ull << lane) - 1ull));
                        if (take && slot < w.r) agent_store(&w.keys[static_cast<size_t>(q0 + q) * w.r + slot], make_key(qd, static_cast<uint32_t>(i)));
                    }
                }
            }
        }
    }
    if (MODE == kTieCount && lane == 0) {
#pragma unroll
        for (int q = 0; q < QT; ++q)
            if (q < nqt) agent_store(&w.tie[static_cast<size_t>(q0 + q) * nunits + u], aux[q]);
    }
}

// The three passes and the sort for the flagged queries qlist[0 .. *nflag), in one launch: as four of them, where nothing is flagged, which is
// the rule, each took 4.5 us.
// Items are handed out in order -- the histogram's of all query tiles, then the tie counts', the collection's, the queries
// to sort -- by one counter, and an item waits for those of the pass before it: these have been handed out already, to workgroups that are running
// and wait, if at all, for items handed out earlier still, so that every wait ends whatever number of workgroups the chip holds at a time.
// (Should the counters not be this call's own, it is given up; redo_wait.h.  Queries that were not finished then get the first r ids.)
// What one item leaves for another goes through device-scope atomics, stores and loads, and is in place before the item is counted as done, or the word that
// others look at is set: the threshold of a query, which says whether it and the quotas are there.  (Those who wait look at it and not at the counts, whose
// additions their loads would queue.)
// done: items of a tile that are done, of all passes; ticket: the counter; thresholds and these are at zero on entry.
// An item is a share of the units, those a share's distance apart, of which a wavefront has one at most: as many shares as there are sixteens of units, and so
// many more, down to four units each, as fill the last round of workgroups.
// What bounds it: for few queries the latency of the loads of a unit, 64 codes of 64 to 256 groups one after the other, so that groups are loaded four at a time (two with
// longer codes); for many the table gathers and histogram counts in LDS.  Tiles of eight queries (four, two with longer codes) let two workgroups share a CU up
// to m = 8; with tiles of sixteen the three passes in one kernel ran out of registers.  N = 4.2e6, m = 8, of 130 queries 1 / 16 / 130 redone: 223 / 996 / 2223 us
// with those, a group at a time, 104 / 375 / 1550 so; m = 16, 9 of 100: 778 and 410.
template <int M, int QT, typename CodeT>
__global__ __launch_bounds__(kRedoThreads, 4 * redo_per_cu(M)) void scan_redo_kernel(const CodeT *__restrict__ codes, uint64_t n_codes, uint32_t unit, uint32_t nunits,
                                                              const uint32_t *__restrict__ nflag, const ScanArrays w, uint32_t *done, unsigned long long *ticket,
                                                              uint32_t n_pow2, int use_lds, uint64_t *__restrict__ spill, uint32_t *__restrict__ cand_id,
                                                              uint8_t *__restrict__ cand_qd)
{
    const uint32_t nq = *nflag;
    if (nq == 0) return;
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ unsigned long long s_item;
    __shared__ uint64_t s_thr[QT];
    __shared__ uint32_t s_last, s_there;
    uint32_t *lhist = reinterpret_cast<uint32_t *>(smem + QT * M * 256);      // [QT][256] behind the tables
    uint64_t *thr = reinterpret_cast<uint64_t *>(w.thr);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t tiles = (nq + QT - 1) / QT, sixteens = (nunits + kRedoWaves - 1) / kRedoWaves;
    constexpr uint32_t SLOTS = 256 * redo_per_cu(M);
    const uint64_t rounds = (static_cast<uint64_t>(tiles) * sixteens + SLOTS - 1) / SLOTS;
    const uint32_t parts = static_cast<uint32_t>(min(static_cast<uint64_t>((nunits + 3) / 4), rounds * SLOTS / tiles));       // ... of a tile; sixteens or more
    const uint64_t per = static_cast<uint64_t>(tiles) * parts, all = 3 * per + nq;
    const auto pause = [] { __builtin_amdgcn_s_sleep(16); };
    // thresholds of the tile's queries, once they say that `what` is there
    auto wait_for_thresholds = [&](uint32_t q0, uint32_t nqt, uint64_t what) {
        if (wave == 0) {
            uint64_t t = what;
            const bool there = wait_until([&] {
                if (static_cast<uint32_t>(lane) < nqt) t = agent_load(&thr[q0 + lane]);
                return static_cast<uint32_t>(__popcll(__ballot((t & what) != 0)));
            }, pause, 64, kRedoPatience);
            if (static_cast<uint32_t>(lane) < nqt) s_thr[lane] = t;
            if (lane == 0) {
                s_there = there;
                if (!there) atomicOr(ticket, kRedoGivenUp);
            }
        }
        __syncthreads();
        return s_there != 0;
    };
    auto wait_for_count = [&](const uint32_t *count, uint32_t n) {
        if (tid == 0) {
            s_there = wait_until([count] { return agent_load(count); }, pause, n, kRedoPatience);
            if (!s_there) atomicOr(ticket, kRedoGivenUp);
        }
        __syncthreads();
        return s_there != 0;
    };
    // counts the item; true for the last of its pass and tile
    auto finished = [&](uint32_t tile, uint32_t pass) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(&done[tile], 1u) == (pass + 1) * parts - 1;
        __syncthreads();
        return s_last != 0;
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
            const uint32_t pass = static_cast<uint32_t>(item / per), in_pass = static_cast<uint32_t>(item % per), tile = in_pass / parts, u = in_pass % parts + wave * parts;
            const uint32_t q0 = tile * QT, nqt = min(static_cast<uint32_t>(QT), nq - q0);
            constexpr uint32_t ROWS = M * 256 / 16;                   // tables of a query, in sixteen bytes
            for (uint32_t t = tid; t < nqt * ROWS; t += kRedoThreads)
                reinterpret_cast<uint4 *>(smem)[t] = reinterpret_cast<const uint4 *>(w.qtab + static_cast<size_t>(w.qlist[q0 + t / ROWS]) * M * 256)[t % ROWS];
            if (pass == 0) {
                for (uint32_t t = tid; t < nqt * 256; t += kRedoThreads) lhist[t] = 0;
            } else {
                if (!wait_for_thresholds(q0, nqt, pass == 1 ? kThresholdThere : kQuotasThere)) continue;       // uniform
            }
            __syncthreads();
            auto walk = [&](auto mode) __attribute__((always_inline)) {
                if (u < nunits) redo_unit<M, QT, decltype(mode)::value, CodeT>(codes, n_codes, unit, nunits, u, q0, nqt, w, smem, lhist, s_thr);
            };
            if (pass == 0) {
                walk(std::integral_constant<int, kHist>{});
                __syncthreads();
                for (uint32_t t = tid; t < nqt * 256; t += kRedoThreads)
                    if (lhist[t]) atomicAdd(&w.hist[static_cast<size_t>(q0) * 256 + t], lhist[t]);
                if (finished(tile, 0) && static_cast<uint32_t>(wave) < nqt) {
                    uint64_t *to = thr + q0 + wave;
                    exact_threshold(w.hist + static_cast<size_t>(q0 + wave) * 256, w.r,
                                    [to](uint32_t t, uint32_t need) { agent_store(to, static_cast<uint64_t>(need) << 32 | kThresholdThere | t); });
                }
            } else if (pass == 1) {
                walk(std::integral_constant<int, kTieCount>{});
                if (finished(tile, 1) && static_cast<uint32_t>(wave) < nqt) {
                    tie_quotas(w.tie + static_cast<size_t>(q0 + wave) * nunits, nunits, static_cast<uint32_t>(s_thr[wave] >> 32));
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                    if (lane == 0) agent_store(thr + q0 + wave, s_thr[wave] | kQuotasThere);
                }
            } else {
                walk(std::integral_constant<int, kCollect>{});
                finished(tile, 2);
            }
            continue;
        }
        const uint32_t p = static_cast<uint32_t>(item - 3 * per);
        const size_t out = static_cast<size_t>(w.qlist[p]) * w.r;
        if (given_up || !wait_for_count(&done[p / QT], 3 * parts)) {  // uniform
            for (uint32_t t = tid; t < w.r; t += kRedoThreads) { cand_id[out + t] = t; cand_qd[out + t] = 255; }
            continue;
        }
        uint64_t *a = use_lds ? reinterpret_cast<uint64_t *>(smem) : spill + static_cast<size_t>(p) * n_pow2;
        for (uint32_t t0 = tid; t0 < n_pow2; t0 += 4 * kRedoThreads) {
            uint64_t key[4];
#pragma unroll
            for (int z = 0; z < 4; ++z) key[z] = t0 + z * kRedoThreads < w.r ? agent_load(&w.keys[static_cast<size_t>(p) * w.r + t0 + z * kRedoThreads]) : ~0ull;
#pragma unroll
            for (int z = 0; z < 4; ++z)
                if (t0 + z * kRedoThreads < n_pow2) a[t0 + z * kRedoThreads] = key[z];
        }
        bitonic_sort(a, n_pow2);
        for (uint32_t t = tid; t < w.r; t += kRedoThreads) {
            cand_id[out + t] = static_cast<uint32_t>(a[t]);
            cand_qd[out + t] = static_cast<uint8_t>(a[t] >> 32);
        }
    }
}

// Thresholds and quotas as kernels of their own, a wavefront per query: for three passes over
// all queries of a batch, where the launches are worth it (each tile's queries would wait for the one workgroup that ends
// it: 21 queries over 1.6 M codes of one sub-code 738 us, 153 this way; 138 queries over 0.26 M 153 and 140).
__global__ __launch_bounds__(256) void threshold_kernel(const uint32_t *__restrict__ hist, int nq, uint32_t r, uint32_t *__restrict__ thr)
{
    const int q = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (q < nq) exact_threshold(hist + static_cast<size_t>(q) * 256, r, thr + 2 * q);
}

__global__ __launch_bounds__(64) void tie_quota_kernel(uint32_t *__restrict__ tie, uint32_t nunits, const uint32_t *__restrict__ thr)
{
    const int q = blockIdx.x;
    tie_quotas(tie + static_cast<size_t>(q) * nunits, nunits, thr[2 * q + 1]);
}

// Sort the r collected keys of each query by (qd, id) and split them into the two outputs.
// use_lds: the padded array fits the dynamic LDS allocation; otherwise it is sorted in `spill`.
__global__ __launch_bounds__(1024) void sort_candidates_kernel(const uint64_t *__restrict__ keys, uint32_t r, uint32_t n_pow2, int use_lds,
                                                              uint64_t *__restrict__ spill, uint32_t *__restrict__ cand_id, uint8_t *__restrict__ cand_qd)
{
    extern __shared__ __align__(16) uint8_t smem[];
    const int q = blockIdx.x;
    uint64_t *a = use_lds ? reinterpret_cast<uint64_t *>(smem) : spill + static_cast<size_t>(q) * n_pow2;
    for (uint32_t t = threadIdx.x; t < n_pow2; t += blockDim.x)
        a[t] = t < r ? keys[static_cast<size_t>(q) * r + t] : ~0ull;
    bitonic_sort(a, n_pow2);
    for (uint32_t t = threadIdx.x; t < r; t += blockDim.x) {
        const uint64_t key = a[t];
        cand_id[static_cast<size_t>(q) * r + t] = static_cast<uint32_t>(key);
        cand_qd[static_cast<size_t>(q) * r + t] = static_cast<uint8_t>(key >> 32);
    }
}

// Clears `n` 32-bit words (a fill kernel rather than a memset node, so that the call sequence
// stays safe to capture into a HIP graph).
__global__ void zero_words_kernel(uint32_t *p, size_t n)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

__global__ void fill_u64_kernel(uint64_t *p, size_t n, uint64_t v)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

int launch_zero_words(uint32_t *p, size_t nwords, hipStream_t st)
{
    if (!nwords) return DCPQ_OK;
    DCPQ_LAUNCH(kStageMisc, st, zero_words_kernel, dim3((nwords + 255) / 256), dim3(256), 0, p, nwords);
    DCPQ_CHECK_LAUNCH("zero_words_kernel");
    return DCPQ_OK;
}

__global__ void zero_and_fill_kernel(uint64_t *z, size_t nz, uint64_t *p, size_t n, uint64_t v)
{
    const size_t i = static_cast<size_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < nz) z[i] = 0;
    else if (i - nz < n) p[i - nz] = v;
}

int launch_zero_and_fill(uint64_t *z, size_t nz, uint64_t *p, size_t n, uint64_t v, hipStream_t st)
{
    DCPQ_LAUNCH(kStageMisc, st, zero_and_fill_kernel, dim3((nz + n + 255) / 256), dim3(256), 0, z, nz, p, n, v);
    DCPQ_CHECK_LAUNCH("zero_and_fill_kernel");
    return DCPQ_OK;
}

int launch_fill_u64(uint64_t *p, size_t n, uint64_t v, hipStream_t st)
{
    if (!n) return DCPQ_OK;
    DCPQ_LAUNCH(kStageMisc, st, fill_u64_kernel, dim3((n + 255) / 256), dim3(256), 0, p, n, v);
    DCPQ_CHECK_LAUNCH("fill_u64_kernel");
    return DCPQ_OK;
}

int launch_threshold(const uint32_t *hist, int nq, uint32_t r, uint32_t *thr, hipStream_t st)
{
    DCPQ_LAUNCH(kStageSelect, st, threshold_kernel, dim3((nq + 3) / 4), dim3(256), 0, hist, nq, r, thr);
    DCPQ_CHECK_LAUNCH("threshold_kernel");
    return DCPQ_OK;
}

int launch_tie_quota(uint32_t *tie, uint32_t nunits, int nq, const uint32_t *thr, hipStream_t st)
{
    DCPQ_LAUNCH(kStageSelect, st, tie_quota_kernel, dim3(nq), dim3(64), 0, tie, nunits, thr);
    DCPQ_CHECK_LAUNCH("tie_quota_kernel");
    return DCPQ_OK;
}

int launch_sort_candidates(const uint64_t *keys, int nq, uint32_t r, uint64_t *spill, uint32_t *cand_id, uint8_t *cand_qd, hipStream_t st)
{
    const uint32_t np2 = next_pow2(r);
    const bool use_spill = np2 > kSortLdsKeys;
    DCPQ_LAUNCH(kStageSelect, st, sort_candidates_kernel, dim3(nq), dim3(1024), use_spill ? 0 : sizeof(uint64_t) * np2,
                keys, r, np2, use_spill ? 0 : 1, spill, cand_id, cand_qd);
    DCPQ_CHECK_LAUNCH("sort_candidates_kernel");
    return DCPQ_OK;
}

constexpr int scan_qt(int m) { return m <= 8 ? 16 : 128 / m; }   // tables of a tile: <= 32 KiB of LDS

// Queries per tile of the single-pass kernel.  Large batches take the largest tile (most queries per
// byte of code stream); for m = 8 a batch that fits a smaller tile takes that one, so that a small
// batch does not pay for absent queries and the scan runs at the speed of the code stream.
int fast_query_tile(int m, int nq, int mode)
{
    if (mode == DCPQ_SCAN_TILE16 || mode == DCPQ_SCAN_TILE32 || mode == DCPQ_SCAN_TILE64) {
        const int qt = mode == DCPQ_SCAN_TILE16 ? 16 : mode == DCPQ_SCAN_TILE32 ? 32 : 64;
        return fast_table_bytes(m, qt) ? qt : 0;
    }
    switch (m) {
        case 4: return 64;
        case 8: return nq <= 16 ? 16 : nq <= 32 ? 32 : 64;
        case 16: return 32;
        case 32: return 16;
        default: return 0;
    }
}

ScanPlan plan_scan(uint64_t n_codes, int m, int nq, uint32_t r, int mode, size_t room)
{
    ScanPlan p{};
    p.qt = scan_qt(m);
    // Unit: enough wavefronts to fill the chip (256 CUs) several times over, 64..16384 codes each.
    const uint64_t qtiles = (static_cast<uint64_t>(nq) + p.qt - 1) / p.qt;
    uint64_t unit = 16384;
    while (unit > 64 && (n_codes + unit - 1) / unit * (qtiles ? qtiles : 1) < 8192) unit >>= 1;
    p.unit = static_cast<uint32_t>(unit);
    p.nunits = static_cast<uint32_t>((n_codes + unit - 1) / unit);
    const uint32_t np2 = next_pow2(r);
    const size_t Q = static_cast<size_t>(nq);
    size_t off = 0;
    p.off_hist = off;    off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
    p.off_thr = off;     off = align_up(off + sizeof(uint32_t) * 2 * Q, 256);
    p.off_counter = off; off = align_up(off + sizeof(uint32_t) * Q, 256);
    p.off_done = off;    off = align_up(off + sizeof(uint32_t) * 3 * qtiles, 256);
    p.fqt = static_cast<uint32_t>(mode == DCPQ_SCAN_THREE_PASS ? 0 : fast_query_tile(m, nq, mode));
    p.fast = p.fqt != 0;
    if (p.fast) {
        p.ntiles = static_cast<uint32_t>((Q + p.fqt - 1) / p.fqt);
        // workgroups along the codes, of 16 Ki codes and more (fewer, down to 4 Ki, on short arrays)
        const uint64_t rest = n_codes;
        // (a single tile does the same work in every workgroup, and one round of the 256 CUs measured
        // fastest for it; with several tiles the work per workgroup varies and more rounds even it out)
        // Several tiles: whole rounds of the 256 CUs (the tables of a tile leave a CU room for one workgroup; 11 tiles in
        // 1034 workgroups, 10 more than four rounds, take 1.10 ms, in 2035 0.99, in 1023 0.955).  64 workgroups per tile and
        // four rounds at least: a workgroup loads its tables and ends with its appends while its CU does nothing else (16 tiles,
        // N = 1e7: 1.54 ms with 128 per tile, 1.49 with 64).  Twice as many where they would be longer than 2^20 codes, since
        // the rounds end unevenly, the more so the longer a workgroup runs (64 tiles, N = 1e8: 41.1 ms with 128, 41.7 with 64, 43.5 with 32).
        const uint64_t lots = rest > (64ull << 20) ? 2 : 1;
        const uint64_t total = lots * (64ull * p.ntiles > 1024 ? 64ull * p.ntiles : 1024);
        const uint64_t want = p.ntiles == 1 ? 256 : ((total + 255) / 256 * 256) / p.ntiles;
        // (down to 4096 codes where the chip would be left half empty: 100 queries over 1 M codes are 2 tiles)
        uint64_t least = 16384;
        while (least > 4096 && (rest + least - 1) / least * p.ntiles < 192) least >>= 1;
        const uint64_t most = (rest + least - 1) / least;
        uint64_t fb = want < most ? want : most;
        if (fb < 1) fb = 1;
        uint64_t cpb = (rest + fb - 1) / fb;
        cpb = (cpb + 1023) / 1024 * 1024;
        p.codes_per_block = static_cast<uint32_t>(cpb);
        p.fblocks = static_cast<uint32_t>((rest + cpb - 1) / cpb);
        // (no more slices than stretches of 16 Ki codes: a slice has room for 1024 candidates or more, whatever r is)
        const uint64_t long_blocks = (rest + 16383) / 16384;
        p.slices = p.fblocks < static_cast<uint32_t>(kFastSlices) ? p.fblocks : kFastSlices;
        if (p.slices > long_blocks) p.slices = static_cast<uint32_t>(long_blocks);
        p.off_fzero = off;
        p.off_fcount = off;  off = align_up(off + sizeof(uint32_t) * Q * p.slices, 256);
        p.off_chist = off;   off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
        p.off_shist = off;   off = align_up(off + sizeof(uint32_t) * 256 * Q, 256);
        p.fzero_bytes = off - p.off_fzero;
        p.off_nflag = off;   off = align_up(off + 256, 256);
    }
    p.zero_bytes = off;
    p.off_tie = off;     off = align_up(off + sizeof(uint32_t) * Q * p.nunits, 256);
    p.off_keys = off;    off = align_up(off + sizeof(uint64_t) * Q * r, 256);
    p.off_spill = off;   // sort area in global memory, only when r keys do not fit the LDS sort
    if (np2 > kSortLdsKeys) off = align_up(off + sizeof(uint64_t) * Q * np2, 256);

    if (p.fast) {
        {
            const uint64_t share = 32ull * r / p.slices;         // 32 r per query in all: twice the even share
            p.cap = static_cast<uint32_t>(share < 1024 ? 1024 : share);
        }
        p.upd = r / 16 < 16 ? 16 : r / 16;                   // appends to one slice between bound updates
        const uint32_t want_sort = next_pow2(2 * r);
        p.sortcap = want_sort < kSortLdsKeys ? kSortLdsKeys : want_sort;
        // Sample: runs of 256 codes spread evenly over the array.  The larger it is, the closer the starting bound and the
        // fewer candidates are noted, but its cost grows with the number of queries: 32 r codes, 64 r for few
        // queries, and no more than holds 256 of the r wanted codes (the slack of the starting bound is a
        // third then), but at least 64 Ki.
        uint64_t mul = 4096 / (Q ? Q : 1);
        mul = mul < 32 ? 32 : mul > 64 ? 64 : mul;
        uint64_t s_codes = mul * r;
        const uint64_t enough = 256 * (n_codes / r);
        if (s_codes > enough) s_codes = enough;
        if (s_codes < 65536) s_codes = 65536;
        // With a pilot pass (below; worth its three extra launches when the histogram of the sample would take more
        // than 30 to 40 microseconds: searches of 300 queries over 1e7 codes 607 us without and 577 with it, 600 over 2e7 1179 and
        // 1134, 440 over 1e6 247 and 225; m = 16 at 1.6e8 and 2.3e8 of the product below, 150 and 220 queries over 1e6 codes: 178 and 184, 196 and
        // 190; m = 32 at 1.6e8 and 3.1e8, 77 and 148 queries: 234 and 242, 324 and 341; at m = 4 so many codes tie: 1000 queries over
        // 4e6 skewed codes 798 without it) the sample costs several times less per code, and is taken twice as large where it holds
        // few of the wanted codes (measured at N = 1e8, r = 4000, 4096 queries: sample and
        // scan together 41.25, 40.93, 40.72, 40.90 ms with 1, 2, 4, 8 times the sample; at N = 1e7, r = 5000
        // the larger sample costs what it saves).
        const uint64_t pilot_from = m == 8 ? 150000000ull : m == 16 ? 220000000ull : 330000000ull;
        const bool want_pilot = s_codes * Q * static_cast<uint64_t>(m) >= pilot_from;
        if (want_pilot && s_codes < 32 * (n_codes / r)) s_codes *= 2;
        if (s_codes > n_codes) s_codes = n_codes;
        p.s_unit = 256;
        p.s_nunits = static_cast<uint32_t>((s_codes + 255) / 256);
        p.s_stride = n_codes / p.s_nunits;
        if (p.s_stride < p.s_unit) p.s_stride = p.s_unit;
        // Pilot pass.  The histogram kernel gathers bytes and is an order of magnitude slower per (code, query)
        // than the single-pass kernel, so on a large array it reads only one run in kPilotEvery of the sample;
        // its histogram gives a bound below which the WHOLE sample is then counted by the single-pass kernel
        // itself (a few hundred hits per query), and those exact counts give the starting bound of the scan.
        p.s_count = static_cast<uint64_t>(p.s_nunits - 1) * p.s_unit;
        {
            const uint64_t last = static_cast<uint64_t>(p.s_nunits - 1) * p.s_stride;
            p.s_count += n_codes - last < p.s_unit ? n_codes - last : p.s_unit;
        }
        p.pilot = want_pilot && p.s_nunits >= 4 * kPilotEvery && p.s_count * 4 <= n_codes && p.s_stride >= p.s_unit;
        p.s1_nunits = p.pilot ? p.s_nunits / kPilotEvery : p.s_nunits;
        p.pilot_r = r;
        p.pilot_blocks = p.pilot_runs = 0;
        if (p.pilot) {
            const double e = static_cast<double>(r) * static_cast<double>(p.s_count) / static_cast<double>(n_codes);
            const double want = e + 5.0 * sqrt(e) + 5.0;            // as in sample_threshold_kernel
            if (want < static_cast<double>(r)) p.pilot_r = static_cast<uint32_t>(want) + 1u;
            // at least 16 runs (4096 codes) per workgroup against the cost of loading the tile's tables, about
            // 1024 workgroups in all
            uint32_t pb = p.s_nunits / 16;
            const uint32_t most = 1024 / p.ntiles ? 1024 / p.ntiles : 1;
            pb = pb > most ? most : pb;
            p.pilot_runs = (p.s_nunits + pb - 1) / pb;
            p.pilot_blocks = (p.s_nunits + p.pilot_runs - 1) / p.pilot_runs;
        }
        if (off - p.off_tie >= sizeof(Bound) * Q) {
            p.off_bound = p.off_tie;
        } else {                                             // r = 1 and a single unit
            p.off_bound = off;   off = align_up(off + sizeof(Bound) * Q, 256);
        }
        p.off_flags = off;   off = align_up(off + sizeof(uint32_t) * Q, 256);
        p.off_qlist = off;   off = align_up(off + sizeof(int32_t) * Q, 256);
        p.off_qsw = off;     off = align_up(off + static_cast<size_t>(p.ntiles) * fast_table_bytes(m, p.fqt), 256);
        p.off_fkeys = off;   off = align_up(off + sizeof(uint64_t) * Q * p.slices * p.cap, 256);
        p.off_fsort = off;
        if (p.sortcap > kSortLdsKeys) off = align_up(off + sizeof(uint64_t) * Q * p.sortcap, 256);
        // Room for the candidates that a wavefront notes for the end of its workgroup: two and a half times its even share of
        // r (of the rank wanted in the sample) candidates per query; what does not fit is appended one by one.
        {
            const uint64_t tile_q = Q < p.fqt ? Q : p.fqt;
            uint64_t share = tile_q * r / (static_cast<uint64_t>(p.fblocks) * kNoteWaves);
            if (p.pilot) {
                const uint64_t ps = tile_q * p.pilot_r / (static_cast<uint64_t>(p.pilot_blocks) * kNoteWaves);
                share = ps > share ? ps : share;
            }
            uint64_t w = (5 * share / 2 + 127) / 64 * 64;
            p.wcap = static_cast<uint32_t>(w > 4096 ? 4096 : w);
            const uint64_t blocks = p.fblocks > p.pilot_blocks ? p.fblocks : p.pilot_blocks;
            // a smaller workspace holds fewer of them, or none (every candidate is then appended by itself)
            const uint64_t fit = (room > off ? room - off : 0) / (sizeof(uint64_t) * p.ntiles * blocks * kNoteWaves) / 64 * 64;
            if (fit < p.wcap) p.wcap = static_cast<uint32_t>(fit);
            p.off_notes = off; off = align_up(off + sizeof(uint64_t) * p.ntiles * blocks * kNoteWaves * p.wcap, 256);
        }
    }
    p.total = off;
    return p;
}

template <int M, int MODE, int WAVES = kScanWaves, typename CodeT>
static void launch_scan_pass(int stage, const CodeT *codes, uint64_t n_codes, uint32_t unit, uint32_t nunits, uint64_t stride, int nq, const ScanArrays &w,
                             const TileEnd &end_of, hipStream_t st)
{
    constexpr int QT = scan_qt(M);
    const uint64_t nxb = (nunits + WAVES - 1) / WAVES;
    const uint64_t items = static_cast<uint64_t>((nq + QT - 1) / QT) * nxb, most = 1u << 20;
    const uint32_t grid = static_cast<uint32_t>(items < most ? (items ? items : 1) : most);
    const size_t lds = static_cast<size_t>(QT) * M * 256 + (MODE == kHist ? QT * 256 * 4 : 0);
    DCPQ_LAUNCH(stage, st, (scan_kernel<M, QT, MODE, CodeT, WAVES>), dim3(grid), dim3(64 * WAVES), lds, codes, n_codes, unit, nunits, stride, nq, w, end_of);
}

static ScanArrays redo_arrays(const uint8_t *qtab, const int *qlist, uint32_t r, uint8_t *base, const ScanPlan &p)
{
    auto words = [&](size_t off) { return reinterpret_cast<uint32_t *>(base + off); };
    return ScanArrays{qtab, qlist, r, words(p.off_hist), words(p.off_thr), words(p.off_tie), words(p.off_counter), reinterpret_cast<uint64_t *>(base + p.off_keys)};
}

// The three passes for all nq queries.  The counters (zero_bytes of the workspace) are at zero.
template <int M, typename CodeT>
static int launch_three_pass(const CodeT *codes, uint64_t n_codes, const uint8_t *qtab, int nq, uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, uint8_t *base,
                             const ScanPlan &p, hipStream_t st)
{
    const ScanArrays w = redo_arrays(qtab, nullptr, r, base, p);
    launch_scan_pass<M, kHist>(kStageScanHist, codes, n_codes, p.unit, p.nunits, p.unit, nq, w, TileEnd{}, st);
    DCPQ_CHECK_LAUNCH("scan_kernel<hist>");
    int rc = launch_threshold(w.hist, nq, r, w.thr, st);
    if (rc) return rc;
    launch_scan_pass<M, kTieCount>(kStageScanTieCount, codes, n_codes, p.unit, p.nunits, p.unit, nq, w, TileEnd{}, st);
    DCPQ_CHECK_LAUNCH("scan_kernel<tiecount>");
    rc = launch_tie_quota(w.tie, p.nunits, nq, w.thr, st);
    if (rc) return rc;
    launch_scan_pass<M, kCollect>(kStageScanCollect, codes, n_codes, p.unit, p.nunits, p.unit, nq, w, TileEnd{}, st);
    DCPQ_CHECK_LAUNCH("scan_kernel<collect>");
    return launch_sort_candidates(w.keys, nq, r, reinterpret_cast<uint64_t *>(base + p.off_spill), cand_id, cand_qd, st);
}

// The same for the queries that the single pass has flagged.
template <int M, typename CodeT>
static int launch_redo(const CodeT *codes, uint64_t n_codes, const uint8_t *qtab, int nq, uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, uint8_t *base,
                       const ScanPlan &p, hipStream_t st)
{
    constexpr int QT = redo_qt(M);
    static_assert(2 * QT >= scan_qt(M), "tiles of the redo have counters in two of the rows for tiles of scan_qt(M) queries");
    const ScanArrays w = redo_arrays(qtab, reinterpret_cast<const int *>(base + p.off_qlist), r, base, p);
    const uint32_t np2 = next_pow2(r);
    const bool spill = np2 > kSortLdsKeys;
    size_t lds = static_cast<size_t>(QT) * M * 256 + QT * 256 * 4;
    if (!spill && sizeof(uint64_t) * np2 > lds) lds = sizeof(uint64_t) * np2;
    const int rc = allow_dynamic_lds(reinterpret_cast<const void *>(&scan_redo_kernel<M, QT, CodeT>), static_cast<int>(lds));
    if (rc) return rc;
    // as many workgroups as the chip holds at once (more would come when there is nothing left to hand out)
    const size_t qtiles = (static_cast<size_t>(nq) + p.qt - 1) / p.qt;
    uint32_t *nflag = reinterpret_cast<uint32_t *>(base + p.off_nflag), *done = reinterpret_cast<uint32_t *>(base + p.off_done) + qtiles;
    DCPQ_LAUNCH(kStageScanCollect, st, (scan_redo_kernel<M, QT, CodeT>), dim3(512), dim3(kRedoThreads), lds, codes, n_codes, p.unit,
                p.nunits, nflag, w, done, reinterpret_cast<unsigned long long *>(nflag + 2), np2, spill ? 0 : 1,
                reinterpret_cast<uint64_t *>(base + p.off_spill), cand_id, cand_qd);
    DCPQ_CHECK_LAUNCH("scan_redo_kernel");
    return DCPQ_OK;
}

// The sample's histogram: wavefronts per workgroup.  They share the tables of a tile, 48 KB of LDS with the counts at m = 8: with four of them a CU holds 12,
// with 16 as many as it can.  But a CU that gets one workgroup more than the others is the last one: the fewest units per CU
// decide, and more wavefronts per workgroup where these are equal (251 queries, 65536 codes, m = 8: 46 us with four, 33 with 16; 136 queries, m = 16, 17 tiles
// of 256 units, where 16 make 272 workgroups: 12 us more).
static int sample_waves(uint64_t tiles, uint64_t units)
{
    auto per_cu = [&](uint64_t waves) { return (tiles * ((units + waves - 1) / waves) + 255) / 256 * waves; };
    const uint64_t c4 = per_cu(4), c8 = per_cu(8), c16 = per_cu(16);
    return c16 <= c8 && c16 <= c4 ? 16 : c8 <= c4 ? 8 : 4;
}

template <int M, typename CodeT>
static int launch_sample_hist_m(const CodeT *codes, uint64_t n_codes, const uint8_t *qtab, int nq, uint32_t r,
                                uint32_t *shist, const ScanPlan &p, const TileEnd &end_of, hipStream_t st)
{
    // (with a pilot pass: runs 0, kPilotEvery, 2 kPilotEvery, ... of the sample)
    const uint64_t stride = p.pilot ? p.s_stride * kPilotEvery : p.s_stride;
    ScanArrays w{};
    w.qtab = qtab;
    w.r = r;
    w.hist = shist;
    auto launch = [&](auto waves) {
        launch_scan_pass<M, kHist, decltype(waves)::value>(kStageScanHist, codes, n_codes, p.s_unit, p.s1_nunits, stride, nq, w, end_of, st);
    };
    switch (sample_waves((nq + scan_qt(M) - 1) / scan_qt(M), p.s1_nunits)) {
    case 16: launch(std::integral_constant<int, 16>{}); break;
    case 8: launch(std::integral_constant<int, 8>{}); break;
    default: launch(std::integral_constant<int, kScanWaves>{});
    }
    DCPQ_CHECK_LAUNCH("scan_kernel<sample hist>");
    return DCPQ_OK;
}

// want_r, want_n, crowded: rank wanted, size of the array the sample stands for, what becomes of crowded buckets (see starting_bound)
template <typename CodeT>
int launch_sample_hist(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r,
                       uint32_t *shist, const ScanPlan &p, uint32_t want_r, uint64_t want_n, Crowded crowded, bool guess, Bound *bound,
                       uint32_t *done, hipStream_t st)
{
    TileEnd e{};
    e.done = done;
    e.bound = bound;
    e.crowded = crowded;
    e.guess = guess;
    e.want_r = want_r;
    e.want_n = want_n;
    switch (m) {
        case 4: return launch_sample_hist_m<4, CodeT>(codes, n_codes, qtab, nq, r, shist, p, e, st);
        case 8: return launch_sample_hist_m<8, CodeT>(codes, n_codes, qtab, nq, r, shist, p, e, st);
        case 16: return launch_sample_hist_m<16, CodeT>(codes, n_codes, qtab, nq, r, shist, p, e, st);
        case 32: return launch_sample_hist_m<32, CodeT>(codes, n_codes, qtab, nq, r, shist, p, e, st);
        default: return fail(DCPQ_EUNSUPPORTED, "sample histogram: m=%d not supported", m);
    }
}

template int launch_sample_hist<uint16_t>(const uint16_t *, uint64_t, int, const uint8_t *, int, uint32_t, uint32_t *,
                                          const ScanPlan &, uint32_t, uint64_t, Crowded, bool, Bound *, uint32_t *, hipStream_t);
template int launch_sample_hist<uint8_t>(const uint8_t *, uint64_t, int, const uint8_t *, int, uint32_t, uint32_t *,
                                         const ScanPlan &, uint32_t, uint64_t, Crowded, bool, Bound *, uint32_t *, hipStream_t);

template <int M, typename CodeT>
static int launch_scan_m(const CodeT *codes, uint64_t n_codes, const uint8_t *qtab, int nq, uint32_t r,
                         uint32_t *cand_id, uint8_t *cand_qd, void *ws, size_t room, int mode, bool cleared, hipStream_t st, const CellsArea *cells)
{
    const ScanPlan p = plan_scan(n_codes, M, nq, r, mode, room);
    uint8_t *base = static_cast<uint8_t *>(ws);
    int rc = DCPQ_OK;
    if (!cleared) rc = launch_zero_words(reinterpret_cast<uint32_t *>(base), p.zero_bytes / sizeof(uint32_t), st);
    if (rc) return rc;
    if (!p.fast)
        return launch_three_pass<M, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, base, p, st);
    rc = launch_scan_fast(codes, n_codes, M, qtab, nq, r, cand_id, cand_qd, base, p, cells, st);
    if (rc) return rc;
    // queries the single pass could not finish (their count is known on the device only)
    if constexpr (M >= 4) return launch_redo<M, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, base, p, st);
    return DCPQ_OK;
}

template <typename CodeT>
static int launch_scan_any(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r,
                           uint32_t *cand_id, uint8_t *cand_qd, void *ws, size_t room, int mode, bool cleared, hipStream_t st, const CellsArea *cells)
{
    if (nq == 0) return DCPQ_OK;
    switch (m) {
        case 1: return launch_scan_m<1, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        case 2: return launch_scan_m<2, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        case 4: return launch_scan_m<4, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        case 8: return launch_scan_m<8, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        case 16: return launch_scan_m<16, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        case 32: return launch_scan_m<32, CodeT>(codes, n_codes, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
        default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
    }
}

// Enough for every algorithm the caller may ask for, in a workspace of `room` bytes.
static size_t scan_bytes_of_all_modes(uint64_t n_codes, int m, int nq, uint32_t r, size_t room)
{
    size_t most = 0;
    const int modes[] = {DCPQ_SCAN_AUTO, DCPQ_SCAN_THREE_PASS, DCPQ_SCAN_TILE16, DCPQ_SCAN_TILE32, DCPQ_SCAN_TILE64};
    for (int mode : modes) {
        const size_t t = plan_scan(n_codes, m, nq, r, mode, room).total;
        most = t > most ? t : most;
    }
    return most;
}

size_t scan_least_bytes(uint64_t n_codes, int m, int nq, uint32_t r) { return scan_bytes_of_all_modes(n_codes, m, nq, r, 0); }

size_t scan_clear_words(uint64_t n_codes, int m, int nq, uint32_t r, int mode) { return plan_scan(n_codes, m, nq, r, mode).zero_bytes / sizeof(uint32_t); }

int launch_scan(const uint16_t *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r,
                uint32_t *cand_id, uint8_t *cand_qd, void *ws, size_t room, int mode, bool cleared, hipStream_t st, const CellsArea *cells)
{
    return launch_scan_any(codes, n_codes, m, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
}

int launch_scan(const uint8_t *plane, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r,
                uint32_t *cand_id, uint8_t *cand_qd, void *ws, size_t room, int mode, bool cleared, hipStream_t st, const CellsArea *cells)
{
    return launch_scan_any(plane, n_codes, m, qtab, nq, r, cand_id, cand_qd, ws, room, mode, cleared, st, cells);
}

}  // namespace dcpq

using namespace dcpq;

extern "C" int dcpq_scan_query_tile(int m)
{
    if (!m_supported(m)) return 0;
    const int f = fast_query_tile(m, 1 << 30, DCPQ_SCAN_AUTO);
    return f ? f : scan_qt(m);
}

extern "C" int dcpq_scan_plan(uint64_t n_codes, int m, int nq, uint32_t r, int mode, uint64_t *info, int ninfo)
{
    clear_error();
    DCPQ_REQUIRE(info && ninfo >= 6, "scan_plan: info must hold 6 values");
    DCPQ_REQUIRE(nq >= 1 && n_codes >= 1 && r >= 1, "scan_plan: empty problem");
    if (!m_supported(m)) return fail(DCPQ_EUNSUPPORTED, "scan_plan: m=%d not supported", m);
    const ScanPlan p = plan_scan(n_codes, m, nq, r, mode);
    info[0] = p.fast ? p.fqt : p.qt;
    info[1] = p.fast ? p.ntiles : (static_cast<uint64_t>(nq) + p.qt - 1) / p.qt;
    info[2] = p.fast ? p.fblocks : 0;
    info[3] = p.fast ? p.codes_per_block : p.unit;
    info[4] = p.fast ? p.slices : 0;
    info[5] = p.fast ? p.cap : 0;
    if (ninfo >= 10) {
        info[6] = p.fast ? p.s_nunits : 0;
        info[7] = p.fast ? p.s_stride : 0;
        info[8] = p.fast && p.pilot ? kPilotEvery : (p.fast ? 1 : 0);
        info[9] = p.fast ? p.pilot_r : 0;
    }
    if (ninfo >= 11) info[10] = scan_least_bytes(n_codes, m, nq, r);
    return DCPQ_OK;
}

extern "C" size_t dcpq_scan_workspace_bytes(uint64_t n_codes, int m, int nq, uint32_t r)
{
    if (nq <= 0 || !m_supported(m) || n_codes == 0 || r == 0 || r > (1u << 26)) return 0;
    return scan_bytes_of_all_modes(n_codes, m, nq, r, ~static_cast<size_t>(0));
}

template <typename CodeT>
static int scan_checked(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r,
                        uint32_t *cand_id, uint8_t *cand_qd, void *workspace, size_t workspace_bytes, int mode,
                        void *stream)
{
    clear_error();
    DCPQ_REQUIRE(nq >= 0, "scan_candidates: nq=%d", nq);
    DCPQ_REQUIRE(mode == DCPQ_SCAN_AUTO || mode == DCPQ_SCAN_THREE_PASS || mode == DCPQ_SCAN_TILE16 ||
                     mode == DCPQ_SCAN_TILE32 || mode == DCPQ_SCAN_TILE64,
                 "scan_candidates: mode=%d", mode);
    if (!m_supported(m)) return fail(DCPQ_EUNSUPPORTED, "scan_candidates: m=%d not supported", m);
    if (mode >= DCPQ_SCAN_TILE16 && fast_query_tile(m, nq, mode) == 0)
        return fail(DCPQ_EUNSUPPORTED, "scan_candidates: no single-pass kernel for m=%d with the tile of mode %d", m, mode);
    DCPQ_REQUIRE(n_codes >= 1 && n_codes < (1ull << 32), "scan_candidates: n_codes=%llu must be in [1, 2^32)",
                 static_cast<unsigned long long>(n_codes));
    DCPQ_REQUIRE(r >= 1 && r <= n_codes, "scan_candidates: r=%u must be in [1, n_codes]", r);
    DCPQ_REQUIRE(r <= (1u << 26), "scan_candidates: r=%u above the supported 2^26", r);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(codes && qtab && cand_id && cand_qd && workspace, "scan_candidates: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "scan_candidates: workspace must be 256-byte aligned");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(codes) & 15) == 0 && (reinterpret_cast<uintptr_t>(qtab) & 15) == 0,
                 "scan_candidates: codes (or their plane) and qtab must be 16-byte aligned");
    const size_t need = scan_least_bytes(n_codes, m, nq, r);
    if (workspace_bytes < need)
        return fail(DCPQ_EWORKSPACE, "scan_candidates: workspace %zu < %zu bytes", workspace_bytes, need);
    return launch_scan(codes, n_codes, m, qtab, nq, r, cand_id, cand_qd, workspace, workspace_bytes, mode, false, as_stream(stream));
}

extern "C" int dcpq_scan_candidates(const uint16_t *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq,
                                    uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, void *workspace,
                                    size_t workspace_bytes, void *stream)
{
    return scan_checked(codes, n_codes, m, qtab, nq, r, cand_id, cand_qd, workspace, workspace_bytes,
                        DCPQ_SCAN_AUTO, stream);
}

extern "C" int dcpq_scan_candidates_packed(const uint8_t *plane, uint64_t n_codes, int m, const uint8_t *qtab, int nq,
                                           uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, void *workspace,
                                           size_t workspace_bytes, int mode, void *stream)
{
    return scan_checked(plane, n_codes, m, qtab, nq, r, cand_id, cand_qd, workspace, workspace_bytes, mode, stream);
}

extern "C" int dcpq_scan_candidates_mode(const uint16_t *codes, uint64_t n_codes, int m, const uint8_t *qtab,
                                         int nq, uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, void *workspace,
                                         size_t workspace_bytes, int mode, void *stream)
{
    return scan_checked(codes, n_codes, m, qtab, nq, r, cand_id, cand_qd, workspace, workspace_bytes, mode, stream);
}

// ---- the entry point that allocates nothing ------------------------------------------------------
// For callers that cannot call hipMalloc (code under graph capture, tight serving loops, harnesses
// that forbid allocation) and have no workspace to hand over: the scan's workspace is this array,
// which every GPU the library runs on holds from the first call until the process ends.
constexpr size_t kStaticScratchBytes = DCPQ_STATIC_SCRATCH_BYTES;
// (the counters of finished workgroups and, at r = 1, the bounds come on top of what the stated size has always admitted)
constexpr size_t kStaticRoom = kStaticScratchBytes + (256u << 10);
static __device__ __align__(256) unsigned char scratch[kStaticRoom];

namespace {
constexpr int kMostDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMostDevices];      // device address of `scratch` on each GPU (the array's name is only a host-side stand-in)

// Device address of the current device's copy of the array, looked up once per device.
int static_scratch(void **out)
{
    int dev = 0;
    DCPQ_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMostDevices) return fail(DCPQ_EUNSUPPORTED, "scan_candidates_static: device %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        DCPQ_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(DCPQ_EHIP, "scan_candidates_static: no device address for the static scratch array");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return DCPQ_OK;
}
}  // namespace

extern "C" size_t dcpq_static_scratch_bytes(void) { return kStaticScratchBytes; }

extern "C" int dcpq_scan_candidates_static(const uint16_t *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq,
                                           uint32_t r, uint32_t *cand_id, uint8_t *cand_qd, void *stream)
{
    clear_error();
    // the size check comes first: a problem that does not fit is refused before the device is touched
    if (nq > 0 && m_supported(m) && n_codes >= 1 && r >= 1 && r <= (1u << 26)) {
        const size_t need = scan_least_bytes(n_codes, m, nq, r);
        if (need > kStaticRoom)
            return fail(DCPQ_EWORKSPACE, "scan_candidates_static: the scan needs %zu bytes of scratch, the static array holds %zu",
                        need, kStaticRoom);
    }
    void *ws = nullptr;
    if (nq > 0) {
        const int rc = static_scratch(&ws);
        if (rc) return rc;
    }
    // every counter the kernels expect at zero is cleared by the scan itself (a fill kernel, so the
    // call may be captured), whatever the previous call left in the array
    return scan_checked(codes, n_codes, m, qtab, nq, r, cand_id, cand_qd, ws, kStaticRoom, DCPQ_SCAN_AUTO, stream);
}

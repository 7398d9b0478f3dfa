// Pass one over codes sorted into cells (m = 8): the same candidate set as the other forms of the scan, without looking at
// every (query, code) pair.
//
// The low bytes of a sub-quantizer name up to 256 derived centroids; those are split into 16 groups of near ones (by distance,
// once per call).  For a query, the smallest quantized entry of a group is a lower bound of the entries in it, and the sum
// of these over a code's groups (its 4-bit group numbers, "nibbles") is a lower bound of its integer distance.
// The codes are sorted by the nibbles of their first five sub-quantizers (the "cell"), so that a query tests whole cells: a
// cell whose bound, with the smallest entry of every other sub-quantizer added, lies above the query's bucket bound holds
// no candidate.  Of the codes of the other cells the remaining three nibbles are looked up, and the codes whose lower bound is
// within the bucket bound -- little more than the candidates themselves -- get their integer distance from the 256-entry
// tables, as in the other scans.  Nothing is approximate: what is skipped is proven to lie above the bound.
// Of 1e8 random codes 1.6 % are looked up for a query and 1.1e-4 settled (r = 4000); of 1e7 encoded vectors 0.2 % and 5e-4.
//
// Where the groups say little (codebooks without near centroids, a bound that most cells are within) this saves nothing:
// cells_decide_kernel estimates both costs on a sample of the codes and sets the flag by which either these kernels or the
// single-pass scan return at once (no host synchronization).  A batch that is not served pays about 60 us for that
// (the median of 73 searches, timed twice; single ones of a millisecond up to 110).
//
// Measured, whole searches, on codebooks of 16 parents per sub-quantizer, which the groups meet: N = 1e8, 4096 queries,
// r = 4000: 41.1 -> 8.6 to 9.1 ms (sorting 1.8, scan 4.4 to 5, pass two 1.5); N = 1e7 encoded vectors, 1000 queries, r = 2000: 1.49 -> 0.72 ms
// (sorting 0.21, scan 0.20).  On quantizers trained by Alg. 2 it depends on the vectors: of a mixture of 1024 tight components in
// 128 dimensions 1.2e7 codes, 4096 queries, r = 2000 7.1 -> 2.5 ms, 4.2e6 codes, 2000 queries 1.86 -> 1.58; of Gaussian vectors, Gaussian ones
// with a decaying spectrum and normalised ones of 4096 wide components every batch was declined (2 to 6 % of 1.05 to 1.5 ms, 1 to 2 % of 6).
#include "lds_access.h"
#include "scan_internal.h"

namespace dcpq {

constexpr int kM = 8;
constexpr int kGroupsPerSub = 16;            // a nibble
constexpr int kKeyNibbles = 5, kKeyBits = 4 * kKeyNibbles;     // the cells: 2^20
constexpr int kBinBits = kKeyBits / 2;       // both passes of the sort
constexpr uint32_t kSampleCodes = 1024;      // codes the decision looks at ...

constexpr uint32_t kSampleQueries = 256;     // ... of no more queries than these

// counters of a call, all zero at its start
struct CellsCtl {
    uint32_t use;                        // set by the decision: the cells serve this batch
    uint32_t pad;
    // of the decision: (query, sample code) pairs within the bound (bits 0 .. 23), in cells to be looked at (24 .. 47), and
    // workgroups that have added theirs (48 ..)
    unsigned long long sums;
};

// ---- groups of near derived centroids --------------------------------------------------------------
// One workgroup per sub-quantizer, four threads per derived centroid: 16 seeds, each the centroid farthest from those before
// it, then one round of {mean, nearest mean}.  Whatever the split, the bounds taken from it hold; it only decides how tight
// they are.  A chain of short steps: the rows lie in LDS, 16 bytes a read, at an odd number of 16-byte units, and a step is a
// reduction without the LDS inside a wavefront and one atomic for each of these (dsub = 16: 18 us; 26 with shuffles of 64-bit keys through the
// LDS, 52 with a thread per centroid and single floats, two rounds).  Workgroups m and above clear the counters of the call.
__host__ __device__ inline int group_pitch(int dsub) { return ((dsub + 3) / 4 | 1) * 4; }      // floats
// v of the lane that is N lanes on, around the row of 16; of the lane whose number differs in the bits of X, within four.
template <int N>
__device__ inline uint32_t around_row(uint32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, true); }
template <int X>
__device__ inline float within_four(float v)
{
    constexpr int perm = (0 ^ X) | (1 ^ X) << 2 | (2 ^ X) << 4 | (3 ^ X) << 6;
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), perm, 0xF, 0xF, true));
}

__global__ __launch_bounds__(1024) void cells_group_kernel(const float *__restrict__ derived, int m, int dsub, int small_bits,
                                                           uint8_t *__restrict__ map, uint32_t *__restrict__ clear, uint32_t nclear)
{
    const int tid = threadIdx.x;
    if (static_cast<int>(blockIdx.x) >= m) {
        const uint32_t nb = gridDim.x - m;
        for (uint32_t t = (blockIdx.x - m) * 1024 + tid; t < nclear / 4; t += nb * 1024) reinterpret_cast<uint4 *>(clear)[t] = make_uint4(0, 0, 0, 0);
        return;
    }
    extern __shared__ __align__(16) float group_lds[];
    __shared__ uint32_t far[kGroupsPerSub];                      // the centroid farthest from its seed: distance (24 bits), 255 - number
    __shared__ int cnt[kGroupsPerSub];
    const int j = blockIdx.x, ks = 1 << small_bits, pitch = group_pitch(dsub), nv = (dsub + 3) / 4;
    float *rows = group_lds, *mean = group_lds + ks * pitch;                 // [ks][pitch], [16][pitch]
    const int e = (tid >> 2) & (ks - 1), part = tid & 3;
    for (int t = tid; t < ks * pitch; t += 1024) {
        const int te = t / pitch, d = t - te * pitch;
        rows[t] = d < dsub ? derived[(static_cast<size_t>(j) * ks + te) * dsub + d] : 0.0f;
    }
    for (int t = tid; t < kGroupsPerSub * pitch; t += 1024) mean[t] = 0.0f;
    if (tid < kGroupsPerSub) { far[tid] = 0; cnt[tid] = 0; }
    __syncthreads();
    const float4 *row = reinterpret_cast<const float4 *>(rows + e * pitch);
    auto distance = [&](const float *to) {
        const float4 *c = reinterpret_cast<const float4 *>(to);
        float s = 0.0f;
        for (int v = part; v < nv; v += 4) {
            const float4 a = row[v], b = c[v];
            s += (a.x - b.x) * (a.x - b.x) + (a.y - b.y) * (a.y - b.y) + (a.z - b.z) * (a.z - b.z) + (a.w - b.w) * (a.w - b.w);
        }
        s += within_four<1>(s);
        return s + within_four<2>(s);
    };
    float best = 3.0e38f;
    int label = 0, seed = 0;                                     // (the first seed: centroid 0)
    for (int g = 0; g < kGroupsPerSub; ++g) {
        const float s = distance(rows + seed * pitch);
        if (s < best) { best = s; label = g; }
        uint32_t key = (__float_as_uint(best) & ~255u) | static_cast<uint32_t>(255 - e);       // (distances are >= +0: they order like their bits)
        key = max(key, around_row<4>(key));
        key = max(key, around_row<8>(key));
        const uint32_t farthest = max(max(__builtin_amdgcn_readlane(key, 0), __builtin_amdgcn_readlane(key, 16)),
                                      max(__builtin_amdgcn_readlane(key, 32), __builtin_amdgcn_readlane(key, 48)));
        if ((tid & 63) == 0) atomicMax(&far[g], farthest);
        __syncthreads();
        seed = 255 - static_cast<int>(far[g] & 255u);
    }
    if (tid < 4 * ks) {
        if (part == 0) atomicAdd(&cnt[label], 1);
        for (int d = part; d < dsub; d += 4) atomicAdd(&mean[label * pitch + d], rows[e * pitch + d]);
    }
    __syncthreads();
    for (int t = tid; t < kGroupsPerSub * pitch; t += 1024) mean[t] /= static_cast<float>(max(cnt[t / pitch], 1));
    __syncthreads();
    best = 3.0e38f;
    for (int g = 0; g < kGroupsPerSub; ++g) {
        const float s = distance(mean + g * pitch);
        if (cnt[g] && s < best) { best = s; label = g; }
    }
    if (part == 0) map[j * 256 + (tid >> 2)] = static_cast<uint8_t>(label);      // (numbers beyond ks repeat the label of their low bits)
}

// The nibbles of a code's first eight sub-quantizers, number 0 in the top bits.
__device__ inline uint32_t nibble_word(const uint32_t (&low)[kM], const uint8_t *lmap)
{
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) w |= static_cast<uint32_t>(lmap[j * 256 + low[j]]) << (28 - 4 * j);
    return w;
}

// Sums of a wavefront's values.
__device__ inline uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
    return v;
}

// G[j][g] = smallest quantized entry among the centroids of group g of sub-quantizer j (255 where it has none), by a workgroup.
// tab, map: [kM][256], 4-byte aligned.
__device__ inline void group_minima(const uint8_t *tab, const uint8_t *map, uint32_t *G)
{
    for (int t = threadIdx.x; t < kM * kGroupsPerSub; t += blockDim.x) G[t] = 255u;
    __syncthreads();
    for (int t = threadIdx.x; t < kM * 64; t += blockDim.x) {
        const uint32_t v = reinterpret_cast<const uint32_t *>(tab)[t], g = reinterpret_cast<const uint32_t *>(map)[t];
#pragma unroll
        for (int b = 0; b < 4; ++b) atomicMin(&G[(t >> 6) * kGroupsPerSub + ((g >> (8 * b)) & 255u)], (v >> (8 * b)) & 255u);
    }
    __syncthreads();
}

// ---- do the cells pay? --------------------------------------------------------------------------
// A workgroup per query of a sample of the queries: every stride-th code, its cell tested and its lower bound taken.  The
// last workgroup compares the estimated cost with that of looking at every pair.
template <typename CodeT>
__global__ __launch_bounds__(256) void cells_decide_kernel(const CodeT *__restrict__ codes, uint64_t n_codes, const uint8_t *__restrict__ qtab,
                                                           int nq, uint32_t every, const uint8_t *__restrict__ map, const Bound *__restrict__ bound,
                                                           float fixed_cost, float code_cost, float cell_cost, float hit_cost, float scan_cost,
                                                           CellsCtl *ctl)
{
    __shared__ __align__(16) uint8_t lmap[kM * 256];
    __shared__ uint32_t G[kM * kGroupsPerSub];
    __shared__ uint32_t red[8];
    const int q = blockIdx.x * every, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int t = tid; t < kM * 64; t += 256) reinterpret_cast<uint32_t *>(lmap)[t] = reinterpret_cast<const uint32_t *>(map)[t];
    __syncthreads();
    group_minima(qtab + static_cast<size_t>(q) * (kM * 256), lmap, G);
    uint32_t rest = 0;                                           // smallest entries of the sub-quantizers outside the key
    for (int j = kKeyNibbles; j < kM; ++j) {
        uint32_t least = 255;
        for (int g = 0; g < kGroupsPerSub; ++g) least = min(least, G[j * kGroupsPerSub + g]);
        rest += least;
    }
    const int t = bound[q].guess;
    const uint64_t stride = n_codes / kSampleCodes;
    uint32_t ncodes = 0, nhits = 0;
    for (uint32_t s = tid; s < kSampleCodes; s += 256) {
        uint32_t low[kM], key = 0, all = 0;
        load_low_bytes<kM>(codes, s * stride, low);
#pragma unroll
        for (int j = 0; j < kM; ++j) {
            all += G[j * kGroupsPerSub + lmap[j * 256 + low[j]]];
            if (j + 1 == kKeyNibbles) key = all;
        }
        ncodes += static_cast<int>(key + rest) <= t ? 1u : 0u;
        nhits += static_cast<int>(all) <= t ? 1u : 0u;
    }
    ncodes = wave_sum(ncodes);
    nhits = wave_sum(nhits);
    if (lane == 0) { red[wave] = ncodes; red[4 + wave] = nhits; }
    __syncthreads();
    if (tid == 0) {
        const unsigned long long mine = static_cast<unsigned long long>(red[0] + red[1] + red[2] + red[3]) << 24 | (red[4] + red[5] + red[6] + red[7]) | 1ull << 48;
        const unsigned long long sums = atomicAdd(&ctl->sums, mine) + mine;
        if (sums >> 48 == gridDim.x) {
            const float per = static_cast<float>(n_codes) / static_cast<float>(kSampleCodes) * static_cast<float>(nq) / static_cast<float>(gridDim.x);
            const float c = static_cast<float>(sums >> 24 & 0xFFFFFFu) * per, h = static_cast<float>(sums & 0xFFFFFFu) * per;
            // (cells within the bound: as many as if the codes lay evenly in all of them)
            const float cells = c * fminf(1.0f, static_cast<float>(1u << kKeyBits) / static_cast<float>(n_codes));
            ctl->use = fixed_cost + code_cost * c + cell_cost * cells + hit_cost * h < scan_cost ? 1u : 0u;
        }
    }
}

// ---- sorting the codes into cells ---------------------------------------------------------------
// Two counting passes over ten bits each, of a 4-byte word of nibbles and the id.  Bound by memory: 1e8 codes in 1.8 ms (0.41 the
// words, 0.67 and 0.48 the passes, 0.22 the counts of the second) for 5 GB read and written; one pass over 2^20 cells would
// write lines of which it fills a fraction.
// Codes to nibble words, and how many fall into each bin of the first pass (the top bits of the word).
template <typename CodeT>
__global__ __launch_bounds__(512) void cells_pack_kernel(const CodeT *__restrict__ codes, uint32_t n, const uint8_t *__restrict__ map,
                                                         uint32_t *__restrict__ words, uint32_t *__restrict__ bins, const CellsCtl *__restrict__ ctl)
{
    if (!ctl->use) return;
    __shared__ __align__(16) uint8_t lmap[8 * 256];
    __shared__ uint32_t h[1 << kBinBits];
    const int tid = threadIdx.x;
    for (int t = tid; t < 8 * 64; t += 512) reinterpret_cast<uint32_t *>(lmap)[t] = reinterpret_cast<const uint32_t *>(map)[t];
    for (int t = tid; t < (1 << kBinBits); t += 512) h[t] = 0;
    __syncthreads();
#pragma unroll 2
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * 512 + tid; i < n; i += static_cast<uint64_t>(gridDim.x) * 512) {
        uint32_t low[kM];
        load_low_bytes<kM>(codes, i, low);
        const uint32_t w = nibble_word(low, lmap);
        words[i] = w;
        atomicAdd(&h[w >> (32 - kBinBits)], 1u);
    }
    __syncthreads();
    for (int t = tid; t < (1 << kBinBits); t += 512)
        if (h[t]) atomicAdd(&bins[t], h[t]);
}

// Exclusive prefix of one value per thread over a workgroup of 1024 threads; wsum: 16 words of LDS.
__device__ inline uint32_t block_prefix(uint32_t v, uint32_t *wsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl(incl, lane >= d ? lane - d : lane);
        if (lane >= d) incl += o;
    }
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - v;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    return before;
}

constexpr uint32_t kSortTile = 8192;         // elements a workgroup sorts in LDS at a time

// Tile `t` of the second pass: the bins of the first pass cut into tiles of their own.  s_tile: bin, first element, count
// (count 0: no such tile).
__device__ inline void find_tile(const uint32_t *bins, uint32_t t, uint32_t *wsum, uint32_t *s_tile)
{
    const uint32_t tid = threadIdx.x;
    if (tid == 0) s_tile[2] = 0;
    const uint32_t c = bins[tid];
    const uint32_t nt = (c + kSortTile - 1) / kSortTile;
    const uint32_t base = block_prefix(c, wsum), tbase = block_prefix(nt, wsum);
    if (t >= tbase && t < tbase + nt) {                          // one thread at most
        const uint32_t at = (t - tbase) * kSortTile;
        s_tile[0] = tid; s_tile[1] = base + at; s_tile[2] = min(kSortTile, c - at);
    }
    __syncthreads();
}

// Consecutive tiles belong to one bin; workgroups are handed to the XCDs in turn, so each XCD takes a stretch of tiles and
// the scattered writes of a bin meet in one L2.
__device__ inline uint32_t tile_of_block()
{
    const uint32_t per = (gridDim.x + 7) / 8;
    return (blockIdx.x & 7u) * per + (blockIdx.x >> 3);
}

// How many codes fall into each cell.
constexpr uint32_t kBins = 1u << kBinBits, kBinMask = kBins - 1u;
static_assert(kBins == 1024, "a bin, or a cell of a bin, per thread of a workgroup");
__global__ __launch_bounds__(1024) void cells_count_kernel(const uint32_t *__restrict__ words, const uint32_t *__restrict__ bins,
                                                           uint32_t *__restrict__ cells, const CellsCtl *__restrict__ ctl)
{
    if (!ctl->use) return;
    __shared__ uint32_t wsum[16], s_tile[3], h[kBins];
    const int tid = threadIdx.x;
    h[tid] = 0;
    find_tile(bins, tile_of_block(), wsum, s_tile);
    const uint32_t bin = s_tile[0], first = s_tile[1], count = s_tile[2];
    if (count == 0) return;                                      // uniform
    for (uint32_t i = tid; i < count; i += 1024) atomicAdd(&h[(words[first + i] >> (32 - kKeyBits)) & kBinMask], 1u);
    __syncthreads();
    if (h[tid]) atomicAdd(&cells[(bin << kBinBits) + tid], h[tid]);
}

// First element of every cell, and the end of the last one; a bit for every cell of four nibbles that holds a code.
__global__ __launch_bounds__(1024) void cells_offsets_kernel(const uint32_t *__restrict__ bins, const uint32_t *__restrict__ cells,
                                                             uint32_t *__restrict__ offs, uint64_t *__restrict__ filled, uint32_t n,
                                                             const CellsCtl *__restrict__ ctl)
{
    if (!ctl->use) return;
    __shared__ uint32_t wsum[16], s_base, s_any[64];
    const uint32_t tid = threadIdx.x, bin = blockIdx.x;
    if (tid < 64) s_any[tid] = 0;
    const uint32_t base = block_prefix(bins[tid], wsum);
    if (tid == bin) s_base = base;
    __syncthreads();
    const uint32_t cell = (bin << kBinBits) + tid, c = cells[cell];
    const uint32_t before = block_prefix(c, wsum);
    offs[cell] = s_base + before;
    if (c) s_any[tid >> 4] = 1;                                  // benign race: every writer stores 1
    __syncthreads();
    if (tid < 64) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(s_any[tid] != 0);
        if (tid == 0) filled[bin] = mask;
    }
    if (bin == 0 && tid == 0) offs[1u << kKeyBits] = n;
}

// One pass of the sort: a workgroup orders a tile by bin in LDS, takes the room for each bin's elements with one atomic
// and writes them out bin by bin.  SECOND: the bins are the cells of one bin of the first pass, and what is written is what
// the scan reads (the low 16 bits of the words, and the ids).
template <bool SECOND>
__global__ __launch_bounds__(1024) void cells_sort_kernel(const uint32_t *__restrict__ words, const uint32_t *__restrict__ ids, uint32_t n,
                                                          const uint32_t *__restrict__ bins, const uint32_t *__restrict__ offs,
                                                          uint32_t *__restrict__ cursor, uint32_t *__restrict__ out, uint16_t *__restrict__ out16,
                                                          uint32_t *__restrict__ out_ids, const CellsCtl *__restrict__ ctl)
{
    if (!ctl->use) return;
    constexpr int PER = kSortTile / 1024, SHIFT = SECOND ? 32 - kKeyBits : 32 - kBinBits;
    extern __shared__ __align__(16) uint32_t dyn[];
    uint32_t *sw = dyn, *sid = dyn + kSortTile;
    __shared__ uint32_t wsum[16], s_tile[3], h[kBins], gofs[kBins];
    const uint32_t tid = threadIdx.x;
    h[tid] = 0;
    uint32_t first, count, bin = 0;
    if constexpr (SECOND) {
        find_tile(bins, tile_of_block(), wsum, s_tile);
        bin = s_tile[0]; first = s_tile[1]; count = s_tile[2];
    } else {
        first = blockIdx.x * kSortTile;
        count = min(kSortTile, n - first);
        __syncthreads();
    }
    if (count == 0) return;                                      // uniform
    uint32_t w[PER], rank[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t i = tid + p * 1024;
        w[p] = i < count ? words[first + i] : 0u;
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t i = tid + p * 1024;
        rank[p] = i < count ? atomicAdd(&h[(w[p] >> SHIFT) & kBinMask], 1u) : 0u;
    }
    __syncthreads();
    const uint32_t c = h[tid];
    uint32_t base;                                               // where the bin starts in the output
    if constexpr (SECOND) base = offs[(bin << kBinBits) + tid];
    else base = block_prefix(bins[tid], wsum);
    const uint32_t start = block_prefix(c, wsum);
    if (c) base += atomicAdd(&cursor[SECOND ? (bin << kBinBits) + tid : tid], c);
    h[tid] = start;
    gofs[tid] = base - start;
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const uint32_t i = tid + p * 1024;
        if (i < count) {
            const uint32_t at = h[(w[p] >> SHIFT) & kBinMask] + rank[p];
            sw[at] = w[p];
            sid[at] = SECOND ? ids[first + i] : first + i;
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < count; i += 1024) {
        const uint32_t x = sw[i], to = gofs[(x >> SHIFT) & kBinMask] + i;
        if constexpr (SECOND) out16[to] = static_cast<uint16_t>(x);
        else out[to] = x;
        out_ids[to] = sid[i];
    }
}

// ---- the scan ---------------------------------------------------------------------------------------
// `parts` workgroups per query, each with some of the values of the first two nibbles, the nearest first (so that the
// bound is lowered early).  In rounds: (1) cells of four nibbles within the bound; (2) of those, the cells of five nibbles
// within the bound leave the stretch of their codes in a queue of the workgroup; (3) the stretches are walked by groups of
// lanes, as many as suit their length, sixteen codes per lane at a time, the next ones on their way while these are looked up;
// codes whose lower bound is within the bound go to a second queue; (4) when that is full, and at the end: id, code and
// integer distance of the queued codes, four per thread, and those within the bound are appended to the query's buffer.
// Bound by lines of memory: 1e8 codes, 4096 queries read 30 GB (stretches of 95 codes touch 2.5 lines, a settled code
// another) in 4.3 to 4.9 ms, beside 75 % of the vector issue slots; three steps under way instead of one changed nothing, nor did
// stretches cut into equal units for every lane group (half of the instructions then went into finding the next unit).
struct CellCfg {
    static constexpr int THREADS = 512, WAVES = THREADS / 64;
    static constexpr uint32_t SEGS = 3072, CELLS = 768, HITS = 4 * THREADS;      // queue entries
    static constexpr uint32_t SHORT = 128;                       // codes of a stretch that a few lanes walk in one step
    static constexpr uint32_t SPLIT = 4;                         // cells of four nibbles that a lane group of step (2) looks at together
    // byte offsets in LDS; the table of the last three nibbles lies at 0 (the kernel has no static LDS), so that a nibble triple
    // is its address
    static constexpr int O_TAB = 0, O_QT = O_TAB + 4096, O_G = O_QT + kM * 256, O_HIST = O_G + kM * 16 * 4, O_AT = O_HIST + 1024;
    static constexpr int O_LEN = O_AT + SEGS * 4, O_V = O_LEN + SEGS * 4, O_CELL = O_V + SEGS * 2;
    static constexpr int O_HIT = O_CELL + CELLS * 4, O_LIST = O_HIT + HITS * 4, O_VARS = O_LIST + 256, BYTES = O_VARS + 256;
};

template <typename CodeT>
__global__ __launch_bounds__(CellCfg::THREADS, 6) void scan_cells_kernel(
    const CodeT *__restrict__ codes, const uint8_t *__restrict__ qtab, const uint8_t *__restrict__ map, const uint32_t *__restrict__ offs,
    const uint64_t *__restrict__ filled, const uint16_t *__restrict__ rem16, const uint32_t *__restrict__ ids, const Bound *__restrict__ bound,
    uint32_t r, uint32_t parts, uint32_t nslices, uint32_t cap, uint32_t most_hits, uint32_t *__restrict__ fcount, uint32_t *__restrict__ chist,
    uint64_t *__restrict__ keys, uint32_t *__restrict__ first_counts, int again, const CellsCtl *__restrict__ ctl)
{
    if (!ctl->use) return;
    using C = CellCfg;
    extern __shared__ __align__(16) uint8_t smem[];
    struct Vars {
        int t;
        uint32_t next, ncell, celltaken, nshort, nlong, codes, total, hits, nhit, paused, nlist, least[kM];
    };
    static_assert(sizeof(Vars) <= 256, "room at the end");
    Vars &sh = *reinterpret_cast<Vars *>(smem + C::O_VARS);
    uint8_t *s_list = smem + C::O_LIST;
    uint8_t *tab = smem + C::O_TAB, *qt = smem + C::O_QT;
    uint32_t *G = reinterpret_cast<uint32_t *>(smem + C::O_G), *hist = reinterpret_cast<uint32_t *>(smem + C::O_HIST);
    // stretches of codes: first code, number, bound of the nibbles of the cell; short ones from the front, long ones from the back
    uint32_t *seg_at = reinterpret_cast<uint32_t *>(smem + C::O_AT), *seg_len = reinterpret_cast<uint32_t *>(smem + C::O_LEN);
    uint16_t *seg_v = reinterpret_cast<uint16_t *>(smem + C::O_V);
    uint32_t *cellq = reinterpret_cast<uint32_t *>(smem + C::O_CELL), *hitq = reinterpret_cast<uint32_t *>(smem + C::O_HIT);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t q = blockIdx.x / parts, part = blockIdx.x % parts;

    const Bound bd = bound[q];
    if (bd.t >= 255) {                                           // no bound: the redo path takes the query
        if (tid == 0 && part == 0) fcount[static_cast<size_t>(q) * nslices] = cap + 1;
        return;
    }
    // candidates are the codes with above < qd <= T: up to the guessed bucket at first, the rest of those up to the bound the
    // second time, for queries with fewer than r so far
    int T = min(bd.guess, bd.t), above = -1;
    if (again) {
        if (first_counts[q] >= r || T >= bd.t) return;           // uniform
        above = T;
        T = bd.t;
    }
    const int first_t = T;
    for (int t = tid; t < kM * 64; t += C::THREADS)
        reinterpret_cast<uint32_t *>(qt)[t] = reinterpret_cast<const uint32_t *>(qtab + static_cast<size_t>(q) * (kM * 256))[t];
    if (tid < 256) hist[tid] = 0;
    if (tid == 0) {
        sh.t = T;
        sh.next = sh.ncell = sh.celltaken = sh.nshort = sh.nlong = sh.codes = sh.total = sh.hits = sh.nhit = sh.paused = sh.nlist = 0;
    }
    __syncthreads();
    group_minima(qt, map, G);
    // sums of three nibbles' entries, capped at 127 (a lower bound still)
    for (int t = tid; t < 4096; t += C::THREADS)
        tab[t] = static_cast<uint8_t>(min(127u, G[5 * 16 + (t >> 8)] + G[6 * 16 + ((t >> 4) & 15)] + G[7 * 16 + (t & 15)]));
    if (tid < kM) {
        uint32_t least = 255;
        for (int g = 0; g < 16; ++g) least = min(least, G[tid * 16 + g]);
        sh.least[tid] = least;
    }
    uint32_t *p01 = seg_at;
    if (tid < 256) p01[tid] = (G[tid >> 4] + G[16 + (tid & 15)]) << 8 | tid;
    __syncthreads();
    int rest2 = 0, rest4 = 0, rest5 = 0;                         // smallest sums of the sub-quantizers from 2, 4 and 5 on
#pragma unroll
    for (int j = 2; j < kM; ++j) {
        const int least = static_cast<int>(sh.least[j]);
        rest2 += least;
        if (j >= 4) rest4 += least;
        if (j >= 5) rest5 += least;
    }
    rest2 = __builtin_amdgcn_readfirstlane(rest2);
    rest4 = __builtin_amdgcn_readfirstlane(rest4);
    rest5 = __builtin_amdgcn_readfirstlane(rest5);
    // the values of the first two nibbles that hold cells within the bound, the nearest first
    // (dealt out to the workgroups in that order)
    if (tid < 256 && static_cast<int>(p01[tid] >> 8) + rest2 <= first_t) {
        const uint32_t mine = p01[tid];
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t t = 0; t < 256; ++t) rank += p01[t] < mine ? 1u : 0u;
        if (rank % parts == part) {
            s_list[rank / parts] = static_cast<uint8_t>(tid);    // (those beyond the bound come after all of these)
            atomicAdd(&sh.nlist, 1u);
        }
    }
    __syncthreads();
    const uint32_t nlist = __builtin_amdgcn_readfirstlane(sh.nlist);

    auto rank_in = [](uint64_t mask) __attribute__((always_inline)) {
        return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32), __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
    };
    auto uniform_load = [](uint32_t *p) __attribute__((always_inline)) {
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    struct __attribute__((packed, aligned(4))) Pair { uint32_t start, end; };
    // eight codes per lane from element `at` on (a multiple of 8; the array is readable a little past its end).  Lanes without
    // codes read the first ones: a load behind a branch would be waited for where the paths join.
    auto load8 = [&](uint32_t at, bool live) __attribute__((always_inline)) {
        return *reinterpret_cast<const uint4 *>(rem16 + (live ? at : 0u));
    };
    uint32_t sl = (blockIdx.x + static_cast<uint32_t>(wave)) % nslices;      // slice of this wavefront's next append

    // counts per bucket: in LDS, and where several workgroups work on a query added to those in memory after every settling
    const bool shared_hist = parts > 1;
    uint32_t *counts = chist + static_cast<size_t>(q) * 256;
    // the first n entries of the second queue, by all threads: their integer distances, and those within the bound to the query's buffer
    auto settle = [&](uint32_t n) __attribute__((always_inline)) {
        constexpr int PER = C::HITS / C::THREADS;
        uint32_t id[PER], low[PER][kM], qd[PER], cnt = 0, rank[PER];
        bool keep[PER];
#pragma unroll
        for (int z = 0; z < PER; ++z) {
            const uint32_t e = hitq[min(static_cast<uint32_t>(z * C::THREADS + tid), n - 1)];
            keep[z] = static_cast<uint32_t>(z * C::THREADS + tid) < n;
            id[z] = ids[keep[z] ? e : 0u];
        }
#pragma unroll
        for (int z = 0; z < PER; ++z) load_low_bytes<kM>(codes, id[z], low[z]);
#pragma unroll
        for (int z = 0; z < PER; ++z) {
            uint32_t sum = 0;
#pragma unroll
            for (int j = 0; j < kM; ++j) sum += qt[j * 256 + low[z][j]];
            qd[z] = min(sum, 255u);
            keep[z] = keep[z] && static_cast<int>(qd[z]) <= T && static_cast<int>(qd[z]) > above && !(qd[z] == bd.t0 && id[z] > bd.last);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(keep[z]);
            rank[z] = cnt + rank_in(mask);
            cnt += __popcll(mask);
        }
        if (cnt) {                                               // uniform
            uint32_t pos = 0;
            if (lane == 0) {
                pos = atomicAdd(&fcount[static_cast<size_t>(q) * nslices + sl], cnt);
                atomicAdd(&sh.total, cnt);
            }
            pos = __builtin_amdgcn_readfirstlane(pos);
            uint64_t *to = keys + (static_cast<size_t>(q) * nslices + sl) * cap;
#pragma unroll
            for (int z = 0; z < PER; ++z) {
                if (!keep[z]) continue;
                if (pos + rank[z] < cap) to[pos + rank[z]] = make_key(qd[z], id[z]);
                atomicAdd(&hist[qd[z]], 1u);
            }
            sl = sl + 1 < nslices ? sl + 1 : 0;
        }
    };

    bool over = false;
    while (!over) {
        // (1) cells of four nibbles, 64 at a time
        while (uniform_load(&sh.ncell) <= C::CELLS - C::THREADS) {
            uint32_t u = 0;
            if (lane == 0) u = atomicAdd(&sh.next, 1u);
            u = __builtin_amdgcn_readfirstlane(u);
            if (u >= 4 * nlist) break;
            const uint32_t a = s_list[u >> 2], b = 64 * (u & 3u) + lane;
            const uint64_t some = filled[4 * a + (u & 3u)];
            const uint32_t s = G[a >> 4] + G[16 + (a & 15)] + G[32 + (b >> 4)] + G[48 + (b & 15)];
            const bool have = static_cast<int>(s) + rest4 <= T && (some >> lane & 1u);
            const uint64_t mask = __builtin_amdgcn_ballot_w64(have);
            if (!mask) continue;
            uint32_t to = 0;
            if (lane == 0) to = atomicAdd(&sh.ncell, static_cast<uint32_t>(__popcll(mask)));
            to = __builtin_amdgcn_readfirstlane(to);
            if (have) cellq[to + rank_in(mask)] = s << 16 | a << 8 | b;
        }
        __syncthreads();
        // (2) the sixteen cells of five nibbles of each, a lane per cell
        const uint32_t ncell = uniform_load(&sh.ncell);
        while (uniform_load(&sh.nshort) + uniform_load(&sh.nlong) <= C::SEGS - C::SPLIT * C::THREADS) {
            uint32_t i = 0;
            if (lane == 0) i = atomicAdd(&sh.celltaken, 4 * C::SPLIT);
            i = __builtin_amdgcn_readfirstlane(i);
            if (i >= ncell) break;
            i += static_cast<uint32_t>(lane) >> 4;
            uint32_t start[C::SPLIT], len[C::SPLIT], v[C::SPLIT], cell[C::SPLIT], to[C::SPLIT], cnt = 0, big = 0, mine = 0;
            bool have[C::SPLIT];
#pragma unroll
            for (uint32_t z = 0; z < C::SPLIT; ++z) {
                const uint32_t e = cellq[min(i + 4 * z, ncell - 1)];
                v[z] = (e >> 16) + G[64 + (lane & 15)];
                have[z] = i + 4 * z < ncell && static_cast<int>(v[z]) + rest5 <= T;
                cell[z] = have[z] ? (e & 0xFFFFu) << 4 | (lane & 15) : 0u;
            }
#pragma unroll
            for (uint32_t z = 0; z < C::SPLIT; ++z) {
                const Pair p = *reinterpret_cast<const Pair *>(offs + cell[z]);
                start[z] = p.start;
                len[z] = have[z] ? p.end - p.start : 0u;
            }
#pragma unroll
            for (uint32_t z = 0; z < C::SPLIT; ++z) {
                const bool small = len[z] != 0 && len[z] <= C::SHORT;
                const uint64_t ms = __builtin_amdgcn_ballot_w64(small), ml = __builtin_amdgcn_ballot_w64(len[z] > C::SHORT);
                to[z] = small ? cnt + rank_in(ms) : big + rank_in(ml);
                cnt += __popcll(ms);
                big += __popcll(ml);
                mine += small ? len[z] : 0u;
            }
            if (!(cnt + big)) continue;
            mine = wave_sum(mine);
            uint32_t base = 0, back = 0;
            if (lane == 0) {
                base = atomicAdd(&sh.nshort, cnt);
                back = atomicAdd(&sh.nlong, big);
                atomicAdd(&sh.codes, mine);
            }
            base = __builtin_amdgcn_readfirstlane(base);
            back = __builtin_amdgcn_readfirstlane(back);
#pragma unroll
            for (uint32_t z = 0; z < C::SPLIT; ++z)
                if (len[z]) {
                    const uint32_t e = len[z] <= C::SHORT ? base + to[z] : C::SEGS - 1 - (back + to[z]);
                    seg_at[e] = start[z];
                    seg_len[e] = len[z];
                    seg_v[e] = static_cast<uint16_t>(v[z]);
                }
        }
        __syncthreads();
        const uint32_t nshort = uniform_load(&sh.nshort), nlong = uniform_load(&sh.nlong), ncodes = uniform_load(&sh.codes);
        const bool cells_left = uniform_load(&sh.celltaken) < ncell;
        const bool last = !cells_left && uniform_load(&sh.next) >= 4 * nlist;
        // (3) short stretches by 2, 4 or 8 lanes, so that one step covers most of them; long ones by 64
        int gbits = 1;
        while (gbits < 3 && nshort * (12u << gbits) < ncodes) ++gbits;
        uint32_t block = static_cast<uint32_t>(wave);            // the 64 >> gbits stretches that come next
        bool far = false;                                        // among the long ones
        uint32_t start = 0, end = 0, at = 0, limit = 0;
        auto open = [&]() __attribute__((always_inline)) {       // false: there are none left
            if (!far && block << (6 - gbits) >= nshort) { far = true; gbits = 6; block = static_cast<uint32_t>(wave); }
            const uint32_t n = far ? nlong : nshort;
            const uint32_t s = (block << (6 - gbits)) + (static_cast<uint32_t>(lane) >> gbits);
            const bool have = s < n;
            const uint32_t e = have ? (far ? C::SEGS - 1 - s : s) : 0u;
            start = seg_at[e];
            const uint32_t len = seg_len[e];
            const int v = seg_v[e];
            at = (start & ~7u) + 16u * (static_cast<uint32_t>(lane) & ((1u << gbits) - 1u));
            end = have ? start + len : 0u;
            // entry <= thr as the top bit of thr + 128 - entry, four codes at a time (thr = 127 lets every capped entry through)
            limit = static_cast<uint32_t>(min(max(T - v, -1), 127) + 128) * 0x01010101u;
            const bool any = block << (6 - gbits) < n;
            block += C::WAVES;
            return any;
        };
        bool more = open();
        uint4 f = load8(at, at < end), g = load8(at + 8, at + 8 < end);
        uint32_t hits = 0, hit_at = 0;
        // queued by every lane for itself; true: some lane found no room and waits until the queue has been settled
        auto queue = [&]() __attribute__((always_inline)) {
            if (hits) {
                uint32_t to = atomicAdd(&sh.nhit, static_cast<uint32_t>(__popc(hits)));
                while (hits && to < C::HITS) {
                    const uint32_t t = __builtin_ctz(hits);
                    hitq[to++] = hit_at + ((t >> 3) << 2) + (t & 3u);
                    hits &= hits - 1;
                }
            }
            return __builtin_amdgcn_ballot_w64(hits != 0) != 0;
        };
        for (;;) {
            bool full = queue();
            while (more && !full) {                              // uniform
                const uint32_t k = limit, start0 = start, end0 = end;
                const uint4 f0 = f, g0 = g;
                hit_at = at;
                // the next codes of the stretches, or the next stretches
                at += 16u << gbits;
                if (!__builtin_amdgcn_ballot_w64(at < end)) more = open();       // uniform
                f = load8(at, at < end);
                g = load8(at + 8, at + 8 < end);
                const uint32_t x[8] = {f0.x, f0.y, f0.z, f0.w, g0.x, g0.y, g0.z, g0.w};
                uint32_t e[16];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    e[2 * c] = lds_read_u8(C::O_TAB + (x[c] & 0xFFFu));
                    e[2 * c + 1] = lds_read_u8(C::O_TAB + ((x[c] >> 16) & 0xFFFu));
                }
                // bit 8 b + i: code 4 b + i of this lane's sixteen is within the bound
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t p = ((e[12 + i] << 8 | e[8 + i]) << 8 | e[4 + i]) << 8 | e[i];
                    hits |= (k - p) >> (7 - i) & (0x01010101u << i);
                }
                if (hits) {                                      // those of the stretch
                    auto below = [](int n) { return n >= 16 ? ~0u : (1u << (2 * (n & ~3) + (n & 3))) - 1u; };
                    hits &= below(end0 > hit_at ? static_cast<int>(min(end0 - hit_at, 16u)) : 0);
                    if (hit_at < start0) hits &= ~below(static_cast<int>(min(start0 - hit_at, 16u)));
                }
                full = queue();
            }
            if (full) sh.paused = 1;
            __syncthreads();
            const bool paused = uniform_load(&sh.paused) != 0;
            const uint32_t n = min(uniform_load(&sh.nhit), C::HITS);
            const bool due = n && (paused || last || n > C::HITS / 2);
            if (due) settle(n);                                  // (4)
            __syncthreads();
            if (due && shared_hist && tid < 256) {
                if (hist[tid]) atomicAdd(&counts[tid], hist[tid]);
                hist[tid] = 0;
            }
            if (wave == 0) {
                if (lane == 0) {
                    sh.paused = 0;
                    if (due) { sh.nhit = 0; sh.hits += n; }
                    if (!paused) {
                        sh.nshort = sh.nlong = sh.codes = 0;
                        if (!cells_left) sh.ncell = sh.celltaken = 0;    // (every cell of the queue has been split)
                    }
                }
                // the bound is lowered to the bucket of the r-th best candidate so far
                if (due && (shared_hist || uniform_load(&sh.total) >= r)) {
                    uint32_t c4[4], mine = 0;
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        c4[z] = shared_hist ? __hip_atomic_load(&counts[4 * lane + z], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : hist[4 * lane + z];
                        mine += c4[z];
                    }
                    uint32_t incl = mine;
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const uint32_t o = __shfl(incl, lane >= d ? lane - d : lane);
                        if (lane >= d) incl += o;
                    }
                    uint32_t cum = incl - mine;
                    if (cum < r && incl >= r) {                  // at most one lane
                        int tn = 4 * lane;
#pragma unroll
                        for (int z = 0; z < 3; ++z) {
                            cum += c4[z];
                            if (cum < r) tn = 4 * lane + z + 1;
                        }
                        sh.t = min(tn, T);
                    }
                }
            }
            __syncthreads();
            T = static_cast<int>(uniform_load(reinterpret_cast<uint32_t *>(&sh.t)));
            over = uniform_load(&sh.hits) > most_hits;
            if (!paused || over) break;
        }
        if (last) break;
    }
    if (tid == 0) {
        if (!again) atomicAdd(&first_counts[q], sh.total);
        if (over) atomicMax(&fcount[static_cast<size_t>(q) * nslices], cap + 1);     // too many codes to look at: the redo path takes the query
    }
    if (tid < 256 && !shared_hist) counts[tid] += hist[tid];
}

// ---- host side ------------------------------------------------------------------------------------
struct CellsPlan {
    size_t off_ctl, off_bins, off_cursor1, off_cells, off_cursor2, off_first, clear_words, off_map, off_offs, off_filled;
    size_t off_words, off_sorted, off_sorted_ids, off_rem, off_ids, total;
};

static CellsPlan plan_cells(uint64_t n, int m, int nq)
{
    CellsPlan p{};
    constexpr size_t cells = static_cast<size_t>(1) << kKeyBits;
    constexpr size_t slack = 64;                                 // elements readable past the end
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
    p.off_ctl = take(sizeof(CellsCtl));
    p.off_bins = take(4 * kBins);
    p.off_cursor1 = take(4 * kBins);
    p.off_cells = take(4 * cells);
    p.off_cursor2 = take(4 * cells);
    p.off_first = take(4 * static_cast<size_t>(nq));
    p.clear_words = off / 4;                                     // all of the above is zero at the start of a call
    p.off_map = take(static_cast<size_t>(m) * 256);
    p.off_offs = take(4 * (cells + 1));
    p.off_filled = take(8 * kBins);
    p.off_ids = take(4 * (n + slack));
    p.off_words = p.off_ids;                                     // (the words are read for the last time before the ids are written)
    p.off_rem = take(2 * (n + slack));
    p.off_sorted = take(4 * (n + slack));
    p.off_sorted_ids = take(4 * (n + slack));
    p.total = off;
    return p;
}

size_t cells_bytes(uint64_t n, int m, int nq) { return plan_cells(n, m, nq).total; }

// (Fewer than 2^31 codes: a lane steps up to 1024 positions past the end of its stretch, and tiles are counted in 32 bits.)
// (Nor where a query wants more than a thousandth of the codes: with 420 and 840 codes to each that is wanted the decision declined for every
// kind of codebook and codes that it was tried on, at 1200 and 2100 it served some: 9.7 -> 4.5 ms and 1.65 -> 0.87.)
bool cells_may_pay(uint64_t n, int m, int nq, uint32_t r)
{
    return m == 8 && n >= (4ull << 20) && n < (1ull << 31) && static_cast<double>(n) * nq >= 8.0e9 && n >= 1000ull * r;
}

template <typename CodeT>
static int launch_cells(const CodeT *codes, uint64_t n_codes, const uint8_t *qtab, int nq, uint32_t r, const CellsArea &area, const Bound *bound,
                          uint32_t nslices, uint32_t cap, uint32_t *fcount, uint32_t *chist, uint64_t *keys, const uint32_t **used, hipStream_t st)
{
    const CellsPlan p = plan_cells(n_codes, kM, nq);
    uint8_t *base = static_cast<uint8_t *>(area.ptr);
    auto words = [&](size_t off) { return reinterpret_cast<uint32_t *>(base + off); };
    CellsCtl *ctl = reinterpret_cast<CellsCtl *>(base + p.off_ctl);
    uint8_t *map = base + p.off_map;
    uint64_t *filled = reinterpret_cast<uint64_t *>(base + p.off_filled);
    uint16_t *rem = reinterpret_cast<uint16_t *>(base + p.off_rem);
    uint32_t *bins = words(p.off_bins), *offs = words(p.off_offs);
    const uint32_t n = static_cast<uint32_t>(n_codes);
    *used = &ctl->use;

    const size_t group_lds = sizeof(float) * group_pitch(area.dsub) * ((static_cast<size_t>(1) << area.small_bits) + kGroupsPerSub);
    constexpr int sort_lds = kSortTile * 8;
    int rc = allow_dynamic_lds(reinterpret_cast<const void *>(&cells_group_kernel), static_cast<int>(group_lds));
    if (!rc) rc = allow_dynamic_lds(reinterpret_cast<const void *>(&cells_sort_kernel<false>), sort_lds);
    if (!rc) rc = allow_dynamic_lds(reinterpret_cast<const void *>(&cells_sort_kernel<true>), sort_lds);
    if (!rc) rc = allow_dynamic_lds(reinterpret_cast<const void *>(&scan_cells_kernel<CodeT>), CellCfg::BYTES, true);
    if (rc) return rc;
    DCPQ_LAUNCH(kStageCellsSort, st, cells_group_kernel, dim3(kM + 64), dim3(1024), group_lds, area.derived, kM, area.dsub, area.small_bits, map,
                words(0), static_cast<uint32_t>(p.clear_words));
    DCPQ_CHECK_LAUNCH("cells_group_kernel");
    // Costs in picoseconds, from N = 1e8, 4096 queries (sorting 1.8 ms, scan 4.9 ms for 6.6e9 codes in 7.4e7 cells and 4.5e7 settled
    // codes; single-pass scan 40.7 ms) and N = 2e6, 4096 queries (4.2 ms for 1.8e8 cells of one or two codes; 1.37 ms).  They leave a margin:
    // of 171 searches of 4.2e6 to 4e7 codes, 210 to 20000 queries, r = 200 to 10000 on eight kinds of codebooks and codes the 56 that were served
    // took 0.15 to 0.89 of the time of the single-pass scan.
    const float pairs = static_cast<float>(n_codes) * static_cast<float>(nq);
    const uint32_t every = (static_cast<uint32_t>(nq) + kSampleQueries - 1) / kSampleQueries;
    DCPQ_LAUNCH(kStageCellsSort, st, (cells_decide_kernel<CodeT>), dim3((nq + every - 1) / every), dim3(256), 0, codes, n_codes, qtab, nq, every, map, bound,
                18.0f * static_cast<float>(n_codes) + 1.0e8f, 0.45f, 20.0f, 15.0f, 0.1f * pairs, ctl);
    DCPQ_CHECK_LAUNCH("cells_decide_kernel");
    DCPQ_LAUNCH(kStageCellsSort, st, (cells_pack_kernel<CodeT>), dim3(2048), dim3(512), 0, codes, n, map, words(p.off_words), bins, ctl);
    DCPQ_CHECK_LAUNCH("cells_pack_kernel");
    const uint32_t tiles = (n + kSortTile - 1) / kSortTile;
    DCPQ_LAUNCH(kStageCellsSort, st, cells_sort_kernel<false>, dim3(tiles), dim3(1024), sort_lds, words(p.off_words), nullptr, n, bins, nullptr,
                words(p.off_cursor1), words(p.off_sorted), nullptr, words(p.off_sorted_ids), ctl);
    DCPQ_CHECK_LAUNCH("cells_sort_kernel<first>");
    const uint32_t tiles2 = (tiles + kBins + 7) / 8 * 8;         // every bin may end in a part of a tile
    DCPQ_LAUNCH(kStageCellsSort, st, cells_count_kernel, dim3(tiles2), dim3(1024), 0, words(p.off_sorted), bins, words(p.off_cells), ctl);
    DCPQ_CHECK_LAUNCH("cells_count_kernel");
    DCPQ_LAUNCH(kStageCellsSort, st, cells_offsets_kernel, dim3(kBins), dim3(1024), 0, bins, words(p.off_cells), offs, filled, n, ctl);
    DCPQ_CHECK_LAUNCH("cells_offsets_kernel");
    DCPQ_LAUNCH(kStageCellsSort, st, cells_sort_kernel<true>, dim3(tiles2), dim3(1024), sort_lds, words(p.off_sorted), words(p.off_sorted_ids), n, bins,
                offs, words(p.off_cursor2), nullptr, rem, words(p.off_ids), ctl);
    DCPQ_CHECK_LAUNCH("cells_sort_kernel<second>");
    uint32_t parts = 1;
    while (parts * 2 * static_cast<uint32_t>(nq) <= 2048 && parts < 16) parts *= 2;
    const uint64_t hits = 64ull * r + n_codes / 64;
    const uint32_t most = static_cast<uint32_t>(hits > 0x7FFFFFFFull ? 0x7FFFFFFFull : hits);
    for (int again = 0; again < 2; ++again) {
        // few queries are left: more workgroups for each.  (Fewer workgroups that look for the pairs that are left return sooner where none
        // is, 5 us instead of 23 with 4096 queries, but take 205 us instead of 162 where 94 are.)
        if (again && parts < 8) parts = 8;
        DCPQ_LAUNCH(kStageScanCells, st, (scan_cells_kernel<CodeT>), dim3(nq * parts), dim3(CellCfg::THREADS), CellCfg::BYTES, codes, qtab,
                    map, offs, filled, rem, words(p.off_ids), bound, r, parts, nslices, cap, most, fcount, chist, keys, words(p.off_first), again, ctl);
        DCPQ_CHECK_LAUNCH("scan_cells_kernel");
    }
    return DCPQ_OK;
}

template <typename CodeT>
int launch_scan_cells(const CodeT *codes, uint64_t n_codes, int m, const uint8_t *qtab, int nq, uint32_t r, const CellsArea &area, const Bound *bound,
                      uint32_t nslices, uint32_t cap, uint32_t *fcount, uint32_t *chist, uint64_t *keys, const uint32_t **used, hipStream_t st)
{
    if (m == 8) return launch_cells<CodeT>(codes, n_codes, qtab, nq, r, area, bound, nslices, cap, fcount, chist, keys, used, st);
    return fail(DCPQ_EUNSUPPORTED, "scan over cells: m=%d not supported", m);
}

template int launch_scan_cells<uint16_t>(const uint16_t *, uint64_t, int, const uint8_t *, int, uint32_t, const CellsArea &, const Bound *, uint32_t,
                                         uint32_t, uint32_t *, uint32_t *, uint64_t *, const uint32_t **, hipStream_t);
template int launch_scan_cells<uint8_t>(const uint8_t *, uint64_t, int, const uint8_t *, int, uint32_t, const CellsArea &, const Bound *, uint32_t,
                                        uint32_t, uint32_t *, uint32_t *, uint64_t *, const uint32_t **, hipStream_t);

}  // namespace dcpq

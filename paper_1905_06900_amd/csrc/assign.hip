// Nearest centroid of every sub-vector (encoding, the assignment step of k-means): the smallest
// (squared distance, index) with distances in double precision.
//
// Small codebooks, and few points with long sub-vectors, take all products on the double-precision matrix pipe
// (assign_f64_kernel; f64_is_faster says where), many points with sub-vectors of 5 to 64 components a filter with one fp16 product
// (assign_half_kernel; the rule is in launch_assign_ks).  The others are computed in two steps with the result of one.  A filter evaluates |c|^2 - 2 <x, c> for all centroids on
// the bf16 matrix cores with every fp32 number split into two bf16 numbers (x = xh + xl + an error of at most
// 2^-17 |x|; the three products xh ch + xl ch + xh cl, and xl cl where it costs no further matrix instruction, lie
// side by side along the K dimension of one matrix product whose accumulators start from |c|^2), and keeps per
// point the three smallest minima over cells of 16, 32 or 64 centroids (16 of every 32 that a cell spans).  A bound on the filter's error, from the norms at hand, says which cells can hold the nearest
// centroid: those, almost always one or two, are evaluated in double precision.  A point with more such cells
// than were kept (or whose values are not finite) is compared with all centroids in double precision.  That is
// most of the time where a codebook repeats itself, and with sub-vectors of one or two components.
//
// What bounds it: matrix and vector instructions, which leave a SIMD 6 % of its cycles if they do not overlap: the
// matrix pipe (KS instructions of 32 cycles per 32 x 32 distances, KS = ceil(3 d / 16)) is busy 0.56 of the time, and 16
// vector instructions per 32 x 32 distances (9 for the minima, the rest the conversion of the centroids, shared by the
// points of a workgroup) 0.38; the LDS 0.22.  250007 vectors, 8
// sub-quantizers of 16 components and 65536 centroids: 11.3 ms = 1.1 PFLOP/s of bf16 products, what a large library
// matrix product reaches here (1.16); with all distances on the double-precision matrix pipe 97 ms.
#include <type_traits>

#include "common.h"
#include "assign.h"
#include "f64_tile.h"

namespace dcpq {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

struct __attribute__((packed, aligned(4))) f4_any { float v[4]; };

// Comparison of points with all centroids in double precision: components staged together, in rows of an odd number of
// 16-byte units; up to kFewHard points are taken one by one, by all threads (0.115 ms each at 65536 x 16, 32 together 1.3 ms).
constexpr int kTileComps = 16;
constexpr int kTileStride = 4 * kTileComps + 16;
constexpr uint32_t kFewHard = 8;

// KS: steps of 16 along K.  P: tiles of 32 points per wavefront.  SPLIT: the four wavefronts share the points
// and split the centroids (else every wavefront has points of its own).  RS: centroids staged together.
template <int KS, int P, bool SPLIT>
struct AssignCfg {
    static constexpr int RS = KS <= 6 ? 128 : 64;              // centroids per stage
    static constexpr int AHEAD = KS * P <= 12 ? 2 : 1;              // operand sets of a tile (2: read one tile ahead)
    // steps from a product to its minimum (registers for LAG + 1 results; at KS = 1 those of a third would leave room for two wavefronts
    // per SIMD instead of three: 140000 points, 2 sub-quantizers of 4 components, 256 centroids 97 us so, 63 with LAG = 1)
    static constexpr int LAG = AHEAD == 2 && P == 4 && KS > 1 ? 2 : 1;
    static constexpr int TPC = SPLIT ? 1 : RS / 32;            // tiles of 32 centroids per cell
    static constexpr int TPR = 256 / RS;                       // threads that convert one centroid
    static constexpr int DPMAX = 16 * KS / 3 & ~3;             // largest padded sub-vector length
    // steps that hold the products xh ch and xh cl, and xh ch alone: all there is to add up where xl, or both xl and cl, are zero
    static constexpr int KS2 = (2 * DPMAX + 15) / 16, KS1 = (DPMAX + 15) / 16;
    // ... which is looked for with sub-vectors of up to 32 components, and not with few points: registers are scarce in the others
    static constexpr bool LOOK = !SPLIT && KS <= 6 && KS2 < KS;
    static constexpr int NG = (DPMAX / 4 + TPR - 1) / TPR;     // groups of 4 components per thread
    static constexpr int STRIDE = KS * 32 + 16;                // bytes per staged row (an odd number of 16-byte units)
    static constexpr int PTS = SPLIT ? 32 * P : 128 * P;       // points per workgroup
    static constexpr int NE = SPLIT ? 8 : 2;                   // lanes that hold minima of one point
    static constexpr int BUF_BYTES = RS * STRIDE + RS * 4;     // the rows, then |c|^2 of every row
    static constexpr int STAGE_BYTES = 2 * BUF_BYTES;
    static constexpr int LIST_BYTES = 3 * PTS * 4;             // three lists of points, behind them the minima ...
    static constexpr int ENT_BYTES = LIST_BYTES + PTS * NE * 5 * 4;
    // The full comparison: points per wavefront and centroids per lane, points and centroids at a time.  (The tiles that split
    // the centroids are for few points: registers for more at a time would halve the wavefronts in flight there.)
    static constexpr int PER_WAVE = SPLIT ? 4 : 8, PER_LANE = SPLIT ? 1 : 4;
    static constexpr int TOGETHER = 4 * PER_WAVE, ROWS = 64 * PER_LANE;
    static constexpr bool ROWS_IN_LDS = KS > 1;                // ... and in place of the minima its rows and points
    static constexpr int ROW_BYTES = ROWS_IN_LDS ? ROWS * kTileStride : 0;
    static constexpr int LAST_BYTES = LIST_BYTES + ROW_BYTES + DPMAX * TOGETHER * 8;
    static constexpr int USED_BYTES = ENT_BYTES > LAST_BYTES ? ENT_BYTES : LAST_BYTES;
    static constexpr int LDS_BYTES = STAGE_BYTES > USED_BYTES ? STAGE_BYTES : USED_BYTES;
    static_assert(!SPLIT || RS == 128, "one 32-centroid tile per wavefront and stage");
};

// Squared distance of two sub-vectors in double precision (components in increasing order).
__device__ inline double exact_distance(const float *__restrict__ x, const float *__restrict__ c, int dsub)
{
    double acc = 0.0;
    int t = 0;
    for (; t + 4 <= dsub; t += 4) {
        const f4_any a = *reinterpret_cast<const f4_any *>(x + t), b = *reinterpret_cast<const f4_any *>(c + t);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double u = static_cast<double>(a.v[e]) - static_cast<double>(b.v[e]);
            acc = fma(u, u, acc);
        }
    }
    for (; t < dsub; ++t) {
        const double u = static_cast<double>(x[t]) - static_cast<double>(c[t]);
        acc = fma(u, u, acc);
    }
    return acc;
}

// Smaller of two (value, index) pairs; equal values -> smaller index.
__device__ inline void take_smaller(double &v, uint32_t &i, double ov, uint32_t oi)
{
    if (ov < v || (ov == v && oi < i)) { v = ov; i = oi; }
}

// Nearest centroid of one point by a workgroup of 256, all distances in double precision; thread 0 has it.  red_v, red_i: four in LDS.
__device__ inline void nearest_of_all(const float *__restrict__ x, const float *__restrict__ cbj, int dsub, int ncent, double *red_v, uint32_t *red_i, double &best,
                                      uint32_t &bi)
{
    const int tid = threadIdx.x;
    best = INFINITY;
    bi = 0xFFFFFFFFu;
    for (int c = tid; c < ncent; c += 256) take_smaller(best, bi, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const double ov = __shfl_xor(best, off);
        const uint32_t oi = __shfl_xor(bi, off);
        take_smaller(best, bi, ov, oi);
    }
    if ((tid & 63) == 0) { red_v[tid >> 6] = best; red_i[tid >> 6] = bi; }
    __syncthreads();
    if (tid == 0)
        for (int w = 1; w < 4; ++w) take_smaller(best, bi, red_v[w], red_i[w]);
    __syncthreads();
}

__device__ inline void store_label(void *labels, int label_bytes, size_t o, uint32_t i)
{
    if (label_bytes == 1) static_cast<uint8_t *>(labels)[o] = static_cast<uint8_t>(i);
    else if (label_bytes == 2) static_cast<uint16_t *>(labels)[o] = static_cast<uint16_t>(i);
    else static_cast<uint32_t *>(labels)[o] = i;
}

// Nearest centroid of the j-th sub-vector of a workgroup's points, whose numbers are at(0), at(1), ... at(np - 1).  points: rows of
// `ld` floats; sub-vector j starts at column j * dsub.  labels: [n][m].  dist (optional): [n][m] fp32 squared distance.
// dp: dsub rounded up to a multiple of 4, 3 dp <= 16 KS (4 dp <= 16 KS: all four products, half the filter's error).  FOURS: dsub is
// one (a kernel of its own: with both ways of reading the centroids in one, the compiler moved the load that they share before the
// branch and waited for it before the products; 300 points, 65536 centroids of 3 components: 0.30 ms so and 0.26 apart; of 8 0.38 and 0.28, of 21 0.73 and 0.64, of 32 0.75 and 0.52).
template <int KS, int P, bool SPLIT, bool FOURS, typename At>
__device__ __forceinline__ void nearest_by_split_products(uint8_t *smem, At at, uint32_t np, const float *__restrict__ points, int ld,
                                                          const float *__restrict__ cbj, int j, int m, int dsub, int dp, int ncent,
                                                          void *__restrict__ labels, int label_bytes, float *__restrict__ dist)
{
    using C = AssignCfg<KS, P, SPLIT>;
    __shared__ __align__(16) float mu[128];
    __shared__ float s_cmax[4];
    __shared__ float xnorm2[C::PTS];
    __shared__ uint32_t s_count[3];                                 // points in the lists below
    __shared__ uint32_t s_whole, s_xlow, s_clow[3];                 // set: large components in mu; an xl, a cl (of a stage) that is not zero
    __shared__ double red_v[4];
    __shared__ uint32_t red_i[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const bool four = KS <= 3 && 4 * dp <= 16 * KS;                 // K has room for the product xl cl (sub-vectors of up to 12)

    // A reference vector subtracted from points and centroids: distances do not change, norms (and with them the
    // filter's error) shrink.  The mean of up to 64 centroids spread over the codebook; any vector would do.  One with large
    // components is rounded to whole numbers: points that are whole numbers (vectors of bytes) then stay so, and where they
    // are below 256 in all components xh = x, and the product with xl, a third of the matrix instructions, is left out (of whole
    // centroids, training's first ones, that with cl too).
    if (tid == 0) s_whole = s_xlow = s_clow[0] = s_clow[1] = s_clow[2] = 0;
    __syncthreads();
    if (tid < 128) {
        float sum = 0.0f;
        const int ns = ncent < 64 ? ncent : 64, step = ncent / ns;
        if (tid < dsub)
            for (int s = 0; s < ns; ++s) {
                const int c = s * step + s % step;
                sum += cbj[static_cast<size_t>(c) * dsub + tid];
            }
        mu[tid] = sum / static_cast<float>(ns);
        if (fabsf(mu[tid]) >= 8.0f) s_whole = 1;
    }
    __syncthreads();
    if (tid < 128 && s_whole) mu[tid] = rintf(mu[tid]);
    if (tid < 3) s_count[tid] = 0;
    for (int t = tid; t < C::STAGE_BYTES / 16; t += 256) reinterpret_cast<uint4 *>(smem)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();

    const int srow = tid / C::TPR, spart = tid % C::TPR;
    // The point side of the product: column `col` of B, K positions 16 ks + 8 half + e:
    // [ -2 xh | -2 xh | -2 xl | 0 ... ] against the centroids' [ ch | cl | ch | 0 ... ]; with room for four products
    // [ -2 xh | -2 xh | -2 xl | -2 xl | 0 ... ] against [ ch | cl | ch | cl | 0 ... ].
    // Converted in rows by the whole workgroup, RS points at a time, and read back as operands.
    v8bf bq[P][KS];
    bool low = false;
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll 1
        for (int sub = 0; sub < (SPLIT ? 1 : 128 / C::RS); ++sub) {
            const uint32_t pt = p * (SPLIT ? 32 : 128) + sub * C::RS + srow;
            const float *x = points + static_cast<size_t>(at(pt < np ? pt : np - 1)) * ld + j * dsub;
            uint8_t *row = smem + srow * C::STRIDE;
            float norm = 0.0f;
#pragma unroll 1
            for (int g = 0; g < C::NG; ++g) {
                const int o = 4 * (spart + C::TPR * g);
                if (o < dp) {
                    v4bf h, l;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int t = o + e < dsub ? o + e : dsub - 1;
                        const float u = o + e < dsub ? x[t] - mu[t] : 0.0f, v = -2.0f * u;
                        h[e] = static_cast<__bf16>(v);
                        l[e] = static_cast<__bf16>(v - static_cast<float>(h[e]));
                        norm = fmaf(u, u, norm);
                        low = low || static_cast<float>(l[e]) != 0.0f;
                    }
                    *reinterpret_cast<v4bf *>(row + 2 * o) = h;
                    *reinterpret_cast<v4bf *>(row + 2 * (dp + o)) = h;
                    *reinterpret_cast<v4bf *>(row + 2 * (2 * dp + o)) = l;
                    if (four) *reinterpret_cast<v4bf *>(row + 2 * (3 * dp + o)) = l;
                }
            }
#pragma unroll
            for (int off = 1; off < C::TPR; off <<= 1) norm += __shfl_xor(norm, off);
            if (spart == 0 && pt < C::PTS) xnorm2[pt] = norm;
            __syncthreads();
            if (SPLIT || wave * 32 / C::RS == sub) {
                const uint8_t *b = smem + ((SPLIT ? 0 : wave * 32 % C::RS) + col) * C::STRIDE + half * 16;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) bq[p][ks] = *reinterpret_cast<const v8bf *>(b + ks * 32);
            }
            __syncthreads();
        }
    }

    if (low) s_xlow = 1;
    __syncthreads();
    const bool low_points = !C::LOOK || __builtin_amdgcn_readfirstlane(s_xlow) != 0;          // uniform

    // staging: TPR threads convert one centroid
    float pre[C::NG][4];
    auto load_stage = [&](int c0) {
        const int c = c0 + srow;
        const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
        if constexpr (FOURS) {
#pragma unroll
            for (int g = 0; g < C::NG; ++g) {
                const int o = 4 * (spart + C::TPR * g);
                const f4_any v = *reinterpret_cast<const f4_any *>(src + (o < dsub ? o : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) pre[g][e] = v.v[e];
            }
        } else {
#pragma unroll
            for (int g = 0; g < C::NG; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int o = 4 * (spart + C::TPR * g) + e;
                    pre[g][e] = src[o < dsub ? o : 0];               // (past the last: set to zero when the stage is stored, not waited for here)
                }
        }
    };
    float cmax2 = 0.0f;                       // largest |c|^2 among the centroids this thread converted
    auto store_stage = [&](auto whole, int s, uint8_t *buf) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;               // the points are: look at cl
        const int c0 = s * C::RS;
        uint8_t *row = buf + srow * C::STRIDE;
        float norm = 0.0f;
        bool low = false;
        if constexpr (!FOURS) {                                      // (mu is zero there)
#pragma unroll
            for (int g = 0; g < C::NG; ++g)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (4 * (spart + C::TPR * g) + e >= dsub) pre[g][e] = 0.0f;
        }
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 4 * (spart + C::TPR * g);
            if (o < dp) {
                v4bf h, l;
                const float4 mv = *reinterpret_cast<const float4 *>(mu + o);
                const float ref[4] = {mv.x, mv.y, mv.z, mv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = pre[g][e] - ref[e];
                    h[e] = static_cast<__bf16>(v);
                    l[e] = static_cast<__bf16>(v - static_cast<float>(h[e]));
                    norm = fmaf(v, v, norm);
                }
                if (WHOLE) low = low || (__builtin_bit_cast(uint64_t, l) & 0x7FFF7FFF7FFF7FFFull) != 0;
                *reinterpret_cast<v4bf *>(row + 2 * o) = h;
                *reinterpret_cast<v4bf *>(row + 2 * (dp + o)) = l;
                *reinterpret_cast<v4bf *>(row + 2 * (2 * dp + o)) = h;
                if (four) *reinterpret_cast<v4bf *>(row + 2 * (3 * dp + o)) = l;
            }
        }
#pragma unroll
        for (int off = 1; off < C::TPR; off <<= 1) norm += __shfl_xor(norm, off);
        if (c0 + srow < ncent) cmax2 = norm < INFINITY ? fmaxf(cmax2, norm) : INFINITY;      // (NaN counts as infinite)
        else norm = INFINITY;                                                               // past the last centroid: never the nearest
        if (spart == 0) reinterpret_cast<float *>(buf + C::RS * C::STRIDE)[srow] = norm;
        if (WHOLE) {                                                 // (the flag of the stage after this one is cleared: it is read no more)
            if (low) s_clow[s % 3] = 1;
            if (tid == 0) s_clow[(s + 1) % 3] = 0;
        }
    };

    // three smallest cell minima of each of this lane's points, and the cells of the first two
    float b1[P], b2[P], b3[P];
    uint32_t i1[P], i2[P];
#pragma unroll
    for (int p = 0; p < P; ++p) { b1[p] = b2[p] = b3[p] = INFINITY; i1[p] = i2[p] = 0; }
    float mn[P];                              // minimum of the cell so far
    // One wavefront's tiles of a stage.  Short operands of a tile are read one tile ahead; the minimum over the 16 filter
    // values of one tile of points (row 8 (v / 4) + 4 half + v % 4 in value v) is taken while the matrix
    // instructions of the next run.
    auto read_tile = [&](const uint8_t *buf, int t, auto &a, v16f &norm) __attribute__((always_inline)) {
        constexpr int K = sizeof(a) / sizeof(v8bf);
        const uint8_t *ra = buf + (t * 32 + col) * C::STRIDE + half * 16;
#pragma unroll
        for (int ks = 0; ks < K; ++ks) a[ks] = *reinterpret_cast<const v8bf *>(ra + ks * 32);
        const float *nr = reinterpret_cast<const float *>(buf + C::RS * C::STRIDE) + t * 32 + 4 * half;
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(nr + 2 * v);
            norm[v] = x.x; norm[v + 1] = x.y; norm[v + 2] = x.z; norm[v + 3] = x.w;
        }
    };
    auto minimum = [](const v16f &acc) {
        float m0 = fminf(fminf(acc[0], acc[1]), acc[2]), m1 = fminf(fminf(acc[3], acc[4]), acc[5]);
#pragma unroll
        for (int v = 6; v < 14; v += 4) {
            m0 = fminf(fminf(acc[v], acc[v + 1]), m0);
            m1 = fminf(fminf(acc[v + 2], acc[v + 3]), m1);
        }
        m0 = fminf(fminf(acc[14], acc[15]), m0);
        return fminf(m0, m1);
    };
    auto compute_cell = [&](auto steps, const uint8_t *buf, int t0) __attribute__((always_inline)) {
        constexpr int K = decltype(steps)::value;                     // steps added up
        constexpr int AH = C::AHEAD;
        v8bf a[AH][K];
        v16f norm[AH], acc[C::LAG + 1];
        if constexpr (AH == 2) read_tile(buf, t0, a[0], norm[0]);
#pragma unroll
        for (int x = 0; x < C::TPC * P + C::LAG; ++x) {               // step x: products of (tile x / P, points x % P), minimum of step x - LAG
            const int t = x / P, p = x % P;
            if (x < C::TPC * P) {
                if constexpr (AH == 2) {
                    if (p == 0 && t + 1 < C::TPC) read_tile(buf, t0 + t + 1, a[(t + 1) & 1], norm[(t + 1) & 1]);
                } else {
                    if (p == 0) read_tile(buf, t0 + t, a[0], norm[0]);
                }
#pragma unroll
                for (int ks = 0; ks < K; ++ks)
                    acc[x % (C::LAG + 1)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t % AH][ks], bq[p][ks], ks == 0 ? norm[t % AH] : acc[x % (C::LAG + 1)], 0, 0, 0);
            }
            if (x >= C::LAG) {
                const int q = (x - C::LAG) % P;
                const float v = minimum(acc[(x - C::LAG) % (C::LAG + 1)]);
                mn[q] = x - C::LAG < P ? v : fminf(mn[q], v);
                asm volatile("" : "+v"(mn[q]));                       // (keeps it here: its use is behind a branch)
            }
#pragma unroll
            for (int ks = 0; ks < K; ++ks) {                          // matrix and vector instructions in turn
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, (9 + K - 1) / K, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto enter = [&](uint32_t cell) {         // entering the three smallest becomes rare as the walk goes on
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (!__builtin_amdgcn_ballot_w64(mn[p] < b3[p])) continue;          // uniform
            const bool c1 = mn[p] < b1[p], c2 = mn[p] < b2[p];
            const uint32_t second = c2 ? cell : i2[p];
            i2[p] = c1 ? i1[p] : second;
            i1[p] = c1 ? cell : i1[p];
            b3[p] = __builtin_amdgcn_fmed3f(b2[p], b3[p], mn[p]);
            b2[p] = __builtin_amdgcn_fmed3f(b1[p], b2[p], mn[p]);
            b1[p] = fminf(b1[p], mn[p]);
        }
    };
    const int nst = (ncent + C::RS - 1) / C::RS;
    auto walk = [&](auto whole) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        load_stage(0);
        store_stage(whole, 0, smem);
        __syncthreads();
        for (int s = 0; s < nst; ++s) {                               // uniform
            if (s + 1 < nst) load_stage((s + 1) * C::RS);
            const uint8_t *buf = smem + (s & 1) * C::BUF_BYTES;
            const int t0 = SPLIT ? wave : 0;
            if constexpr (!WHOLE) {
                compute_cell(std::integral_constant<int, KS>{}, buf, t0);
            } else if (C::KS1 == C::KS2 || __builtin_amdgcn_readfirstlane(s_clow[s % 3])) {      // uniform
                compute_cell(std::integral_constant<int, C::KS2>{}, buf, t0);
            } else {
                compute_cell(std::integral_constant<int, C::KS1>{}, buf, t0);
            }
            enter(SPLIT ? s * (C::RS / 32) + wave : s);
            if (s + 1 < nst) store_stage(whole, s + 1, smem + ((s + 1) & 1) * C::BUF_BYTES);
            __syncthreads();
        }
    };
    if constexpr (!C::LOOK) {
        walk(std::false_type{});
    } else {
        if (low_points) walk(std::false_type{});
        else walk(std::true_type{});
    }

    // hand the minima over: ent[point][lane that held them][b1, b2, b3, i1, i2]
    float *ent = reinterpret_cast<float *>(smem + C::LIST_BYTES);
    uint32_t *list[3];                        // points with one cell to look at, with several, and for the full comparison
#pragma unroll
    for (int k = 0; k < 3; ++k) list[k] = reinterpret_cast<uint32_t *>(smem) + k * C::PTS;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int pt = SPLIT ? p * 32 + col : p * 128 + wave * 32 + col;
        float *e = ent + (pt * C::NE + (SPLIT ? wave * 2 : 0) + half) * 5;
        e[0] = b1[p]; e[1] = b2[p]; e[2] = b3[p];
        e[3] = __uint_as_float(i1[p]); e[4] = __uint_as_float(i2[p]);
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) cmax2 = fmaxf(cmax2, __shfl_xor(cmax2, off));
    if (lane == 0) s_cmax[wave] = cmax2;
    __syncthreads();
    const float cmax = sqrtf(fmaxf(fmaxf(s_cmax[0], s_cmax[1]), fmaxf(s_cmax[2], s_cmax[3]))) * 1.001f;

    // Error of a filter value, |c| <= c1.  bf16 has 8 significant bits: for 2^e <= |x| < 2^(e+1) the first rounding
    // leaves |xl| <= 2^(e-8) and the second, of a number in a binade below that (or exactly on it, and then without
    // error), at most 2^(e-17).  So |xl| <= 2^-8 |x|, x - xh - xl is at most 2^-17 |x|, and what the product of two
    // numbers loses is xl cl (2^-16) and what the two remainders multiply (2^-17 each): 2^-15 |x| |c|, twice that in
    // 2 |<x, c>|, 16 / 2^18; without the loss of xl cl half as much (15.91 and 7.98 are reached).  The K additions
    // (with the roundings of x - mu, c - mu and |c|^2 counted among them) lose at most 2^-23 of the sum of the
    // magnitudes each.  The last term covers values that vanish below the smallest bf16 numbers.  With xl = 0 the remainder of c is
    // all that is lost: 2^-17 |x| |c|, twice.
    constexpr float kSplit3 = 16.2f / 262144.0f, kSplit4 = 8.1f / 262144.0f, kSplit2 = 4.05f / 262144.0f, kAdd = (16.0f * KS + 16.0f) / 8388608.0f;
    const float split = !low_points ? kSplit2 : four ? kSplit4 : kSplit3;
    auto filter_error = [split](float xn, float c1) {
        return xn * c1 * (split + 2.1f * kAdd) + c1 * c1 * (1.1f * kAdd) + 1e-35f * (1.0f + xn + c1);
    };
    // Largest filter value a nearest centroid can have.  The nearest centroid is no farther than the one with the
    // smallest filter value, so its norm is at most |x| plus that distance.
    auto threshold = [&](int pt) {
        const float *e = ent + pt * C::NE * 5;
        const float xn = sqrtf(xnorm2[pt]) * 1.001f;
        float gmin = INFINITY;
#pragma unroll
        for (int k = 0; k < C::NE; ++k) gmin = fminf(gmin, e[k * 5]);
        const float d2 = fmaxf(xn * xn + gmin + filter_error(xn, cmax), 0.0f);
        const float c1 = fminf(cmax, (xn + sqrtf(d2)) * 1.001f);
        return gmin + 2.0f * filter_error(xn, c1);
    };
    for (int pt = tid; pt < C::PTS; pt += 256) {
        if (static_cast<uint32_t>(pt) >= np) break;
        const float *e = ent + pt * C::NE * 5;
        const float thr = threshold(pt);
        bool full = !(thr < 1e37f);
        int cells = 0, last = 0;
#pragma unroll
        for (int k = 0; k < C::NE; ++k) {
            full = full || e[k * 5 + 2] <= thr;
            if (e[k * 5] <= thr) { ++cells; last = 2 * k; }
            if (e[k * 5 + 1] <= thr) { ++cells; last = 2 * k + 1; }
        }
        const int kind = full ? 2 : cells == 1 ? 0 : 1;
        list[kind][atomicAdd(&s_count[kind], 1u)] = static_cast<uint32_t>(pt) | static_cast<uint32_t>(last) << 16;
    }
    __syncthreads();
    const int l16 = tid & 15;
    // centroid of 16-lane group position l16 in tile t of the cell of entry k of a point
    auto cell_centroid = [&](const float *e, int k, int t) {
        const int h = C::NE == 2 ? k >> 1 : (k >> 1) & 1;
        const uint32_t cell = __float_as_uint(e[(k >> 1) * 5 + 3 + (k & 1)]);
        return (cell * C::TPC + t) * 32 + 8 * (l16 >> 2) + 4 * h + (l16 & 3);
    };
    auto put = [&](uint64_t q, double best, uint32_t bi) {
        const size_t o = static_cast<size_t>(q) * m + j;
        store_label(labels, label_bytes, o, bi);
        if (dist) dist[o] = static_cast<float>(best);
    };
    // One cell: distances in fp32 from the differences are within (dsub + 4) 2^-23 of themselves, so usually one
    // centroid is left; only where several are (or the distance itself is wanted) is double precision needed.
    // 16 lanes per point.
    const float near = 1.0f + 2.2f * static_cast<float>(dsub + 4) / 8388608.0f;
    const uint32_t n_one = s_count[0], n_several = s_count[1], n_hard = s_count[2];
    for (uint32_t t0 = tid >> 4; t0 < n_one; t0 += 16) {
        const uint32_t rec = list[0][t0];
        const int pt = static_cast<int>(rec & 0xFFFFu), k = static_cast<int>(rec >> 16);
        const uint64_t q = at(pt);
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub, *e = ent + pt * C::NE * 5;
        uint32_t c[C::TPC];
        const float *row[C::TPC];
        float v[C::TPC];
#pragma unroll
        for (int t = 0; t < C::TPC; ++t) {
            c[t] = cell_centroid(e, k, t);
            row[t] = cbj + static_cast<size_t>(c[t] < static_cast<uint32_t>(ncent) ? c[t] : ncent - 1) * dsub;
            v[t] = 0.0f;
        }
        int d0 = 0;
#pragma unroll 4
        for (; d0 + 4 <= dsub; d0 += 4) {
            const f4_any a = *reinterpret_cast<const f4_any *>(x + d0);
#pragma unroll
            for (int t = 0; t < C::TPC; ++t) {
                const f4_any b = *reinterpret_cast<const f4_any *>(row[t] + d0);
#pragma unroll
                for (int i = 0; i < 4; ++i) { const float u = a.v[i] - b.v[i]; v[t] = fmaf(u, u, v[t]); }
            }
        }
        for (; d0 < dsub; ++d0)
#pragma unroll
            for (int t = 0; t < C::TPC; ++t) { const float u = x[d0] - row[t][d0]; v[t] = fmaf(u, u, v[t]); }
        float mn = INFINITY;
#pragma unroll
        for (int t = 0; t < C::TPC; ++t) {
            if (c[t] >= static_cast<uint32_t>(ncent)) v[t] = INFINITY;
            mn = fminf(mn, v[t]);
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) mn = fminf(mn, __shfl_xor(mn, off));
        const float lim = mn * near + 1e-34f;
        int left = 0;
        uint32_t bi = 0xFFFFFFFFu;
#pragma unroll
        for (int t = 0; t < C::TPC; ++t)
            if (v[t] <= lim) { ++left; bi = min(bi, c[t]); }
        int total = left;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) total += __shfl_xor(total, off);
        if (total == 1 && !dist) {
            if (left) put(q, 0.0, bi);
            continue;
        }
        double best = INFINITY;
        bi = 0xFFFFFFFFu;
#pragma unroll
        for (int t = 0; t < C::TPC; ++t)
            if ((v[t] <= lim || !(lim < INFINITY)) && c[t] < static_cast<uint32_t>(ncent)) take_smaller(best, bi, exact_distance(x, row[t], dsub), c[t]);
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const double ov = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            take_smaller(best, bi, ov, oi);
        }
        if (l16 == 0) put(q, best, bi);
    }
    // several cells
    for (uint32_t t0 = tid >> 4; t0 < n_several; t0 += 16) {
        const int pt = static_cast<int>(list[1][t0] & 0xFFFFu);
        const uint64_t q = at(pt);
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub, *e = ent + pt * C::NE * 5;
        const float thr = threshold(pt);
        double best = INFINITY;
        uint32_t bi = 0xFFFFFFFFu;
#pragma unroll 1
        for (int k = 0; k < 2 * C::NE; ++k)
            if (e[(k >> 1) * 5 + (k & 1)] <= thr) {
#pragma unroll
                for (int t = 0; t < C::TPC; ++t) {
                    const uint32_t c = cell_centroid(e, k, t);
                    if (c < static_cast<uint32_t>(ncent)) take_smaller(best, bi, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
                }
            }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const double ov = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            take_smaller(best, bi, ov, oi);
        }
        if (l16 == 0) put(q, best, bi);
    }
    // Points whose cells are not all known are compared with every centroid.  They are few where centroids are well
    // apart; where a codebook repeats itself, or its sub-vectors are so short that the filter cannot tell its centroids
    // apart, they are most.
    // (the thread's number is taken afresh, so that nothing derived from it is kept, spilled, over the loop above)
    int tid_now = tid;
    asm volatile("" : "+v"(tid_now));
    if (n_hard > kFewHard) {                                          // uniform
        const int tid = tid_now, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        // 32 points at a time: their components lie in LDS in double precision, [component][point]; a wavefront takes 8 of
        // them against 4 centroids per lane, so that eight components read serve 32 products (bound by the
        // double-precision vector instructions, two per component: seven tenths of their rate).  The centroids' rows reach the
        // lanes through LDS, 16 components at a time, read one step ahead; rows of up to 4 components are read where they
        // are.  20000 x 8 x 16, all centroids equal: 18 ms, an eighth of points and centroids zeros: 3.2 ms (one point at a
        // time: 88 and 11.9; all distances on the double-precision matrix pipe: 8.0 both); 20000 x 32 x 1: 15.6 (82; 17.5).
        uint8_t *tile = smem + C::LIST_BYTES;
        double *xd = reinterpret_cast<double *>(tile + C::ROW_BYTES);
        constexpr int LOADS = C::PER_LANE;                               // 16-byte parts of a tile per thread
        float4 ahead[LOADS];
        auto load_rows = [&](int c0, int o0) {                        // (4 lanes per row)
#pragma unroll
            for (int i = 0; i < LOADS; ++i) {
                const int f = tid + 256 * i, c = c0 + (f >> 2), o = o0 + 4 * (f & 3);
                const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
                if (o + 4 <= dsub) {
                    const f4_any v = *reinterpret_cast<const f4_any *>(src + o);
                    ahead[i] = make_float4(v.v[0], v.v[1], v.v[2], v.v[3]);
                } else {
                    ahead[i] = make_float4(o < dsub ? src[o] : 0.0f, o + 1 < dsub ? src[o + 1] : 0.0f, o + 2 < dsub ? src[o + 2] : 0.0f, 0.0f);
                }
            }
        };
        const int last = (ncent - 1) / C::ROWS * C::ROWS;
        for (uint32_t h0 = 0; h0 < n_hard; h0 += C::TOGETHER) {         // uniform
            const uint32_t nh = min(n_hard - h0, static_cast<uint32_t>(C::TOGETHER));
            __syncthreads();                                          // the minima and the previous points are no longer read
            for (int t = tid; t < C::TOGETHER * dsub; t += 256) {
                const int p = t / dsub, o = t % dsub;
                const uint64_t q = at(list[2][h0 + (static_cast<uint32_t>(p) < nh ? p : 0)] & 0xFFFFu);
                xd[o * C::TOGETHER + p] = static_cast<double>(points[static_cast<size_t>(q) * ld + j * dsub + o]);
            }
            const double *xw = xd + wave * C::PER_WAVE;
            double best[C::PER_WAVE];
            uint32_t bi[C::PER_WAVE];
#pragma unroll
            for (int p = 0; p < C::PER_WAVE; ++p) { best[p] = INFINITY; bi[p] = 0xFFFFFFFFu; }
            if constexpr (C::ROWS_IN_LDS) load_rows(last, 0);
            else __syncthreads();
            // (from the last centroid to the first, so that "no farther" leaves the smallest index of equal distances)
            for (int c0 = last; c0 >= 0; c0 -= C::ROWS) {           // uniform
                double acc[C::PER_LANE][C::PER_WAVE];                              // (as exact_distance adds them up)
#pragma unroll
                for (int k = 0; k < C::PER_LANE; ++k)
#pragma unroll
                    for (int p = 0; p < C::PER_WAVE; ++p) acc[k][p] = 0.0;
                for (int o0 = 0; o0 < dsub; o0 += kTileComps) {       // uniform
                    if constexpr (C::ROWS_IN_LDS) {
                        __syncthreads();                              // the rows before these are no longer read
#pragma unroll
                        for (int i = 0; i < LOADS; ++i)
                            *reinterpret_cast<float4 *>(tile + ((tid + 256 * i) >> 2) * kTileStride + 16 * (tid & 3)) = ahead[i];
                        __syncthreads();                              // (also publishes the points)
                        const bool more = o0 + kTileComps < dsub;
                        if (more || c0 > 0) load_rows(more ? c0 : c0 - C::ROWS, more ? o0 + kTileComps : 0);
                    }
#pragma unroll 1
                    for (int o = o0; o < o0 + kTileComps && o < dsub; o += 4) {        // uniform
                        float b[C::PER_LANE][4];
#pragma unroll
                        for (int k = 0; k < C::PER_LANE; ++k) {
                            if constexpr (C::ROWS_IN_LDS) {
                                const float4 v = *reinterpret_cast<const float4 *>(tile + (64 * k + lane) * kTileStride + 4 * (o - o0));
                                b[k][0] = v.x; b[k][1] = v.y; b[k][2] = v.z; b[k][3] = v.w;
                            } else {
                                const int c = c0 + 64 * k + lane;
                                const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
#pragma unroll
                                for (int e = 0; e < 4; ++e) b[k][e] = src[e < dsub ? e : 0];
                            }
                        }
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            if (o + e >= dsub) break;                 // uniform
#pragma unroll
                            for (int k = 0; k < C::PER_LANE; ++k) {
                                const double cv = static_cast<double>(b[k][e]);
#pragma unroll
                                for (int p = 0; p < C::PER_WAVE; ++p) {
                                    const double u = xw[(o + e) * C::TOGETHER + p] - cv;
                                    acc[k][p] = fma(u, u, acc[k][p]);
                                }
                            }
                        }
                    }
                }
#pragma unroll
                for (int k = C::PER_LANE - 1; k >= 0; --k) {
                    const int c = c0 + 64 * k + lane;
                    if (c >= ncent) continue;
#pragma unroll
                    for (int p = 0; p < C::PER_WAVE; ++p) {
                        const bool take = acc[k][p] <= best[p];
                        best[p] = take ? acc[k][p] : best[p];
                        bi[p] = take ? static_cast<uint32_t>(c) : bi[p];
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < C::PER_WAVE; ++p) {
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const double ov = __shfl_xor(best[p], off);
                    const uint32_t oi = __shfl_xor(bi[p], off);
                    take_smaller(best[p], bi[p], ov, oi);
                }
                const uint32_t h = wave * C::PER_WAVE + p;
                if (lane == 0 && h < nh) put(at(list[2][h0 + h] & 0xFFFFu), best[p], bi[p]);
            }
        }
        return;
    }
    for (uint32_t hi = 0; hi < n_hard; ++hi) {                        // uniform
        const uint64_t q = at(list[2][hi] & 0xFFFFu);
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub;
        double best;
        uint32_t bi;
        nearest_of_all(x, cbj, dsub, ncent, red_v, red_i, best, bi);
        if (tid == 0) put(q, best, bi);
    }
}

template <int KS, int P, bool SPLIT, bool FOURS>
__global__ __launch_bounds__(256, KS <= 3 && P == 2 ? 3 : KS <= 16 ? 2 : 1) void assign_kernel(const float *__restrict__ points, uint64_t n, int ld,
                                                     const float *__restrict__ cb, int m, int dsub, int dp, int ncent,
                                                     void *__restrict__ labels, int label_bytes, float *__restrict__ dist)
{
    using C = AssignCfg<KS, P, SPLIT>;
    extern __shared__ __align__(16) uint8_t smem[];
    const int j = blockIdx.y;
    const uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * C::PTS;
    const uint32_t np = n - q0 < C::PTS ? static_cast<uint32_t>(n - q0) : C::PTS;
    nearest_by_split_products<KS, P, SPLIT, FOURS>(smem, [q0](uint32_t pt) { return q0 + pt; }, np, points, ld, cb + static_cast<size_t>(j) * ncent * dsub, j, m,
                                                   dsub, dp, ncent, labels, label_bytes, dist);
}

// ---- many points, sub-vectors of 5 to 64 components ------------------------------------------------------------
// The same result, with ONE fp16 product in the filter where the form above takes three or four bf16 ones: fp16 keeps 11 significant
// bits, and the window that this leaves around the smallest filter value holds 1.05 to 1.25 centroids on average (65536 centroids of 12 to
// 60 components, encoded data as well as Gaussian).  It is proven as above: from |x|, |c| and the lengths of the remainders x - xh and c - ch
// themselves.  Points with four or more cells of one half of a tile in their window, as a rule 1 in 1000 or fewer, are walked again, 32 or 128 at a time, the
// wavefronts sharing the centroids, and now that the window is known every centroid in it is listed and compared in double precision.  Where
// the windows hold too many for that (more than 32 to 128 centroids closer together than 2^-11 of their distance from the reference vector), the points
// left go through the split products.
//
// Scale: points and centroids are multiplied by a power of two that brings the largest component of 64 centroids to 2^4; it follows no other number, so that
// what lies far out takes no window but its own.  Points some thousand times farther out than those 64 overflow: they go through the split products.  Centroids as far out
// have no part in the filter: a centroid of length c is at least c - |x| away, which rules them out for every point whose nearest of the others is closer than that (the
// rest have no window either).  What falls below the normal numbers, 2^-14, is counted with the remainders whether the
// matrix pipe keeps it or not.
//
// What bounds it (KS = 3, the common case of up to 16 components): a tile of 32 x 32 distances is one matrix instruction and eight for its minima; together, with random
// numbers and nothing else to do, 29 ns per SIMD (21 and 16 each alone: the clock falls to 1.9 GHz meanwhile).  The walk takes 37 ns: another 1.3 vector instructions for the conversion of the
// centroids, 1 for the cells, and the barriers between the stages (29 ns without these three).  1024 points per workgroup: the operands and norms of the
// centroids, 40 clocks of the LDS per tile, then serve eight tiles of points.  250007 vectors, 8 sub-quantizers: 5.4 ms, of which the
// walk 4.7, the cells 0.35, the second walk 0.35; the numbers of the cells in the low bits of their minima leave four of these per point and lane room in
// the registers (three with a register each for their numbers: 1 % of the points were left open, and every workgroup walked again).
constexpr float kFarNorm = 4.0e9f;            // |c|^2 of a centroid too far out: a component of 65504 and above would be infinite in fp16
constexpr uint32_t kFewFar = 2;               // points without a window that are compared with all centroids one by one
constexpr uint32_t kCells = 512;              // cells of a codebook, at most: their numbers take nine bits
template <int KS, int P>
struct HalfCfg {
    static constexpr int DPMAX = 16 * KS / 3 & ~3;
    static constexpr int KH = (DPMAX + 15) / 16;                    // steps of 16 along K
    static constexpr bool TWO = 2 * DPMAX <= 16 * KH;               // room for the product xl ch
    static constexpr int RS = KH == 1 ? 256 : 128, TPR = 256 / RS, NG = (DPMAX / 4 + TPR - 1) / TPR;      // (as in AssignCfg)
    static constexpr int TPC = 4;                                   // tiles of 32 centroids per cell
    static constexpr int AHEAD = KH <= 4 ? 2 : 1, LAG = 2;
    static constexpr int STRIDE = KH * 32 + 16, PTS = 128 * P, NE = 2;
    static constexpr int BUF_BYTES = RS * STRIDE + RS * 4, STAGE_BYTES = 2 * BUF_BYTES;
    // minima of a point: KEEP by each of the two lanes that held them, and what became of them
    static constexpr int KEEP = 4, SLOTS = NE * KEEP;
    static constexpr uint32_t ITEMS = 2 * PTS;                      // cells that are looked at for all points together, at most
    static constexpr int ENT_BYTES = 2 * ITEMS * 2 + PTS * SLOTS * 4 + PTS * 5;
    // the second walk: centroids listed for 32 points,
    static constexpr int TILES2 = 4;                                // ... or for so many times 32
    static constexpr uint32_t FOUND = 4096;
    static constexpr int FOUND_BYTES = STAGE_BYTES + FOUND * 4 + 32 * TILES2 * 12;
    // the rest: up to 32 points whose centroids are split between the wavefronts, or each wavefront with points of its own
    static constexpr bool SPLIT = KS <= 6;
    static constexpr int MANY_P = KS <= 12 ? 2 : 1;
    using Few = AssignCfg<KS, 1, SPLIT>;
    using Many = AssignCfg<KS, MANY_P, false>;
    static constexpr int max4(int a, int b, int c, int d) { return (a > b ? a : b) > (c > d ? c : d) ? (a > b ? a : b) : (c > d ? c : d); }
    static constexpr int LDS_BYTES = max4(STAGE_BYTES > Few::LDS_BYTES ? STAGE_BYTES : Few::LDS_BYTES, ENT_BYTES, FOUND_BYTES, Many::LDS_BYTES);
};

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));

// v of the lane whose number differs in the bits of X, within four.
template <int X>
__device__ inline float other_of_four(float v)
{
    constexpr int perm = (0 ^ X) | (1 ^ X) << 2 | (2 ^ X) << 4 | (3 ^ X) << 6;
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), perm, 0xF, 0xF, true));
}

template <int KS, int P, bool FOURS>
__global__ __launch_bounds__(256, 2) void assign_half_kernel(const float *__restrict__ points, uint64_t n, int ld, const float *__restrict__ cb,
                                                             int m, int dsub, int dp, int ncent, void *__restrict__ labels, int label_bytes,
                                                             float *__restrict__ dist)
{
    using C = HalfCfg<KS, P>;
    constexpr int KH = C::KH;
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ __align__(16) float mus[128];                        // minus the reference vector, scaled
    __shared__ float mu[128], s_cmax[4], s_crest[4], xnorm2[C::PTS], xrest2[C::PTS];
    __shared__ uint32_t s_count[6], s_whole, s_cabs, s_cfar;
    __shared__ uint16_t open[C::PTS];                               // points that the first walk has left open; those without a window from the end
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = blockIdx.y;
    const uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * C::PTS;
    const uint32_t np = n - q0 < C::PTS ? static_cast<uint32_t>(n - q0) : C::PTS;
    const float *cbj = cb + static_cast<size_t>(j) * ncent * dsub;
    const int col = lane & 31, half = lane >> 5;

    // reference vector and scale
    if (tid == 0) s_whole = s_cabs = s_cfar = 0;
    if (tid < 6) s_count[tid] = tid == 4 ? C::ITEMS : 0;             // items, slow points, open points with a window, (second walk) centroids found; items that there are; open points without
    __syncthreads();
    if (tid < 128) {
        float sum = 0.0f, lo = 0.0f, hi = 0.0f;
        const int ns = ncent < 64 ? ncent : 64, step = ncent / ns;
        if (tid < dsub)
            for (int s = 0; s < ns; ++s) {
                const float v = cbj[static_cast<size_t>(s * step + s % step) * dsub + tid];
                sum += v;
                lo = s ? fminf(lo, v) : v;
                hi = s ? fmaxf(hi, v) : v;
            }
        const float mean = sum / static_cast<float>(ns);
        mu[tid] = mean;
        if (fabsf(mean) >= 8.0f) s_whole = 1;
        const float far = fmaxf(fabsf(hi - mean), fabsf(lo - mean)) + 1.0f * (fabsf(mean) >= 8.0f);
        if (far < INFINITY) atomicMax(&s_cabs, __float_as_uint(far));
    }
    for (int t = tid; t < C::STAGE_BYTES / 16; t += 256) reinterpret_cast<uint4 *>(smem)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (tid < 128 && s_whole) mu[tid] = rintf(mu[tid]);
    __syncthreads();
    const int ec = static_cast<int>(s_cabs >> 23) - 126;              // (x < 2^(exponent - 126) for the exponent field of x)
    const float scale = __uint_as_float(static_cast<uint32_t>(min(max(4 - ec, -120), 120) + 127) << 23);
    if (tid < 128) mus[tid] = -mu[tid] * scale;
    __syncthreads();

    const int srow = tid / C::TPR, spart = tid % C::TPR;
    // The point side of the product, as in the other form: [ -2 xh | 0 ... ], with room for two products [ -2 xh | -2 xl | 0 ... ].  One row
    // of LDS, by C::TPR threads; norm, rest: |x|^2 and the square of what is left out of x, of this thread's components
    auto convert_point = [&](uint8_t *row, uint64_t q, float &norm, float &rest) __attribute__((always_inline)) {
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub;
        norm = rest = 0.0f;
#pragma unroll 1
        for (int g = 0; g < C::NG; ++g) {
            const int o = 4 * (spart + C::TPR * g);
            if (o < dp) {
                v4h h, l;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int t = o + e < dsub ? o + e : dsub - 1;
                    const float u = o + e < dsub ? (x[t] - mu[t]) * scale : 0.0f, v = -2.0f * u;
                    h[e] = static_cast<_Float16>(v);
                    float left = v - static_cast<float>(h[e]);
                    if (C::TWO) {
                        l[e] = static_cast<_Float16>(left);
                        left -= static_cast<float>(l[e]);
                    }
                    norm = fmaf(u, u, norm);
                    rest = fmaf(0.25f * left, left, rest);
                }
                *reinterpret_cast<v4h *>(row + 2 * o) = h;
                if (C::TWO) *reinterpret_cast<v4h *>(row + 2 * (dp + o)) = l;
            }
        }
#pragma unroll
        for (int off = 1; off < C::TPR; off <<= 1) { norm += __shfl_xor(norm, off); rest += __shfl_xor(rest, off); }
    };
    v8h bq[P][KH];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        if (srow < 128) {                                             // (whole wavefronts)
            const uint32_t pt = p * 128 + srow;
            float norm, rest;
            convert_point(smem + srow * C::STRIDE, q0 + (pt < np ? pt : np - 1), norm, rest);
            if (spart == 0) { xnorm2[pt] = norm; xrest2[pt] = rest; }
        }
        __syncthreads();
        const uint8_t *b = smem + (wave * 32 + col) * C::STRIDE + half * 16;
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) bq[p][ks] = *reinterpret_cast<const v8h *>(b + ks * 32);
        __syncthreads();
    }

    // staging: TPR threads convert one centroid
    float pre[C::NG][4];
    auto load_stage = [&](int c0) __attribute__((always_inline)) {
        const int c = c0 + srow;
        const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 4 * (spart + C::TPR * g);
            if constexpr (FOURS) {
                const f4_any v = *reinterpret_cast<const f4_any *>(src + (o < dsub ? o : 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) pre[g][e] = v.v[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) pre[g][e] = src[o + e < dsub ? o + e : 0];       // (past the last: set to zero when the stage is stored)
            }
        }
    };
    float cmax2 = 0.0f, crest2 = 0.0f;        // largest |c|^2 and |c - ch|^2 among the centroids this thread converted
    bool cfar = false;                        // one of them is too far out
    auto store_stage = [&](int c0, uint8_t *buf) __attribute__((always_inline)) {
        uint8_t *row = buf + srow * C::STRIDE;
        float norm = 0.0f, rest = 0.0f;
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 4 * (spart + C::TPR * g);
            if (o < dp) {
                v4h h;
                const float4 mv = *reinterpret_cast<const float4 *>(mus + o);
                const float ref[4] = {mv.x, mv.y, mv.z, mv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float v = fmaf(pre[g][e], scale, ref[e]);        // (pre - mu), rounded once, scaled
                    if (!FOURS && o + e >= dsub) v = 0.0f;
                    h[e] = static_cast<_Float16>(v);
                    norm = fmaf(v, v, norm);
                    const float left = v - static_cast<float>(h[e]);
                    rest = fmaf(left, left, rest);
                }
                *reinterpret_cast<v4h *>(row + 2 * o) = h;
                if (C::TWO) *reinterpret_cast<v4h *>(row + 2 * (dp + o)) = h;
            }
        }
#pragma unroll
        for (int off = 1; off < C::TPR; off <<= 1) { norm += __shfl_xor(norm, off); rest += __shfl_xor(rest, off); }
        if (!(norm < kFarNorm)) {                                    // (NaN too)
            cfar = true;
            norm = 3.0e38f;                                          // never the nearest (finite: the number of a cell goes into its minimum)
#pragma unroll
            for (int g = 0; g < C::NG; ++g) {
                const int o = 4 * (spart + C::TPR * g);
                if (o < dp) {
                    *reinterpret_cast<v4h *>(row + 2 * o) = v4h{};
                    if (C::TWO) *reinterpret_cast<v4h *>(row + 2 * (dp + o)) = v4h{};
                }
            }
        } else {
            crest2 = fmaxf(crest2, rest);                             // (rows past the last repeat it)
            cmax2 = fmaxf(cmax2, norm);
        }
        if (c0 + srow >= ncent) norm = 3.0e38f;
        if (spart == 0) reinterpret_cast<float *>(buf + C::RS * C::STRIDE)[srow] = norm;
    };

    // the four smallest cell minima of each of this lane's points, in increasing order; the low bits hold the number of the cell
    constexpr int KEEP = C::KEEP;
    float best4[P][KEEP];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int i = 0; i < KEEP; ++i) best4[p][i] = INFINITY;
    float mn[P];                              // minimum of the cell so far
    auto read_tile = [&](const uint8_t *buf, int t, v8h (&a)[KH], v16f &norm) __attribute__((always_inline)) {
        const uint8_t *ra = buf + (t * 32 + col) * C::STRIDE + half * 16;
#pragma unroll
        for (int ks = 0; ks < KH; ++ks) a[ks] = *reinterpret_cast<const v8h *>(ra + ks * 32);
        const float *nr = reinterpret_cast<const float *>(buf + C::RS * C::STRIDE) + t * 32 + 4 * half;
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(nr + 2 * v);
            norm[v] = x.x; norm[v + 1] = x.y; norm[v + 2] = x.z; norm[v + 3] = x.w;
        }
    };
    // minimum of 16 filter values and `with`, in eight instructions
    auto minimum = [](const v16f &acc, float with) __attribute__((always_inline)) {
        float m0 = fminf(fminf(acc[0], acc[1]), acc[2]), m1 = fminf(fminf(acc[3], acc[4]), acc[5]);
#pragma unroll
        for (int v = 6; v < 14; v += 4) {
            m0 = fminf(fminf(acc[v], acc[v + 1]), m0);
            m1 = fminf(fminf(acc[v + 2], acc[v + 3]), m1);
        }
        m0 = fminf(fminf(acc[14], acc[15]), m0);
        return fminf(fminf(m0, m1), with);
    };
    // One wavefront's tiles of a stage, as in the other form: the minimum of step x - LAG while the products of step x run
    auto compute_cell = [&](const uint8_t *buf, int t0) __attribute__((always_inline)) {
        constexpr int AH = C::AHEAD;
        v8h a[AH][KH];
        v16f norm[AH], acc[C::LAG + 1];
        if constexpr (AH == 2) read_tile(buf, t0, a[0], norm[0]);
#pragma unroll
        for (int x = 0; x < C::TPC * P + C::LAG; ++x) {
            const int t = x / P, p = x % P;
            if (x < C::TPC * P) {
                if constexpr (AH == 2) {
                    if (p == 0 && t + 1 < C::TPC) read_tile(buf, t0 + t + 1, a[(t + 1) & 1], norm[(t + 1) & 1]);
                } else {
                    if (p == 0) read_tile(buf, t0 + t, a[0], norm[0]);
                }
#pragma unroll
                for (int ks = 0; ks < KH; ++ks)
                    acc[x % (C::LAG + 1)] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[t % AH][ks], bq[p][ks], ks == 0 ? norm[t % AH] : acc[x % (C::LAG + 1)], 0, 0, 0);
            }
            if (x >= C::LAG) {
                const int q = (x - C::LAG) % P;
                mn[q] = minimum(acc[(x - C::LAG) % (C::LAG + 1)], x - C::LAG < P ? INFINITY : mn[q]);
                asm volatile("" : "+v"(mn[q]));                       // (keeps it here: its use is behind a branch)
            }
#pragma unroll
            for (int ks = 0; ks < KH; ++ks) {                         // matrix and vector instructions in turn
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, (8 + KH - 1) / KH, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto enter = [&](uint32_t cell) __attribute__((always_inline)) {
        asm volatile("" : "+v"(cell));                                // (in a vector register: one instruction for mask and number)
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const float v = __uint_as_float((__float_as_uint(mn[p]) & ~(kCells - 1u)) | cell);
#pragma unroll
            for (int i = KEEP - 1; i >= 0; --i) best4[p][i] = __builtin_amdgcn_fmed3f(i ? best4[p][i - 1] : -INFINITY, best4[p][i], v);
        }
    };
    bool any = false;                                                 // a point that does not overflow (without one there is nothing to walk for)
    for (uint32_t pt = tid; pt < np; pt += 256) any = any || xrest2[pt] < INFINITY;
    const int nst = __syncthreads_or(any) ? (ncent + C::RS - 1) / C::RS : 0;
    load_stage(0);
    store_stage(0, smem);
    __syncthreads();
    for (int s = 0; s < nst; ++s) {                                   // uniform
        if (s + 1 < nst) load_stage((s + 1) * C::RS);
#pragma unroll 1
        for (int h = 0; h < C::RS / (32 * C::TPC); ++h) {
            compute_cell(smem + (s & 1) * C::BUF_BYTES, h * C::TPC);
            enter(s * (C::RS / (32 * C::TPC)) + h);
        }
        if (s + 1 < nst) store_stage((s + 1) * C::RS, smem + ((s + 1) & 1) * C::BUF_BYTES);
        __syncthreads();
    }

    // hand the minima over: ent[point][half that held them][KEEP]
    float *ent = reinterpret_cast<float *>(smem);
    uint16_t *items = reinterpret_cast<uint16_t *>(ent + C::PTS * C::SLOTS), *res = items + C::ITEMS;        // cells to look at: (point, slot); what was found
    uint16_t *first = res + C::ITEMS, *slow = first + C::PTS;         // first item of a point; points that need double precision
    uint8_t *has = reinterpret_cast<uint8_t *>(slow + C::PTS);        // the slots of a point that are looked at
#pragma unroll
    for (int p = 0; p < P; ++p) {
        float *e = ent + (p * 128 + wave * 32 + col) * C::SLOTS + half * KEEP;
#pragma unroll
        for (int i = 0; i < KEEP; ++i) e[i] = best4[p][i];
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { cmax2 = fmaxf(cmax2, __shfl_xor(cmax2, off)); crest2 = fmaxf(crest2, __shfl_xor(crest2, off)); }
    if (lane == 0) { s_cmax[wave] = cmax2; s_crest[wave] = crest2; }
    if (cfar) s_cfar = 1;
    __syncthreads();
    const float farthest = s_cfar ? 0.996f * sqrtf(kFarNorm) : INFINITY;          // centroids this long are not among the cells
    const float crest = sqrtf(fmaxf(fmaxf(s_crest[0], s_crest[1]), fmaxf(s_crest[2], s_crest[3]))) * 1.001f;
    const float cmax = sqrtf(fmaxf(fmaxf(s_cmax[0], s_cmax[1]), fmaxf(s_cmax[2], s_cmax[3]))) * 1.001f;

    // Error of a filter value, |c| <= c1: <x, c> - <xh, ch> = <x - xh, c> + <xh, c - ch>, doubled, with remainders of known lengths (fp16 has
    // 11 significant bits: they are 2^-11 of the whole at most, and 0.4 of that as a rule).  A component below 2^-14 may lose all of it in the
    // matrix pipe: `tiny` for dp of them.  The additions as in the other form.
    constexpr float kNumber = kCells / 8388608.0f, kAddHalf = (16.0f * KH + 16.0f) / 8388608.0f;
    const float tiny = sqrtf(static_cast<float>(dp)) * (1.01f / 16384.0f);
    auto filter_error = [tiny, crest](float xn, float xr, float c1) {
        return 2.0f * ((xn + xr) * (fminf(crest, c1 * (1.001f / 2048.0f)) + tiny) + xr * c1) + (xn * 2.1f + c1 * 1.1f) * c1 * kAddHalf + 1e-35f * (1.0f + xn + c1);
    };
    // Largest filter value a nearest centroid can have (as in the other form).
    for (uint32_t pt = tid; pt < np; pt += 256) {
        const float *e = ent + pt * C::SLOTS;
        const float xn = sqrtf(xnorm2[pt]) * 1.001f, xr = sqrtf(xrest2[pt]) * 1.001f + tiny;
        const float gmin = fminf(e[0], e[KEEP]);
        const float d2 = fmaxf(xn * xn + gmin + (1.1f * kNumber) * fabsf(gmin) + filter_error(xn, xr, cmax), 0.0f);
        const float reach = (xn + sqrtf(d2)) * 1.001f, c1 = fminf(cmax, reach);
        const float window = 2.0f * filter_error(xn, xr, c1);
        const float thr = reach < farthest ? gmin + window + (2.1f * kNumber) * (fabsf(gmin) + window) : INFINITY;      // (what the number of a cell takes of the value)
        xnorm2[pt] = thr;                                             // (the norm is needed no more)
        uint32_t slots = 0;
#pragma unroll
        for (int k = 0; k < C::SLOTS; ++k) slots |= (e[k] <= thr ? 1u : 0u) << k;
        constexpr uint32_t kLast = 1u << (KEEP - 1) | 1u << (C::SLOTS - 1);
        bool left = !(thr < 1e37f) || (slots & kLast);
        uint32_t to = 0;
        if (!left) {
            to = atomicAdd(&s_count[0], static_cast<uint32_t>(__popc(slots)));
            left = to + __popc(slots) > C::ITEMS;
            if (left) atomicMin(&s_count[4], to);
        }
        if (left) {
            if (thr < 1e37f) open[atomicAdd(&s_count[2], 1u)] = static_cast<uint16_t>(pt);
            else open[C::PTS - 1 - atomicAdd(&s_count[5], 1u)] = static_cast<uint16_t>(pt);
            slots = 0;
        }
        has[pt] = static_cast<uint8_t>(slots);
        first[pt] = static_cast<uint16_t>(to);
        for (; slots; slots &= slots - 1) items[to++] = static_cast<uint16_t>(pt * C::SLOTS + __builtin_ctz(slots));
    }
    __syncthreads();
    auto put = [&](uint64_t q, double best, uint32_t bi) {
        const size_t o = static_cast<size_t>(q) * m + j;
        store_label(labels, label_bytes, o, bi);
        if (dist) dist[o] = static_cast<float>(best);
    };
    // The 64 centroids of a cell, 16 lanes per cell: four lanes read a row together, 16 components at a time (a lane per row has four
    // times as many requests to the first-level cache, as many as the whole walk can hide).  Distances in fp32
    // from the differences are within (dsub + 4) 2^-23 of themselves, so usually one centroid is left; only where several are (or the
    // distance itself is wanted) is double precision needed.
    const float near = 1.0f + 2.2f * static_cast<float>(dsub + 4) / 8388608.0f;
    const int l4 = tid & 3, quad = (tid >> 2) & 3;
    constexpr int ROWS = 4 * C::TPC;                                  // rows per lane quad
    // row i of a quad in a cell; half: of the lane that held its minimum
    auto row_of = [](uint32_t cell, int half, int i, int quad) { return (cell * C::TPC + (i >> 2)) * 32 + 8 * (i & 3) + 4 * half + quad; };
    auto distances = [&](const float *x, uint32_t cell, int half, float (&v)[ROWS]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i) v[i] = 0.0f;
#pragma unroll 1
        for (int o = 4 * l4; o < dsub; o += 16) {
            float a[4];
            f4_any b[ROWS];
            const bool whole = FOURS || o + 4 <= dsub;
#pragma unroll
            for (int c = 0; c < 4; ++c) a[c] = whole || o + c < dsub ? x[o + c] : 0.0f;
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                const uint32_t c = row_of(cell, half, i, quad);
                const float *row = cbj + static_cast<size_t>(c < static_cast<uint32_t>(ncent) ? c : ncent - 1) * dsub + o;
                if (whole) b[i] = *reinterpret_cast<const f4_any *>(row);
                else {
#pragma unroll
                    for (int z = 0; z < 4; ++z) b[i].v[z] = o + z < dsub ? row[z] : 0.0f;
                }
            }
#pragma unroll
            for (int i = 0; i < ROWS; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) { const float u = a[c] - b[i].v[c]; v[i] = fmaf(u, u, v[i]); }
        }
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            v[i] += other_of_four<1>(v[i]);
            v[i] += other_of_four<2>(v[i]);
            if (row_of(cell, half, i, quad) >= static_cast<uint32_t>(ncent)) v[i] = INFINITY;
        }
    };
    // every cell: its smallest distance (in place of the filter's), and (bits 9 ..) the row that has it: 4 i + quad, or 64 where
    // several are too close to tell
    const uint32_t n_items = min(s_count[0], s_count[4]), n_open = s_count[2], n_no_window = s_count[5];
    for (uint32_t t0 = tid >> 4; t0 < n_items; t0 += 16) {
        const uint32_t item = items[t0], pt = item / C::SLOTS, slot = item % C::SLOTS, cell = __float_as_uint(ent[item]) & (kCells - 1u);
        float v[ROWS];
        distances(points + static_cast<size_t>(q0 + pt) * ld + j * dsub, cell, slot / KEEP, v);
        float least = v[0];
#pragma unroll
        for (int i = 1; i < ROWS; ++i) least = fminf(least, v[i]);
        least = fminf(least, __shfl_xor(least, 4));
        least = fminf(least, __shfl_xor(least, 8));
        const float lim = least * near + 1e-34f;
        uint32_t found = 0;                                           // number << 16 | sum of their rows
#pragma unroll
        for (int i = 0; i < ROWS; ++i) found += v[i] <= lim ? 0x10000u + 4 * i + quad : 0u;
        found += __shfl_xor(found, 4);
        found += __shfl_xor(found, 8);
        if ((tid & 15) == 0) {
            ent[item] = least;
            res[t0] = static_cast<uint16_t>(cell | (found >> 16 == 1 ? found & 63u : 64u) << 9);
        }
    }
    __syncthreads();
    // every point: done where one centroid is left
    auto centroid_of = [&](uint32_t r, uint32_t slot) { const uint32_t row = r >> 9; return row_of(r & (kCells - 1u), slot / KEEP, row >> 2, row & 3); };
    for (uint32_t pt = tid; pt < np; pt += 256) {
        const uint32_t slots = has[pt];
        if (!slots) continue;
        const float *e = ent + pt * C::SLOTS;
        float least = INFINITY;
#pragma unroll
        for (int k = 0; k < C::SLOTS; ++k) least = slots >> k & 1u ? fminf(least, e[k]) : least;
        const float lim = least * near + 1e-34f;
        uint32_t close = 0;
#pragma unroll
        for (int k = 0; k < C::SLOTS; ++k) close |= (slots >> k & 1u) && e[k] <= lim ? 1u << k : 0u;
        const uint32_t slot = __builtin_ctz(close), r = res[first[pt] + __popc(slots & ((1u << slot) - 1u))];
        if ((close & (close - 1)) == 0 && r >> 9 < 64) {
            const uint32_t c = centroid_of(r, slot);
            const uint64_t q = q0 + pt;
            put(q, dist ? exact_distance(points + static_cast<size_t>(q) * ld + j * dsub, cbj + static_cast<size_t>(c) * dsub, dsub) : 0.0, c);
        } else {
            xnorm2[pt] = lim;
            slow[atomicAdd(&s_count[1], 1u)] = static_cast<uint16_t>(pt);
        }
    }
    __syncthreads();
    const uint32_t n_slow = s_count[1];
    for (uint32_t t0 = tid >> 4; t0 < n_slow; t0 += 16) {
        const uint32_t pt = slow[t0];
        const uint64_t q = q0 + pt;
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub;
        const float lim = xnorm2[pt];
        double best = INFINITY;
        uint32_t bi = 0xFFFFFFFFu;
        uint32_t t = first[pt];
        for (uint32_t slots = has[pt]; slots; slots &= slots - 1, ++t) {         // (the same for the 16 lanes)
            const uint32_t slot = __builtin_ctz(slots), r = res[t];
            if (!(ent[pt * C::SLOTS + slot] <= lim)) continue;
            if (r >> 9 < 64) {
                const uint32_t c = centroid_of(r, slot);
                take_smaller(best, bi, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
                continue;
            }
            const uint32_t cell = r & (kCells - 1u);
            float v[ROWS];
            distances(x, cell, slot / KEEP, v);
            uint32_t take = 0;
#pragma unroll
            for (int i = 0; i < ROWS; ++i) take |= v[i] <= lim ? 1u << i : 0u;
            for (; take; take &= take - 1) {
                const uint32_t c = row_of(cell, slot / KEEP, __builtin_ctz(take), quad);
                if (c < static_cast<uint32_t>(ncent)) take_smaller(best, bi, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
            }
        }
#pragma unroll
        for (int off = 4; off < 16; off <<= 1) {
            const double ov = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            take_smaller(best, bi, ov, oi);
        }
        if ((tid & 15) == 0) put(q, best, bi);
    }
    if (n_open + n_no_window == 0) return;                            // uniform

    // ---- the second walk --------------------------------------------------------------------------------------
    // 32 points at a time, or 128 where more are open (all of them with 4096 clusters of 16 centroids, 250007 x 8 x 16: 17.3 ms; with split products for more than a
    // sixteenth of a workgroup's points 30.2, for all without this filter 19.0; 140000 x 4 x 32 9.8, 12.1 and 8.0).  A walk that finds more than there is room for ends at once.
    uint32_t done = 0;
    auto walk_again = [&](auto tiles) __attribute__((always_inline)) {
        constexpr int W = decltype(tiles)::value, MOST = 32 * W;
        uint32_t *found = reinterpret_cast<uint32_t *>(smem + C::STAGE_BYTES);                    // (point << 16) | centroid
        unsigned long long *nearest = reinterpret_cast<unsigned long long *>(found + C::FOUND);       // of every point: distance, then ...
        uint32_t *which = reinterpret_cast<uint32_t *>(nearest + MOST);                           // ... centroid
        const uint32_t mine = min(static_cast<uint32_t>(MOST), n_open - done);
        __syncthreads();                                              // (the minima, or what the points before these left, are no longer read)
        for (int t = tid; t < MOST * C::STRIDE / 16; t += 256) reinterpret_cast<uint4 *>(smem)[t] = make_uint4(0, 0, 0, 0);        // rows: zero past dp
        __syncthreads();
        if (srow < MOST) {
            float norm, rest;
            convert_point(smem + srow * C::STRIDE, q0 + open[done + min(static_cast<uint32_t>(srow), mine - 1)], norm, rest);
        }
        if (tid < MOST) { nearest[tid] = ~0ull; which[tid] = 0xFFFFFFFFu; }
        if (tid == 0) s_count[3] = 0;
        __syncthreads();
        v8h bx[W][KH];
        float window[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
#pragma unroll
            for (int ks = 0; ks < KH; ++ks) bx[w][ks] = *reinterpret_cast<const v8h *>(smem + (32 * w + col) * C::STRIDE + half * 16 + ks * 32);
            window[w] = static_cast<uint32_t>(32 * w + col) < mine ? xnorm2[open[done + 32 * w + col]] : -INFINITY;
        }
        // (a wavefront reads the centroids of its tiles itself, AHEAD2 tiles ahead, and needs nothing from the others: with stages of the
        // workgroup as above every one of them waited for its loads, 0.25 ms a walk of 65536)
        constexpr int AHEAD2 = KH == 1 ? 4 : KH == 2 ? 2 : 1, G = W == 1 ? AHEAD2 : 1;            // G: tiles of centroids whose products run together
        const int ntiles = (ncent + 31) / 32;
        float *wnorm = reinterpret_cast<float *>(smem) + wave * 32 * AHEAD2;                // |c|^2 of these tiles
        float raw[AHEAD2][KH][8];
        auto component = [&](int ks, int e) { return (C::TWO ? 0 : 16 * ks + 8 * half) + e; };       // of K position 16 ks + 8 half + e
        auto load_tile = [&](int t, float (&r)[KH][8]) __attribute__((always_inline)) {
            const int c = t * 32 + col;
            const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
#pragma unroll
            for (int ks = 0; ks < KH; ++ks)
#pragma unroll
                for (int e = 0; e < 8; e += 4) {
                    const int o = component(ks, e);
                    if constexpr (FOURS) {
                        const f4_any v = *reinterpret_cast<const f4_any *>(src + (o < dsub ? o : 0));
#pragma unroll
                        for (int z = 0; z < 4; ++z) r[ks][e + z] = v.v[z];
                    } else {
#pragma unroll
                        for (int z = 0; z < 4; ++z) r[ks][e + z] = src[o + z < dsub ? o + z : 0];
                    }
                }
        };
        __syncthreads();                                              // the points' rows are no longer read
        bool full = false;                                            // more are found than there is room for
#pragma unroll
        for (int d = 0; d < AHEAD2; ++d) load_tile(wave + 4 * d, raw[d]);
        for (int t0 = wave; t0 < ntiles && !full; t0 += 4 * AHEAD2) { // uniform
            v8h a[AHEAD2][KH];
            float norm[AHEAD2];
#pragma unroll
            for (int d = 0; d < AHEAD2; ++d) {
                norm[d] = 0.0f;
#pragma unroll
                for (int ks = 0; ks < KH; ++ks)
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int o = component(ks, e);
                        float v = fmaf(raw[d][ks][e], scale, mus[o]);
                        if (o >= dsub) v = 0.0f;
                        a[d][ks][e] = static_cast<_Float16>(v);
                        norm[d] = fmaf(v, v, norm[d]);
                    }
                load_tile(t0 + 4 * (d + AHEAD2), raw[d]);
            }
#pragma unroll
            for (int d = 0; d < AHEAD2; ++d) {
                if (!C::TWO) norm[d] += __shfl_xor(norm[d], 32);
                if (!(norm[d] < kFarNorm)) {
                    norm[d] = 3.0e38f;
#pragma unroll
                    for (int ks = 0; ks < KH; ++ks) a[d][ks] = v8h{};
                }
                if (half == 0) wnorm[32 * d + col] = (t0 + 4 * d) * 32 + col < ncent ? norm[d] : 3.0e38f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int d0 = 0; d0 < AHEAD2; d0 += G) {
                v16f acc[G][W];
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int v = 0; v < 16; v += 4) {
                        const float4 x = *reinterpret_cast<const float4 *>(wnorm + 32 * (d0 + g) + 4 * half + 2 * v);
#pragma unroll
                        for (int w = 0; w < W; ++w) { acc[g][w][v] = x.x; acc[g][w][v + 1] = x.y; acc[g][w][v + 2] = x.z; acc[g][w][v + 3] = x.w; }
                    }
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int w = 0; w < W; ++w)
#pragma unroll
                        for (int ks = 0; ks < KH; ++ks) acc[g][w] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[d0 + g][ks], bx[w][ks], acc[g][w], 0, 0, 0);
                uint32_t most = 0;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    float least = INFINITY;
#pragma unroll
                    for (int g = 0; g < G; ++g) least = minimum(acc[g][w], least);
                    if (!__builtin_amdgcn_ballot_w64(least <= window[w])) continue;      // uniform
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        uint32_t in = 0;                              // (a branch for every value is twice as long)
#pragma unroll
                        for (int v = 0; v < 16; ++v) in |= acc[g][w][v] <= window[w] ? 1u << v : 0u;          // (not past the last centroid: the window is below 1e37)
                        for (; in; in &= in - 1) {
                            const uint32_t v = __builtin_ctz(in);
                            most = atomicAdd(&s_count[3], 1u);
                            if (most < C::FOUND)
                                found[most] = static_cast<uint32_t>(32 * w + col) << 16 | static_cast<uint32_t>((t0 + 4 * (d0 + g)) * 32 + 8 * (v >> 2) + 4 * half + (v & 3));
                        }
                    }
                }
                full = full || __builtin_amdgcn_ballot_w64(most >= C::FOUND);
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
        __syncthreads();
        const uint32_t nfound = s_count[3];
        if (nfound > C::FOUND) return false;                          // uniform
        auto distance = [&](uint32_t f) {
            return static_cast<unsigned long long>(__double_as_longlong(         // (distances are >= +0: they order like their bits)
                exact_distance(points + static_cast<size_t>(q0 + open[done + (f >> 16)]) * ld + j * dsub, cbj + static_cast<size_t>(f & 0xFFFFu) * dsub, dsub)));
        };
#pragma unroll 1
        for (uint32_t t = tid; t < nfound; t += 256) atomicMin(&nearest[found[t] >> 16], distance(found[t]));
        __syncthreads();
#pragma unroll 1
        for (uint32_t t = tid; t < nfound; t += 256)
            if (distance(found[t]) == nearest[found[t] >> 16]) atomicMin(&which[found[t] >> 16], found[t] & 0xFFFFu);
        __syncthreads();
        if (tid < static_cast<int>(mine)) put(q0 + open[done + tid], __longlong_as_double(static_cast<long long>(nearest[tid])), which[tid]);
        done += mine;
        return true;
    };
    for (bool goes = true; goes && done < n_open;)                    // uniform
        goes = n_open - done <= 32 ? walk_again(std::integral_constant<int, 1>{}) : walk_again(std::integral_constant<int, C::TILES2>{});
    // (those without a window: one by one 0.12 ms each with 65536 centroids of 16 components; the walk with split products 0.3, above 32 components 2)
    uint32_t rest = n_open + n_no_window;
    if (n_no_window <= kFewFar) {                                     // uniform
        rest = n_open;
        __syncthreads();                                              // what the walks have in LDS is no longer read
        for (uint32_t i = 0; i < n_no_window; ++i) {
            const uint64_t q = q0 + open[C::PTS - 1 - i];
            double best;
            uint32_t bi;
            nearest_of_all(points + static_cast<size_t>(q) * ld + j * dsub, cbj, dsub, ncent, reinterpret_cast<double *>(smem), reinterpret_cast<uint32_t *>(smem + 32), best, bi);
            if (tid == 0) put(q, best, bi);
        }
    }
    while (done < rest) {                                             // uniform
        const uint32_t left = rest - done, base = done;
        const auto at = [&, base](uint32_t pt) { const uint32_t i = base + pt; return q0 + open[i < n_open ? i : C::PTS - 1 - (i - n_open)]; };
        __syncthreads();
        if (left <= C::Few::PTS) {
            nearest_by_split_products<KS, 1, C::SPLIT, FOURS>(smem, at, left, points, ld, cbj, j, m, dsub, dp, ncent, labels, label_bytes, dist);
            done += left;
        } else {
            const uint32_t mine = min(left, static_cast<uint32_t>(C::Many::PTS));
            nearest_by_split_products<KS, C::MANY_P, false, FOURS>(smem, at, mine, points, ld, cbj, j, m, dsub, dp, ncent, labels, label_bytes, dist);
            done += mine;
        }
    }
}

template <int KS, int P, bool SPLIT, bool FOURS>
static int launch_assign_f(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                           void *labels, int label_bytes, float *dist, hipStream_t st)
{
    using C = AssignCfg<KS, P, SPLIT>;
    const auto kernel = &assign_kernel<KS, P, SPLIT, FOURS>;
    const int arc = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), C::LDS_BYTES);
    if (arc) return arc;
    DCPQ_LAUNCH(kStageTrain, st, (assign_kernel<KS, P, SPLIT, FOURS>), dim3(static_cast<unsigned>((n + C::PTS - 1) / C::PTS), m), dim3(256),
                C::LDS_BYTES, points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist);
    DCPQ_CHECK_LAUNCH("assign_kernel");
    return DCPQ_OK;
}

template <int KS, int P, bool SPLIT>
static int launch_assign_t(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                           void *labels, int label_bytes, float *dist, hipStream_t st)
{
    if (dp == dsub) return launch_assign_f<KS, P, SPLIT, true>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return launch_assign_f<KS, P, SPLIT, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
}

template <int KS, int P, bool FOURS>
static int launch_half_f(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                         void *labels, int label_bytes, float *dist, hipStream_t st)
{
    using C = HalfCfg<KS, P>;
    const auto kernel = &assign_half_kernel<KS, P, FOURS>;
    const int arc = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), C::LDS_BYTES);
    if (arc) return arc;
    DCPQ_LAUNCH(kStageTrain, st, (assign_half_kernel<KS, P, FOURS>), dim3(static_cast<unsigned>((n + C::PTS - 1) / C::PTS), m), dim3(256),
                C::LDS_BYTES, points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist);
    DCPQ_CHECK_LAUNCH("assign_half_kernel");
    return DCPQ_OK;
}

template <int KS, int P>
static int launch_half(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                       void *labels, int label_bytes, float *dist, hipStream_t st)
{
    if (dp == dsub) return launch_half_f<KS, P, true>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return launch_half_f<KS, P, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
}

template <int KS>
static int launch_assign_ks(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                            void *labels, int label_bytes, float *dist, hipStream_t st)
{
    // The largest tile of points that still gives two workgroups per CU (the centroids are converted once per
    // workgroup and read from LDS once per wavefront, so large tiles are cheaper: 204 cycles per 32 x 32 distances with
    // 512 points at d = 16, 290 with 256); below that the four wavefronts split the centroids (2000 points, 8 x 16
    // components: 0.50 ms; 1.3 ms with 256-point tiles, which leave most CUs without work).
    auto enough = [&](int pts) { return (n + pts - 1) / pts * static_cast<uint64_t>(m) >= 512; };
    // One fp16 product in the filter, where two workgroups per CU can have 512 points or more (256 with sub-vectors above 32 components), of 1024
    // where these leave no more of the last round idle.  Rows of up to four components have all four bf16 products in one matrix
    // instruction as it is; above 64 both forms take the same time (30000 x 4 of 84: 7.0 and 6.9 ms, of 128: 13.3 both).  Split products
    // and this form, 65536 centroids, ms: 250007 x 8 of 16 components (whole numbers) 8.67 and 5.46; 250000 x 8 of 12 10.8 and 5.65; 70000 x 8 of 8 2.53
    // and 1.87, of 24 5.5 and 3.2; 140000 x 4 of 32 7.6 and 4.15; 30000 x 8 of 64 5.8 and 3.5; 20000 x 16 of 60 9.8 and 5.5; 1024 centroids: 250000 x 8
    // of 16 0.93 and 0.86.  Where every centroid repeats, or hundreds are closer together than both forms can tell, 4 to 7 % slower (repeated 16 times 186 and 195);
    // clusters of 16 that the split products can tell 0.9 to 1.25 of the time; half of the points 1e6 times farther out than the centroids as long, with 64 components 1.3.
    if constexpr (KS > 1 && KS <= 12) {
        constexpr int P = KS <= 3 ? 8 : KS <= 6 ? 4 : 2, PTS = HalfCfg<KS, P>::PTS;
        auto rounds = [&](int pts) { return ((n + pts - 1) / pts * static_cast<uint64_t>(m) + 511) / 512; };
        if (ncent <= static_cast<int>(kCells * 32 * HalfCfg<KS, P>::TPC)) {
            if constexpr (P == 8) {
                if (enough(PTS / 2) && (!enough(PTS) || rounds(PTS / 2) * 11 < rounds(PTS) * 20)) return launch_half<KS, P / 2>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
            }
            if (enough(PTS)) return launch_half<KS, P>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
        }
    }
    if constexpr (KS <= 6) {
        if (enough(AssignCfg<KS, 4, false>::PTS)) return launch_assign_t<KS, 4, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    }
    if (enough(AssignCfg<KS, KS <= 12 ? 2 : 1, false>::PTS) || KS > 6)
        return launch_assign_t<KS, KS <= 12 ? 2 : 1, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if constexpr (KS <= 6) return launch_assign_t<KS, 1, true>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return DCPQ_OK;
}

// The kernels of longer sub-vectors are compiled by themselves, by files that include this one as far as here: together they take the compiler six
// minutes, apart a bit more than two.
#ifndef DCPQ_ASSIGN_KERNELS_ONLY

int launch_assign_short(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                        void *labels, int label_bytes, float *dist, hipStream_t st)
{
    const int ks = (3 * dp + 15) / 16;
    if (ks <= 1) return launch_assign_ks<1>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 2) return launch_assign_ks<2>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return launch_assign_ks<3>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
}

// The same result with all inner products on the double-precision matrix pipe (f64_is_faster: where).  A workgroup takes kF64Points points and walks the centroids in steps of
// kF64Cents; |c|^2 - 2 <x, c> and the distance by difference are each within (dsub + 8) 2^-53 of the magnitudes they are
// made of, so a smallest value that no other comes near is the nearest centroid in either form.  Where another does (equal
// centroids above all), or a value is not finite, a wavefront compares the point with every centroid by difference.
// What bounds it: the matrix pipe for long rows (250000 x 4 points, 1024 centroids of 128 components: 4.5 ms, 0.75 of its
// peak; of 60 components half, of 16 a third), and the more the shorter they are what is done with each value, eight vector
// instructions.  Two wavefronts per SIMD, which is what 256 registers leave; without that bound the compiler takes 272, and
// with one wavefront it takes up to 1.8 times as long.
constexpr int kF64Points = 32, kF64Cents = 256;

__global__ __launch_bounds__(256, 2) void assign_f64_kernel(const float *__restrict__ points, uint64_t n, int ld,
                                                         const float *__restrict__ cb, int m, int dsub, int ncent,
                                                         void *__restrict__ labels, int label_bytes, float *__restrict__ dist)
{
    constexpr int MT = kF64Points / 16;
    __shared__ double red_v[4][kF64Points], norm[kF64Points], limit[kF64Points], red_c[4];
    __shared__ uint32_t red_i[4][kF64Points], close[kF64Points];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = blockIdx.y, lr = lane & 15, lk = lane >> 4;
    const uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * kF64Points;
    const float *cbj = cb + static_cast<size_t>(j) * ncent * dsub;

    // value v of the result tile (mt, nt): point 16 mt + 4 v + l / 16, centroid 4 (l % 16) + nt of the wavefront's 64
    double best[MT][4], na[MT], cmax = 0.0;
    // Of the second smallest value the upper word is kept.  Upper words of numbers below 2^1017 are ordered as floats of the
    // same bits are (2^265 is the largest magnitude that finite fp32 inputs give).
    float second[MT][4];
    auto upper = [](double x) { return __uint_as_float(static_cast<uint32_t>(__double_as_longlong(x) >> 32)); };
    uint32_t bi[MT][4];
    const float *ap[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) { best[mt][v] = INFINITY; second[mt][v] = 3.4e38f; bi[mt][v] = 0xFFFFFFFFu; }
        na[mt] = 0.0;
        const uint64_t q = q0 + mt * 16 + lr;
        ap[mt] = points + static_cast<size_t>(q < n ? q : n - 1) * ld + j * dsub;
    }
    for (int c0 = 0; c0 < ncent; c0 += kF64Cents) {                   // uniform
        const int cw = c0 + wave * 64;
        if (cw >= ncent) break;                                       // uniform (the first wavefront takes the points' norms)
        double4_t acc[MT][4];
        double nb[4] = {0.0, 0.0, 0.0, 0.0};
        const float *bp[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][nt] = double4_t{0.0, 0.0, 0.0, 0.0};
            const int c = cw + lr * 4 + nt;
            bp[nt] = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
        }
        f64_tile_products<MT>(ap, bp, dsub, lk, c0 == 0, acc, na, nb);
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            nb[nt] += __shfl_xor(nb[nt], 16);
            nb[nt] += __shfl_xor(nb[nt], 32);
            const int c = cw + lr * 4 + nt;
            if (c >= ncent) continue;
            cmax = nb[nt] < INFINITY ? fmax(cmax, nb[nt]) : INFINITY;            // (NaN counts as infinite)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const double val = fma(-2.0, acc[mt][nt][v], nb[nt]);
                    const bool better = val < best[mt][v];
                    const float other = better ? upper(best[mt][v]) : upper(val);
                    second[mt][v] = other < second[mt][v] ? other : second[mt][v];        // (that of infinity is not a number here)
                    best[mt][v] = better ? val : best[mt][v];
                    bi[mt][v] = better ? static_cast<uint32_t>(c) : bi[mt][v];
                }
        }
    }
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) cmax = fmax(cmax, __shfl_xor(cmax, off));
    if (lane == 0) red_c[wave] = cmax;
    double own[MT][4];                                                // the smallest value of this lane
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            own[mt][v] = best[mt][v];
#pragma unroll
            for (int off = 1; off < 16; off <<= 1) {
                const double ov = __shfl_xor(best[mt][v], off);
                const uint32_t oi = __shfl_xor(bi[mt][v], off);
                take_smaller(best[mt][v], bi[mt][v], ov, oi);
            }
            const int p = mt * 16 + v * 4 + lk;
            if (lr == 0) { red_v[wave][p] = best[mt][v]; red_i[wave][p] = bi[mt][v]; }
        }
        na[mt] += __shfl_xor(na[mt], 16);
        na[mt] += __shfl_xor(na[mt], 32);
        if (wave == 0 && lk == 0) norm[mt * 16 + lr] = na[mt];
    }
    __syncthreads();
    double v = INFINITY;
    uint32_t i = 0xFFFFFFFFu;
    if (tid < kF64Points) {
        for (int w = 0; w < 4; ++w) take_smaller(v, i, red_v[w][tid], red_i[w][tid]);
        // both forms' errors for two centroids, of magnitudes up to (|x| + |c|)^2 <= 2 |x|^2 + 2 |c|^2 (infinite, or not
        // a number, where any value is not finite)
        const double c2 = fmax(fmax(red_c[0], red_c[1]), fmax(red_c[2], red_c[3]));
        limit[tid] = v + (dsub + 8) * 0x1p-50 * (norm[tid] + c2);
        close[tid] = 0;
    }
    __syncthreads();
    // the values that lie within the limit: the smallest one itself, and any other
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int p = mt * 16 + v * 4 + lk;
            const double lim = limit[p];
            const uint32_t up = __float_as_uint(second[mt][v]);        // the smallest number of this upper word:
            const double low = __longlong_as_double(static_cast<long long>(static_cast<uint64_t>(up) << 32 | (up >> 31 ? 0xFFFFFFFFu : 0u)));
            if (own[mt][v] <= lim) atomicAdd(&close[p], low <= lim ? 2u : 1u);
        }
    __syncthreads();
    auto put = [&](uint64_t q, double d, uint32_t i) {
        const size_t o = static_cast<size_t>(q) * m + j;
        store_label(labels, label_bytes, o, i);
        if (dist) dist[o] = static_cast<float>(d);
    };
    auto sure = [&](int p) { return close[p] == 1 && limit[p] < INFINITY; };
    if (tid < kF64Points && q0 + tid < n && sure(tid)) {
        const uint64_t q = q0 + tid;
        put(q, dist ? exact_distance(points + static_cast<size_t>(q) * ld + j * dsub, cbj + static_cast<size_t>(i) * dsub, dsub) : 0.0, i);
    }
    for (int p = wave; p < kF64Points; p += 4) {                      // uniform
        if (q0 + p >= n || sure(p)) continue;                        // uniform
        const float *x = points + static_cast<size_t>(q0 + p) * ld + j * dsub;
        double d = INFINITY;
        uint32_t i = 0xFFFFFFFFu;
        for (int c = lane; c < ncent; c += 64) take_smaller(d, i, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double ov = __shfl_xor(d, off);
            const uint32_t oi = __shfl_xor(i, off);
            take_smaller(d, i, ov, oi);
        }
        if (lane == 0) put(q0 + p, d, i);
    }
}

// Which kernel.  The filter saves products, and what follows it costs each point the reading of a few rows one by one, 256
// to 512 points to a workgroup; the double-precision products cost more per distance but nothing after them, and take
// points in tens.  So they are the faster where centroids are few, or points so few that the filter's tiles leave the chip
// idle, and the longer the rows the more so.  Measured with 4 sub-quantizers, filter against products, in us: 1000 points,
// 256 centroids of 8 components 18 and 11, of 32 24 and 12, of 60 84 and 17, of 128 127 and 18; 12000 points, 256 of 16
// 41 and 34 (512: 45 and 44); 250000 points, 256 of 16 385 and 608, of 32 1150 and 736 (rows of 128 bytes meet in the
// same sets of the first-level cache; of 28: 668 and 780), of 60 1037 and 1070 (with distances 0.74 of the time), of 128
// 3531 and 1412; 1024 of 128 4790 and 4550, of 60 1516 and 3100; 65536 of 128, 1000 points 4933 and 2516, 6000 4770 and 6900.
static bool f64_is_faster(uint64_t sub_vectors, int dsub, int ncent, bool want_dist)
{
    const uint64_t pairs = sub_vectors * static_cast<uint64_t>(ncent);
    if (dsub > 32) {
        if (sub_vectors <= 4096 || pairs <= 1u << 25) return true;
        return ncent <= 256 ? dsub > 64 || want_dist : ncent <= 512 && dsub > 96;
    }
    if (dsub <= 2 && ncent <= (dsub == 1 ? 4096 : 1024)) return sub_vectors <= 16384;        // (the filter cannot tell many apart)
    if (ncent > 512) return false;
    return dsub == 32 || pairs <= (dsub <= 8 ? 1u << 22 : 1u << 23);
}

int launch_assign(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int ncent, void *labels,
                  int label_bytes, float *dist, hipStream_t st)
{
    if (n == 0) return DCPQ_OK;
    if (f64_is_faster(n * static_cast<uint64_t>(m), dsub, ncent, dist != nullptr)) {
        DCPQ_LAUNCH(kStageTrain, st, assign_f64_kernel, dim3(static_cast<unsigned>((n + kF64Points - 1) / kF64Points), m), dim3(256),
                    0, points, n, ld, cb, m, dsub, ncent, labels, label_bytes, dist);
        DCPQ_CHECK_LAUNCH("assign_f64_kernel");
        return DCPQ_OK;
    }
    const int dp = (dsub + 3) & ~3, ks = (3 * dp + 15) / 16;
    if (ks <= 3) return launch_assign_short(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 6) return launch_assign_middle(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if (ks <= 24) return launch_assign_long(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return fail(DCPQ_EUNSUPPORTED, "assign: dsub=%d not supported", dsub);
}

#endif

}  // namespace dcpq

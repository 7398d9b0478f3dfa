// Nearest centroid of every sub-vector (encoding, the assignment step of k-means): the smallest
// (squared distance, index) with distances in double precision.
//
// Computed in two steps with the result of one.  A filter evaluates |c|^2 - 2 <x, c> for all centroids on
// the bf16 matrix cores with every fp32 number split into two bf16 numbers (x = xh + xl + an error of at most
// 2^-18 |x|; three products xh ch + xl ch + xh cl, and |c|^2 as three bf16 numbers against ones, all along the
// K dimension of one matrix product), and keeps per point the three smallest minima over cells of 16
// centroids.  A bound on the filter's error, from the norms at hand, says which cells can hold the nearest
// centroid: those, almost always one or two, are evaluated in double precision.  A point with more such cells
// than were kept (or whose values are not finite) is compared with all centroids in double precision.
//
// What bounds it: the matrix pipe (KS instructions of 32 cycles per 32 x 32 distances, KS = ceil((3 d + 4) / 16)),
// beside 1.0 vector instruction per lane and distance for the minima.
#include "common.h"
#include "assign.h"

namespace dcpq {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

struct __attribute__((packed, aligned(4))) f4_any { float v[4]; };

// KS: steps of 16 along K.  P: tiles of 32 points per wavefront.  SPLIT: the four wavefronts share the points
// and split the centroids (else every wavefront has points of its own).  RS: centroids staged together.
template <int KS, int P, bool SPLIT>
struct AssignCfg {
    static constexpr int RS = KS <= 7 ? 128 : 32;              // centroids per stage
    static constexpr int TPR = 256 / RS;                       // threads that convert one centroid
    static constexpr int DPMAX = (16 * KS - 4) / 3 & ~3;       // largest padded sub-vector length
    static constexpr int NG = (DPMAX / 4 + TPR - 1) / TPR;     // groups of 4 components per thread
    static constexpr int STRIDE = KS * 32 + 16;                // bytes per staged row (an odd number of 16-byte units)
    static constexpr int PTS = SPLIT ? 32 * P : 128 * P;       // points per workgroup
    static constexpr int NE = SPLIT ? 8 : 2;                   // lanes that hold minima of one point
    static constexpr int STAGE_BYTES = 2 * RS * STRIDE;
    static constexpr int ENT_BYTES = PTS * NE * 5 * 4 + PTS * 4;
    static constexpr int LDS_BYTES = STAGE_BYTES > ENT_BYTES ? STAGE_BYTES : ENT_BYTES;
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

__device__ inline void store_label(void *labels, int label_bytes, size_t o, uint32_t i)
{
    if (label_bytes == 1) static_cast<uint8_t *>(labels)[o] = static_cast<uint8_t>(i);
    else if (label_bytes == 2) static_cast<uint16_t *>(labels)[o] = static_cast<uint16_t>(i);
    else static_cast<uint32_t *>(labels)[o] = i;
}

// Nearest centroid of the j-th sub-vector of every point, j = blockIdx.y.  points: rows of `ld` floats;
// sub-vector j starts at column j * dsub.  labels: [n][m].  dist (optional): [n][m] fp32 squared distance.
// dp: dsub rounded up to a multiple of 4, 3 dp + 4 <= 16 KS.
template <int KS, int P, bool SPLIT>
__global__ __launch_bounds__(256) void assign_kernel(const float *__restrict__ points, uint64_t n, int ld,
                                                     const float *__restrict__ cb, int m, int dsub, int dp, int ncent,
                                                     void *__restrict__ labels, int label_bytes, float *__restrict__ dist)
{
    using C = AssignCfg<KS, P, SPLIT>;
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ float mu[128];
    __shared__ float s_cmax[4];
    __shared__ uint32_t s_nhard;
    __shared__ double red_v[4];
    __shared__ uint32_t red_i[4];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = blockIdx.y;
    const uint64_t q0 = static_cast<uint64_t>(blockIdx.x) * C::PTS;
    const float *cbj = cb + static_cast<size_t>(j) * ncent * dsub;
    const int col = lane & 31, half = lane >> 5;

    // A reference vector subtracted from points and centroids: distances do not change, norms (and with them the
    // filter's error) shrink.  The mean of up to 64 centroids spread over the codebook; any vector would do.
    if (tid < 128) {
        float sum = 0.0f;
        const int ns = ncent < 64 ? ncent : 64, step = ncent / ns;
        if (tid < dsub)
            for (int s = 0; s < ns; ++s) {
                const int c = s * step + s % step;
                sum += cbj[static_cast<size_t>(c) * dsub + tid];
            }
        mu[tid] = sum / static_cast<float>(ns);
    }
    if (tid == 0) s_nhard = 0;
    for (int t = tid; t < C::STAGE_BYTES / 16; t += 256) reinterpret_cast<uint4 *>(smem)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();

    const int srow = tid / C::TPR, spart = tid % C::TPR;
    // The point side of the product: column `col` of B, K positions 16 ks + 8 half + e:
    // [ -2 xh | -2 xl | -2 xh | 1 1 1 | 0 ... ] against the centroids' [ ch | ch | cl | |c|^2 in three parts | 0 ... ].
    // Converted in rows by the whole workgroup, RS points at a time, and read back as operands.
    v8bf bq[P][KS];
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll 1
        for (int sub = 0; sub < (SPLIT ? 1 : 128 / C::RS); ++sub) {
            const uint64_t q = q0 + p * (SPLIT ? 32 : 128) + sub * C::RS + srow;
            const float *x = points + static_cast<size_t>(q < n ? q : n - 1) * ld + j * dsub;
            uint8_t *row = smem + srow * C::STRIDE;
#pragma unroll 1
            for (int g = 0; g < C::NG; ++g) {
                const int o = 4 * (spart + C::TPR * g);
                if (o < dp) {
                    v4bf h, l;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int t = o + e < dsub ? o + e : dsub - 1;
                        const float v = o + e < dsub ? -2.0f * (x[t] - mu[t]) : 0.0f;
                        h[e] = static_cast<__bf16>(v);
                        l[e] = static_cast<__bf16>(v - static_cast<float>(h[e]));
                    }
                    *reinterpret_cast<v4bf *>(row + 2 * o) = h;
                    *reinterpret_cast<v4bf *>(row + 2 * (dp + o)) = l;
                    *reinterpret_cast<v4bf *>(row + 2 * (2 * dp + o)) = h;
                }
            }
            if (spart == 0) {
                const __bf16 one = static_cast<__bf16>(1.0f);
                *reinterpret_cast<v4bf *>(row + 6 * dp) = v4bf{one, one, one, static_cast<__bf16>(0.0f)};
            }
            __syncthreads();
            if (SPLIT || wave * 32 / C::RS == sub) {
                const uint8_t *b = smem + ((SPLIT ? 0 : wave * 32 % C::RS) + col) * C::STRIDE + half * 16;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) bq[p][ks] = *reinterpret_cast<const v8bf *>(b + ks * 32);
            }
            __syncthreads();
        }
    }

    // staging: TPR threads convert one centroid
    float pre[C::NG][4];
    auto load_stage = [&](int c0) {
        const int c = c0 + srow;
        const float *src = cbj + static_cast<size_t>(c < ncent ? c : ncent - 1) * dsub;
        if ((dsub & 3) == 0) {
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
                    pre[g][e] = src[o < dsub ? o : 0];
                }
        }
    };
    float cmax2 = 0.0f;                       // largest |c|^2 among the centroids this thread converted
    auto store_stage = [&](int c0, uint8_t *buf) {
        uint8_t *row = buf + srow * C::STRIDE;
        float norm = 0.0f;
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 4 * (spart + C::TPR * g);
            if (o < dp) {
                v4bf h, l;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float v = o + e < dsub ? pre[g][e] - mu[o + e] : 0.0f;
                    h[e] = static_cast<__bf16>(v);
                    l[e] = static_cast<__bf16>(v - static_cast<float>(h[e]));
                    norm = fmaf(v, v, norm);
                }
                *reinterpret_cast<v4bf *>(row + 2 * o) = h;
                *reinterpret_cast<v4bf *>(row + 2 * (dp + o)) = h;
                *reinterpret_cast<v4bf *>(row + 2 * (2 * dp + o)) = l;
            }
        }
#pragma unroll
        for (int off = 1; off < C::TPR; off <<= 1) norm += __shfl_xor(norm, off);
        if (spart == 0) {
            v4bf nn;
            if (c0 + srow < ncent) {
                cmax2 = fmaxf(cmax2, norm);
                if (!(norm < INFINITY)) cmax2 = INFINITY;            // (also NaN)
                nn[0] = static_cast<__bf16>(norm);
                const float r1 = norm - static_cast<float>(nn[0]);
                nn[1] = static_cast<__bf16>(r1);
                nn[2] = static_cast<__bf16>(r1 - static_cast<float>(nn[1]));
            } else {                                                 // past the last centroid: never the nearest
                nn[0] = static_cast<__bf16>(3e38f);
                nn[1] = nn[2] = static_cast<__bf16>(0.0f);
            }
            nn[3] = static_cast<__bf16>(0.0f);
            *reinterpret_cast<v4bf *>(row + 6 * dp) = nn;
        }
    };

    // three smallest cell minima of each of this lane's points, and the cells of the first two
    float b1[P], b2[P], b3[P];
    uint32_t i1[P], i2[P];
#pragma unroll
    for (int p = 0; p < P; ++p) { b1[p] = b2[p] = b3[p] = INFINITY; i1[p] = i2[p] = 0; }
    auto compute_tile = [&](const uint8_t *buf, int t, uint32_t cell) {
        const uint8_t *a = buf + (t * 32 + col) * C::STRIDE + half * 16;
        v16f acc[P];
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[p][v] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const v8bf av = *reinterpret_cast<const v8bf *>(a + ks * 32);
#pragma unroll
            for (int p = 0; p < P; ++p) acc[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bq[p][ks], acc[p], 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float mn = acc[p][0];
#pragma unroll
            for (int v = 1; v + 1 < 16; v += 2) mn = fminf(fminf(acc[p][v], acc[p][v + 1]), mn);
            mn = fminf(mn, acc[p][15]);
            const bool c1 = mn < b1[p], c2 = mn < b2[p];
            i2[p] = c1 ? i1[p] : c2 ? cell : i2[p];
            i1[p] = c1 ? cell : i1[p];
            b3[p] = __builtin_amdgcn_fmed3f(b2[p], b3[p], mn);
            b2[p] = __builtin_amdgcn_fmed3f(b1[p], b2[p], mn);
            b1[p] = fminf(b1[p], mn);
        }
    };
    const int nst = (ncent + C::RS - 1) / C::RS;
    load_stage(0);
    store_stage(0, smem);
    __syncthreads();
    for (int s = 0; s < nst; ++s) {                                   // uniform
        const uint8_t *buf = smem + (s & 1) * (C::RS * C::STRIDE);
        if (s + 1 < nst) load_stage((s + 1) * C::RS);
        if constexpr (SPLIT) compute_tile(buf, wave, s * (C::RS / 32) + wave);
        else {
#pragma unroll 1
            for (int t = 0; t < C::RS / 32; ++t) compute_tile(buf, t, s * (C::RS / 32) + t);
        }
        if (s + 1 < nst) store_stage((s + 1) * C::RS, smem + ((s + 1) & 1) * (C::RS * C::STRIDE));
        __syncthreads();
    }

    // hand the minima over: ent[point][lane that held them][b1, b2, b3, i1, i2]
    float *ent = reinterpret_cast<float *>(smem);
    uint32_t *hard = reinterpret_cast<uint32_t *>(smem + C::PTS * C::NE * 20);        // points for the full comparison
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

    // Error of a filter value, |c| <= c1:  2 |<x, c>| has 3 dropped products of relative size 2^-18 each; the K additions
    // (with the roundings of x - mu, c - mu and |c|^2 counted among them) lose at most 2^-23 of the sum of the
    // magnitudes each.  The last term covers values that vanish below the smallest bf16 numbers.
    constexpr float kSplit = 6.2f / 262144.0f, kAdd = (16.0f * KS + 16.0f) / 8388608.0f;
    auto filter_error = [](float xn, float c1) {
        return xn * c1 * (kSplit + 2.1f * kAdd) + c1 * c1 * (1.1f * kAdd) + 1e-35f * (1.0f + xn + c1);
    };
    const int l16 = tid & 15;
    for (int pt = tid >> 4; pt < C::PTS; pt += 16) {                  // 16 lanes per point
        const uint64_t q = q0 + pt;
        if (q >= n) break;
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub;
        float xn2 = 0.0f;
        for (int t = l16; t < dsub; t += 16) { const float v = x[t] - mu[t]; xn2 = fmaf(v, v, xn2); }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) xn2 += __shfl_xor(xn2, off);
        const float xn = sqrtf(xn2) * 1.001f;
        const float *e = ent + pt * C::NE * 5;
        float gmin = INFINITY;
#pragma unroll
        for (int k = 0; k < C::NE; ++k) gmin = fminf(gmin, e[k * 5]);
        // The nearest centroid is no farther than the one with the smallest filter value, so its norm is at
        // most |x| plus that distance.
        const float d2 = fmaxf(xn * xn + gmin + filter_error(xn, cmax), 0.0f);
        const float c1 = fminf(cmax, (xn + sqrtf(d2)) * 1.001f);
        const float thr = gmin + 2.0f * filter_error(xn, c1);
        bool full = !(thr < 1e37f);
#pragma unroll
        for (int k = 0; k < C::NE; ++k) full = full || e[k * 5 + 2] <= thr;
        if (full) {
            if (l16 == 0) hard[atomicAdd(&s_nhard, 1u)] = static_cast<uint32_t>(pt);
            continue;
        }
        double best = INFINITY;
        uint32_t bi = 0xFFFFFFFFu;
#pragma unroll 1
        for (int k = 0; k < 2 * C::NE; ++k) {
            const float *ek = e + (k >> 1) * 5;
            if (ek[k & 1] <= thr) {
                const int h = C::NE == 2 ? k >> 1 : (k >> 1) & 1;
                const uint32_t cell = __float_as_uint(ek[3 + (k & 1)]);
                const uint32_t c = cell * 32 + 8 * (l16 >> 2) + 4 * h + (l16 & 3);
                if (c < static_cast<uint32_t>(ncent)) {
                    const double v = exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub);
                    take_smaller(best, bi, v, c);
                }
            }
        }
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) {
            const double ov = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            take_smaller(best, bi, ov, oi);
        }
        if (l16 == 0) {
            const size_t o = static_cast<size_t>(q) * m + j;
            store_label(labels, label_bytes, o, bi);
            if (dist) dist[o] = static_cast<float>(best);
        }
    }
    __syncthreads();
    const uint32_t nhard = s_nhard;
    for (uint32_t hi = 0; hi < nhard; ++hi) {                         // uniform
        const uint64_t q = q0 + hard[hi];
        const float *x = points + static_cast<size_t>(q) * ld + j * dsub;
        double best = INFINITY;
        uint32_t bi = 0xFFFFFFFFu;
        for (int c = tid; c < ncent; c += 256) take_smaller(best, bi, exact_distance(x, cbj + static_cast<size_t>(c) * dsub, dsub), c);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double ov = __shfl_xor(best, off);
            const uint32_t oi = __shfl_xor(bi, off);
            take_smaller(best, bi, ov, oi);
        }
        if (lane == 0) { red_v[wave] = best; red_i[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 4; ++w) take_smaller(best, bi, red_v[w], red_i[w]);
            const size_t o = static_cast<size_t>(q) * m + j;
            store_label(labels, label_bytes, o, bi);
            if (dist) dist[o] = static_cast<float>(best);
        }
        __syncthreads();
    }
}

template <int KS, int P, bool SPLIT>
static int launch_assign_t(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                           void *labels, int label_bytes, float *dist, hipStream_t st)
{
    using C = AssignCfg<KS, P, SPLIT>;
    const auto kernel = &assign_kernel<KS, P, SPLIT>;
    const int arc = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), C::LDS_BYTES);
    if (arc) return arc;
    DCPQ_LAUNCH(kStageTrain, st, (assign_kernel<KS, P, SPLIT>), dim3(static_cast<unsigned>((n + C::PTS - 1) / C::PTS), m), dim3(256),
                C::LDS_BYTES, points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist);
    DCPQ_CHECK_LAUNCH("assign_kernel");
    return DCPQ_OK;
}

template <int KS>
static int launch_assign_ks(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int dp, int ncent,
                            void *labels, int label_bytes, float *dist, hipStream_t st)
{
    // two rounds of the 256 CUs with tiles that large, else the tile that gives more workgroups
    auto enough = [&](int pts) { return (n + pts - 1) / pts * static_cast<uint64_t>(m) >= 512; };
    if constexpr (KS <= 5) {
        if (enough(AssignCfg<KS, 4, false>::PTS)) return launch_assign_t<KS, 4, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    }
    if (enough(AssignCfg<KS, KS <= 16 ? 2 : 1, false>::PTS) || KS > 7)
        return launch_assign_t<KS, KS <= 16 ? 2 : 1, false>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    if constexpr (KS <= 7) return launch_assign_t<KS, 1, true>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    return DCPQ_OK;
}

int launch_assign(const float *points, uint64_t n, int ld, const float *cb, int m, int dsub, int ncent, void *labels,
                  int label_bytes, float *dist, hipStream_t st)
{
    if (n == 0) return DCPQ_OK;
    const int dp = (dsub + 3) & ~3, ks = (3 * dp + 4 + 15) / 16;
#define DCPQ_ASSIGN_KS(K) \
    if (ks <= K) return launch_assign_ks<K>(points, n, ld, cb, m, dsub, dp, ncent, labels, label_bytes, dist, st);
    DCPQ_ASSIGN_KS(1) DCPQ_ASSIGN_KS(2) DCPQ_ASSIGN_KS(3) DCPQ_ASSIGN_KS(4) DCPQ_ASSIGN_KS(5) DCPQ_ASSIGN_KS(7)
    DCPQ_ASSIGN_KS(9) DCPQ_ASSIGN_KS(12) DCPQ_ASSIGN_KS(13) DCPQ_ASSIGN_KS(16) DCPQ_ASSIGN_KS(20) DCPQ_ASSIGN_KS(25)
#undef DCPQ_ASSIGN_KS
    return fail(DCPQ_EUNSUPPORTED, "assign: dsub=%d not supported", dsub);
}

}  // namespace dcpq

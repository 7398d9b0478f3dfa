// Index step for many queries: the nprobe nearest cell centres without the double-precision distance of every (query, centre).
//
// probe_filter_kernel estimates all squared distances on the fp16 matrix cores, one product, with a proven error bound, and leaves them in fp16
// with the smallest of every 32 centres in fp32; probe_pick_kernel takes from the smallest ones of the groups what the nprobe-th distance can be at most, and works
// out in double precision the distances of the centres that can be within it, one or two more than are wanted.  They are compared after
// rounding to fp32, by (distance, centre), as those of the other form are (distances of every centre on the fp64 matrix pipe, 0.69 of its peak, and a selection
// that walks them three times: 1024 queries, 65536 centres of 128 components 312 + 115 us).
//
// The estimate.  Queries and centres are taken relative to a reference vector (the mean of 32 centres), multiplied by a power of two that
// brings the largest component of those centres to 2^4, and rounded to fp16.  (Queries do not have a say in it: one that is thousands of times farther out has no estimates, whatever the
// scale, since these end at 65504, and would take those of its neighbours.)
// What the product loses is bounded by the lengths at hand: the remainder of the query is known, that of a centre is at most 2^-11 of its length
// (components below 2^-14 may be lost whole).  A centre of length c is at least |c - x| away, so that the centres that matter are not longer than a bound that follows from
// the estimate itself.  Where the bound leaves more centres than there is room for, or values are not finite, a query is left to two more launches, which as a rule
// find nothing to do (5 to 10 us): probe_left_kernel works out all its distances, and they are selected from as in the other form.
#include "common.h"
#include "device_util.h"
#include "ivf_select.h"

namespace dcpq {

typedef _Float16 ph8 __attribute__((ext_vector_type(8)));
typedef _Float16 ph4 __attribute__((ext_vector_type(4)));
typedef float pf16 __attribute__((ext_vector_type(16)));

constexpr int kProbeGroup = 32;              // centres of a group: a tile of the matrix product
constexpr int kProbeRows = 64;               // centres per stage
constexpr int kProbeMostTiles = 32;          // tiles per workgroup
constexpr uint32_t kProbeCand = 2048;        // centres that are worked out for a query, at most
constexpr uint32_t kProbeGroups = 1024;      // groups looked at, at most

template <int KH, int P>
struct ProbeCfg {
    static constexpr int DP = 16 * KH, STRIDE = KH * 32 + 16, QPW = 4 * P * 32;      // queries per workgroup
    static constexpr int BUF_BYTES = kProbeRows * STRIDE + kProbeRows * 4;
    static constexpr int LDS_BYTES = 2 * BUF_BYTES + QPW * (kProbeMostTiles + 1) * 4;
    static constexpr int NG = DP / 16;       // vectors of 4 components per thread and row (4 threads a row)
};

// A query's part of the workspace, nlist * 4 bytes: estimates (fp16 [nlist]), smallest of every group (float [nlist / 32, rounded up]), then
// |x| and |x - xh|.
__host__ __device__ inline size_t probe_min_offset(int nlist) { return (static_cast<size_t>(nlist) * 2 + 15) & ~static_cast<size_t>(15); }
__host__ __device__ inline size_t probe_info_offset(int nlist) { return probe_min_offset(nlist) + 4 * ((static_cast<size_t>(nlist) + kProbeGroup - 1) / kProbeGroup); }

template <int KH, int P>
__global__ __launch_bounds__(256, 2) void probe_filter_kernel(const float *__restrict__ queries, int nq, int D, const float *__restrict__ coarse, int nlist,
                                                             int tiles_per_block, uint8_t *__restrict__ out)
{
    using C = ProbeCfg<KH, P>;
    extern __shared__ __align__(16) uint8_t smem[];
    __shared__ __align__(16) float mu[C::DP], mus[C::DP];
    __shared__ float xnorm2[C::QPW], xrest2[C::QPW];
    __shared__ uint32_t s_cabs;
    float *gmin = reinterpret_cast<float *>(smem + 2 * C::BUF_BYTES);        // [QPW][kProbeMostTiles + 1]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5, srow = tid >> 2, spart = tid & 3;
    const int q0 = blockIdx.y * C::QPW;
    if (tid == 0) s_cabs = 0;
    for (int t = tid; t < 2 * C::BUF_BYTES / 16; t += 256) reinterpret_cast<uint4 *>(smem)[t] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (tid < C::DP) {
        float sum = 0.0f, lo = 0.0f, hi = 0.0f;
        const int step = nlist / 32;
        if (tid < D) {
            float v[32];
#pragma unroll
            for (int s = 0; s < 32; ++s) v[s] = coarse[static_cast<size_t>(s * step + s % step) * D + tid];
            lo = hi = v[0];
#pragma unroll
            for (int s = 0; s < 32; ++s) { sum += v[s]; lo = fminf(lo, v[s]); hi = fmaxf(hi, v[s]); }
        }
        const float mean = sum / 32.0f, far = fmaxf(fabsf(hi - mean), fabsf(lo - mean));
        mu[tid] = fabsf(mean) < INFINITY ? mean : 0.0f;
        if (far < INFINITY) atomicMax(&s_cabs, __float_as_uint(far));
    }
    __syncthreads();
    const int ec = static_cast<int>(s_cabs >> 23) - 126;                // (x < 2^(exponent - 126))
    const float scale = __uint_as_float(static_cast<uint32_t>(min(max(4 - ec, -120), 120) + 127) << 23);
    if (tid < C::DP) mus[tid] = -mu[tid] * scale;
    __syncthreads();

    // the queries: column `col` of B, [ -2 xh ], converted 64 at a time and read back by the wavefront that has them
    ph8 bq[P][KH];
    float xn2[P];
    for (int r0 = 0; r0 < C::QPW; r0 += 64) {                         // uniform
        const int qq = r0 + srow, q = q0 + qq < nq ? q0 + qq : nq - 1;
        float norm = 0.0f, rest = 0.0f;
#pragma unroll 1
        for (int o = 4 * spart; o < D; o += 16) {
            const float4 x = *reinterpret_cast<const float4 *>(queries + static_cast<size_t>(q) * D + o), m = *reinterpret_cast<const float4 *>(mu + o);
            const float u[4] = {(x.x - m.x) * scale, (x.y - m.y) * scale, (x.z - m.z) * scale, (x.w - m.w) * scale};
            ph4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float v = -2.0f * u[e];
                h[e] = static_cast<_Float16>(v);
                const float left = 0.5f * (v - static_cast<float>(h[e]));
                norm = fmaf(u[e], u[e], norm);
                rest = fmaf(left, left, rest);
            }
            *reinterpret_cast<ph4 *>(smem + srow * C::STRIDE + 2 * o) = h;
        }
        norm += __shfl_xor(norm, 1); norm += __shfl_xor(norm, 2);
        rest += __shfl_xor(rest, 1); rest += __shfl_xor(rest, 2);
        if (spart == 0) { xnorm2[qq] = norm; xrest2[qq] = rest; }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < P; ++p)
            if ((wave * P + p) * 32 / 64 * 64 == r0) {                // uniform
                const uint8_t *b = smem + ((wave * P + p) * 32 % 64 + col) * C::STRIDE + half * 16;
#pragma unroll
                for (int ks = 0; ks < KH; ++ks) bq[p][ks] = *reinterpret_cast<const ph8 *>(b + ks * 32);
            }
        __syncthreads();
    }
    // (a workgroup whose queries are all so far out that no estimate is below 60000, unless a centre is as well, leaves them at once)
    bool near = false;
    for (int qq = tid; qq < C::QPW && q0 + qq < nq; qq += 256) near = near || xnorm2[qq] < 250000.0f;
    const bool any = __syncthreads_or(near);
#pragma unroll
    for (int p = 0; p < P; ++p) xn2[p] = xnorm2[(wave * P + p) * 32 + col];
    if (blockIdx.x == 0)
        for (int qq = tid; qq < C::QPW && q0 + qq < nq; qq += 256) {
            float *info = reinterpret_cast<float *>(out + static_cast<size_t>(q0 + qq) * nlist * 4 + probe_info_offset(nlist));
            info[0] = any ? sqrtf(xnorm2[qq]) * 1.001f : INFINITY;
            info[1] = sqrtf(xrest2[qq]) * 1.001f;
        }
    if (!any) return;                                                 // uniform

    const int ntiles = (nlist + kProbeGroup - 1) / kProbeGroup, tile0 = blockIdx.x * tiles_per_block, tiles = min(tiles_per_block, ntiles - tile0);
    if (tiles <= 0) return;                                           // uniform
    // stages of two tiles, four threads a row
    float4 pre[C::NG];
    auto load_stage = [&](int s) __attribute__((always_inline)) {
        const int c = (tile0 + 2 * s) * kProbeGroup + srow;
        const float *row = coarse + static_cast<size_t>(c < nlist ? c : nlist - 1) * D;
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 16 * g + 4 * spart;
            pre[g] = *reinterpret_cast<const float4 *>(row + (o < D ? o : 0));
        }
    };
    auto store_stage = [&](int s, uint8_t *buf) __attribute__((always_inline)) {
        const int c = (tile0 + 2 * s) * kProbeGroup + srow;
        float norm = 0.0f;
#pragma unroll
        for (int g = 0; g < C::NG; ++g) {
            const int o = 16 * g + 4 * spart;
            if (o < D) {
                const float4 m = *reinterpret_cast<const float4 *>(mus + o);
                const float v[4] = {fmaf(pre[g].x, scale, m.x), fmaf(pre[g].y, scale, m.y), fmaf(pre[g].z, scale, m.z), fmaf(pre[g].w, scale, m.w)};
                ph4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) { h[e] = static_cast<_Float16>(v[e]); norm = fmaf(v[e], v[e], norm); }
                *reinterpret_cast<ph4 *>(buf + srow * C::STRIDE + 2 * o) = h;
            }
        }
        norm += __shfl_xor(norm, 1);
        norm += __shfl_xor(norm, 2);
        if (spart == 0) reinterpret_cast<float *>(buf + kProbeRows * C::STRIDE)[srow] = c < nlist && norm < 4.0e9f ? norm : INFINITY;      // (a component of 65504 and above would be infinite in fp16)
    };
    const int stages = (tiles + 1) / 2;
    load_stage(0);
    store_stage(0, smem);
    __syncthreads();
    for (int s = 0; s < stages; ++s) {                                // uniform
        if (s + 1 < stages) load_stage(s + 1);
        const uint8_t *buf = smem + (s & 1) * C::BUF_BYTES;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            ph8 a[KH];
            pf16 norm;
            const uint8_t *ra = buf + (t * 32 + col) * C::STRIDE + half * 16;
#pragma unroll
            for (int ks = 0; ks < KH; ++ks) a[ks] = *reinterpret_cast<const ph8 *>(ra + ks * 32);
            const float *nr = reinterpret_cast<const float *>(buf + kProbeRows * C::STRIDE) + t * 32 + 4 * half;
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const float4 x = *reinterpret_cast<const float4 *>(nr + 2 * v);
                norm[v] = x.x; norm[v + 1] = x.y; norm[v + 2] = x.z; norm[v + 3] = x.w;
            }
#pragma unroll
            for (int p = 0; p < P; ++p) {
                pf16 acc = norm;
#pragma unroll
                for (int ks = 0; ks < KH; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], bq[p][ks], acc, 0, 0, 0);
                const int qq = (wave * P + p) * 32 + col, tile = tile0 + 2 * s + t, l0 = tile * kProbeGroup + 4 * half;
                float least = INFINITY;
                ph4 h[4];
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    float d = acc[v] + xn2[p];
                    d = d < 0.0f ? 0.0f : d;
                    least = fminf(least, d);                          // (what is not a number counts as far)
                    h[v >> 2][v & 3] = static_cast<_Float16>(fminf(d, 65504.0f));
                }
                least = fminf(least, __shfl_xor(least, 32));
                if (half == 0) gmin[qq * (kProbeMostTiles + 1) + 2 * s + t] = least;
                if (q0 + qq < nq) {
                    _Float16 *to = reinterpret_cast<_Float16 *>(out + static_cast<size_t>(q0 + qq) * nlist * 4);
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        if (l0 + 8 * g + 3 < nlist) *reinterpret_cast<ph4 *>(to + l0 + 8 * g) = h[g];
                }
            }
        }
        if (s + 1 < stages) store_stage(s + 1, smem + ((s + 1) & 1) * C::BUF_BYTES);
        __syncthreads();
    }
    for (int t = tid; t < C::QPW * tiles; t += 256) {
        const int qq = t / tiles, x = t % tiles;
        if (q0 + qq < nq)
            reinterpret_cast<float *>(out + static_cast<size_t>(q0 + qq) * nlist * 4 + probe_min_offset(nlist))[tile0 + x] = gmin[qq * (kProbeMostTiles + 1) + x];
    }
}

// One workgroup per query (see above).
__global__ __launch_bounds__(1024) void probe_pick_kernel(const float *__restrict__ queries, int D, const float *__restrict__ coarse, int nlist, int nprobe,
                                                         int kh, uint8_t *__restrict__ est, int32_t *__restrict__ probe)
{
    __shared__ uint32_t steps[2048], s_lo, s_hi, s_step, s_ngroup, s_ncand, wsum[16];
    __shared__ uint64_t sel[kProbeCand];
    __shared__ uint32_t cand[kProbeCand];
    __shared__ uint16_t group[kProbeGroups];
    __shared__ float s_v;
    const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint8_t *row = est + static_cast<size_t>(q) * nlist * 4;
    const float *x = queries + static_cast<size_t>(q) * D;
    const int ngroups = (nlist + kProbeGroup - 1) / kProbeGroup;
    const float *gm = reinterpret_cast<const float *>(row + probe_min_offset(nlist));
    const float xn = reinterpret_cast<const float *>(row + probe_info_offset(nlist))[0], xr0 = reinterpret_cast<const float *>(row + probe_info_offset(nlist))[1];

    if (!(xn < INFINITY)) {                                           // uniform: no estimates
        if (tid == 0) probe[static_cast<size_t>(q) * nprobe] = -1;
        return;
    }
    // an upper bound v of the nprobe-th smallest of the groups' smallest estimates: the largest in the step of equal width that has it
    uint32_t lo = 0xFFFFFFFFu, hi = 0;
    for (int t = tid; t < ngroups; t += 1024) {
        const uint32_t key = __float_as_uint(gm[t]);
        lo = min(lo, key);
        if (key < 0x7F800000u) hi = max(hi, key);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        lo = min(lo, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), o)));
        hi = max(hi, static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), o)));
    }
    if (tid == 0) { s_lo = 0xFFFFFFFFu; s_hi = 0; s_step = 2048; s_ngroup = s_ncand = 0; s_v = 0.0f; }
    for (uint32_t t = tid; t < 2048; t += 1024) steps[t] = 0;
    __syncthreads();
    if (lane == 0) { atomicMin(&s_lo, lo); atomicMax(&s_hi, hi); }
    __syncthreads();
    const float dlo = __uint_as_float(s_lo), dhi = __uint_as_float(s_hi), scale = 2048.0f / fmaxf(dhi - dlo, 1e-30f);
    auto step_of = [&](float d) -> uint32_t { const float y = (d - dlo) * scale; return y < 2047.0f ? static_cast<uint32_t>(y) : 2047u; };
    for (int t = tid; t < ngroups; t += 1024) atomicAdd(&steps[step_of(gm[t])], 1u);
    __syncthreads();
    {
        const uint32_t h0 = steps[2 * tid], h1 = steps[2 * tid + 1], want = static_cast<uint32_t>(nprobe);
        uint32_t incl = h0 + h1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t other = __shfl(incl, lane >= o ? lane - o : lane);
            if (lane >= o) incl += other;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint32_t before = incl - (h0 + h1);
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (before < want && before + h0 + h1 >= want) s_step = before + h0 >= want ? 2 * tid : 2 * tid + 1;      // exactly one thread
    }
    __syncthreads();
    const uint32_t step = s_step;
    for (int t = tid; t < ngroups; t += 1024) {
        const float d = gm[t];
        if (step_of(d) <= step) atomicMax(reinterpret_cast<uint32_t *>(&s_v), __float_as_uint(d));
    }
    __syncthreads();
    const float v = s_v;
    // error(c) = a + b c + k1 c c of an estimate for a centre of length c (h: a centre's remainder; the additions, the norms' among them: (16 KH + 16) 2^-23 of
    // what is added up, |x|^2 too; tiny: what may be lost below 2^-14)
    const float tiny = sqrtf(static_cast<float>(16 * kh)) * (1.01f / 16384.0f), h = 1.001f / 2048.0f, kadd = (16.0f * kh + 16.0f) / 8388608.0f;
    const float xr = xr0 + tiny, a = 2.0f * (xn + xr) * tiny + 1.1f * xn * xn * kadd + 1e-30f, b = 2.0f * ((xn + xr) * h + xr) + 2.1f * xn * kadd, k1 = 1.1f * kadd;
    // (c - xn)^2 <= v + error(c): the longest centre whose estimate can be v or less, and the longest that can be as near as the nprobe-th
    auto longest = [&](float d) {
        const float B = 2.0f * xn + b, A = 1.0f - k1;
        return (B + sqrtf(fmaxf(B * B - 4.0f * A * (xn * xn - d - a), 0.0f))) / (2.0f * A) * 1.001f;
    };
    auto error = [&](float c) { return a + b * c + k1 * c * c; };
    const float nth = v + error(longest(v));                          // the nprobe-th distance is no larger
    const float limit = nth + error((xn + sqrtf(nth)) * 1.001f), limit16 = limit * (1.0f + 1.0f / 1024.0f) + 1e-7f;
    bool done = limit16 < 60000.0f && nprobe <= ngroups && step < 2048;       // (estimates end at 65504; not so for what is not a number)
    if (done) {                                                       // uniform
        for (int t = tid; t < ngroups; t += 1024)
            if (gm[t] <= limit) {
                const uint32_t to = atomicAdd(&s_ngroup, 1u);
                if (to < kProbeGroups) group[to] = static_cast<uint16_t>(t);
            }
        __syncthreads();
        done = s_ngroup <= kProbeGroups;
    }
    if (done) {                                                       // uniform
        const uint32_t n = s_ngroup * kProbeGroup;
        for (uint32_t t = tid; t < n; t += 1024) {
            const uint32_t l = group[t / kProbeGroup] * kProbeGroup + t % kProbeGroup;
            if (l < static_cast<uint32_t>(nlist) && static_cast<float>(reinterpret_cast<const _Float16 *>(row)[l]) <= limit16) {
                const uint32_t to = atomicAdd(&s_ncand, 1u);
                if (to < kProbeCand) cand[to] = l;
            }
        }
        __syncthreads();
        done = s_ncand <= kProbeCand && s_ncand >= static_cast<uint32_t>(nprobe);
    }
    // squared distance of centre l in double precision, by 16 lanes
    auto distance = [&](uint32_t l) {
        const float *c = coarse + static_cast<size_t>(l) * D;
        double s = 0.0;
        for (int o = 4 * (tid & 15); o < D; o += 64) {
            const float4 u = *reinterpret_cast<const float4 *>(x + o), w = *reinterpret_cast<const float4 *>(c + o);
            const double e0 = static_cast<double>(u.x) - w.x, e1 = static_cast<double>(u.y) - w.y, e2 = static_cast<double>(u.z) - w.z, e3 = static_cast<double>(u.w) - w.w;
            s = fma(e0, e0, s); s = fma(e1, e1, s); s = fma(e2, e2, s); s = fma(e3, e3, s);
        }
        s += __shfl_xor(s, 1); s += __shfl_xor(s, 2); s += __shfl_xor(s, 4); s += __shfl_xor(s, 8);
        return s;
    };
    if (!done) {                                                      // uniform
        if (tid == 0) probe[static_cast<size_t>(q) * nprobe] = -1;    // left
        return;
    }
    const uint32_t n = s_ncand;
    uint32_t np2 = 2;
    while (np2 < n) np2 <<= 1;
    for (uint32_t t = n + tid; t < np2; t += 1024) sel[t] = ~0ull;
    for (uint32_t t0 = 0; t0 < n; t0 += 64) {                         // uniform
        const uint32_t t = t0 + (tid >> 4);
        const double d = distance(cand[t < n ? t : n - 1]);
        if ((tid & 15) == 0 && t < n) sel[t] = make_key(__float_as_uint(static_cast<float>(d)), cand[t]);
    }
    if (np2 <= 256) {                                                 // uniform: the place of a key is the number of smaller ones
        __syncthreads();
        const uint32_t own = tid >> 3;
        for (uint32_t t = own; t < n; t += 128) {
            const uint64_t key = sel[t];
            uint32_t rank = 0;
            for (uint32_t y = 2 * (tid & 7); y < np2; y += 16) rank += (sel[y] < key ? 1u : 0u) + (sel[y + 1] < key ? 1u : 0u);
            rank += __shfl_xor(rank, 1);
            rank += __shfl_xor(rank, 2);
            rank += __shfl_xor(rank, 4);
            if ((tid & 7) == 0 && rank < static_cast<uint32_t>(nprobe)) probe[static_cast<size_t>(q) * nprobe + rank] = static_cast<int32_t>(key & 0xFFFFFFFFu);
        }
        return;
    }
    bitonic_sort(sel, np2);
    for (int t = tid; t < nprobe; t += 1024) probe[static_cast<size_t>(q) * nprobe + t] = static_cast<int32_t>(sel[t] & 0xFFFFFFFFu);
}

// The distances of the queries that are left (a negative number in the place of their first list), by difference in double precision, into their part of the
// workspace.  A workgroup takes kLeftCents centres, two a thread, sixteen components at a time through LDS, and those of 64 queries that are left, kLeftTogether
// at a time, from scalar registers.  Bound by the two double-precision instructions per component and pair and the conversions (2.6 of them in all).  1024 queries, 65536 centres of 128
// components, the whole call: one query left 0.17 ms, a tenth 0.27, all 1.08 (0.11 where none is; 1.01, 1.25 and 2.5 with a workgroup a query, each reading all centres).
constexpr int kLeftTogether = 8, kLeftCents = 512, kLeftStride = 20;
__global__ __launch_bounds__(256) void probe_left_kernel(const float *__restrict__ queries, int nq, int D, const float *__restrict__ coarse, int nlist, int nprobe,
                                                        const int32_t *__restrict__ probe, float *__restrict__ dist)
{
    __shared__ __align__(16) float cents[kLeftCents * kLeftStride];
    __shared__ int left[64];
    __shared__ uint32_t s_n;
    const int tid = threadIdx.x;
    const int q0 = blockIdx.y * 64, c0 = blockIdx.x * kLeftCents;
    if (tid < 64) {
        const bool is = q0 + tid < nq && probe[static_cast<size_t>(q0 + tid) * nprobe] < 0;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(is);
        if (is) left[__popcll(mask & ((1ull << tid) - 1ull))] = q0 + tid;
        if (tid == 0) s_n = __popcll(mask);
    }
    __syncthreads();
    const int n = static_cast<int>(s_n);
    if (n == 0) return;                                               // uniform
    for (int g = 0; g < n; g += kLeftTogether) {                      // uniform
        const float *x[kLeftTogether];                                // (in scalar registers)
#pragma unroll
        for (int i = 0; i < kLeftTogether; ++i) x[i] = queries + static_cast<size_t>(__builtin_amdgcn_readfirstlane(left[g + i < n ? g + i : n - 1])) * D;
        double sum[kLeftTogether][2];
#pragma unroll
        for (int i = 0; i < kLeftTogether; ++i) sum[i][0] = sum[i][1] = 0.0;
        for (int o = 0; o < D; o += 16) {                             // uniform
            __syncthreads();
            for (int t = tid; t < kLeftCents * 4; t += 256) {
                const int c = c0 + t / 4;
                *reinterpret_cast<float4 *>(cents + t / 4 * kLeftStride + t % 4 * 4) =
                    *reinterpret_cast<const float4 *>(coarse + static_cast<size_t>(c < nlist ? c : nlist - 1) * D + o + t % 4 * 4);
            }
            __syncthreads();
#pragma unroll 1
            for (int e = 0; e < 16; e += 4) {
                const float4 a = *reinterpret_cast<const float4 *>(cents + tid * kLeftStride + e), b = *reinterpret_cast<const float4 *>(cents + (tid + 256) * kLeftStride + e);
                const double ca[4] = {a.x, a.y, a.z, a.w}, cb[4] = {b.x, b.y, b.z, b.w};
                float xv[kLeftTogether][4];
#pragma unroll
                for (int i = 0; i < kLeftTogether; ++i)
#pragma unroll
                    for (int z = 0; z < 4; ++z) xv[i][z] = x[i][o + e + z];
#pragma unroll
                for (int i = 0; i < kLeftTogether; ++i)
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const double v = xv[i][z], da = v - ca[z], db = v - cb[z];
                        sum[i][0] = fma(da, da, sum[i][0]);
                        sum[i][1] = fma(db, db, sum[i][1]);
                    }
            }
        }
#pragma unroll
        for (int i = 0; i < kLeftTogether; ++i)
#pragma unroll
            for (int z = 0; z < 2; ++z)
                if (g + i < n && c0 + tid + 256 * z < nlist) dist[static_cast<size_t>(left[g + i]) * nlist + c0 + tid + 256 * z] = static_cast<float>(sum[i][z]);
    }
}

// Rows of whole 64-byte pieces up to 256 components, read 16 bytes at a time (a query's part of the workspace too: lists in fours); a cut that
// leaves few groups of 32 (eight times the probed lists are groups); and pairs enough that the estimate pays.  Against the distances of all
// centres in double precision, D = 128: 4096 lists x 1024 queries 0.97 of the time, 16384 x 256 0.91, 65536 x 64 0.82, x 256 0.46, x 1024
// 0.28 (427 -> 119 us); below 2^22 pairs the launches' latency is all there is (4096 lists x 1024 queries of 96 components 43 and 45 us).  Batches that are left whole are slower than without
// estimates: 65536 x 1024, all queries far out 0.43 and 1.08 ms; all centres equal, where the selection takes most of it, 1.70 and 1.69.
bool probe_filter_serves(const float *queries, int nq, int D, const float *coarse, int nlist, int nprobe)
{
    return D % 16 == 0 && D <= 256 && nlist >= 4096 && nlist % 4 == 0 && nlist <= kProbeGroup * 65536 && nprobe * 8 <= nlist / kProbeGroup &&
           static_cast<uint64_t>(nq) * nlist >= (4ull << 20) && ((reinterpret_cast<uintptr_t>(queries) | reinterpret_cast<uintptr_t>(coarse)) & 15) == 0;
}

template <int KH, int P>
static int launch_filter(const float *queries, int nq, int D, const float *coarse, int nlist, uint8_t *est, hipStream_t st)
{
    using C = ProbeCfg<KH, P>;
    const int rc = allow_dynamic_lds(reinterpret_cast<const void *>(&probe_filter_kernel<KH, P>), C::LDS_BYTES);
    if (rc) return rc;
    // two workgroups per CU, of 32 tiles at most
    const int groups = (nq + C::QPW - 1) / C::QPW, ntiles = (nlist + kProbeGroup - 1) / kProbeGroup;
    int per = static_cast<int>((static_cast<int64_t>(ntiles) * groups + 511) / 512);
    per = (per + 1) / 2 * 2;
    per = per < 2 ? 2 : per > kProbeMostTiles ? kProbeMostTiles : per;
    DCPQ_LAUNCH(kStageIvfProbe, st, (probe_filter_kernel<KH, P>), dim3((ntiles + per - 1) / per, groups), dim3(256), C::LDS_BYTES, queries, nq, D, coarse, nlist, per, est);
    DCPQ_CHECK_LAUNCH("probe_filter_kernel");
    return DCPQ_OK;
}

// (leaves queries that have a negative number in the place of their first list, and the distances of all centres in their part of the workspace)
int launch_probe_filter(const float *queries, int nq, int D, const float *coarse, int nlist, int nprobe, void *ws, int32_t *probe, hipStream_t st)
{
    uint8_t *est = static_cast<uint8_t *>(ws);
    const int kh = D / 16, used = kh <= 4 ? 4 : kh <= 6 ? 6 : kh <= 8 ? 8 : kh <= 12 ? 12 : 16;
    int rc = DCPQ_OK;
    switch (used) {
    case 4: rc = launch_filter<4, 2>(queries, nq, D, coarse, nlist, est, st); break;
    case 6: rc = launch_filter<6, 2>(queries, nq, D, coarse, nlist, est, st); break;
    case 8: rc = launch_filter<8, 2>(queries, nq, D, coarse, nlist, est, st); break;
    case 12: rc = launch_filter<12, 1>(queries, nq, D, coarse, nlist, est, st); break;
    default: rc = launch_filter<16, 1>(queries, nq, D, coarse, nlist, est, st); break;
    }
    if (rc) return rc;
    DCPQ_LAUNCH(kStageIvfProbe, st, probe_pick_kernel, dim3(nq), dim3(1024), 0, queries, D, coarse, nlist, nprobe, used, est, probe);
    DCPQ_CHECK_LAUNCH("probe_pick_kernel");
    DCPQ_LAUNCH(kStageIvfProbe, st, probe_left_kernel, dim3((nlist + kLeftCents - 1) / kLeftCents, (nq + 63) / 64), dim3(256), 0, queries, nq, D, coarse, nlist, nprobe,
                probe, static_cast<float *>(ws));
    DCPQ_CHECK_LAUNCH("probe_left_kernel");
    return DCPQ_OK;
}

}  // namespace dcpq

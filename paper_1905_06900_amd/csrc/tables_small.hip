// Derived codebooks (Sec. 3.2) and the small-table / quantization stage of Alg. 3 (Sec. 3.3,
// "Tables step").  Everything here feeds an integer decision, so the arithmetic is plain fp32
// with one rounding per operation in a fixed order: no FMA contraction (explicit *_rn
// intrinsics), correctly rounded division, sequential accumulation.
#include "common.h"
#include "device_util.h"

namespace dcpq {

// derived[j][l][t] = (sum_i cb[j][(i << bbar) | l][t]) / 2^(b - bbar), i = 0 .. 2^(b - bbar) - 1 increasing
// (Sec. 3.2: the derived centroid is the mean of the group of centroids that share the low bbar
// bits).  One thread per output element; for a fixed i the threads of a block read one contiguous
// run of 2^bbar * dsub floats, so the loads coalesce.
__global__ __launch_bounds__(256) void derive_kernel(const float *__restrict__ cb, int dsub, int full_size,
                                                     int small_bits, float *__restrict__ derived)
{
    const int j = blockIdx.y;
    const int per_sub = dsub << small_bits;                // floats in one derived codebook
    const int groups = full_size >> small_bits;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;   // l * dsub + t
    if (e >= per_sub) return;
    const float *base = cb + static_cast<size_t>(j) * full_size * dsub + e;
    float acc = 0.0f;
    for (int i = 0; i < groups; ++i)
        acc = __fadd_rn(acc, base[static_cast<size_t>(i) * per_sub]);
    derived[static_cast<size_t>(j) * per_sub + e] = __fdiv_rn(acc, static_cast<float>(groups));
}

// A workgroup takes QPB queries.  LDS: the queries (D floats each) and their m * 2^bbar small-table entries.
// The quantized tables are written with 256 entries each whatever bbar is: entry e holds the
// quantized distance of derived centroid (e mod 2^bbar), so that a scan which looks a table up by
// the low BYTE of a sub-code gets the entry of its low bbar BITS (property P1 of Sec. 3.1 for any
// bbar <= 8).  `small`, when asked for, keeps the 2^bbar floating-point entries as they are.
// Bound by reading the derived codebooks (one row per thread, out of the L2) and the table gathers of the walk for qmax:
// two queries share every row and every code where there are enough queries (512 queries of 16 x 60 components: 60 us with a
// workgroup of 256 threads per query, 78 with 1024 threads per query, 51 with two queries, 54 with four); with few queries
// it is a chain of memory round trips, which 1024 threads shorten (251 queries of 8 x 16, r = 10000: 23 -> 12 us).
constexpr int kSmallTabThreads = 1024;

// floats of the tables, up to a whole 16-byte vector (one query, one sub-quantizer and bbar = 1 make two floats)
__host__ __device__ inline int table_floats(int qpb, int m, int small_bits) { return ((qpb * m << small_bits) + 3) & ~3; }

template <int M, int QPB, typename CodeT>
__global__ __launch_bounds__(kSmallTabThreads) void small_tables_kernel(
    const float *__restrict__ queries, int nq, const float *__restrict__ derived, int dsub, int small_bits,
    const CodeT *__restrict__ codes, uint32_t n_first, uint8_t *__restrict__ qtab,
    float *__restrict__ bounds, float *__restrict__ small, uint32_t *__restrict__ clear, size_t clear_words)
{
    extern __shared__ __align__(16) float lds[];
    const int q0 = blockIdx.x * QPB, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int D = M * dsub;
    const int ks = 1 << small_bits, mask = ks - 1;
    float *ltab = lds;                     // [QPB][M][2^bbar]
    float *ly = lds + table_floats(QPB, M, small_bits);        // [QPB][M*dsub], 16-byte aligned (it is read in vectors)
    __shared__ float red[QPB][16];
    for (size_t w = static_cast<size_t>(blockIdx.x) * kSmallTabThreads + tid; w < clear_words / 4; w += static_cast<size_t>(gridDim.x) * kSmallTabThreads)
        reinterpret_cast<uint4 *>(clear)[w] = make_uint4(0u, 0u, 0u, 0u);
    for (int t = tid; t < QPB * D; t += kSmallTabThreads) {
        const int q = q0 + t / D;          // (past the last query: any valid one)
        ly[t] = queries[static_cast<size_t>(q < nq ? q : nq - 1) * D + t % D];
    }
    __syncthreads();

    // minimum or maximum over the workgroup, one value per query; the barriers also order the LDS accesses around it
    auto reduce = [&](float (&v)[QPB], bool want_max) {
#pragma unroll
        for (int p = 0; p < QPB; ++p)
            for (int off = 32; off > 0; off >>= 1) {
                const float o = __shfl_xor(v[p], off, kWave);
                v[p] = want_max ? fmaxf(v[p], o) : fminf(v[p], o);
            }
        __syncthreads();
        if (lane == 0)
#pragma unroll
            for (int p = 0; p < QPB; ++p) red[p][wave] = v[p];
        __syncthreads();
#pragma unroll
        for (int p = 0; p < QPB; ++p) {
            v[p] = red[p][0];
            for (int w = 1; w < kSmallTabThreads / kWave; ++w) v[p] = want_max ? fmaxf(v[p], red[p][w]) : fminf(v[p], red[p][w]);
        }
    };

    // Eq. 1 on the derived codebooks: a thread owns entries (j, i) and works them out for all QPB queries, the squares
    // added one by one in ascending t.
    const bool vec4 = (dsub & 3) == 0 && (reinterpret_cast<uintptr_t>(derived) & 15) == 0;      // uniform
    float lo[QPB];
#pragma unroll
    for (int p = 0; p < QPB; ++p) lo[p] = INFINITY;
    for (int e = tid; e < M * ks; e += kSmallTabThreads) {
        const int j = e >> small_bits;
        const float *c = derived + static_cast<size_t>(e) * dsub, *y = ly + j * dsub;
        float acc[QPB];
#pragma unroll
        for (int p = 0; p < QPB; ++p) acc[p] = 0.0f;
        if (vec4) {
#pragma unroll 4
            for (int t = 0; t < dsub; t += 4) {
                const float4 c4 = *reinterpret_cast<const float4 *>(c + t);
                const float cv[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
                for (int p = 0; p < QPB; ++p) {
                    const float4 y4 = *reinterpret_cast<const float4 *>(y + p * D + t);
                    const float yv[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const float diff = __fsub_rn(yv[z], cv[z]);
                        acc[p] = __fadd_rn(acc[p], __fmul_rn(diff, diff));
                    }
                }
            }
        } else {
            for (int t = 0; t < dsub; ++t) {
                const float cv = c[t];
#pragma unroll
                for (int p = 0; p < QPB; ++p) {
                    const float diff = __fsub_rn(y[p * D + t], cv);
                    acc[p] = __fadd_rn(acc[p], __fmul_rn(diff, diff));
                }
            }
        }
#pragma unroll
        for (int p = 0; p < QPB; ++p) {
            ltab[p * M * ks + e] = acc[p];
            lo[p] = fminf(lo[p], acc[p]);
        }
    }
    reduce(lo, false);                     // (also publishes ltab)

    // qmax: largest small-table distance to the first n_first codes, sum over j increasing.
    float hi[QPB];
#pragma unroll
    for (int p = 0; p < QPB; ++p) hi[p] = -INFINITY;
    for (uint32_t i = tid; i < n_first; i += kSmallTabThreads) {
        const CodeT *c = codes + static_cast<size_t>(i) * M;
        float d[QPB];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const int e = j * ks + (c[j] & mask);
#pragma unroll
            for (int p = 0; p < QPB; ++p) d[p] = j == 0 ? ltab[p * M * ks + e] : __fadd_rn(d[p], ltab[p * M * ks + e]);
        }
#pragma unroll
        for (int p = 0; p < QPB; ++p) hi[p] = fmaxf(hi[p], d[p]);
    }
    reduce(hi, true);

    for (int v = tid; v < QPB * M * kSmallSize; v += kSmallTabThreads) {
        const int p = v / (M * kSmallSize), e = v % (M * kSmallSize);
        if (q0 + p >= nq) break;           // (increasing in v)
        const int j = e / kSmallSize, i = e % kSmallSize;
        float qmin = lo[0], qmax = hi[0];
#pragma unroll
        for (int x = 1; x < QPB; ++x)
            if (p == x) { qmin = lo[x]; qmax = hi[x]; }
        const float val = ltab[(p * M + j) * ks + (i & mask)];
        qtab[static_cast<size_t>(q0 + p) * M * kSmallSize + e] = quantize_entry(val, qmin, qmax);
        if (small && i < ks) small[(static_cast<size_t>(q0 + p) * M + j) * ks + i] = val;
    }
    if (tid < QPB && q0 + tid < nq) {
        float qmin = lo[0], qmax = hi[0];
#pragma unroll
        for (int x = 1; x < QPB; ++x)
            if (tid == x) { qmin = lo[x]; qmax = hi[x]; }
        bounds[2 * (q0 + tid)] = qmin;
        bounds[2 * (q0 + tid) + 1] = qmax;
    }
}

template <int M, int QPB, typename CodeT>
static int launch_small_tables_m(const float *queries, int nq, const float *derived, int dsub, int small_bits, const CodeT *codes,
                                 uint32_t n_first, uint8_t *qtab, float *bounds, float *small, hipStream_t st, uint32_t *clear,
                                 size_t clear_words)
{
    const size_t lds = sizeof(float) * (static_cast<size_t>(QPB) * M * dsub + table_floats(QPB, M, small_bits));
    const int arc = allow_dynamic_lds(reinterpret_cast<const void *>(&small_tables_kernel<M, QPB, CodeT>), static_cast<int>(lds));
    if (arc) return arc;
    DCPQ_LAUNCH(kStageSmallTables, st, (small_tables_kernel<M, QPB, CodeT>), dim3((nq + QPB - 1) / QPB), dim3(kSmallTabThreads), lds,
                queries, nq, derived, dsub, small_bits, codes, n_first, qtab, bounds, small, clear, clear_words);
    DCPQ_CHECK_LAUNCH("small_tables_kernel");
    return DCPQ_OK;
}

template <typename CodeT>
static int launch_small_tables_t(const float *queries, int nq, const float *derived, int m, int dsub, int small_bits,
                                 const CodeT *codes, uint64_t n_codes, uint32_t r, uint8_t *qtab,
                                 float *bounds, float *small, hipStream_t st, uint32_t *clear, size_t clear_words)
{
    if (nq == 0) return DCPQ_OK;
    const uint32_t n_first = static_cast<uint32_t>(r < n_codes ? r : n_codes);
#define DCPQ_LAUNCH_SMALL(MV)                                                                                 \
    case MV:                                                                                                  \
        if (nq >= 500) /* a workgroup per CU and more */                                                      \
            return launch_small_tables_m<MV, 2, CodeT>(queries, nq, derived, dsub, small_bits, codes, n_first, qtab, bounds, small, st, clear, clear_words); \
        return launch_small_tables_m<MV, 1, CodeT>(queries, nq, derived, dsub, small_bits, codes, n_first, qtab, bounds, small, st, clear, clear_words);
    switch (m) {
        DCPQ_LAUNCH_SMALL(1) DCPQ_LAUNCH_SMALL(2) DCPQ_LAUNCH_SMALL(4) DCPQ_LAUNCH_SMALL(8)
        DCPQ_LAUNCH_SMALL(16) DCPQ_LAUNCH_SMALL(32)
        default: return fail(DCPQ_EUNSUPPORTED, "m=%d not supported", m);
    }
#undef DCPQ_LAUNCH_SMALL
}

int launch_small_tables(const float *queries, int nq, const float *derived, int m, int dsub, int small_bits,
                        const void *codes, int code_bytes, uint64_t n_codes, uint32_t r, uint8_t *qtab,
                        float *bounds, float *small, hipStream_t st, uint32_t *clear, size_t clear_words)
{
    if (code_bytes == 1)
        return launch_small_tables_t(queries, nq, derived, m, dsub, small_bits, static_cast<const uint8_t *>(codes),
                                     n_codes, r, qtab, bounds, small, st, clear, clear_words);
    return launch_small_tables_t(queries, nq, derived, m, dsub, small_bits, static_cast<const uint16_t *>(codes),
                                 n_codes, r, qtab, bounds, small, st, clear, clear_words);
}

int launch_derive(const float *codebooks, int m, int dsub, int full_bits, int small_bits, float *derived, hipStream_t st)
{
    const int per_sub = dsub << small_bits;
    hipLaunchKernelGGL(derive_kernel, dim3((per_sub + 255) / 256, m), dim3(256), 0, st, codebooks, dsub, 1 << full_bits,
                       small_bits, derived);
    DCPQ_CHECK_LAUNCH("derive_kernel");
    return DCPQ_OK;
}

}  // namespace dcpq

using namespace dcpq;

extern "C" int dcpq_shape_supported(int m, int dsub)
{
    return (m_supported(m) && dsub >= 1 && dsub <= 128) ? 1 : 0;
}

extern "C" int dcpq_bits_supported(int b, int bbar)
{
    return ((b == 8 || b == 16) && bbar >= 1 && bbar <= 8 && bbar <= b) ? 1 : 0;
}

extern "C" int dcpq_derive_codebooks_bits(const float *codebooks, int m, int dsub, int b, int bbar, float *derived,
                                          void *stream)
{
    clear_error();
    DCPQ_REQUIRE(codebooks && derived, "derive_codebooks: null pointer");
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "derive_codebooks: m=%d dsub=%d not supported", m, dsub);
    if (!dcpq_bits_supported(b, bbar)) return fail(DCPQ_EUNSUPPORTED, "derive_codebooks: b=%d bbar=%d not supported", b, bbar);
    return launch_derive(codebooks, m, dsub, b, bbar, derived, as_stream(stream));
}

extern "C" int dcpq_derive_codebooks(const float *codebooks, int m, int dsub, float *derived, void *stream)
{
    return dcpq_derive_codebooks_bits(codebooks, m, dsub, kFullBits, kSmallBits, derived, stream);
}

extern "C" int dcpq_build_small_tables_bits(const float *queries, int nq, const float *derived, int m, int dsub,
                                            int bbar, const void *codes, int code_bytes, uint64_t n_codes, uint32_t r,
                                            uint8_t *qtab, float *bounds, float *small, void *stream)
{
    clear_error();
    DCPQ_REQUIRE(nq >= 0, "build_small_tables: nq=%d", nq);
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "build_small_tables: m=%d dsub=%d not supported", m, dsub);
    DCPQ_REQUIRE(code_bytes == 1 || code_bytes == 2, "build_small_tables: code_bytes=%d (1 or 2)", code_bytes);
    if (!dcpq_bits_supported(8 * code_bytes, bbar))
        return fail(DCPQ_EUNSUPPORTED, "build_small_tables: bbar=%d with %d-byte sub-codes not supported", bbar, code_bytes);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && derived && qtab && bounds, "build_small_tables: null pointer");
    DCPQ_REQUIRE(r >= 1 && n_codes >= 1 && codes, "build_small_tables: needs r >= 1 and at least one code (qmax is taken over the first r codes)");
    return launch_small_tables(queries, nq, derived, m, dsub, bbar, codes, code_bytes, n_codes, r, qtab, bounds, small,
                               as_stream(stream));
}

extern "C" int dcpq_build_small_tables(const float *queries, int nq, const float *derived, int m, int dsub,
                                       const uint16_t *codes, uint64_t n_codes, uint32_t r, uint8_t *qtab,
                                       float *bounds, float *small, void *stream)
{
    return dcpq_build_small_tables_bits(queries, nq, derived, m, dsub, kSmallBits, codes, 2, n_codes, r, qtab, bounds,
                                        small, stream);
}

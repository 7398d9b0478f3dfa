// 8-bit sub-codes with derived codebooks of at most 16 centroids: two sub-codes look up 16 entries each, so the low halves of
// two neighbours are one byte that looks up the sum of both entries in a table of 256.  An integer distance is the sum of the
// entries, capped at 255; capping the sums of two at 255 first changes nothing.  The scan then runs over codes of half
// as many sub-quantizers: half of the rows per (query, code) pair.
#include "common.h"

namespace dcpq {

// Two neighbouring sub-codes to one byte, the first in the low half; 16 bytes to 8 a thread.  Bound by memory: 160 MB to 80 MB
// in 37 us.
__global__ __launch_bounds__(256) void pair_codes_kernel(const uint8_t *__restrict__ codes, size_t nbytes, uint8_t *__restrict__ plane)
{
    auto pairs_of = [](uint32_t w) {                             // four sub-codes to two bytes
        w &= 0x0F0F0F0Fu;
        w = (w | w >> 4) & 0x00FF00FFu;
        return (w | w >> 8) & 0xFFFFu;
    };
    const size_t n = nbytes / 16, step = static_cast<size_t>(gridDim.x) * 256, first = static_cast<size_t>(blockIdx.x) * 256 + threadIdx.x;
#pragma unroll 4
    for (size_t i = first; i < n; i += step) {
        const uint4 x = reinterpret_cast<const uint4 *>(codes)[i];
        reinterpret_cast<uint2 *>(plane)[i] = make_uint2(pairs_of(x.x) | pairs_of(x.y) << 16, pairs_of(x.z) | pairs_of(x.w) << 16);
    }
    if (first == 0 && nbytes % 16) {                             // an odd number of codes of 8 bytes: one half of a vector left
        const uint2 x = *reinterpret_cast<const uint2 *>(codes + 16 * n);
        *reinterpret_cast<uint32_t *>(plane + 8 * n) = pairs_of(x.x) | pairs_of(x.y) << 16;
    }
}

// Tables of the pairs, a workgroup per query.
__global__ __launch_bounds__(256) void pair_tables_kernel(const uint8_t *__restrict__ qtab, int m, uint8_t *__restrict__ ptab)
{
    __shared__ uint8_t low[32 * 16];                             // the first 16 entries of every table (the others repeat them)
    const uint8_t *in = qtab + static_cast<size_t>(blockIdx.x) * m * 256;
    uint32_t *out = reinterpret_cast<uint32_t *>(ptab + static_cast<size_t>(blockIdx.x) * (m / 2) * 256);
    for (int t = threadIdx.x; t < m * 16; t += 256) low[t] = in[(t >> 4) * 256 + (t & 15)];
    __syncthreads();
    for (int t = threadIdx.x; t < m / 2 * 64; t += 256) {
        const uint8_t *a = low + (t >> 6) * 32, *b = a + 16;
        const uint32_t hi = b[(t & 63) >> 2];
        uint32_t w = 0;
#pragma unroll
        for (int z = 0; z < 4; ++z) w |= min(255u, a[4 * (t & 3) + z] + hi) << (8 * z);
        out[t] = w;
    }
}

// Whether 8-bit codes are scanned as pairs where bbar <= 4 (the workspace has room for the plane of pairs then).  Searches with
// pairs against single sub-codes, in us: m = 16, N = 1e7, 500 queries, r = 500: 757 and 1235, r = 10000: 1173 and 1673; 333 queries,
// r = 2000: 692 and 958; 128 queries: 395 and 439, 96: 404 and 378 (two tiles of 64 against three of 32); N = 5e6, 100 queries: 276 and
// 299; N = 1e6, 500: 279 and 313.  m = 8, N = 1e7, 500 queries: 606 and 714; N = 1e6: 248 and 247.  m = 32, N = 5e6, 100 queries: 327 and 602.
bool pairs_pay(uint64_t n_codes, int m, int nq)
{
    return (m == 8 || m == 16 || m == 32) && nq >= 100 && static_cast<double>(n_codes) * nq >= 5.0e8;
}

int launch_pair_codes(const uint8_t *codes, uint64_t n_codes, int m, uint8_t *plane, hipStream_t st)
{
    const size_t nbytes = n_codes * m;
    const size_t blocks = (nbytes / 16 + 1023) / 1024;
    DCPQ_LAUNCH(kStageMisc, st, pair_codes_kernel, dim3(static_cast<uint32_t>(blocks < 8192 ? (blocks ? blocks : 1) : 8192)), dim3(256), 0, codes, nbytes, plane);
    DCPQ_CHECK_LAUNCH("pair_codes_kernel");
    return DCPQ_OK;
}

int launch_pair_tables(const uint8_t *qtab, int nq, int m, uint8_t *ptab, hipStream_t st)
{
    DCPQ_LAUNCH(kStageMisc, st, pair_tables_kernel, dim3(nq), dim3(256), 0, qtab, m, ptab);
    DCPQ_CHECK_LAUNCH("pair_tables_kernel");
    return DCPQ_OK;
}

}  // namespace dcpq

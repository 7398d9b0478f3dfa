// Selection of the nearest cell centres of a query from its row of distances, shared by the two forms of the Index step (HIP translation
// units only).
#pragma once

#include "common.h"
#include "device_util.h"

namespace dcpq {

constexpr int kIvfMaxProbe = 512;         // probed lists per query, at most
constexpr uint32_t kProbeSteps = 2048;   // histogram steps of the cut by value (two per thread)

// The nprobe smallest of a row of nlist distances (non-negative, fp32), by (distance, list id), by a workgroup of 1024 threads: a cut by value, or a 4-level
// radix select on the bit patterns (non-negative floats order like their bits), ties at the cut taken in id order.
__device__ inline void select_probe_of_row(const float *__restrict__ dist, int nlist, int nprobe, int32_t *__restrict__ probe)
{
    __shared__ uint32_t hist[256];
    __shared__ uint32_t s_prefix, s_need, s_pos;
    __shared__ uint32_t part[16];
    __shared__ uint64_t sel[kIvfMaxProbe * 2];
    const int tid = threadIdx.x;
    const uint32_t *d = reinterpret_cast<const uint32_t *>(dist);

    // Cut by value first: a histogram over kProbeSteps equal steps between the smallest and the largest
    // distance locates the step that holds the nprobe-th smallest; the keys up to that step (a superset of
    // the nprobe smallest, usually little more) are gathered and sorted by (distance, id).  The radix
    // select below remains for inputs where that superset is large (many equal distances) or the
    // distances span no finite range.  (Its first levels put all keys into a handful of counters, since
    // distances of similar size share their top bits, which serializes the LDS atomics.)
    {
        __shared__ uint32_t steps[kProbeSteps];
        __shared__ uint32_t s_lo, s_hi, s_step, s_n, wsum[16];
        const int lane = tid & 63, wave = tid >> 6;
        uint32_t lo = 0xFFFFFFFFu, hi = 0;
        // (the row is walked three times, four keys per lane and load where its length allows: 16 instead of 64
        // dependent rounds per walk at 65536 lists)
        const bool vec = (nlist & 3) == 0 && (reinterpret_cast<uintptr_t>(dist) & 15) == 0;    // uniform
        auto for_each_key = [&](auto &&f) {
            if (vec) {
                const uint4 *d4 = reinterpret_cast<const uint4 *>(d);
                for (int l4 = tid; l4 < nlist / 4; l4 += 1024) {
                    const uint4 k4 = d4[l4];
                    f(k4.x, 4 * l4); f(k4.y, 4 * l4 + 1); f(k4.z, 4 * l4 + 2); f(k4.w, 4 * l4 + 3);
                }
            } else {
                for (int l = tid; l < nlist; l += 1024) f(d[l], l);
            }
        };
        for_each_key([&](uint32_t key, int) { lo = min(lo, key); hi = max(hi, key); });
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            lo = min(lo, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lo), o)));
            hi = max(hi, static_cast<uint32_t>(__shfl_xor(static_cast<int>(hi), o)));
        }
        if (tid == 0) { s_lo = 0xFFFFFFFFu; s_hi = 0; s_step = kProbeSteps; s_n = 0; }
        for (uint32_t t = tid; t < kProbeSteps; t += 1024) steps[t] = 0;
        __syncthreads();
        if (lane == 0) { atomicMin(&s_lo, lo); atomicMax(&s_hi, hi); }
        __syncthreads();
        const float dlo = __uint_as_float(s_lo), dhi = __uint_as_float(s_hi);
        const float scale = static_cast<float>(kProbeSteps) / (dhi - dlo);
        // non-decreasing in the distance, so "step <= s" keeps every key below some value
        auto step_of = [&](uint32_t key) -> uint32_t {
            const float x = (__uint_as_float(key) - dlo) * scale;
            return x < static_cast<float>(kProbeSteps - 1) ? static_cast<uint32_t>(x) : kProbeSteps - 1;
        };
        bool cut = scale > 0.0f && scale < INFINITY;
        if (cut) {                                               // uniform
            for_each_key([&](uint32_t key, int) { atomicAdd(&steps[step_of(key)], 1u); });
            __syncthreads();
            const uint32_t h0 = steps[2 * tid], h1 = steps[2 * tid + 1];      // kProbeSteps = 2 x 1024 threads
            uint32_t incl = h0 + h1;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t other = __shfl(incl, lane >= o ? lane - o : lane);
                if (lane >= o) incl += other;
            }
            if (lane == 63) wsum[wave] = incl;
            __syncthreads();
            uint32_t before = incl - (h0 + h1);
            for (int w2 = 0; w2 < wave; ++w2) before += wsum[w2];
            const uint32_t want = static_cast<uint32_t>(nprobe);
            if (before < want && before + h0 + h1 >= want) {      // exactly one thread (nprobe <= nlist)
                const bool first = before + h0 >= want;
                s_step = first ? 2 * tid : 2 * tid + 1;
                s_n = first ? before + h0 : before + h0 + h1;
            }
            __syncthreads();
            cut = s_step < kProbeSteps && s_n <= kIvfMaxProbe * 2;
        }
        if (cut) {                                               // uniform
            const uint32_t step = s_step, nkeep = s_n;
            uint32_t nf = 1;
            while (nf < nkeep) nf <<= 1;
            __syncthreads();
            if (tid == 0) s_n = 0;
            for (uint32_t t = tid; t < nf; t += 1024) sel[t] = ~0ull;
            __syncthreads();
            for_each_key([&](uint32_t key, int l) {
                if (step_of(key) <= step) {
                    const uint32_t pos = atomicAdd(&s_n, 1u);
                    if (pos < nf) sel[pos] = make_key(key, static_cast<uint32_t>(l));
                }
            });
            bitonic_sort(sel, nf);
            for (int t = tid; t < nprobe; t += 1024)
                probe[t] = static_cast<int32_t>(sel[t] & 0xFFFFFFFFu);
            return;
        }
        __syncthreads();
    }

    // value of the nprobe-th smallest key, one byte at a time from the top
    uint32_t prefix = 0, need = nprobe;
    for (int level = 3; level >= 0; --level) {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        const uint32_t shift = 8 * level;
        const uint32_t hi_mask = level == 3 ? 0u : ~0u << (shift + 8);
        for (int l = tid; l < nlist; l += 1024) {
            const uint32_t key = d[l], digit = (key >> shift) & 255u;
            const bool in = (key & hi_mask) == prefix;
            const uint64_t mask = __builtin_amdgcn_ballot_w64(in);
            if (!mask) continue;                                     // (the same for all of a wavefront's lanes that are here)
            // (equal keys, which is what gets here, are counted together: their additions queue for one word)
            const int first = __builtin_ctzll(mask);
            const uint32_t common = __builtin_amdgcn_readlane(digit, first);
            const uint64_t same = __builtin_amdgcn_ballot_w64(in && digit == common);
            if ((tid & 63) == first) atomicAdd(&hist[common], static_cast<uint32_t>(__popcll(same)));
            if (in && digit != common) atomicAdd(&hist[digit], 1u);
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t cum = 0, b = 0;
            for (; b < 256; ++b) {
                if (cum + hist[b] >= need) break;
                cum += hist[b];
            }
            s_prefix = prefix | (b << shift);
            s_need = need - cum;
        }
        __syncthreads();
        prefix = s_prefix;
        need = s_need;
        __syncthreads();
    }
    const uint32_t kth = prefix;          // exact key of the nprobe-th smallest; `need` of the equal keys are taken
    if (tid == 0) s_pos = 0;
    __syncthreads();
    auto take = [&](uint32_t key, int l) {
        const uint32_t pos = atomicAdd(&s_pos, 1u);
        if (pos < static_cast<uint32_t>(nprobe)) sel[pos] = make_key(key, static_cast<uint32_t>(l));
    };
    for (int l = tid; l < nlist; l += 1024)
        if (d[l] < kth) take(d[l], l);
    // the first `need` of the equal ones, 1024 lists at a time (65536 lists, 1024 queries, all distances equal: 1.38 ms with a stretch of the row per thread and
    // without counting equal keys together above, 0.6 so)
    for (int base = 0; base < nlist && need; base += 1024) {           // uniform
        const int l = base + tid, lane = tid & 63;
        const bool equal = l < nlist && d[l] == kth;
        const uint64_t mask = __builtin_amdgcn_ballot_w64(equal);
        if (lane == 0) part[tid >> 6] = __popcll(mask);
        __syncthreads();
        uint32_t before = __popcll(mask & ((1ull << lane) - 1ull)), all = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < tid >> 6) before += part[w];
            all += part[w];
        }
        if (equal && before < need) take(kth, l);
        need -= min(need, all);
        __syncthreads();
    }
    __syncthreads();
    uint32_t np2 = 1;
    while (np2 < static_cast<uint32_t>(nprobe)) np2 <<= 1;
    for (uint32_t t = nprobe + tid; t < np2; t += 1024) sel[t] = ~0ull;
    bitonic_sort(sel, np2);
    for (int t = tid; t < nprobe; t += 1024) probe[t] = static_cast<int32_t>(sel[t] & 0xFFFFFFFFu);
}

}  // namespace dcpq

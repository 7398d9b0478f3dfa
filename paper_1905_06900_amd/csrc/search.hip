// Alg. 3 nns_derived end to end (no index): Tables -> Scan -> Refine for a batch of queries,
// in chunks so that the full 2^b-entry tables of one chunk fit the workspace.  b (bits of a sub-code,
// 16 or 8) and bbar (bits of a derived-codebook index, 1..8) are run-time parameters (the PQ m x bbar,b
// family of Sec. 3.1); sub-codes are stored in 2 bytes for b = 16 and in 1 byte for b = 8.
#include "common.h"

namespace dcpq {

struct SearchPlan {
    int chunk;
    size_t off_qtab, off_bounds, off_cand_id, off_cand_qd, off_tables, tables_bytes, off_scan, off_refine;
    size_t least, total;       // bytes a workspace must hold, and does best with
    size_t off_pairs, off_pair_tab;      // 8-bit sub-codes scanned in pairs (off_pairs 0: not at these sizes); the scan's arrays end there
};

static SearchPlan plan_search(uint64_t n_codes, int m, int nq, uint32_t r, int full_bits, int chunk_queries)
{
    SearchPlan p{};
    int chunk = chunk_queries;
    if (chunk <= 0) {   // default: about 8 GiB of full tables per chunk (sized for a 288 GB device; the larger
                        // the chunk, the fewer launches share the scan's start-up and tail)
        const size_t per_q = sizeof(float) * (static_cast<size_t>(m) << full_bits);
        chunk = static_cast<int>((static_cast<size_t>(8) << 30) / per_q);
        if (chunk < 64) chunk = 64;
    }
    if (chunk > nq) chunk = nq;
    p.chunk = chunk;
    size_t off = 0;
    p.off_qtab = off;    off = align_up(off + static_cast<size_t>(chunk) * m * kSmallSize, 256);
    p.off_bounds = off;  off = align_up(off + sizeof(float) * 2 * static_cast<size_t>(chunk), 256);
    p.off_cand_id = off; off = align_up(off + sizeof(uint32_t) * static_cast<size_t>(chunk) * r, 256);
    p.off_cand_qd = off; off = align_up(off + static_cast<size_t>(chunk) * r, 256);
    // The scan and the refinement lay their scratch out for the number of queries they are given, and
    // a smaller batch does not always need less (fewer queries can mean more units or slices), so
    // the regions hold the larger of what a full chunk and what the ragged last chunk need: those
    // are the only two batch sizes the loop below ever passes.
    const int tail = nq % chunk;
    size_t scan_bytes = dcpq_scan_workspace_bytes(n_codes, m, chunk, r), least_bytes = scan_least_bytes(n_codes, m, chunk, r);
    size_t refine_bytes = dcpq_refine_workspace_bytes(chunk, r);
    if (tail) {
        const size_t st = dcpq_scan_workspace_bytes(n_codes, m, tail, r), rt = dcpq_refine_workspace_bytes(tail, r);
        const size_t lt = scan_least_bytes(n_codes, m, tail, r);
        scan_bytes = st > scan_bytes ? st : scan_bytes;
        least_bytes = lt > least_bytes ? lt : least_bytes;
        refine_bytes = rt > refine_bytes ? rt : refine_bytes;
    }
    p.off_refine = off;  off = align_up(off + refine_bytes, 256);
    // the full tables of a chunk (table mode), or the codebooks with their rows padded to whole 64-byte units
    // (on-demand mode with rows shorter than that; 16 floats per row), or the sub-code planes and entries of the
    // split on-demand mode (used only where they fit): the region holds the larger of the first two
    {
        const size_t tables = sizeof(float) * ((static_cast<size_t>(chunk) * m) << full_bits);
        const size_t padded = sizeof(float) * ((static_cast<size_t>(m) * 16) << full_bits);
        p.tables_bytes = tables > padded ? tables : padded;
        p.off_tables = off;  off = align_up(off + p.tables_bytes, 256);
    }
    p.off_scan = off;    // last: the scan's own last array is as long as the workspace allows
    p.least = align_up(off + least_bytes, 256);
    p.total = align_up(off + scan_bytes, 256);
    // (not where the codes can be sorted into cells)
    if (full_bits == 8 && pairs_pay(n_codes, m, chunk) && !(cells_may_pay(n_codes, m, chunk, r) && cells_bytes(n_codes, m, chunk) <= p.tables_bytes)) {
        size_t pair_bytes = dcpq_scan_workspace_bytes(n_codes, m / 2, chunk, r);
        if (tail) {
            const size_t st = dcpq_scan_workspace_bytes(n_codes, m / 2, tail, r);
            pair_bytes = st > pair_bytes ? st : pair_bytes;
        }
        p.off_pairs = align_up(off + pair_bytes, 256);
        p.off_pair_tab = align_up(p.off_pairs + n_codes * (m / 2), 256);
        const size_t t = align_up(p.off_pair_tab + static_cast<size_t>(chunk) * (m / 2) * kSmallSize, 256);
        p.total = t > p.total ? t : p.total;
    }
    // small problems take the two-kernel form where its arrays fit, over the tables (which it does not use) and the scan's
    // (asked of the chunk: a batch of one chunk reserves no more than one with a ragged chunk behind it)
    if (small_search_pays(n_codes, m, chunk)) {
        const size_t t = align_up(p.off_tables + small_search_bytes(n_codes, chunk, r), 256);
        p.total = t > p.total ? t : p.total;
    }
    return p;
}

}  // namespace dcpq

using namespace dcpq;

extern "C" int dcpq_search_bits_chunk(int m, int nq, int b, int chunk_queries)
{
    if (nq <= 0 || !m_supported(m) || !dcpq_bits_supported(b, 1)) return 0;
    return plan_search(1, m, nq, 1, b, chunk_queries).chunk;
}

extern "C" int dcpq_search_chunk(int m, int nq, int chunk_queries) { return dcpq_search_bits_chunk(m, nq, kFullBits, chunk_queries); }

extern "C" size_t dcpq_search_bits_workspace_bytes(uint64_t n_codes, int m, int nq, uint32_t r, int b, int chunk_queries)
{
    if (nq <= 0 || !m_supported(m) || n_codes == 0 || r == 0 || r > (1u << 26) || !dcpq_bits_supported(b, 1)) return 0;
    return plan_search(n_codes, m, nq, r, b, chunk_queries).total;
}

extern "C" size_t dcpq_search_workspace_bytes(uint64_t n_codes, int m, int nq, uint32_t r, int chunk_queries)
{
    return dcpq_search_bits_workspace_bytes(n_codes, m, nq, r, kFullBits, chunk_queries);
}

// How pass two gets its table entries: looked up in full tables built first (DCPQ_REFINE_TABLES), or computed
// on demand, in one kernel (DCPQ_REFINE_DIRECT) or split by sub-quantizer (DCPQ_REFINE_SPLIT).  Measured on MI355X,
// microseconds for tables / one kernel / split:
//   m = 8, dsub = 12, random codes: 300 queries, r = 9000: 734 / 712 / 242;  16 queries, r = 4000: 87 / 181 / 37;  2 queries, r = 1000: 45 / 51 / 27
//   m = 8, dsub = 16, encoded codes: 251, r = 10000: 376 / 232 / 178;  1000, r = 2000: 691 / 118 / 169
//   m = 16, dsub = 60, encoded codes: 512, r = 5000, N = 10 M: 1850 / 139 / 267;  N = 3 M: 1850 / 1358 / 351;  3, r = 6000: 285 / 15 / 40
//   m = 4, dsub = 32, random codes: 1000, r = 1000: 607 / 124 / 104;  100, r = 10000: 168 / 231 / 103
//   b = 8 (tables of 256 entries), m = 16, dsub = 8: 333, r = 2000: 47 / 97 / -
// The one-kernel form wins where the candidates of a query name few enough sub-codes to memoize their entries, and loses
// widely where they do not; that shows on the device only.  So with 16-bit sub-codes: split where a sub-codebook
// (two for m = 16, four for m = 32) is smaller than one XCD's 4 MB cache (dsub < 16 at m = 8: the split form is never far
// behind there), where there is nothing to memoize, or where the batch is small (below 2^18 candidates the attempt costs what
// it can save: 50 queries, r = 3000: 33 one kernel, 35 split, 50 one after the other); else the one-kernel form first, and the split form for the queries
// that it gives up.  A query with a few candidates (an entry per thread of its workgroup at most) is worked out in one kernel at
// once, where that reads the codebooks in place (m = 8, dsub = 16, r = 10, searches of 20 / 300 / 1000 queries: 78 / 168 / 278 us
// against 82 / 172 / 285 split; r = 100: 90 / 198 / 330 and 94 / 199 / 329; r = 400: 89 / 230 / 404 and 89 / 222 / 381).  Tables for 8-bit sub-codes, and where the split form's arrays do not fit and r > 2^b / 8 (a gathered row
// costs about 8 ps more than a table lookup and a 2^16-entry table 60 to 200 ns to build).
static bool split_possible(const SearchPlan &p, int m, int b, int nq, uint32_t r, const float *queries)
{
    // (its kernels read query sub-vectors 16 bytes at a time from where the caller keeps them)
    return static_cast<uint64_t>(nq) * r < (1ull << 32) && refine_split_bytes(nq, r, m, b / 8) <= p.tables_bytes &&
           (reinterpret_cast<uintptr_t>(queries) & 15) == 0;
}

// the split form at once, without an attempt to memoize?
static bool split_first(int m, int dsub, int b, int nq, uint32_t r)
{
    const size_t sub = (sizeof(float) * static_cast<size_t>(dsub)) << b;
    return sub * ((m + 7) / 8) < (4u << 20) || refine_memo_slots(m, dsub, r) == 0 || static_cast<uint64_t>(nq) * r < (1u << 18);
}

// rows that the one-kernel form reads from a copy (see below)
static bool pads_rows(int dsub) { return dsub < 16 && 16 % dsub != 0; }

// What a chunk of nq queries runs.
enum Form { kTables, kOneKernel, kSplit, kOneKernelThenSplit };
static Form refine_form(int requested, const SearchPlan &p, int m, int dsub, int b, int nq, uint32_t r, const float *queries)
{
    if (requested != DCPQ_REFINE_AUTO) return requested == DCPQ_REFINE_TABLES ? kTables : requested == DCPQ_REFINE_DIRECT ? kOneKernel : kSplit;
    if (b != 16 || !split_possible(p, m, b, nq, r, queries)) return r > (1u << b) / 8 ? kTables : kOneKernel;
    if (static_cast<uint64_t>(r) * m <= 1024 && !pads_rows(dsub)) return kOneKernel;
    return split_first(m, dsub, b, nq, r) ? kSplit : kOneKernelThenSplit;
}

// the size rule that dcpq_search_refine_mode reports; a search goes by refine_form
static int refine_mode_for(int requested, const SearchPlan &p, int m, int dsub, int b, int nq, uint32_t r)
{
    if (requested != DCPQ_REFINE_AUTO) return requested;
    if (r > (1u << b) / 8) return DCPQ_REFINE_TABLES;
    const size_t sub = (sizeof(float) * static_cast<size_t>(dsub)) << b;
    const bool pays = sub * ((m + 7) / 8) < (4u << 20) && sub * m > (4u << 20) && static_cast<uint64_t>(nq) * r >= (1u << 16);
    return pays && split_possible(p, m, b, nq, r, nullptr) ? DCPQ_REFINE_SPLIT : DCPQ_REFINE_DIRECT;
}

extern "C" int dcpq_search_bits(const float *queries, int nq, const float *codebooks, const float *derived, int m,
                                int dsub, int b, int bbar, const void *codes, uint64_t n_codes, uint32_t r, uint32_t k,
                                int refine_mode, uint32_t *ids, float *dist, int chunk_queries, void *workspace,
                                size_t workspace_bytes, void *stream)
{
    clear_error();
    DCPQ_REQUIRE(nq >= 0, "search: nq=%d", nq);
    if (!dcpq_shape_supported(m, dsub)) return fail(DCPQ_EUNSUPPORTED, "search: m=%d dsub=%d not supported", m, dsub);
    if (!dcpq_bits_supported(b, bbar)) return fail(DCPQ_EUNSUPPORTED, "search: b=%d bbar=%d not supported", b, bbar);
    DCPQ_REQUIRE(n_codes >= 1 && n_codes < (1ull << 32), "search: n_codes out of range");
    DCPQ_REQUIRE(r >= 1 && r <= n_codes && k >= 1 && k <= r, "search: needs 1 <= k <= r <= n_codes");
    DCPQ_REQUIRE(r <= (1u << 26), "search: r=%u above the supported 2^26", r);
    DCPQ_REQUIRE(refine_mode == DCPQ_REFINE_AUTO || refine_mode == DCPQ_REFINE_TABLES || refine_mode == DCPQ_REFINE_DIRECT ||
                     refine_mode == DCPQ_REFINE_SPLIT,
                 "search: refine_mode=%d", refine_mode);
    if (nq == 0) return DCPQ_OK;
    DCPQ_REQUIRE(queries && codebooks && derived && codes && ids && dist && workspace, "search: null pointer");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(codebooks) & 15) == 0, "search: codebooks must be 16-byte aligned");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(workspace) & 255) == 0, "search: workspace must be 256-byte aligned");
    DCPQ_REQUIRE((reinterpret_cast<uintptr_t>(codes) & 15) == 0, "search: codes must be 16-byte aligned");
    const SearchPlan p = plan_search(n_codes, m, nq, r, b, chunk_queries);
    if (workspace_bytes < p.least)
        return fail(DCPQ_EWORKSPACE, "search: workspace %zu < %zu bytes", workspace_bytes, p.least);
    uint8_t *base = static_cast<uint8_t *>(workspace);
    uint8_t *qtab = base + p.off_qtab;
    float *bounds = reinterpret_cast<float *>(base + p.off_bounds);
    uint32_t *cand_id = reinterpret_cast<uint32_t *>(base + p.off_cand_id);
    uint8_t *cand_qd = base + p.off_cand_qd;
    float *tables = reinterpret_cast<float *>(base + p.off_tables);
    hipStream_t st = as_stream(stream);
    const int D = m * dsub;
    const int code_bytes = b / 8;
    const int tail = nq % p.chunk;
    const Form full = refine_form(refine_mode, p, m, dsub, b, p.chunk, r, queries);
    const Form last = tail ? refine_form(refine_mode, p, m, dsub, b, tail, r, queries) : full;
    if (full == kSplit && !split_possible(p, m, b, p.chunk, r, queries))
        return fail(DCPQ_EINVAL, "search: DCPQ_REFINE_SPLIT: %zu bytes of sub-codes and entries per chunk do not fit the table "
                                 "region (%zu bytes), or chunk * r reaches 2^32, or the queries are not 16-byte aligned",
                    refine_split_bytes(p.chunk, r, m, b / 8), p.tables_bytes);
    // small problems: candidates and their distances in two kernels (entries on demand, as DCPQ_REFINE_DIRECT computes them)
    if (small_search_pays(n_codes, m, nq) && p.chunk == nq && small_search_bytes(n_codes, nq, r) <= workspace_bytes - p.off_tables &&
        (refine_mode == DCPQ_REFINE_AUTO || refine_mode == DCPQ_REFINE_DIRECT)) {
        int rc = launch_small_tables(queries, nq, derived, m, dsub, bbar, codes, code_bytes, n_codes, r, qtab, bounds, nullptr, st,
                                     reinterpret_cast<uint32_t *>(base + p.off_tables), small_search_clear_words(n_codes, nq, r));
        if (rc) return rc;
        const uint64_t *keys = nullptr;
        rc = launch_small_search(queries, nq, codebooks, m, dsub, 1u << b, codes, code_bytes, n_codes, qtab, r, tables, &keys, st);
        if (rc) return rc;
        return launch_topk_of_keys(keys, nq, r, k, ids, dist, base + p.off_refine, st);
    }
    // On demand in one kernel, a candidate gathers m centroid rows; a row shorter than a 64-byte unit that does not divide it
    // lies across two memory lines more often than it has to, so such codebooks are copied once per call into
    // rows of 16 floats (25 -> 33 MB at m = 8, dsub = 12: 30 microseconds, 6 % off the refinement).  Longer rows
    // gain nothing and the copy costs more (measured at dsub = 60), so they are read in place.  The copy lies in the
    // region that the other forms use for arrays of their own: it is made where the whole chunks run this form, and the last
    // chunk, which comes after them, may still read it if it does too.
    const float *rows = codebooks;
    int cstride = dsub;
    if (full == kOneKernel && pads_rows(dsub)) {
        cstride = 16;
        int rc = launch_pad_rows(codebooks, static_cast<size_t>(m) << b, dsub, cstride, tables, st);
        if (rc) return rc;
        rows = tables;
    }
    // up to 16 derived centroids: 8-bit sub-codes are scanned as pairs, where the workspace has room for these
    const bool paired = p.off_pairs && bbar <= 4 && workspace_bytes >= p.off_pair_tab + static_cast<size_t>(p.chunk) * (m / 2) * kSmallSize;
    const size_t room = (paired ? p.off_pairs : workspace_bytes) - p.off_scan;
    uint8_t *plane = base + p.off_pairs, *ptab = base + p.off_pair_tab;
    if (paired) {
        const int rc = launch_pair_codes(static_cast<const uint8_t *>(codes), n_codes, m, plane, st);
        if (rc) return rc;
    }
    const int ms = paired ? m / 2 : m;             // sub-quantizers of the scan
    for (int q0 = 0; q0 < nq; q0 += p.chunk) {
        const int nc = (nq - q0 < p.chunk) ? nq - q0 : p.chunk;
        const float *y = queries + static_cast<size_t>(q0) * D;
        int rc = launch_small_tables(y, nc, derived, m, dsub, bbar, codes, code_bytes, n_codes, r, qtab, bounds, nullptr, st,
                                     reinterpret_cast<uint32_t *>(base + p.off_scan), scan_clear_words(n_codes, ms, nc, r, DCPQ_SCAN_AUTO));
        if (rc) return rc;
        // (the table region is free until pass two: where the codes fit it, the scan may sort them there)
        const CellsArea area{base + p.off_tables, derived, dsub, bbar};
        const CellsArea *cells = rows == codebooks && cells_may_pay(n_codes, m, nc, r) && cells_bytes(n_codes, m, nc) <= p.tables_bytes ? &area : nullptr;
        // the quantized tables have 256 entries whatever bbar is, and 1-byte sub-codes are their own low-byte plane
        if (paired) {
            rc = launch_pair_tables(qtab, nc, m, ptab, st);
            if (rc) return rc;
            rc = launch_scan(plane, n_codes, ms, ptab, nc, r, cand_id, cand_qd, base + p.off_scan, room, DCPQ_SCAN_AUTO, true, st);
        } else if (code_bytes == 1)
            rc = launch_scan(static_cast<const uint8_t *>(codes), n_codes, m, qtab, nc, r, cand_id, cand_qd, base + p.off_scan,
                             room, DCPQ_SCAN_AUTO, true, st, cells);
        else
            rc = launch_scan(static_cast<const uint16_t *>(codes), n_codes, m, qtab, nc, r, cand_id, cand_qd,
                             base + p.off_scan, room, DCPQ_SCAN_AUTO, true, st, cells);
        if (rc) return rc;
        uint32_t *ids_c = ids + static_cast<size_t>(q0) * k;
        float *dist_c = dist + static_cast<size_t>(q0) * k;
        switch (nc == p.chunk ? full : last) {
        case kSplit:
            rc = launch_refine_split(y, codebooks, dsub, 1u << b, codes, code_bytes, n_codes, m, cand_id, nc, r, k, ids_c, dist_c,
                                     tables, base + p.off_refine, st);
            break;
        case kOneKernelThenSplit: {
            // (the integer distances are not needed any more: their place holds the queries left to the split form)
            uint32_t *left = reinterpret_cast<uint32_t *>(cand_qd);
            rc = launch_refine_direct(y, codebooks, dsub, dsub, 1u << b, codes, code_bytes, n_codes, m, cand_id, nc, r, k, ids_c,
                                      dist_c, base + p.off_refine, st, left, tables);
            if (rc) return rc;
            rc = launch_refine_split(y, codebooks, dsub, 1u << b, codes, code_bytes, n_codes, m, cand_id, nc, r, k, ids_c, dist_c,
                                     tables, base + p.off_refine, st, left);
            break;
        }
        case kOneKernel:
            rc = launch_refine_direct(y, rows, dsub, cstride, 1u << b, codes, code_bytes, n_codes, m, cand_id, nc, r, k, ids_c,
                                      dist_c, base + p.off_refine, st);
            break;
        case kTables:
            rc = launch_distance_tables(y, nc, codebooks, m, dsub, 1 << b, tables, kStageFullTables, st);
            if (rc) return rc;
            rc = launch_refine(tables, 1u << b, codes, code_bytes, n_codes, m, cand_id, nc, r, k, ids_c, dist_c,
                               base + p.off_refine, st);
            break;
        }
        if (rc) return rc;
    }
    return DCPQ_OK;
}

extern "C" int dcpq_search(const float *queries, int nq, const float *codebooks, const float *derived, int m,
                           int dsub, const uint16_t *codes, uint64_t n_codes, uint32_t r, uint32_t k,
                           uint32_t *ids, float *dist, int chunk_queries, void *workspace,
                           size_t workspace_bytes, void *stream)
{
    return dcpq_search_bits(queries, nq, codebooks, derived, m, dsub, kFullBits, kSmallBits, codes, n_codes, r, k,
                            DCPQ_REFINE_AUTO, ids, dist, chunk_queries, workspace, workspace_bytes, stream);
}

extern "C" int dcpq_search_refine_mode(int m, int dsub, int b, int nq, uint32_t r, int refine_mode)
{
    if (nq <= 0 || !m_supported(m) || !dcpq_bits_supported(b, 1) || r == 0) return refine_mode;
    const SearchPlan p = plan_search(1, m, nq, r, b, 0);
    return refine_mode_for(refine_mode, p, m, dsub, b, p.chunk, r);
}

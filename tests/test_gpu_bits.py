"""GPU parity tests of the PQ m x bbar,b family (Sec. 3.1 notation): the two-pass search with b-bit
sub-codes (16 or 8) and bbar-bit derived codebooks (4, 5, 6, 8), stage by stage and fused, against
the oracle run with the same widths."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_06900_amd import binding, synth
from parity import to_np, assert_topk_matches

pytestmark = pytest.mark.gpu

DEV = "cuda"


def make_case(m, dsub, b, bbar, N, Q, seed):
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    pbits = min(4, bbar)
    cb = synth.hierarchical_codebooks(m, dsub, b, pbits, lambda shape, gg: 0.3 * torch.randn(
        shape, generator=gg, device=DEV, dtype=torch.float32), 0.05, DEV, seed + 1)
    if b == 16:
        codes = synth.random_codes(N, m, DEV, seed + 2).view(torch.uint16)
    else:
        codes = torch.randint(0, 256, (N, m), generator=g, device=DEV, dtype=torch.uint8)
    queries = 0.3 * torch.randn((Q, m * dsub), generator=g, device=DEV, dtype=torch.float32)
    return cb, codes, queries


CASES = [  # (b, bbar, m, dsub, N, Q, r)
    (16, 8, 4, 8, 60_003, 19, 400),
    (16, 6, 4, 8, 60_003, 19, 400),
    (16, 4, 8, 6, 50_001, 21, 300),
    (8, 4, 8, 6, 70_001, 37, 500),
    (8, 5, 4, 8, 40_003, 9, 300),
    (8, 6, 16, 4, 30_001, 11, 600),      # r m = 9600: the on-demand refinement memoizes (at most 256 distinct sub-codes)
    (8, 8, 8, 6, 30_001, 11, 200),
    (8, 4, 2, 16, 30_001, 5, 100),
    (16, 8, 1, 8, 20_001, 7, 200),
    (16, 8, 32, 4, 20_001, 7, 200),
    (16, 5, 2, 8, 20_001, 7, 200),
]


@pytest.mark.parametrize("b,bbar,m,dsub,N,Q,r", CASES)
def test_two_pass_search_with_these_bit_widths(b, bbar, m, dsub, N, Q, r):
    print("PQ %dx%d,%d dsub=%d N=%d Q=%d r=%d" % (m, bbar, b, dsub, N, Q, r), flush=True)
    k = 50
    cb, codes, queries = make_case(m, dsub, b, bbar, N, Q, 7000 + 10 * b + bbar)
    derived = binding.derive_codebooks(cb, bbar)
    qtab, bounds, small = binding.build_small_tables(queries, derived, codes, r, want_small=True)
    cand_id, cand_qd = binding.scan_candidates(codes, qtab, r)
    tables = binding.build_tables_n(queries, cb)
    ids, dist = binding.refine_topk(tables, codes, cand_id, k)
    fids, fdist = binding.search(queries, cb, derived, codes, r, k, refine_mode=binding.REFINE_TABLES)
    dids, ddist = binding.search(queries, cb, derived, codes, r, k, refine_mode=binding.REFINE_DIRECT)
    # on demand, split by sub-quantizer: the same bits as the one-kernel form; its arrays always fit the table
    # region when r * (4 + b / 8) <= 4 * 2^b, and where they do not fit the mode is refused
    try:
        sids, sdist = binding.search(queries, cb, derived, codes, r, k, refine_mode=binding.REFINE_SPLIT)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(to_np(sids), to_np(dids), err_msg="split on-demand refinement, ids")
        np.testing.assert_array_equal(to_np(sdist), to_np(ddist), err_msg="split on-demand refinement, distances")
    except binding.DcpqError as err:
        assert err.code == binding.EINVAL and r * (4 + b // 8) > 4 << b
    torch.cuda.synchronize()

    cb_np, q_np = to_np(cb), to_np(queries)
    codes_np = to_np(codes).astype(np.uint16)
    der_ref = oracle.derive_codebooks(cb_np, b=b, bbar=bbar)
    ref = oracle.search_flat(cb_np, der_ref, codes_np, q_np, r, k, b=b, bbar=bbar)
    ks = 1 << bbar
    np.testing.assert_array_equal(to_np(derived), der_ref, err_msg="derived codebooks")
    np.testing.assert_array_equal(to_np(small), ref["small"], err_msg="small tables")
    np.testing.assert_array_equal(to_np(bounds), ref["bounds"], err_msg="qmin/qmax")
    qt = to_np(qtab)
    np.testing.assert_array_equal(qt[:, :, :ks], ref["qtab"], err_msg="quantized tables")
    np.testing.assert_array_equal(qt, np.tile(ref["qtab"], (1, 1, 256 // ks)), err_msg="quantized tables, replicas")
    np.testing.assert_array_equal(to_np(cand_id), ref["cand_id"], err_msg="candidate ids")
    np.testing.assert_array_equal(to_np(cand_qd), ref["cand_qd"], err_msg="candidate qd")
    ids, dist = to_np(ids), to_np(dist)
    for q in range(Q):
        exact = oracle.refine(q_np[q], cb_np, codes_np, ids[q], b=b)
        assert_topk_matches(ids[q], dist[q], ref["ids"][q], ref["dist"][q], exact, cand_ref=ref["cand_id"][q],
                            tag="query %d" % q)
    np.testing.assert_array_equal(to_np(fids), ids, err_msg="fused search ids")
    np.testing.assert_array_equal(to_np(fdist), dist, err_msg="fused search distances")
    dids, ddist = to_np(dids), to_np(ddist)
    for q in range(Q):
        exact = oracle.refine(q_np[q], cb_np, codes_np, dids[q], b=b)
        assert_topk_matches(dids[q], ddist[q], ref["ids"][q], ref["dist"][q], exact, cand_ref=ref["cand_id"][q],
                            tag="on-demand refinement, query %d" % q)


def test_unsupported_widths_are_refused():
    assert binding.lib().dcpq_bits_supported(16, 8) == 1 and binding.lib().dcpq_bits_supported(8, 4) == 1
    assert binding.lib().dcpq_bits_supported(12, 8) == 0 and binding.lib().dcpq_bits_supported(8, 9) == 0
    cb = torch.zeros((2, 4096, 4), dtype=torch.float32, device=DEV)      # b = 12
    with pytest.raises(binding.DcpqError):
        binding.derive_codebooks(cb, 8)


@pytest.mark.parametrize("b,bbar,m,dsub,N,Q,r", [
    (16, 8, 8, 12, 4096, 3, 4096),          # r = N, one full step of the first kernel
    (16, 8, 4, 32, 4097, 1, 100),           # one code beyond it
    (16, 8, 1, 7, 130_001, 9, 1),           # ragged last stretch, r = 1
    (16, 8, 16, 5, 300_003, 2, 9000),       # several rounds of candidates per stretch
    (8, 6, 32, 4, 50_001, 5, 700),
    (16, 8, 8, 16, 1_200_003, 1, 12_000),   # a stretch per workgroup (no adding up of histograms)
    (8, 4, 2, 16, 1_000_001, 4, 3000),      # two sub-codes of 16 values each: tens of thousands of ties at the bound
    (16, 4, 1, 6, 1_500_007, 1, 12_000),    # ... and of one: all candidates in the first stretch, more than its list holds
    (16, 1, 8, 8, 700_001, 2, 9000),
    (16, 8, 8, 6, 30_001, 300, 200),        # queries enough for one stretch each
])
def test_small_problems_in_two_kernels(b, bbar, m, dsub, N, Q, r):
    # the same search through the staged calls (scan, full tables, refine)
    print("small PQ %dx%d,%d dsub=%d N=%d Q=%d r=%d" % (m, bbar, b, dsub, N, Q, r), flush=True)
    k = min(100, r)
    cb, codes, queries = make_case(m, dsub, b, bbar, N, Q, 9100 + N % 97)
    derived = binding.derive_codebooks(cb, bbar)
    qtab, _, _ = binding.build_small_tables(queries, derived, codes, r)
    cand_id, _ = binding.scan_candidates(codes, qtab, r)
    want_ids, want_dist = binding.refine_direct_topk(queries, cb, codes, cand_id, k)
    for mode in (binding.REFINE_AUTO, binding.REFINE_DIRECT):
        ids, dist = binding.search(queries, cb, derived, codes, r, k, refine_mode=mode)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(to_np(ids), to_np(want_ids))
        np.testing.assert_array_equal(to_np(dist), to_np(want_dist))
    ids, dist, cb_np, codes_np = to_np(ids), to_np(dist), to_np(cb), to_np(codes).astype(np.uint16)
    for q in {0, Q - 1}:
        y = to_np(queries)[q:q + 1]
        ref = oracle.search_flat(cb_np, to_np(derived), codes_np, y, r, k, b=b, bbar=bbar)
        exact = oracle.refine(y[0], cb_np, codes_np, ids[q], b=b)
        assert_topk_matches(ids[q], dist[q], ref["ids"][0], ref["dist"][0], exact, cand_ref=ref["cand_id"][0], tag="query %d" % q)


@pytest.mark.parametrize("Q", [1, 499, 500, 501])
def test_small_tables_with_one_and_two_queries_per_workgroup(Q):
    m, dsub, b, bbar, N, r = 8, 6, 16, 8, 3000, 700
    cb, codes, queries = make_case(m, dsub, b, bbar, N, Q, 77)
    derived = binding.derive_codebooks(cb, bbar)
    qtab, bounds, small = (to_np(x) for x in binding.build_small_tables(queries, derived, codes, r, want_small=True))
    q_np, d_np, c_np = to_np(queries), to_np(derived), to_np(codes)
    for q in {0, Q // 2, Q - 1}:
        D = oracle.compute_tables_f32(q_np[q], d_np)
        lo, hi = oracle.bounds(D, c_np, r)
        np.testing.assert_array_equal(small[q], D)
        np.testing.assert_array_equal(bounds[q], np.array([lo, hi], np.float32))


def test_more_queries_than_a_grid_has_rows():
    # 8-bit codes leave room for chunks of millions of queries; over so short an array they are a small problem
    m, dsub, N, Q, r, k = 1, 4, 300, 70_001, 20, 5
    print("small problem of %d queries" % Q, flush=True)
    cb, codes, queries = make_case(m, dsub, 8, 8, N, Q, 4711)
    derived = binding.derive_codebooks(cb, 8)
    ids, dist = (to_np(t) for t in binding.search(queries, cb, derived, codes, r, k))
    torch.cuda.synchronize()
    cb_np, c_np, q_np = to_np(cb), to_np(codes), to_np(queries)
    sel = [0, 35_000, 65_535, 65_536, Q - 1]
    ref = oracle.search_flat(cb_np, to_np(derived), c_np, q_np[sel], r, k, 8, 8)
    for a, q in enumerate(sel):
        exact = oracle.refine(q_np[q], cb_np, c_np, ids[q], 8)
        assert_topk_matches(ids[q], dist[q], ref["ids"][a], ref["dist"][a], exact, cand_ref=ref["cand_id"][a], tag="query %d" % q)


@pytest.mark.parametrize("Q,b,dsub", [(1, 16, 4), (7, 8, 8), (499, 16, 4), (501, 16, 12)])
def test_smallest_tables_and_candidate_sets(Q, b, dsub):
    # one sub-quantizer with two derived centroids, and one candidate: two floats of tables, and one key, lie in front of
    # the query in LDS, which is read in 16-byte vectors
    print("smallest tables Q=%d b=%d dsub=%d" % (Q, b, dsub), flush=True)
    cb, codes, queries = make_case(1, dsub, b, 1, 900, Q, 13)
    derived = binding.derive_codebooks(cb, 1)
    qtab, bounds, small = (to_np(x) for x in binding.build_small_tables(queries, derived, codes, 50, want_small=True))
    q_np, d_np, cb_np, c_np = to_np(queries), to_np(derived), to_np(cb), to_np(codes).astype(np.uint16)
    cand = torch.randint(0, 900, (Q, 1), device=DEV, dtype=torch.int32).view(torch.uint32)
    ids, dist = (to_np(x) for x in binding.refine_direct_topk(queries, cb, codes, cand, 1))
    np.testing.assert_array_equal(ids, to_np(cand))
    for q in {0, Q // 2, Q - 1}:
        D = oracle.compute_tables_f32(q_np[q], d_np)
        np.testing.assert_array_equal(small[q], D)
        lo, hi = oracle.bounds(D, c_np, 50, 1)
        np.testing.assert_array_equal(bounds[q], np.array([lo, hi], np.float32))
        np.testing.assert_array_equal(qtab[q], np.tile(oracle.quantize(D, lo, hi), (1, 128)))
        np.testing.assert_allclose(dist[q], oracle.refine(q_np[q], cb_np, c_np, ids[q], b), rtol=1e-6)

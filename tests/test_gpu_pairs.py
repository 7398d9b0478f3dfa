"""8-bit sub-codes scanned as pairs (bbar <= 4, large batches): the same results as with the scan of single sub-codes, which the
other tests hold against the oracle."""
import pytest
import torch

from paper_1905_06900_amd import binding
from test_gpu_bits import make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,dsub,bbar,N,Q,r,chunk", [
    (16, 8, 4, 2_500_003, 203, 2000, 0),
    (16, 4, 1, 1_000_001, 501, 300, 0),      # two derived centroids: nearly all distances equal
    (8, 16, 4, 5_000_001, 100, 1000, 0),     # the smallest batch; an odd number of 8-byte codes
    (8, 5, 3, 5_000_001, 150, 700, 101),     # a ragged last chunk
    (32, 4, 2, 1_000_003, 500, 1, 0),
])
def test_pairs_against_single_sub_codes(m, dsub, bbar, N, Q, r, chunk):
    k = min(r, 50)
    cb, codes, y = make_case(m, dsub, 8, bbar, N, Q, 40 + m + bbar)
    derived = binding.derive_codebooks(cb, bbar)
    full = binding.search_workspace_bytes(N, m, Q, r, chunk, 8)
    ids, dist = binding.search(y, cb, derived, codes, r, k, chunk)
    less = torch.empty(full - 1, dtype=torch.uint8, device=codes.device)      # no room for the pairs
    ids1, dist1 = binding.search(y, cb, derived, codes, r, k, chunk, workspace=less)
    assert torch.equal(ids.view(torch.int32), ids1.view(torch.int32))
    assert torch.equal(dist, dist1)
    qtab, _, _ = binding.build_small_tables(y, derived, codes, r)
    cand, _ = binding.scan_candidates(codes, qtab, r)
    if r > 32:                               # as the search does: tables, or single entries for very few candidates
        ids2, dist2 = binding.refine_topk(binding.build_tables_n(y, cb), codes, cand, k)
    else:
        ids2, dist2 = binding.refine_direct_topk(y, cb, codes, cand, k)
    assert torch.equal(ids.view(torch.int32), ids2.view(torch.int32))
    assert torch.equal(dist, dist2)

"""Search over codes sorted into cells (large batches over large arrays, m = 8): the same results as with the scan that looks at
every pair, which the other tests hold against the oracle."""
import pytest
import torch

from paper_1905_06900_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N, Q = 4_194_307, 2001          # just above the sizes from which the codes are sorted; no tile divides them


def _inputs(kind, dsub, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    parents = 3.0 * torch.randn((8, 16, dsub), generator=g, device=DEV)
    cb = parents.repeat(1, 4096, 1) + 0.3 * torch.randn((8, 65536, dsub), generator=g, device=DEV)
    if kind == "ties":              # 300 different codes: thousands of equal distances at the bound
        base = torch.randint(0, 65536, (300, 8), generator=g, device=DEV, dtype=torch.int32)
        codes = base[torch.randint(0, 300, (N,), generator=g, device=DEV)]
    elif kind == "one_cell":        # all codes in one cell but a few
        codes = torch.randint(0, 4096, (N, 8), generator=g, device=DEV, dtype=torch.int32) * 16
        codes[::1000] = torch.randint(0, 65536, codes[::1000].shape, generator=g, device=DEV, dtype=torch.int32)
    else:                           # mixture: neighbours differ in the high bytes mostly
        base = torch.randint(0, 65536, (1000, 8), generator=g, device=DEV, dtype=torch.int32)
        codes = base[torch.randint(0, 1000, (N,), generator=g, device=DEV)]
        codes ^= torch.randint(0, 256, (N, 8), generator=g, device=DEV, dtype=torch.int32) * 256
        flip = torch.rand((N, 8), generator=g, device=DEV) < 0.02
        codes = torch.where(flip, torch.randint(0, 65536, (N, 8), generator=g, device=DEV, dtype=torch.int32), codes)
    codes = codes.to(torch.int16).contiguous()
    at = codes[torch.randint(0, N, (Q,), generator=g, device=DEV)].long() & 0xFFFF
    y = torch.stack([cb[j][at[:, j]] for j in range(8)], 1).reshape(Q, -1)
    return cb, codes.view(torch.uint16), (y + 0.3 * torch.randn(y.shape, generator=g, device=DEV)).contiguous()


@pytest.mark.parametrize("kind,dsub,r,k,bbar", [
    ("mixture", 16, 2000, 100, 8),
    ("mixture", 5, 1, 1, 8),            # rows that are no whole 16 bytes; a single candidate
    ("mixture", 12, 1501, 100, 6),      # more codes to settle than the queue holds, derived codebooks of 64
    ("mixture", 16, 500, 10, 4),        # as many derived centroids as groups
    ("ties", 16, 1000, 100, 8),
    ("one_cell", 16, 1000, 100, 8),
])
def test_cells_against_the_scan_of_every_pair(kind, dsub, r, k, bbar):
    cb, codes, y = _inputs(kind, dsub, 11)
    derived = binding.derive_codebooks(cb, bbar)
    binding.profile_enable(True)
    ids, dist = binding.search(y, cb, derived, codes, r, k)
    torch.cuda.synchronize()
    stages = binding.profile_read()
    binding.profile_enable(False)
    assert stages["scan_cells"][1] > 0
    if kind == "mixture":               # sorted, and the single-pass scan had nothing to do (over a millisecond otherwise)
        assert stages["scan_fast"][0] < 0.3
    qtab, _, _ = binding.build_small_tables(y, derived, codes, r)
    cand, _ = binding.scan_candidates(codes, qtab, r)
    ids2, dist2 = binding.refine_direct_topk(y, cb, codes, cand, k)
    assert torch.equal(ids.view(torch.int32), ids2.view(torch.int32))
    assert torch.equal(dist, dist2)

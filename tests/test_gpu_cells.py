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


def _check(cb, derived, codes, y, r, k, chunk=0, graph=False):
    """A search that the cells have to serve, against the scan of every pair; returns the profiled stages."""
    Q, n = y.shape[0], codes.shape[0]
    b = 16 if codes.dtype == torch.uint16 else 8
    ws = torch.empty(binding.search_workspace_bytes(n, 8, Q, r, chunk, b), dtype=torch.uint8, device=DEV)
    ids = torch.empty((Q, k), dtype=torch.uint32, device=DEV)
    dist = torch.empty((Q, k), dtype=torch.float32, device=DEV)
    binding.profile_enable(True)
    binding.search(y, cb, derived, codes, r, k, chunk, ws, ids, dist)
    torch.cuda.synchronize()
    stages = binding.profile_read()
    binding.profile_enable(False)
    assert stages["scan_cells"][1] > 0
    assert stages["scan_fast"][0] < 0.3              # served: the single-pass scan had nothing to do
    qtab, _, _ = binding.build_small_tables(y, derived, codes, r)
    cand, _ = binding.scan_candidates(codes, qtab, r)
    if b == 8:                                       # as the search does
        ids2, dist2 = binding.refine_topk(binding.build_tables_n(y, cb), codes, cand, k)
    else:
        ids2, dist2 = binding.refine_direct_topk(y, cb, codes, cand, k)
    assert torch.equal(ids.view(torch.int32), ids2.view(torch.int32))
    assert torch.equal(dist, dist2)
    if graph:
        g, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
        with torch.cuda.stream(side):
            side.wait_stream(torch.cuda.default_stream())
            with torch.cuda.graph(g, stream=side):
                binding.search(y, cb, derived, codes, r, k, chunk, ws, ids, dist)
        for _ in range(3):
            ids.view(torch.int32).fill_(-1)
            dist.fill_(-1.0)
            ws.random_(0, 255)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(ids.view(torch.int32), ids2.view(torch.int32))
            assert torch.equal(dist, dist2)
    return stages


def _mixture(n, q, dsub, seed, b=16):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    parents = 3.0 * torch.randn((8, 16, dsub), generator=g, device=DEV)
    kc = 1 << b
    cb = parents.repeat(1, kc // 16, 1) + 0.3 * torch.randn((8, kc, dsub), generator=g, device=DEV)
    base = torch.randint(0, kc, (1000, 8), generator=g, device=DEV, dtype=torch.int32)
    codes = base[torch.randint(0, 1000, (n,), generator=g, device=DEV)]
    flip = torch.rand((n, 8), generator=g, device=DEV) < 0.02
    codes = torch.where(flip, torch.randint(0, kc, (n, 8), generator=g, device=DEV, dtype=torch.int32), codes)
    if b == 16:
        codes ^= torch.randint(0, 256, (n, 8), generator=g, device=DEV, dtype=torch.int32) * 256
    codes = codes.to(torch.int16 if b == 16 else torch.uint8).contiguous()
    at = codes[torch.randint(0, n, (q,), generator=g, device=DEV)].long() & (kc - 1)
    y = torch.cat([cb[j][at[:, j]] for j in range(8)], 1)
    return cb, codes.view(torch.uint16) if b == 16 else codes, (y + 0.3 * torch.randn(y.shape, generator=g, device=DEV)).contiguous()


@pytest.mark.parametrize("n,q,dsub,r,graph", [
    (8_400_001, 1000, 16, 2000, True),       # two workgroups to a query from the first launch on, counts in memory
    (16_800_013, 500, 4, 1000, False),       # four
])
def test_several_workgroups_to_a_query(n, q, dsub, r, graph):
    cb, codes, y = _mixture(n, q, dsub, 5)
    _check(cb, binding.derive_codebooks(cb), codes, y, r, 100, graph=graph)


def test_chunks_sort_the_codes_again():
    cb, codes, y = _mixture(4_194_307, 3951, 8, 6)           # a last chunk of 1950, which the cells serve too
    _check(cb, binding.derive_codebooks(cb), codes, y, 700, 50, chunk=2001)


@pytest.mark.parametrize("bbar", [4, 6])
def test_eight_bit_codes(bbar):
    cb, codes, y = _mixture(4_194_307, 9001, 8, 7, b=8)      # batches whose tables leave room for the sort
    _check(cb, binding.derive_codebooks(cb, bbar), codes, y, 300, 50)


def test_trained_quantizers():
    g = torch.Generator(device=DEV)
    g.manual_seed(8)
    means = 160.0 * torch.rand((1024, 128), generator=g, device=DEV)

    def draw(n):
        x = means[torch.randint(0, 1024, (n,), generator=g, device=DEV)]
        return (x + 12.0 * torch.randn(x.shape, generator=g, device=DEV)).clamp_(0, 255).round_()

    train = draw(131_072)
    init = torch.stack([train[torch.randperm(131_072, generator=g, device=DEV)[:65536], 16 * j:16 * j + 16] for j in range(8)]).contiguous()
    cb, derived = binding.build_quantizers(train, init, 8, 2, 1)
    codes = torch.cat([binding.encode(draw(1_050_000), cb).view(torch.int16) for _ in range(4)]).contiguous().view(torch.uint16)
    _check(cb, derived, codes, draw(2001), 500, 100)


@pytest.mark.parametrize("r", [100, 1000])
def test_ties_and_queries_that_the_cells_give_up(r):
    # codes with the low bytes of one place, 3 % of all: 126000 equal distances for the queries near it, more than may be looked at
    # (64 r and a 64th of the codes), or, for r = 1000, more than is wanted by far: of these only the first ids are candidates
    cb, codes, y = _mixture(4_194_307, 2001, 16, 9)
    g = torch.Generator(device=DEV)
    g.manual_seed(10)
    some = torch.rand((codes.shape[0],), generator=g, device=DEV) < 0.03
    place = codes.view(torch.int16)[12345] & 255
    high = torch.randint(-128, 128, (int(some.sum()), 8), generator=g, device=DEV, dtype=torch.int16) * 256
    codes.view(torch.int16)[some] = place[None] | high
    at = codes.view(torch.int16)[some][:40].long() & 0xFFFF
    near = torch.cat([cb[j][at[:, j]] for j in range(8)], 1)
    y[:40] = near + 0.05 * torch.randn(near.shape, generator=g, device=DEV)
    stages = _check(cb, binding.derive_codebooks(cb), codes, y, r, 50)
    if r == 100:
        assert stages["scan_collect"][0] > 0.02              # the three passes did the queries that were given up

"""Inverted lists: the forms that only some sizes or inputs take, against each other and against plain torch."""
import pytest
import torch

from paper_1905_06900_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(kind, m, dsub, n, nq, nlist, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    cb = 3.0 * torch.randn((m, 65536, dsub), generator=g, device=DEV)
    coarse = 10.0 * torch.randn((nlist, m * dsub), generator=g, device=DEV)
    codes = synth.random_codes(n, m, DEV, seed + 1).view(torch.int16)
    if kind == "ties":                       # three different codes: full slices, and ties by the thousand at the bound
        codes = codes[:3][torch.randint(0, 3, (n,), generator=g, device=DEV)].contiguous()
    offsets = synth.zipf_list_offsets(nlist, n, DEV, seed + 2)
    queries = coarse[torch.randint(0, nlist, (nq,), generator=g, device=DEV)] + torch.randn((nq, m * dsub), generator=g, device=DEV)
    return cb, coarse, codes.view(torch.uint16), offsets, queries.contiguous()


@pytest.mark.parametrize("kind,m,dsub,n,nq,nlist,nprobe,r,k", [
    ("random", 8, 16, 200_003, 1, 64, 9, 1000, 100),       # one query: a workgroup per sub-quantizer of its tables
    ("random", 4, 6, 50_021, 37, 64, 33, 777, 100),        # codes of 8 bytes; more lists than a wavefront's half
    ("random", 16, 3, 30_011, 300, 32, 5, 129, 129),       # rows that are no whole 16 bytes
    ("random", 8, 16, 3_001, 70, 64, 3, 2000, 60),         # fewer codes than r in the lists: every query is done again, and padded
    ("ties", 8, 4, 400_009, 45, 16, 7, 600, 50),           # quotas for ties
    ("random", 8, 8, 300_007, 5, 32, 8, 20_000, 100),      # keys beyond what is sorted in LDS
    ("random", 32, 2, 20_011, 70, 64, 3, 2000, 60),        # every query done again: long codes, ...
    ("random", 16, 2, 20_011, 600, 64, 3, 2000, 60),       # ... more of them than a pass has items, ...
    ("random", 4, 4, 30_011, 3, 64, 3, 9000, 60),          # ... keys beyond what is sorted in LDS
])
def test_search_equals_its_steps(kind, m, dsub, n, nq, nlist, nprobe, r, k):
    cb, coarse, codes, offsets, queries = _case(kind, m, dsub, n, nq, nlist, 77 + m)
    derived = binding.derive_codebooks(cb)
    ids, dist = binding.ivf_search(queries, coarse, cb, derived, codes, offsets, nprobe, r, k)
    probe = binding.ivf_probe(queries, coarse, nprobe)
    qtab, _ = binding.ivf_build_small_tables(queries, coarse, probe, derived, codes, offsets, r)
    cand, qd, count = binding.ivf_scan_candidates(codes, offsets, probe, qtab, r)
    ids2, dist2 = binding.ivf_refine_topk(queries, coarse, cb, codes, offsets, probe, cand, k)
    assert torch.equal(ids.view(torch.int32), ids2.view(torch.int32))
    assert torch.equal(dist, dist2)
    # the candidates: the r smallest (integer distance, id) of all probed codes
    low = (codes.view(torch.int16).to(torch.int64)) & 255
    for q in range(0, nq, max(1, nq // 9)):
        keys = []
        for p, l in enumerate(probe[q].tolist()):
            a, b = int(offsets[l]), int(offsets[l + 1])
            s = sum(qtab[q, p, j].long()[low[a:b, j]] for j in range(m)).clamp(max=255)
            keys.append(s << 32 | torch.arange(a, b, device=DEV))
        want = torch.cat(keys).sort().values[:r]
        assert int(count[q:q + 1].view(torch.int32)) == want.numel()
        got = (qd[q].long() << 32 | (cand[q].view(torch.int32).long() & 0xFFFFFFFF))[:want.numel()]
        assert torch.equal(got, want)


@pytest.mark.parametrize("nq,r,dsub", [
    (3, 128, 4), (3, 129, 3), (64, 256, 4), (65, 256, 4), (65, 257, 4),      # the sizes from which the keys are worked out on their own
    (65_535, 300, 4), (65_536, 300, 4), (70_001, 300, 3),                    # more queries than a grid takes along y
])
def test_refinement_with_and_without_room_for_the_keys(nq, r, dsub):
    m, nlist, nprobe, k = 4, 16, 2, 3
    cb, coarse, codes, offsets, queries = _case("random", m, dsub, 5_003, nq, nlist, 5)
    g = torch.Generator(device=DEV)
    g.manual_seed(nq)
    probe = torch.rand((nq, nlist), generator=g, device=DEV).argsort(1)[:, :nprobe].to(torch.int32).contiguous()
    cand = torch.randint(0, 5_003, (nq, r), generator=g, device=DEV, dtype=torch.int32)     # (those of other lists are padding)
    L, ptr = binding.lib(), lambda t: t.data_ptr()

    def refine(workspace_bytes):
        ids, dist = torch.zeros((nq, k), dtype=torch.int32, device=DEV), torch.zeros((nq, k), device=DEV)
        ws = torch.empty(max(workspace_bytes, 256), dtype=torch.uint8, device=DEV)
        assert L.dcpq_ivf_refine_topk(ptr(queries), ptr(coarse), nlist, ptr(cb), m, dsub, ptr(codes), ptr(offsets), ptr(probe), nprobe, ptr(cand),
                                      nq, r, k, ptr(ids), ptr(dist), ptr(ws), workspace_bytes, torch.cuda.current_stream().cuda_stream) == 0
        return ids, dist

    ids, dist = refine(8 * nq * r + 256 + L.dcpq_refine_workspace_bytes(nq, r))        # room for the keys
    ids1, dist1 = refine(L.dcpq_ivf_refine_workspace_bytes(nq, r))
    assert torch.equal(ids, ids1) and torch.equal(dist, dist1)

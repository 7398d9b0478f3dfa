"""Scans whose starting bounds come from a pilot pass, with few and with many equal distances at the bound: the candidates of the
three passes over all pairs."""
import pytest
import torch

from paper_1905_06900_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,N,Q,r,different", [
    (8, 2_000_003, 301, 2000, 0),        # just above the sample sizes that take a pilot pass
    (8, 2_000_003, 301, 2000, 300),      # 7000 codes at every distance
    (8, 2_000_003, 333, 1500, 3),        # two thirds of a million
    (16, 1_000_003, 203, 1000, 40),
    (4, 1_500_007, 1300, 3000, 50),
])
def test_candidates_with_ties(m, N, Q, r, different):
    g = torch.Generator(device=DEV)
    g.manual_seed(9 + m)
    codes = synth.random_codes(N, m, DEV, 3).view(torch.int16)
    if different:
        codes = codes[:different][torch.randint(0, different, (N,), generator=g, device=DEV)].contiguous()
    qtab = torch.randint(0, 40, (Q, m, 256), generator=g, device=DEV, dtype=torch.uint8)
    codes = codes.view(torch.uint16)
    ids, qd = binding.scan_candidates(codes, qtab, r)
    ids3, qd3 = binding.scan_candidates(codes, qtab, r, mode=binding.SCAN_THREE_PASS)
    assert torch.equal(ids.view(torch.int32), ids3.view(torch.int32))
    assert torch.equal(qd, qd3)


@pytest.mark.parametrize("m,N,Q,r,different,entries", [
    (8, 1_000_003, 306, 300, 30, 40),        # each of 30 codes is more than the pilot counts: left out of its bound
    (8, 1_000_003, 306, 300, 0, 2),          # crowded from the first buckets on
    (8, 1_000_003, 300, 500, 0, 1),          # all distances 0: nothing lies below the crowded bucket
    (8, 2_000_003, 301, 700, 5, 256),        # distances beyond the last bucket
    (16, 1_000_003, 230, 300, 20, 30),
])
def test_crowded_buckets_are_not_counted_by_the_pilot(m, N, Q, r, different, entries):
    assert binding.scan_plan(N, m, Q, r)["pilot_every"] == 16
    g = torch.Generator(device=DEV)
    g.manual_seed(19 + m + entries)
    codes = synth.random_codes(N, m, DEV, 4).view(torch.int16)
    if different:
        codes = codes[:different][torch.randint(0, different, (N,), generator=g, device=DEV)].contiguous()
    qtab = torch.randint(0, entries, (Q, m, 256), generator=g, device=DEV, dtype=torch.int16).to(torch.uint8)
    codes = codes.view(torch.uint16)
    ids, qd = binding.scan_candidates(codes, qtab, r)
    ids3, qd3 = binding.scan_candidates(codes, qtab, r, mode=binding.SCAN_THREE_PASS)
    assert torch.equal(ids.view(torch.int32), ids3.view(torch.int32))
    assert torch.equal(qd, qd3)

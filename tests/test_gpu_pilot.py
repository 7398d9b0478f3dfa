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

"""Nearest centroid of whole-number points (products with zero low parts left out), tiles and stages of several kinds side by
side, against double precision."""
import pytest
import torch

from paper_1905_06900_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("m,dsub,n,k", [
    (4, 16, 66_001, 1000),      # large tiles of points; a last stage that is not full
    (8, 16, 17_003, 700),       # tiles of 256
    (4, 8, 66_001, 600),
    (4, 32, 66_001, 513),
    (4, 19, 66_001, 600),       # rows that are no whole vectors
    (1, 16, 3_001, 1000),       # few points: the wavefronts split the centroids
])
def test_whole_points_and_centroids(m, dsub, n, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(5 + dsub)
    x = torch.randint(0, 256, (n, m * dsub), generator=g, device=DEV).float()
    x[2 * n // 3:] += 0.37                                           # tiles of other points ...
    x[n // 3:n // 3 + 3] += 300.0                                    # ... of whole numbers with more than eight digits ...
    x[n // 7, :] += 0.25                                         # ... and one among whole ones
    cb = torch.randint(0, 256, (m, k, dsub), generator=g, device=DEV).float()
    cb[:, 256:384] += 0.61                                       # whole centroids, others, and both in one stage
    cb[:, 500] -= 0.123
    cb[:, k - 3:] = cb[:, :3]                                    # equal distances: the smaller index
    labels = binding.assign(x, cb)
    for j in range(m):
        c = cb[j].double()
        for i in range(0, n, 8192):
            p = x[i:i + 8192, j * dsub:(j + 1) * dsub].double()
            d = torch.zeros((p.shape[0], k), dtype=torch.float64, device=DEV)
            for t in range(dsub):
                d += (p[:, t:t + 1] - c[None, :, t]) ** 2
            best = d.min(dim=1, keepdim=True).values
            # (sums of whole numbers are exact; of the others equal up to rounding)
            got = d.gather(1, labels[i:i + 8192, j:j + 1].long())
            assert torch.all(got <= best * (1 + 1e-14))
            first = (d == best).to(torch.uint8).argmax(dim=1)
            whole = (p == p.round()).all(dim=1) & (best[:, 0] == best[:, 0].round())
            assert torch.equal(labels[i:i + 8192, j].long()[whole], first[whole])

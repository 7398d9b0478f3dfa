"""The bound on what the nearest-centroid filter's split products lose (paper_1905_06900_amd/csrc/assign.hip), on the
CPU: every fp32 significand split into two bf16 numbers, and the products that are left out, against the constants of the
kernel's source."""
import os
import re

import numpy as np
import pytest
import torch

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1905_06900_amd", "csrc", "assign.hip")


def bf16(x):
    return torch.from_numpy(x).bfloat16().float().numpy()


@pytest.mark.parametrize("name,all_four", [("kSplit3", False), ("kSplit4", True)])
def test_the_filters_bound_covers_every_significand(name, all_four):
    # Every significand in one binade (the loss does not depend on the exponents), split as the kernel splits it: x = xh + xl + xe.
    x = ((np.arange(1 << 23, dtype=np.int64) + (1 << 23)) / float(1 << 23)).astype(np.float32)
    rest = x - bf16(x)
    xl = bf16(rest)
    low, err = np.abs(xl / x.astype(np.float64)), np.abs((rest.astype(np.float64) - xl) / x)
    # 2 <x, c> loses 2 (xl cl + xe c + x ce) and, with all four products, only the last two; each term is largest where its
    # factors are, and the numbers that make the sum large are among those with large parts
    weight = err + (0.0 if all_four else 2.0 ** -8) * low
    top = np.argsort(-weight)[:2000]
    lost = err[top][:, None] + err[top][None, :] + err[top][:, None] * err[top][None, :]
    if not all_four:
        lost = lost + low[top][:, None] * low[top][None, :]
    worst = 2.0 * lost.max()
    text = open(SOURCE).read()
    bound = float(re.search(name + r" = ([0-9.]+)f / 262144\.0f", text).group(1)) / 262144.0
    assert worst <= bound, "%s = %.4g, products lose up to %.4g" % (name, bound, worst)
    assert worst >= 0.95 * bound             # (and the bound is not looser than it has to be)

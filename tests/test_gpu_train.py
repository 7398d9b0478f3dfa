"""GPU parity tests of training and encoding (Sec. 3.2, Alg. 2) against the oracle: nearest-centroid
assignment and encoding, k-means, same-size k-means (balanced assignment in rounds), the final
codebook order, and all of Alg. 2 in one call."""
import numpy as np
import pytest
import torch

import oracle
from paper_1905_06900_amd import binding, synth
from parity import to_np

pytestmark = pytest.mark.gpu

DEV = "cuda"


def gen(seed):
    g = torch.Generator(device=DEV); g.manual_seed(seed)
    return g


def check_labels(labels, points, cb, ref_labels, tag):
    """Labels equal the oracle's wherever the oracle's best and second-best centroids are apart; where they
    are closer than 1e-9 relative (the two sides add their double-precision terms in different orders) the
    chosen centroid must be as near as the best."""
    labels = labels.astype(np.int64); ref_labels = ref_labels.astype(np.int64)
    diff = np.nonzero(labels != ref_labels)[0]
    assert len(diff) <= max(1, len(labels) // 1000), tag + ": %d labels differ" % len(diff)
    for i in diff:
        x = points[i].astype(np.float64)
        da = ((x - cb[labels[i]].astype(np.float64)) ** 2).sum()
        db = ((x - cb[ref_labels[i]].astype(np.float64)) ** 2).sum()
        assert abs(da - db) <= 1e-9 * max(db, 1e-300), tag + ": point %d got a farther centroid" % i


@pytest.mark.parametrize("n,m,dsub,ncent", [(1000, 2, 6, 1000), (333, 1, 13, 77), (4097, 4, 4, 256), (50, 1, 128, 300)])
def test_assign_against_the_oracle(n, m, dsub, ncent):
    print("assign n=%d m=%d dsub=%d ncent=%d" % (n, m, dsub, ncent), flush=True)
    g = gen(100 + n)
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    cb = torch.randn((m, ncent, dsub), generator=g, device=DEV)
    cb[:, 5] = cb[:, 3]                                          # a duplicate centroid: the smaller index must win
    pts[7, :dsub] = cb[0, 5]
    labels, dist = binding.assign(pts, cb, want_dist=True)
    torch.cuda.synchronize()
    labels, dist, p_np, c_np = to_np(labels), to_np(dist), to_np(pts), to_np(cb)
    assert labels[7, 0] == 3
    for j in range(m):
        ref, rd = oracle.assign(p_np[:, j * dsub:(j + 1) * dsub], c_np[j], want_dist=True)
        check_labels(labels[:, j], p_np[:, j * dsub:(j + 1) * dsub], c_np[j], ref, "sub-quantizer %d" % j)
        # (a point that IS a centroid: the expanded form ||x||^2 + ||c||^2 - 2<x, c> leaves a rounding residue of
        # the order of 1e-16 times the norms instead of an exact zero)
        np.testing.assert_allclose(dist[:, j], rd, rtol=1e-5, atol=1e-12 * float((p_np.astype(np.float64) ** 2).sum(1).max()))


@pytest.mark.parametrize("dsub", [1, 3, 5, 8, 10, 12, 16, 20, 24, 32, 40, 52, 60, 84, 100, 128])
@pytest.mark.parametrize("n,ncent", [(31, 1), (129, 33), (300, 129), (1027, 1000)])
def test_assign_at_the_edges_of_tiles_and_vector_lengths(dsub, n, ncent):
    # every length of the filter's matrix product, tiles of points and centroids that are not full, and (last point
    # and centroids) a large offset with small differences, where the filter's error bound exceeds the distances
    print("assign edges dsub=%d n=%d ncent=%d" % (dsub, n, ncent), flush=True)
    g = gen(17 * dsub + n)
    pts = torch.randn((n, dsub), generator=g, device=DEV)
    cb = torch.randn((1, ncent, dsub), generator=g, device=DEV)
    if ncent > 40:
        cb[0, 20:40] = 3000.0 + 1e-3 * torch.randn((20, dsub), generator=g, device=DEV)
        cb[0, 39] = cb[0, 21]                                   # equal centroids: the smaller index must win
        pts[-1] = 3000.0
        pts[0] = cb[0, 39]
    labels, dist = binding.assign(pts, cb, want_dist=True)
    labels2 = binding.assign(pts, cb)
    torch.cuda.synchronize()
    p_np, c_np = to_np(pts), to_np(cb)[0]
    ref, rd = oracle.assign(p_np, c_np, want_dist=True)
    check_labels(to_np(labels)[:, 0], p_np, c_np, ref, "dsub %d" % dsub)
    np.testing.assert_array_equal(to_np(labels), to_np(labels2))
    np.testing.assert_allclose(to_np(dist)[:, 0], rd, rtol=1e-5, atol=1e-12 * float((p_np.astype(np.float64) ** 2).sum(1).max()))


@pytest.mark.parametrize("dsub,ncent", [(1, 300), (3, 257), (4, 256), (5, 700), (16, 1000), (21, 255), (60, 300), (128, 513)])
@pytest.mark.parametrize("n", [9, 33, 300])
def test_assign_where_most_centroids_repeat(dsub, ncent, n):
    # the filter cannot tell repeated centroids apart, so nearly all points are compared with all centroids: numbers of
    # points and centroids around the tiles of that comparison, the smallest index of equal centroids, and points that
    # are not finite among the others
    print("assign repeats dsub=%d ncent=%d n=%d" % (dsub, ncent, n), flush=True)
    g = gen(31 * dsub + n)
    few = torch.randn((7, dsub), generator=g, device=DEV)
    cb = few[torch.randint(0, 7, (ncent,), generator=g, device=DEV)][None].contiguous()
    pts = few[torch.randint(0, 7, (n,), generator=g, device=DEV)] + 0.01 * torch.randn((n, dsub), generator=g, device=DEV)
    pts[3] = 0.0
    pts[5, dsub // 2] = float("nan")
    pts[7, 0] = float("inf")
    labels, dist = binding.assign(pts, cb, want_dist=True)
    torch.cuda.synchronize()
    labels, dist, p_np, c_np = to_np(labels)[:, 0], to_np(dist)[:, 0], to_np(pts), to_np(cb)[0]
    d2 = ((p_np[:, None].astype(np.float64) - c_np[None]) ** 2).sum(2)
    fine = np.isfinite(p_np).all(1)
    np.testing.assert_array_equal(labels[fine], d2[fine].argmin(1))         # (numpy: the first of equals)
    np.testing.assert_allclose(dist[fine], d2[fine].min(1), rtol=1e-6)
    assert labels[5] == -1 and labels[7] == 0 and np.isinf(dist[7])        # no distance at all; all distances infinite


@pytest.mark.parametrize("n,m,dsub", [(66_000, 8, 4), (140_000, 1, 16), (34_000, 16, 30)])
def test_assign_with_the_large_point_tiles(n, m, dsub):
    print("assign large tiles n=%d m=%d dsub=%d" % (n, m, dsub), flush=True)
    g = gen(n)
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    cb = torch.randn((m, 200, dsub), generator=g, device=DEV)
    labels = to_np(binding.assign(pts, cb))
    p64, c64 = pts.double().cpu(), cb.double().cpu()
    for j in range(m):
        x, c = p64[:, j * dsub:(j + 1) * dsub], c64[j]
        d = (x ** 2).sum(1, keepdim=True) + (c ** 2).sum(1)[None] - 2.0 * (x @ c.T)
        chosen = d.gather(1, torch.from_numpy(labels[:, j].astype(np.int64))[:, None])[:, 0]
        best = d.min(1).values
        assert bool((chosen <= best + 1e-12 * ((x ** 2).sum(1) + float((c ** 2).sum(1).max()))).all()), "sub-quantizer %d" % j


# The components at which a number and the sum of its two bf16 parts are as far apart, and the product of the two second
# parts as large, as they get: just below and just above the middle between two bf16 numbers.
SPLIT_BELOW = 1 + 2.0 ** -8 - 2.0 ** -16 + 2.0 ** -17 - 2.0 ** -23
SPLIT_ABOVE = 1 + 2.0 ** -8 + 2.0 ** -16 - 2.0 ** -17 + 2.0 ** -23


def worst_split_case(dsub, scale):
    """256 centroids, all zero but 1 and 129, and a point along centroid 1 that is nearest to it but whose split products
    favour 129.  scale 1: the point is centroid 1; above: their last components are 0 and just enough to make 129 the farther one."""
    c = np.zeros((256, dsub), np.float32)
    c[1], c[129] = SPLIT_BELOW, SPLIT_ABOVE
    if scale != 1:
        c[[1, 129], -1] = 0.0
    x = np.float32(scale) * c[1:2]
    d2 = lambda i: ((x[0].astype(np.float64) - c[i].astype(np.float64)) ** 2).sum()
    if scale != 1:
        c[129, -1] = np.sqrt(d2(1) - d2(129)) * (1 + 1e-4)
    assert 0.0 <= d2(1) < d2(129) < d2(0)
    return x, c


@pytest.mark.parametrize("dsub,scale", [(1, 1), (2, 1), (4, 1), (8, 1)] + [(d, s) for d in (12, 16, 20) for s in (4, 8, 16, 64)])
def test_assign_where_the_split_products_are_farthest_from_the_product(dsub, scale):
    print("assign worst split dsub=%d scale=%d" % (dsub, scale), flush=True)
    x, c = worst_split_case(dsub, scale)
    pts = torch.from_numpy(np.repeat(x, 40, 0)).to(DEV)
    labels, dist = binding.assign(pts, torch.from_numpy(c)[None].to(DEV), want_dist=True)
    codes = binding.encode(pts, torch.from_numpy(c)[None].to(DEV))
    torch.cuda.synchronize()
    ref, rd = oracle.assign(x, c, want_dist=True)
    assert ref[0] == 1
    np.testing.assert_array_equal(to_np(labels)[:, 0], 1)
    np.testing.assert_array_equal(to_np(codes)[:, 0], 1)
    np.testing.assert_allclose(to_np(dist)[:, 0], rd[0], rtol=1e-6, atol=1e-12)


@pytest.mark.parametrize("dsub", [1, 2, 3, 4, 7, 8, 9, 12, 16, 21, 31, 32, 33, 40, 60, 64, 100, 128])
@pytest.mark.parametrize("data", ["normal", "repeats", "some repeat", "offset", "lattice", "split"])
def test_assign_few_points_and_many_agree(dsub, data):
    # Few points against a small codebook take the products in double precision, many the bf16 filter (rows of 32 components
    # the latter both times, at these sizes): the same labels and the same bits of the distances, which are those of a comparison by
    # difference.  Equal and nearly equal centroids, points half-way between two, and values that are not finite.
    print("assign few and many dsub=%d %s" % (dsub, data), flush=True)
    g = gen(dsub + 1000 * len(data))
    n, ncent = 300, 300 if dsub < 32 else 600
    pts = torch.randn((n, dsub), generator=g, device=DEV)
    cb = torch.randn((ncent, dsub), generator=g, device=DEV)
    if data == "repeats":
        cb = cb[torch.randint(0, 7, (ncent,), generator=g, device=DEV)].contiguous()
        pts[5, dsub // 2], pts[7, 0] = float("nan"), float("inf")
    elif data == "some repeat":                                 # a few to a third of the points of a tile near equal centroids
        cb[1::2] = 20.0 + cb[torch.randint(0, 7, (ncent // 2,), generator=g, device=DEV) * 2]
        pts += 20.0 * (torch.rand((n, 1), generator=g, device=DEV) < torch.arange(n, device=DEV)[:, None] / (3.0 * n))
    elif data == "offset":
        cb = 3000.0 + 1e-3 * cb
        pts = 3000.0 + 1e-3 * pts
        cb[17, 0] = float("nan")
    elif data == "lattice":
        cb = torch.randint(-1, 2, (ncent, dsub), generator=g, device=DEV).float() * 0.1
        pts = torch.randint(-2, 3, (n, dsub), generator=g, device=DEV).float() * 0.05
    elif data == "split":
        x, c = worst_split_case(dsub, 1)
        cb = torch.zeros((ncent, dsub), device=DEV)
        cb[:256] = torch.from_numpy(c).to(DEV)
        pts = torch.from_numpy(np.repeat(x, n, 0)).to(DEV)
    times = 200
    few, few_dist = binding.assign(pts, cb[None], want_dist=True)
    few2 = binding.assign(pts, cb[None])
    many, many_dist = binding.assign(pts.repeat(times, 1), cb[None], want_dist=True)
    many2 = binding.assign(pts.repeat(times, 1), cb[None])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_np(few), to_np(few2))
    np.testing.assert_array_equal(to_np(many), to_np(few.repeat(times, 1)))
    np.testing.assert_array_equal(to_np(many2), to_np(few.repeat(times, 1)))
    np.testing.assert_array_equal(to_np(many_dist), to_np(few_dist.repeat(times, 1)))
    few, few_dist, p_np, c_np = to_np(few)[:, 0], to_np(few_dist)[:, 0], to_np(pts).astype(np.float64), to_np(cb).astype(np.float64)
    d2 = np.zeros((n, ncent))
    for t in range(dsub):
        d2 += (p_np[:, None, t] - c_np[None, :, t]) ** 2
    fine = np.isfinite(p_np).all(1)
    # (the kernels add with fused multiply-adds: (dsub + 1) roundings of 2^-53 on either side, twice)
    best = np.nanmin(d2[fine], 1)
    assert (d2[fine][np.arange(fine.sum()), few[fine]] <= best * (1 + 4 * (dsub + 1) * 2.0 ** -53)).all()
    np.testing.assert_allclose(few_dist[fine], best, rtol=2.0 ** -23)
    if data == "repeats":
        assert few[5] == -1 and few[7] == 0 and np.isinf(few_dist[7])


@pytest.mark.parametrize("b", [16, 8])
def test_encode_against_the_oracle(b):
    m, dsub, n = (4, 8, 3000) if b == 16 else (8, 4, 20000)
    print("encode b=%d m=%d dsub=%d n=%d" % (b, m, dsub, n), flush=True)
    cb = synth.hierarchical_codebooks(m, dsub, b, 4, lambda shape, gg: 3.0 * torch.randn(
        shape, generator=gg, device=DEV, dtype=torch.float32), 0.5, DEV, 4242 + b)
    g = gen(77 + b)
    codes_true = torch.randint(0, 1 << b, (n, m), generator=g, device=DEV)
    x = torch.cat([cb[j][codes_true[:, j]] for j in range(m)], dim=1) + 0.2 * torch.randn((n, m * dsub), generator=g, device=DEV)
    codes = binding.encode(x, cb)
    torch.cuda.synchronize()
    assert codes.dtype == (torch.uint16 if b == 16 else torch.uint8)
    codes, x_np, cb_np = to_np(codes), to_np(x), to_np(cb)
    ref = oracle.encode(x_np, cb_np)
    for j in range(m):
        check_labels(codes[:, j], x_np[:, j * dsub:(j + 1) * dsub], cb_np[j], ref[:, j], "sub-quantizer %d" % j)
    # decodable vectors come back as their own codes
    exact = torch.cat([cb[j][codes_true[:50, j]] for j in range(m)], dim=1).contiguous()
    back = to_np(binding.encode(exact, cb)).astype(np.int64)
    xe = to_np(exact)
    for j in range(m):
        check_labels(back[:, j], xe[:, j * dsub:(j + 1) * dsub], cb_np[j], to_np(codes_true[:50, j]), "decodable, %d" % j)


def test_kmeans_against_the_oracle():
    n, d, k = 20000, 8, 256
    print("kmeans n=%d d=%d k=%d" % (n, d, k), flush=True)
    g = gen(5)
    means = 4.0 * torch.randn((64, d), generator=g, device=DEV)
    x = means[torch.randint(0, 64, (n,), generator=g, device=DEV)] + torch.randn((n, d), generator=g, device=DEV)
    init = x[:k].clone()
    for iters in (0, 1, 4):
        cent, labels = binding.kmeans(x, init, iters)
        torch.cuda.synchronize()
        rc, rl = oracle.kmeans(to_np(x), to_np(init), iters)
        np.testing.assert_allclose(to_np(cent), rc, rtol=1e-5, atol=1e-6, err_msg="centroids after %d iterations" % iters)
        check_labels(to_np(labels), to_np(x), rc, rl, "labels after %d iterations" % iters)


def test_kmeans_centroid_without_members_keeps_its_value():
    x = torch.tensor([[0.0, 0.0], [1.0, 0.0], [2.0, 0.0], [3.0, 0.0]], device=DEV)
    init = torch.tensor([[1.0, 0.0], [100.0, 0.0]], device=DEV)
    cent, labels = binding.kmeans(x, init, 3)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_np(labels), [0, 0, 0, 0])
    np.testing.assert_array_equal(to_np(cent), np.array([[1.5, 0.0], [100.0, 0.0]], np.float32))


@pytest.mark.parametrize("n,d,kbar,iters", [(4096, 6, 16, 2), (1024, 3, 256, 1), (65536, 12, 256, 1)])
def test_same_size_kmeans_against_the_oracle(n, d, kbar, iters):
    print("same-size k-means n=%d d=%d kbar=%d iters=%d" % (n, d, kbar, iters), flush=True)
    g = gen(900 + kbar + n)
    means = 3.0 * torch.randn((40, d), generator=g, device=DEV)
    # lopsided on purpose: most points around a few of the means, so that many groups overflow
    pick = (torch.rand((n,), generator=g, device=DEV) ** 3 * 40).long().clamp(max=39)
    p = (means[pick] + 0.7 * torch.randn((n, d), generator=g, device=DEV)).contiguous()
    init = p[:kbar].clone()
    cent, labels = binding.kmeans_same_size(p, init, iters)
    torch.cuda.synchronize()
    labels, cent = to_np(labels), to_np(cent)
    np.testing.assert_array_equal(np.bincount(labels, minlength=kbar), np.full(kbar, n // kbar))
    rc, rl = oracle.kmeans_same_size(to_np(p), to_np(init), iters)
    np.testing.assert_array_equal(labels, rl.astype(np.int32))
    np.testing.assert_allclose(cent, rc, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n,kbar", [(6, 2), (63, 9), (64, 1), (65, 13), (130, 2), (1000, 250), (4290, 10)])
def test_same_size_kmeans_of_few_points_against_the_oracle(n, kbar):
    # numbers of points around the 64 that propose together, down to one group; most around a few places, so that groups turn points away
    print("same-size k-means of few, n=%d kbar=%d" % (n, kbar), flush=True)
    g = gen(31 * n + kbar)
    p = (4.0 * torch.randint(0, 3, (n, 3), generator=g, device=DEV) + torch.randn((n, 3), generator=g, device=DEV)).contiguous()
    cent, labels = binding.kmeans_same_size(p, p[:kbar].clone(), 1)
    torch.cuda.synchronize()
    rc, rl = oracle.kmeans_same_size(to_np(p), to_np(p[:kbar]), 1)
    np.testing.assert_array_equal(to_np(labels), rl.astype(np.int32))
    np.testing.assert_allclose(to_np(cent), rc, rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("n,kbar", [(4096, 64), (65536, 256), (65536, 16), (65536, 2)])
def test_same_size_kmeans_where_every_group_has_room_for_its_proposers(n, kbar):
    # groups of 64 to 32768 points apart from each other: every proposer is accepted at once, unsorted, by one to all wavefronts of
    # the group's workgroup
    print("same-size k-means, room for all, n=%d kbar=%d" % (n, kbar), flush=True)
    g = gen(n + kbar)
    of = (torch.arange(n, device=DEV) % kbar)[torch.randperm(n, generator=g, device=DEV)]
    p = (100.0 * of[:, None] + torch.rand((n, 3), generator=g, device=DEV)).contiguous()
    init = (100.0 * torch.arange(kbar, device=DEV)[:, None] + 0.5).expand(kbar, 3).contiguous()
    cent, labels = binding.kmeans_same_size(p, init, 8)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_np(labels), to_np(of))
    means = torch.stack([p.double()[of == l].mean(0) for l in range(kbar)])
    np.testing.assert_allclose(to_np(cent), to_np(means), rtol=2.0 ** -23)


def test_final_codebook_against_the_oracle():
    g = gen(31)
    for b, bbar, d in [(8, 3, 5), (16, 8, 12), (8, 8, 4)]:
        k, kbar = 1 << b, 1 << bbar
        labels = torch.arange(kbar, device=DEV, dtype=torch.int32).repeat_interleave(k // kbar)[torch.randperm(k, generator=g, device=DEV)].contiguous()
        temp = torch.randn((k, d), generator=g, device=DEV)
        final, perm = binding.build_final_codebook(temp, labels, bbar)
        torch.cuda.synchronize()
        rf, rp = oracle.build_final_codebook(to_np(temp), to_np(labels), bbar)
        np.testing.assert_array_equal(to_np(perm), rp.astype(np.int32))
        np.testing.assert_array_equal(to_np(final), rf)


def test_all_of_alg2_in_one_call_against_the_oracle_steps():
    m, dsub, b, bbar, n, iters, ss = 2, 4, 8, 4, 6000, 3, 2
    print("build_quantizers m=%d dsub=%d b=%d bbar=%d n=%d" % (m, dsub, b, bbar, n), flush=True)
    g = gen(64)
    means = 5.0 * torch.randn((300, m * dsub), generator=g, device=DEV)
    x = (means[torch.randint(0, 300, (n,), generator=g, device=DEV)] + torch.randn((n, m * dsub), generator=g, device=DEV)).contiguous()
    init = torch.stack([x[:1 << b, j * dsub:(j + 1) * dsub] for j in range(m)]).contiguous()
    cb, derived = binding.build_quantizers(x, init, bbar, iters, ss)
    torch.cuda.synchronize()
    x_np, init_np = to_np(x), to_np(init)
    for j in range(m):
        temp, _ = oracle.kmeans(np.ascontiguousarray(x_np[:, j * dsub:(j + 1) * dsub]), init_np[j], iters)
        cbar, lab = oracle.kmeans_same_size(temp, temp[:1 << bbar].copy(), ss)
        final, _ = oracle.build_final_codebook(temp, lab, bbar)
        np.testing.assert_allclose(to_np(cb)[j], final, rtol=1e-5, atol=1e-6, err_msg="final codebook %d" % j)
        np.testing.assert_allclose(to_np(derived)[j], cbar, rtol=1e-5, atol=1e-6, err_msg="derived codebook %d" % j)
    # the derived codebooks are those of the search path, and the search runs on the trained quantizer
    np.testing.assert_array_equal(to_np(derived), to_np(binding.derive_codebooks(cb, bbar)))
    codes = binding.encode(x, cb)
    ids, dist = binding.search(x[:16].contiguous(), cb, derived, codes, 200, 10)
    torch.cuda.synchronize()
    ref = oracle.search_flat(to_np(cb), to_np(derived), to_np(codes).astype(np.uint16), x_np[:16], 200, 10, b=b, bbar=bbar)
    np.testing.assert_allclose(to_np(dist), ref["dist"], rtol=1e-5, atol=1e-6)


def test_training_argument_errors():
    p = torch.zeros((100, 4), device=DEV)
    with pytest.raises(binding.DcpqError):
        binding.kmeans_same_size(p, p[:8].clone(), 1)            # 100 is not a multiple of 8
    with pytest.raises(binding.DcpqError):
        binding.build_quantizers(p, torch.zeros((1, 4096, 4), device=DEV), 8, 1, 1)     # b = 12


@pytest.mark.parametrize("dsub,m", [(5, 4), (8, 8), (12, 8), (16, 8), (21, 8), (32, 8), (40, 8), (52, 8), (60, 8), (64, 8)])
@pytest.mark.parametrize("data", ["normal", "bytes", "near", "repeats", "offset", "outlier"])
def test_assign_of_many_points_agrees_with_few(dsub, m, data):
    # From 2^18 sub-vectors on (2^17 above 32 components) the filter has one fp16 product; few points take other kernels: the same labels and bits of
    # the distances.  "near": points whose window holds many centroids of many cells (the second walk), "repeats" and "offset": too
    # many for that, values that are not finite; "outlier": a centroid and a point far outside the range of fp16.  Point and centroid
    # counts that no tile divides.
    print("assign many points dsub=%d m=%d %s" % (dsub, m, data), flush=True)
    g = gen(dsub + 1000 * len(data))
    n, ncent = 517, 1337
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    cb = torch.randn((m, ncent, dsub), generator=g, device=DEV)
    if data == "bytes":
        pts = (40 * pts + 120).clamp(0, 255).round()
        cb = (40 * cb + 120).clamp(0, 255).round()
        cb[:, 3:n + 3] = pts.view(n, m, dsub).transpose(0, 1)
    elif data == "near":                                         # 40 centroids all over the codebook within 1e-4 of one of them
        cb[:, 7::33] = 3.0 + cb[:, 7:8] + 1e-4 * torch.randn(cb[:, 7::33].shape, generator=g, device=DEV)
        pts.view(n, m, dsub)[::61] = 3.0 + cb[:, 7][None] + 1e-3 * torch.randn((len(range(0, n, 61)), m, dsub), generator=g, device=DEV)
    elif data == "repeats":
        cb = cb[:, torch.randint(0, 7, (ncent,), generator=g, device=DEV)].contiguous()
        pts[5, dsub // 2], pts[7, 0] = float("nan"), float("inf")
    elif data == "offset":
        cb, pts = 3000.0 + 1e-3 * cb, 3000.0 + 1e-3 * pts
        cb[0, 17, 0] = float("nan")
    elif data == "outlier":
        cb[0, 77] *= 1e6
        pts[3] *= 1e5
    times = ((1 << 18) // m + n) // n + 1 + (300 if data == "normal" else 0)
    few, few_dist = binding.assign(pts, cb, want_dist=True)
    many, many_dist = binding.assign(pts.repeat(times, 1), cb, want_dist=True)
    many2 = binding.assign(pts.repeat(times, 1), cb)
    torch.cuda.synchronize()
    for got in (many, many2):
        np.testing.assert_array_equal(to_np(got), to_np(few.repeat(times, 1)))
    np.testing.assert_array_equal(to_np(many_dist), to_np(few_dist.repeat(times, 1)))
    p64, c64 = pts.double().view(n, m, dsub).cpu(), cb.double().cpu()
    fine = torch.isfinite(p64).all(2).all(1).numpy()
    for j in range(m):
        d2 = ((p64[:, j, None, :] - c64[j][None]) ** 2).sum(2).numpy()[fine]
        best = np.nanmin(d2, 1)
        chosen = d2[np.arange(fine.sum()), to_np(few)[fine, j]]
        assert (chosen <= best * (1 + 4 * (dsub + 1) * 2.0 ** -53)).all(), "sub-quantizer %d" % j


def crowded_codebooks(m, b, dsub, bbar, crowded, seed):
    """Starting centroids; of the sub-quantizers `crowded` 2^bbar groups lie in a row and all other centroids before the first of them, so that a
    round of the balanced assignment fills one group and as many rounds as groups are needed."""
    g = gen(seed)
    init = torch.randint(-300, 300, (m, 1 << b, dsub), generator=g, device=DEV).float() / 64.0        # (sums of these are exact)
    for j in crowded:
        init[j] = 0.0
        init[j, :, 1] = torch.arange(1 << b, device=DEV) / (4.0 * (1 << b))
        init[j, :1 << bbar, 0] = torch.arange(1, (1 << bbar) + 1, device=DEV).float()
    return init, torch.randn((300, m * dsub), generator=g, device=DEV)


@pytest.mark.parametrize("m,dsub,b,bbar,iters_same,crowded", [
    (4, 4, 8, 4, 1, (0, 2)), (4, 4, 8, 4, 2, (0, 2)), (4, 4, 8, 4, 3, (0, 1, 2, 3)),
    (8, 3, 8, 5, 2, (7,)),                                       # 300 training points: labels of several codebooks in the place of theirs
    (32, 2, 8, 4, 2, (0, 13, 31)), (2, 40, 8, 8, 1, (1,)),
    (4, 1, 16, 4, 2, ()), (4, 8, 16, 4, 2, (1, 3)),              # 65536 centroids: a batch of two or more, one with a copy outside the lists
    (2, 40, 16, 4, 2, (0,)), (8, 2, 16, 1, 1, ()),               # lists of proposers too short for a codebook's copy
])
def test_training_where_a_balanced_assignment_takes_more_rounds_than_it_is_given(m, dsub, b, bbar, iters_same, crowded):
    # Twelve rounds are enqueued ahead; the same codebooks as step by step, where every assignment is waited for.
    init, x = crowded_codebooks(m, b, dsub, bbar, crowded, 71)
    cb, derived = binding.build_quantizers(x, init, bbar, 0, iters_same)
    torch.cuda.synchronize()
    for j in range(m):
        _, labels = binding.kmeans_same_size(init[j].contiguous(), init[j, :1 << bbar].contiguous(), iters_same)
        final, _ = binding.build_final_codebook(init[j].contiguous(), labels, bbar)
        np.testing.assert_array_equal(to_np(cb)[j], to_np(final), err_msg="sub-quantizer %d" % j)
        if b == 8:
            lab, _ = oracle.kmeans_same_size(to_np(init[j]), to_np(init[j, :1 << bbar]), iters_same)[::-1]
            np.testing.assert_array_equal(to_np(labels), lab)
    np.testing.assert_array_equal(to_np(derived), to_np(binding.derive_codebooks(cb, bbar)))


def test_training_repeats_no_rounds_of_a_balanced_assignment():
    # Crowded starting centroids: what is enqueued ahead counts, and an assignment that takes more goes on from there.  Fewer launches than step
    # by step, plus what an assignment that is taken up again costs: a distance table, the rooms, and at most as many rounds too many as are enqueued at a time (two launches each).
    m, b, dsub, bbar, iters = 8, 8, 4, 4, 5
    init, x = crowded_codebooks(m, b, dsub, bbar, range(m), 72)
    counts = []
    for whole in (True, False):
        binding.profile_enable(True)
        try:
            if whole:
                binding.build_quantizers(x, init, bbar, 0, iters)
            else:
                for j in range(m):
                    _, labels = binding.kmeans_same_size(init[j].contiguous(), init[j, :1 << bbar].contiguous(), iters)
                    binding.build_final_codebook(init[j].contiguous(), labels, bbar)
            torch.cuda.synchronize()
            counts.append(binding.profile_read()["train"][1])
        finally:
            binding.profile_enable(False)
    assert counts[0] <= counts[1] + m * iters * (2 + 2 * 4)


def check_many_points_against_few(pts, cb, times, tag):
    """Labels and distances of `pts` are those that the same points have `times` over, where their number takes another kernel; and the nearest
    in double precision."""
    n, m, dsub = pts.shape[0], cb.shape[0], cb.shape[2]
    few, few_dist = binding.assign(pts, cb, want_dist=True)
    many, many_dist = binding.assign(pts.repeat(times, 1), cb, want_dist=True)
    many2 = binding.assign(pts.repeat(times, 1), cb)
    assert torch.equal(many, few.repeat(times, 1)) and torch.equal(many2, many), tag
    np.testing.assert_array_equal(to_np(many_dist), to_np(few_dist.repeat(times, 1)), err_msg=tag)
    for j in range(m):
        x, c = pts[:, j * dsub:(j + 1) * dsub].double(), cb[j].double()
        for i in range(0, n, 64):
            d2 = torch.zeros((x[i:i + 64].shape[0], c.shape[0]), dtype=torch.float64, device=DEV)
            for t in range(dsub):
                d2 += (x[i:i + 64, t:t + 1] - c[None, :, t]) ** 2
            d2 = torch.where(d2.isnan(), float("inf"), d2)
            chosen = d2.gather(1, few[i:i + 64, j:j + 1].long())[:, 0]
            assert bool((chosen <= d2.min(1).values * (1 + 4 * (dsub + 1) * 2.0 ** -53)).all()), "%s, sub-quantizer %d" % (tag, j)


@pytest.mark.parametrize("ncent", [65535, 65536, 65537])
@pytest.mark.parametrize("dsub,m", [(8, 4), (12, 4), (16, 4), (20, 4), (23, 4), (32, 4), (40, 4), (64, 4)])
@pytest.mark.parametrize("data", ["normal", "bytes", "near"])
def test_assign_of_many_points_to_the_largest_codebooks(dsub, m, ncent, data):
    # 65536 centroids are as many cells as their numbers have room for in the filter with one fp16 product; one more takes the split products, in the
    # large tiles of points up to 32 components.  Nearest centroids in the first and last cells, and ("near") windows that hold
    # centroids of many cells up to the last (the second walk); "bytes": whole numbers, whose second bf16 parts are zero, and equal distances.
    print("assign to %d centroids dsub=%d m=%d %s" % (ncent, dsub, m, data), flush=True)
    g = gen(dsub + ncent)
    n = 517
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    cb = torch.randn((m, ncent, dsub), generator=g, device=DEV)
    if data == "bytes":
        pts = (40 * pts + 120).clamp(0, 255).round()
        cb = (40 * cb + 120).clamp(0, 255).round()
        cb[:, -9:] = cb[:, :9]
    per_point = pts.view(n, m, dsub)
    places = torch.tensor([0, 31, 127, 128, 32767, 32768, 65407, 65408, 65500, ncent - 65, ncent - 2, ncent - 1], device=DEV)
    step = 0.0 if data == "bytes" else 1e-2
    near = cb[:, places].transpose(0, 1).repeat(20, 1, 1)
    per_point[:near.shape[0]] = near + step * torch.randn(near.shape, generator=g, device=DEV)
    if data == "near":                                           # 50 centroids all over the codebook, the last among them, within 1e-4 of one of them
        at = torch.cat([torch.arange(7, ncent - 1, 1337, device=DEV), torch.tensor([ncent - 1], device=DEV)])
        cb[:, at] = 3.0 + cb[:, 7:8] + 1e-4 * torch.randn((m, at.numel(), dsub), generator=g, device=DEV)
        per_point[::61] = cb[:, ncent - 1][None] + 1e-4 * torch.randn((len(range(0, n, 61)), m, dsub), generator=g, device=DEV)
    # (tiles of 512 points; of 1024 with up to 16 components where the data is "normal")
    check_many_points_against_few(pts, cb, (1 << 19) // (m * n) if dsub <= 16 and data == "normal" else (1 << 18) // (m * n) + 1, "%d centroids" % ncent)


@pytest.mark.parametrize("dsub,m", [(7, 8), (8, 8), (16, 8), (30, 8), (64, 8)])
@pytest.mark.parametrize("which", ["point", "points", "all points", "centroid", "centroids", "both", "not finite"])
def test_assign_of_many_points_where_some_lie_far_out(dsub, m, which):
    # The scale of the fp16 filter follows 64 centroids.  What it makes infinite: points (one or two of a workgroup, more, all), and centroids, which are ruled out by
    # their length, but not for points as far out.
    print("assign far out dsub=%d m=%d %s" % (dsub, m, which), flush=True)
    g = gen(dsub + 7)
    n, ncent = 2003, 1500
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    cb = torch.randn((m, ncent, dsub), generator=g, device=DEV)
    if which in ("point", "both"):
        pts[1001] *= 1e6
        pts[77] *= 3e3
    elif which == "points":
        pts[100::50] *= 10.0 ** torch.linspace(2, 12, len(range(100, n, 50)), device=DEV)[:, None]
    elif which == "all points":
        pts *= 1e6
    if which in ("centroid", "both"):
        cb[:, 1497] *= 1e5
    if which in ("centroids", "both"):
        cb[:, 5::100] *= 1e4
        cb[0, 1400:] = 1e7
        pts[5::64] = cb[:, 1305].reshape(1, m * dsub) + 1e3       # (nearest to a centroid far out)
        pts[6::64] = cb[:, 1305].reshape(1, m * dsub) / 2          # (about as far from it as from the others)
    if which == "not finite":
        cb[:, 9], cb[:, 11] = float("nan"), float("inf")
        cb[:, 1499] = -float("inf")
    check_many_points_against_few(pts, cb, (1 << 18) // (m * n) + 1, which)


def test_assign_beside_centroids_and_points_far_out_takes_as_long():
    # A centroid far out left the filter without windows: 35 times as long (the split products cannot tell centroids apart beside it either).
    n, m, dsub, ncent = 65536, 8, 16, 16384
    g = gen(3)
    pts, cb = torch.randn((n, m * dsub), generator=g, device=DEV), torch.randn((m, ncent, dsub), generator=g, device=DEV)
    far_points, far_centroid = pts.clone(), cb.clone()
    far_points[::2000] *= 1e9
    far_centroid[:, 77] *= 1e6
    ms = []
    for x, c in ((pts, cb), (far_points, cb), (pts, far_centroid)):
        times = []
        for _ in range(6):
            binding.profile_enable(True)
            try:
                binding.assign(x, c)
                torch.cuda.synchronize()
                times.append(binding.profile_read()["train"][0])
            finally:
                binding.profile_enable(False)
        ms.append(min(times))
    print("assign, ms: %.3f, points far out %.3f, a centroid %.3f" % tuple(ms), flush=True)
    assert ms[1] < 2 * ms[0] and ms[2] < 2 * ms[0]


@pytest.mark.parametrize("dsub,m", [(7, 8), (8, 8), (16, 8), (30, 8), (60, 8)])
@pytest.mark.parametrize("members,every", [(16, 1), (16, 3), (16, 11), (31, 2), (40, 2), (300, 1)])
def test_assign_of_many_points_whose_windows_hold_many_centroids(dsub, m, members, every):
    # Clusters of centroids closer together than the filter with one fp16 product can tell, spread over the codebook, and every so many points beside one: they are walked again, 128 at a
    # time, the last 32 or fewer apart, or, where they find more centroids than are listed (about 32 each), go through the split products.  A fifth of a
    # cluster's centroids are equal: the first of them.
    print("assign crowded dsub=%d m=%d members=%d every=%d" % (dsub, m, members, every), flush=True)
    g = gen(dsub + members)
    n, ncent = 2003, 6000
    cluster = torch.arange(ncent, device=DEV) % (ncent // members)
    means = torch.randn((m, ncent // members, dsub), generator=g, device=DEV)
    cb = means[:, cluster] + 2e-3 * torch.randn((m, ncent, dsub), generator=g, device=DEV)
    cb[:, ::5] = means[:, cluster[::5]]
    pts = torch.randn((n, m * dsub), generator=g, device=DEV)
    beside = pts.view(n, m, dsub)[::every]
    beside[:] = means[:, torch.arange(beside.shape[0], device=DEV) % means.shape[1]].transpose(0, 1) + 1e-3 * torch.randn(beside.shape, generator=g, device=DEV)
    check_many_points_against_few(pts, cb, (1 << 18) // (m * n) + 1, "%d members" % members)


def test_assign_to_clusters_of_centroids_is_not_much_slower():
    # 4096 clusters of 16: with every open point left to the split products 5.4 times as long as without clusters; walked again 3.1.
    n, m, dsub, ncent = 70000, 8, 16, 65536
    g = gen(4)
    pts, cb = torch.randn((n, m * dsub), generator=g, device=DEV), torch.randn((m, ncent, dsub), generator=g, device=DEV)
    means = torch.randn((m, 4096, dsub), generator=g, device=DEV)
    clusters = means[:, torch.randint(0, 4096, (ncent,), generator=g, device=DEV)] + 0.03 * torch.randn((m, ncent, dsub), generator=g, device=DEV)
    pick = torch.randint(0, ncent, (n, m), generator=g, device=DEV)
    beside = clusters[torch.arange(m, device=DEV)[None], pick] + 0.03 * torch.randn((n, m, dsub), generator=g, device=DEV)
    ms = []
    for x, c in ((pts, cb), (beside.reshape(n, m * dsub), clusters)):
        times = []
        for _ in range(6):
            binding.profile_enable(True)
            try:
                binding.assign(x, c)
                torch.cuda.synchronize()
                times.append(binding.profile_read()["train"][0])
            finally:
                binding.profile_enable(False)
        ms.append(min(times))
    print("assign, ms: %.3f, clusters %.3f" % tuple(ms), flush=True)
    assert ms[1] < 4.2 * ms[0]

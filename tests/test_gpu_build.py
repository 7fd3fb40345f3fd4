"""Index building on the GPU (dictionaries, leaf centers, encoding, layout) against the oracle, at the sizes where the
kernels' tiles and variants meet their edges."""
import time

import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# points around a workgroup's 256 and a tile's 64, exactly as many points as codewords; every specialised number of
# dimensions per subspace and others; sums too large for one workgroup's LDS (256 codewords of 96 dimensions)
@pytest.mark.parametrize("n,d,M,bits", [(16, 2, 1, 4), (257, 6, 6, 4), (255, 6, 3, 4), (1025, 105, 35, 4), (700, 20, 5, 4),
                                        (513, 35, 7, 4), (256, 10, 5, 8), (1000, 12, 3, 8), (2049, 24, 3, 8), (600, 36, 4, 8),
                                        (900, 96, 1, 8), (70_001, 4, 2, 4)])
@pytest.mark.parametrize("residual", [False, True])
def test_dictionaries_of_all_subspaces_match(n, d, M, bits, residual):
    rng = np.random.default_rng(n + d)
    x = unit_rows(rng, n, d)
    okw = {}
    leaves = 3 if residual else 0
    idx = avq.Index(d, M, bits, kmeans_iters=3, seed=5, n_leaves=leaves, leaf_kmeans_iters=2)
    idx.train(dev(x))
    if residual:
        okw = dict(leaf_centers=idx.get_leaf_centers())
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
    want = oracle.train_pq(x, M, 1 << bits, 3, 5, **okw)
    # fp64 means in another order, rounded to fp32: one unit in the last place of values below 1
    np.testing.assert_allclose(idx.get_codebooks(), want, rtol=0, atol=1.2e-7)


# exact ties, values whose squares leave fp32, distances small against the norms, a point repeated until codewords are equal
def hard_points(rng, n, d, law):
    x, scale = unit_rows(rng, n, d), 1.0
    if law == "lattice":
        x = np.round(x * 4).astype(np.float32)
        scale = 4.0
    elif law in ("tiny", "huge"):
        scale = 1e-22 if law == "tiny" else 1e20
        x = (x * np.float32(scale)).astype(np.float32)
    elif law == "far":
        x = (100.0 + 0.01 * x).astype(np.float32)
        scale = 100.0
    elif law == "equal":
        x[: n * 3 // 4] = x[0]
    return x, scale


def check_dictionaries(n, d, M, bits, law, iters):
    x, scale = hard_points(np.random.default_rng(d + M + bits), n, d, law)
    idx = avq.Index(d, M, bits, kmeans_iters=iters, seed=5)
    idx.train(dev(x))
    # fp64 means in another order, rounded to fp32: one unit in the last place of the largest values
    np.testing.assert_allclose(idx.get_codebooks(), oracle.train_pq(x, M, 1 << bits, iters, 5), rtol=0, atol=1.2e-7 * scale)


@pytest.mark.parametrize("d,M,bits", [(3, 3, 4), (6, 3, 4), (6, 2, 4), (8, 2, 4), (4, 2, 8), (8, 2, 8), (16, 2, 8)])
@pytest.mark.parametrize("law", ["lattice", "tiny", "huge", "far", "equal"])
def test_dictionaries_of_hard_points(d, M, bits, law):
    check_dictionaries(1111, d, M, bits, law, 3)


# The fp32 search of every specialised size against fp64 distances, at two steps a workgroup, from which on there is one: it decides
# most points ("unit"), or little, and is left out from the second iteration on.
@pytest.mark.parametrize("d,M,bits", [(64, 64, 4), (128, 64, 4), (192, 64, 4), (256, 64, 4), (128, 64, 8), (256, 64, 8), (512, 64, 8)])
@pytest.mark.parametrize("law", ["unit", "lattice", "tiny", "huge", "far", "equal"])
def test_dictionaries_of_hard_points_in_several_steps(d, M, bits, law):
    check_dictionaries(9001, d, M, bits, law, 3 if bits == 4 else 2)


def train_seconds(x, M, bits):
    idx = avq.Index(x.shape[1], M, bits, kmeans_iters=10)
    best = float("inf")
    for _ in range(5):
        t = time.perf_counter()
        idx.train(x)
        best = min(best, time.perf_counter() - t)
    return best


# Copies of a row, which fp32 cannot tell apart, against unit vectors: 1.4 and 1.8 times as long with the fp32 search left out, 2.0 and
# 2.8 times with both searches. A few points: all in fp64 0.53 of the time of four times as many, 0.74 with both.
def test_training_time_where_fp32_decides_little():
    x = dev(unit_rows(np.random.default_rng(1), 262_144, 100))
    same = x[:1].repeat(len(x), 1).contiguous()
    assert train_seconds(same, 50, 4) < 1.7 * train_seconds(x, 50, 4)
    assert train_seconds(same, 25, 8) < 2.3 * train_seconds(x, 25, 8)
    assert train_seconds(x[:5000], 25, 8) < 0.64 * train_seconds(x[:20_000], 25, 8)


def leaf_index(d, centers, **kw):
    idx = avq.Index(d, 1, 4, n_leaves=centers.shape[0], **kw)
    idx.set_leaf_centers(centers)
    idx.set_codebooks(np.zeros((1, 16, d), np.float32))
    return idx


# steps of 16 coordinates of the matrix-core kernel (with three for the bias: 13 | 14, 29 | 30, 109 | 110, ...), tiles of
# 32 centers, workgroups of 128 and 256 points; 270 dimensions take the kernel without matrix cores
@pytest.mark.parametrize("n,d,k", [(1, 2, 1), (129, 13, 31), (255, 14, 32), (256, 29, 33), (257, 30, 64), (1000, 64, 65),
                                   (3000, 100, 200), (511, 109, 40), (512, 110, 40), (513, 128, 97), (300, 141, 33),
                                   (640, 192, 50), (700, 205, 129), (385, 256, 300), (260, 269, 31), (260, 270, 31),
                                   # (up to 16,384 points and 1,024 = centers x dimensions take the kernel without matrix cores too)
                                   (1, 2, 600), (129, 13, 90), (255, 14, 80), (256, 29, 40), (300, 32, 32), (300, 32, 33),
                                   (16_384, 8, 16), (16_385, 8, 16)])
@pytest.mark.parametrize("law", ["unit", "far", "lattice", "twins", "scales"])
def test_nearest_leaf_is_that_of_fp64_distances(n, d, k, law):
    rng = np.random.default_rng(n * 7 + d)
    x, c = unit_rows(rng, n, d), unit_rows(rng, k, d)
    if law == "far":            # distances small against the norms: the f16 product leaves every point open
        off = 50.0 * unit_rows(rng, 1, d)
        x, c = (off + 0.1 * x).astype(np.float32), (off + 0.1 * c).astype(np.float32)
    elif law == "lattice":      # many exact ties: the lowest index wins
        x, c = np.round(x * 3).astype(np.float32), np.round(c * 3).astype(np.float32)
    elif law == "twins":        # equal centers, and centers that differ in the last bit
        c[k // 2:] = c[: k - k // 2]
        c[-1] = np.nextafter(c[-1], 2.0)
    elif law == "scales":       # tiny and huge coordinates, points far outside the centers, zero rows
        c *= np.float32(3e-3)
        x *= (10.0 ** rng.uniform(-6, 4, (n, 1))).astype(np.float32)
        x[0] = 0.0
    idx = leaf_index(d, c)
    idx.encode(dev(x))
    np.testing.assert_array_equal(idx.get_leaf_assign(), oracle.assign_nearest(x, c))


# twins a given number of centers apart: in one group of four values (1, 2), in the other half-wave's rows (4), in another group
# (8), in the next tile (32), with a point on each; one and two column tiles per wave, an odd and an even number of tiles
@pytest.mark.parametrize("d", [12, 30, 100, 140, 150, 268])
@pytest.mark.parametrize("k", [96, 128])
@pytest.mark.parametrize("apart", [1, 2, 4, 8, 32])
def test_twin_centers_anywhere_in_a_tile(d, k, apart):
    rng = np.random.default_rng(d * 131 + k + apart)
    c = unit_rows(rng, k, d)
    half = (np.arange(k) // apart) % 2 == 1
    c[half] = c[np.flatnonzero(half) - apart]
    c[half, 0] = np.nextafter(c[half, 0], np.float32(2.0))
    x = np.concatenate([c, unit_rows(rng, 900, d)])
    idx = leaf_index(d, c)
    idx.encode(dev(x))
    np.testing.assert_array_equal(idx.get_leaf_assign(), oracle.assign_nearest(x, c))


# The same with points enough for the kernel of many points and centers (n x tiles of 32 centers above 2^18; the line itself).
@pytest.mark.parametrize("d,k", [(12, 96), (30, 128), (60, 96), (100, 128), (140, 96), (150, 96), (268, 96)])
@pytest.mark.parametrize("apart", [1, 2, 4, 8, 32])
def test_twin_centers_among_many_points(d, k, apart):
    rng = np.random.default_rng(d * 131 + k + apart)
    c = unit_rows(rng, k, d)
    half = (np.arange(k) // apart) % 2 == 1
    c[half] = c[np.flatnonzero(half) - apart]
    c[half, 0] = np.nextafter(c[half, 0], np.float32(2.0))
    few = np.concatenate([c, unit_rows(rng, 900, d)])
    want = oracle.assign_nearest(few, c)
    for n in ((1 << 18) // ((k + 31) // 32), (1 << 18) // ((k + 31) // 32) + 1, 100_000):
        idx = leaf_index(d, c)
        idx.encode(dev(np.resize(few, (n, d))))
        np.testing.assert_array_equal(idx.get_leaf_assign(), np.resize(want, n))


@pytest.mark.parametrize("n,d,k", [(64, 5, 64), (3001, 100, 70), (2000, 36, 300), (1500, 270, 9)])
def test_leaf_centers_match(n, d, k):
    rng = np.random.default_rng(3)
    x = unit_rows(rng, n, d)
    idx = avq.Index(d, 1, 4, n_leaves=k, leaf_kmeans_iters=4, kmeans_iters=0, seed=8)
    idx.train(dev(x))
    # fp64 means in another order, rounded to fp32: one unit in the last place of values below 1
    np.testing.assert_allclose(idx.get_leaf_centers(), oracle.kmeans(x, k, 4, seed=8), rtol=0, atol=1.2e-7)


# leaves of 0, 1, 255, 256, 257 points and one with most of them; fewer and more points than a chunk of 1,024; code sizes
# with and without left-over planes; what a search of every leaf returns depends on every place
@pytest.mark.parametrize("n,d,M,bits,leaves", [(1, 8, 4, 4, 3), (1500, 8, 4, 4, 7), (5000, 10, 5, 8, 2), (2049, 12, 6, 4, 1300)])
def test_points_are_grouped_by_leaf(n, d, M, bits, leaves):
    rng = np.random.default_rng(17)
    x, q = unit_rows(rng, n, d), unit_rows(rng, 3, d)
    cb = oracle.train_pq(np.tile(x, (256 // n + 1, 1)) if n < 256 else x, M, 1 << bits, 1, 3)
    codes = rng.integers(0, 1 << bits, (n, M)).astype(np.uint8)
    centers = unit_rows(rng, leaves, d)
    assign = rng.integers(0, leaves, n).astype(np.int32)
    if n >= 1500 and leaves >= 7:
        assign[:] = 6
        assign[rng.permutation(n)[:769]] = np.repeat([1, 2, 3, 4], [1, 255, 256, 257])
    idx = avq.Index(d, M, bits, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(centers)
    idx.set_database(dev(x), oracle.pack_codes(codes, bits), assign)
    L = min(leaves, 512)
    k = min(n, 60)
    ids, sc = idx.search(dev(q), k, min(n, 100), 0, leaves_to_search=L)
    oi, os_ = oracle.search(x, cb, codes, bits, q, k, min(n, 100), 0, centers=centers, assign=assign, leaves_to_search=L)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)
    assign[n // 2] = leaves
    with pytest.raises(avq.AvqError, match="leaf assignment %d of point %d" % (leaves, n // 2)):
        idx.set_database(dev(x), oracle.pack_codes(codes, bits), assign)


# every specialised number of dimensions per subspace and one without; waves of 64 points that hold 1, 63, 64, 65 points;
# rows of x in LDS copied 64 coordinates at a time, for four, two waves and one of a compute unit (128, 192, 400 dimensions),
# and rows that do not fit it (512 and 1,024: the plain kernel); more points than all resident waves have lanes (262,144), so
# that lanes take further points as theirs finish, in passes of their own
@pytest.mark.parametrize("n,d,M,bits", [(1, 4, 4, 4), (63, 6, 3, 4), (64, 30, 6, 4), (65, 100, 50, 4), (700, 105, 35, 4),
                                        (333, 100, 25, 4), (129, 24, 3, 8), (257, 20, 5, 8), (300, 12, 6, 8), (200, 512, 256, 4),
                                        (70, 1024, 256, 4), (40_000, 8, 4, 4), (130, 128, 64, 4),
                                        (100, 192, 96, 4), (90, 400, 200, 4), (400_000, 16, 8, 4), (300_000, 6, 3, 8),
                                        # (few subspaces take the kernel all in fp64: more of 1, 2 and 4 dimensions; the lines)
                                        (70, 12, 12, 4), (63, 30, 15, 4), (65, 40, 10, 4), (64, 4, 4, 4), (64, 5, 5, 4),
                                        (64, 14, 7, 4), (64, 16, 8, 4), (64, 6, 2, 4), (64, 9, 3, 4), (64, 20, 5, 4),
                                        (64, 24, 6, 4), (64, 4, 2, 8), (64, 8, 2, 8), (64, 8, 4, 8), (64, 12, 3, 8)])
@pytest.mark.parametrize("law", ["unit", "scales", "huge", "tiny", "eta_exact", "eta_explicit", "lattice", "one_pass", "no_pass", "leaves"])
def test_codes_are_those_of_fp64_losses(n, d, M, bits, law):
    if n > 1000 and law not in ("unit", "leaves"):
        pytest.skip("many points: the common law only")
    if law == "leaves" and d > 512:
        pytest.skip("leaf assignment refuses this dimension")
    rng = np.random.default_rng(n + 31 * d)
    x = unit_rows(rng, n, d)
    cb = unit_rows(rng, (1 << bits) * M, d // M).reshape(M, 1 << bits, d // M) * np.float32((M + 0.0) ** -0.5)
    kw, okw = dict(T=0.2, encode_passes=6), dict(T=0.2, passes=6)
    if law == "scales":         # norms from 1e-4 to 1e4 of the codewords' scale
        x *= (10.0 ** rng.uniform(-4, 4, (n, 1))).astype(np.float32)
        x[0] = 0.0
    elif law in ("huge", "tiny"):  # single-precision squares run over, or vanish
        s = np.float32(1e25 if law == "huge" else 1e-25)
        x, cb = x * s, cb * s
        kw["T"] = okw["T"] = float(np.float32(0.2) * s)
    elif law == "eta_exact":
        if n * d > 4000:
            pytest.skip("an integral per point on the CPU")
        kw["eta_mode"], okw["eta_mode"] = avq.ETA_EXACT, 1
    elif law == "eta_explicit":
        kw.update(eta_mode=avq.ETA_EXPLICIT, eta_explicit=37.0)
        okw.update(eta_mode=2, eta_explicit=37.0)
    elif law == "lattice":      # exact ties between the nearest codewords (later passes: ties that rounding breaks)
        x, cb = np.round(x * 4).astype(np.float32), np.round(cb * 8).astype(np.float32)
        kw["encode_passes"] = okw["passes"] = 0
    elif law == "one_pass":
        kw["encode_passes"] = okw["passes"] = 1
    elif law == "no_pass":
        kw["encode_passes"] = okw["passes"] = 0
    if law == "leaves":
        centers = unit_rows(rng, 5, d)
        assign = oracle.assign_nearest(x, centers)
        okw.update(leaf_centers=centers, leaf_assign=assign)
        idx = avq.Index(d, M, bits, n_leaves=5, **kw)
        idx.set_leaf_centers(centers)
    else:
        idx = avq.Index(d, M, bits, **kw)
    idx.set_codebooks(cb)
    idx.encode(dev(x))
    want = oracle.pack_codes(oracle.encode(x, cb, **okw), bits)
    np.testing.assert_array_equal(idx.get_codes(), want)


def random_dictionaries(rng, M, kc, ds):
    return (unit_rows(rng, kc * M, ds).reshape(M, kc, ds) * np.float32(M ** -0.5)).astype(np.float32)


# shapes that the search in fp32 does not take: 16 codewords of 8 dimensions, rows of which LDS does not hold 64 (2 and 4
# dimensions per subspace); workgroups of 128 points
@pytest.mark.parametrize("n,d,M", [(127, 8, 1), (129, 64, 8), (300, 128, 16), (130, 448, 224), (128, 512, 128)])
@pytest.mark.parametrize("leaves", [0, 5])
def test_codes_of_shapes_without_fp32_search(n, d, M, leaves):
    rng = np.random.default_rng(n + d)
    x, cb = unit_rows(rng, n, d), random_dictionaries(rng, M, 16, d // M)
    idx = avq.Index(d, M, 4, T=0.2, encode_passes=6, n_leaves=leaves)
    okw = {}
    if leaves:
        okw["leaf_centers"] = unit_rows(rng, leaves, d)
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
        idx.set_leaf_centers(okw["leaf_centers"])
    idx.set_codebooks(cb)
    idx.encode(dev(x))
    np.testing.assert_array_equal(idx.get_codes(), oracle.pack_codes(oracle.encode(x, cb, T=0.2, passes=6, **okw), 4))


@pytest.mark.parametrize("n,d,M,bits", [(1, 6, 3, 8), (31, 12, 6, 8), (33, 24, 6, 8), (65, 64, 8, 8), (40, 264, 132, 8),
                                        (40, 512, 256, 8), (1, 10, 10, 4), (63, 27, 9, 4), (65, 52, 13, 4), (40, 510, 255, 4)])
@pytest.mark.parametrize("leaves", [0, 3])
def test_codes_at_the_edges_of_a_wave(n, d, M, bits, leaves):
    """Windows of points that are not full, subspaces that are no multiple of four, dictionaries beyond LDS."""
    rng = np.random.default_rng([n, d, M, leaves])
    x = unit_rows(rng, n, d)
    cb = (rng.standard_normal((M, 1 << bits, d // M)) / np.sqrt(d)).astype(np.float32)
    idx = avq.Index(d, M, bits, T=0.2, encode_passes=5, n_leaves=leaves)
    okw = {}
    if leaves:
        cen = unit_rows(rng, leaves, d)
        idx.set_leaf_centers(dev(cen))
        okw = dict(leaf_centers=cen, leaf_assign=oracle.assign_nearest(x, cen))
    idx.set_codebooks(dev(cb))
    idx.encode(dev(x))
    np.testing.assert_array_equal(idx.get_codes(), oracle.pack_codes(oracle.encode(x, cb, T=0.2, passes=5, **okw), bits))


def encode_seconds(n, d, M, bits=4, codewords=None):
    """The fastest of five calls."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(d + M)
    x = torch.nn.functional.normalize(torch.randn((n, d), generator=gen, device="cuda"))
    cb = x[: 1 << bits].reshape(1 << bits, M, d // M).transpose(0, 1).contiguous()
    if codewords is not None:
        cb = codewords(cb).contiguous()
    idx = avq.Index(d, M, bits, T=0.2)
    idx.set_codebooks(cb)
    best = float("inf")
    for _ in range(6):
        t = time.perf_counter()
        idx.encode(x)
        best = min(best, time.perf_counter() - t)
    return best


# A shape without the fp32 search against one with it: 1.4, 4.0 and 3.6 times as long; with nothing known about the
# dimensions per subspace at compile time 11.9, 23.5 and 13.3 times.
@pytest.mark.parametrize("shape,other,most", [((128, 16), (128, 32), 4), ((512, 128), (256, 64), 10), ((512, 256), (256, 128), 7)])
def test_encode_time_of_shapes_without_fp32_search(shape, other, most):
    assert encode_seconds(200_000, *shape) < most * encode_seconds(200_000, *other)


# Equal codewords in every dictionary: fp64 decides at every step, the lower index wins; 16 codewords from registers, 256
# several at a time, the first and last pass and leaf centers
@pytest.mark.parametrize("n,d,M,bits", [(130, 5, 5, 4), (700, 36, 18, 4), (300, 105, 35, 4), (260, 64, 16, 4), (130, 10, 5, 8),
                                        (129, 24, 6, 8), (128, 40, 5, 8)])
@pytest.mark.parametrize("leaves,passes", [(0, 6), (5, 6), (0, 0), (0, 1)])
def test_codes_with_equal_codewords(n, d, M, bits, leaves, passes):
    rng = np.random.default_rng(n + d)
    x, cb = unit_rows(rng, n, d), random_dictionaries(rng, M, 1 << bits, d // M)
    cb[:, 1 << (bits - 1):] = cb[:, : 1 << (bits - 1)]
    idx = avq.Index(d, M, bits, T=0.2, encode_passes=passes, n_leaves=leaves)
    okw = {}
    if leaves:
        okw["leaf_centers"] = unit_rows(rng, leaves, d)
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
        idx.set_leaf_centers(okw["leaf_centers"])
    idx.set_codebooks(cb)
    idx.encode(dev(x))
    want = oracle.encode(x, cb, T=0.2, passes=passes, **okw)
    assert want.max() < 1 << (bits - 1)
    np.testing.assert_array_equal(idx.get_codes(), oracle.pack_codes(want, bits))


# Runs of equal codewords: all of a dictionary, the first five, neighbours, a dictionary and coordinates of zeros of either sign
@pytest.mark.parametrize("d,M,bits", [(12, 12, 4), (36, 18, 4), (45, 15, 4), (64, 16, 4), (24, 6, 8)])
@pytest.mark.parametrize("law", ["all", "five", "neighbours", "zeros"])
@pytest.mark.parametrize("leaves,passes", [(0, 6), (5, 6), (0, 0)])
def test_codes_with_runs_of_equal_codewords(d, M, bits, law, leaves, passes):
    rng = np.random.default_rng(d)
    n, ds = 260, d // M
    x, cb = unit_rows(rng, n, d), random_dictionaries(rng, M, 1 << bits, ds)
    if law == "all":
        cb[::2] = cb[::2, :1]
    elif law == "five":
        cb[:, 3:8] = cb[:, 3:4]
    elif law == "neighbours":
        cb[:, 1::2] = cb[:, ::2]
    else:
        cb[1::3] = 0.0
        cb[1::3, 1::2] = -0.0
        x.reshape(n, M, ds)[:, 1::3] = 0.0
    idx = avq.Index(d, M, bits, T=0.2, encode_passes=passes, n_leaves=leaves)
    okw = {}
    if leaves:
        okw["leaf_centers"] = unit_rows(rng, leaves, d)
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
        idx.set_leaf_centers(okw["leaf_centers"])
    idx.set_codebooks(cb)
    idx.encode(dev(x))
    np.testing.assert_array_equal(idx.get_codes(), oracle.pack_codes(oracle.encode(x, cb, T=0.2, passes=passes, **okw), bits))


# Every step open: 1.7 times as long as with codewords that differ (2.7 times with one codeword loaded at a time)
def test_encode_time_with_equal_codewords():
    def twins(cb):
        return torch.cat([cb[:, :8], cb[:, :8]], dim=1)
    assert encode_seconds(200_000, 100, 50, codewords=twins) < 2.2 * encode_seconds(200_000, 100, 50)


def device_bytes_taken(call):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    call()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0]


# 1,300,000 x 64 points by coordinate are 333 MB of scratch, which go back at the end of the training
def test_training_gives_its_scratch_back():
    x = torch.randn((1_300_000, 64), device="cuda")
    idx = avq.Index(64, 32, 4, kmeans_iters=1)
    assert device_bytes_taken(lambda: idx.train(x)) < 64 << 20


# Leaves of more points than one launch assigns (three launches, the last one short). What stays is bounded: 9,000,000 points
# take 36 MB each of leaves and places and 18 MB of codes, 84 MB of lists of undecided points for a launch (180 for all).
def test_leaves_of_more_points_than_a_launch_assigns():
    rng = np.random.default_rng(4)
    n, d, k = 9_000_000, 4, 3
    x = torch.randn((n, d), device="cuda")
    c = unit_rows(rng, k, d)
    idx = avq.Index(d, 1, 4, n_leaves=k, encode_passes=0)
    idx.set_leaf_centers(c)
    idx.set_codebooks(np.zeros((1, 16, d), np.float32))
    assert device_bytes_taken(lambda: idx.encode(x)) < 230 << 20
    np.testing.assert_array_equal(idx.get_leaf_assign(), oracle.assign_nearest(x.cpu().numpy(), c))


# Less scratch than the fast kernels ask for: ten subspaces take 183 KB (340 with leaves) at once, five 91 (170), two 36 (68),
# one 18 (34); leaf centers, leaves and codes by the kernels that need none
@pytest.mark.parametrize("limit_kb", [900, 100, 40])
@pytest.mark.parametrize("leaves,eta", [(0, "limit"), (7, "limit"), (0, "exact")])
def test_building_within_limited_scratch(limit_kb, leaves, eta):
    rng = np.random.default_rng(6)
    n, d, M = 2000, 20, 10
    x = unit_rows(rng, n, d)
    kw = dict(eta_mode=avq.ETA_EXACT) if eta == "exact" else {}
    idx = avq.Index(d, M, 4, T=0.2, encode_passes=4, kmeans_iters=3, seed=5, n_leaves=leaves, leaf_kmeans_iters=2, **kw)
    idx.set_tuning("scratch_limit_kb", limit_kb)
    idx.train(dev(x))
    okw = {}
    if leaves:
        okw["leaf_centers"] = idx.get_leaf_centers()
        # fp64 means in another order, rounded to fp32: one unit in the last place of values below 1
        np.testing.assert_allclose(okw["leaf_centers"], oracle.kmeans(x[: 256 * leaves], leaves, 2, seed=5), rtol=0, atol=1.2e-7)
        okw["leaf_assign"] = oracle.assign_nearest(x, okw["leaf_centers"])
    cb = idx.get_codebooks()
    np.testing.assert_allclose(cb, oracle.train_pq(x, M, 16, 3, 5, **okw), rtol=0, atol=1.2e-7)
    m = 120 if eta == "exact" else n # (an integral per point on the CPU)
    idx.set_tuning("scratch_limit_kb", 4)
    idx.encode(dev(x[:m]))
    if leaves:
        np.testing.assert_array_equal(idx.get_leaf_assign(), okw["leaf_assign"])
    want = oracle.encode(x[:m], cb, T=0.2, passes=4, **(dict(eta_mode=1) if eta == "exact" else {}), **okw)
    np.testing.assert_array_equal(idx.get_codes(), oracle.pack_codes(want, 4))


# A dimension whose leaves cannot be assigned (l2, anisotropic): the call is refused and the installed database stays
@pytest.mark.parametrize("d,aniso", [(640, 0), (320, 1)])
def test_refused_encode_leaves_the_database(d, aniso):
    rng = np.random.default_rng(2)
    n, M, leaves = 700, d // 4, 3
    x, q, centers = unit_rows(rng, n, d), unit_rows(rng, 2, d), unit_rows(rng, leaves, d)
    codes = rng.integers(0, 16, (n, M)).astype(np.uint8)
    idx = avq.Index(d, M, 4, n_leaves=leaves, leaf_aniso_iters=aniso)
    idx.set_codebooks(random_dictionaries(rng, M, 16, 4))
    idx.set_leaf_centers(centers)
    idx.set_database(dev(x), oracle.pack_codes(codes, 4), rng.integers(0, leaves, n).astype(np.int32))
    before = [t.cpu().numpy() for t in idx.search(dev(q), 10, 50, 0, leaves_to_search=2)]
    with pytest.raises(avq.AvqError, match="too large"):
        idx.encode(dev(x))
    assert idx.n == n
    for b, a in zip(before, idx.search(dev(q), 10, 50, 0, leaves_to_search=2)):
        np.testing.assert_array_equal(a.cpu().numpy(), b)


# 1,000,000 points of 2 subspaces: 92 us (251 where the waves of the fp32 search hand them out one by one), against 580 for 50
# subspaces of a fifth of the points
def test_encode_time_of_few_subspaces():
    assert encode_seconds(1_000_000, 4, 2) < 0.3 * encode_seconds(200_000, 100, 50)

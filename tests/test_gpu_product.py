"""Batches through the product of the queries with the decoded points, against the oracle: where tiles of 32 queries, groups of
32 to 512 points, steps of 16 dimensions, kinds of subspaces and code rows meet their edges; queries that the product decides
nothing for; the rule that picks this path."""
import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def index(x, cb, codes, bits):
    idx = avq.Index(x.shape[1], codes.shape[1], bits)
    idx.set_codebooks(cb)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(oracle.pack_codes(codes, bits)).cuda())
    return idx


def check(x, cb, codes, bits, q, k, R, unverified=0):
    idx = index(x, cb, codes, bits)
    idx.set_tuning("scan_product", 2)
    qd = torch.from_numpy(q).cuda()
    for mode in (avq.LUT_F32, avq.LUT_U8):
        oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, mode)
        for prefilter in (0, 2):  # 2: every odd query goes to the plain scan
            idx.set_tuning("scan_prefilter", prefilter)
            ids, sc = idx.search(qd, k, R, mode)
            np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="tables %d prefilter %d" % (mode, prefilter))
            np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="tables %d prefilter %d" % (mode, prefilter))
            if prefilter == 2:
                assert idx.debug_unverified_queries() >= len(q) // 2
            elif unverified is not None:
                assert idx.debug_unverified_queries() == unverified


def draw(n, d, M, bits, nq, seed=0):
    rng = np.random.default_rng(n + 7 * d + M + nq + seed)
    kc = 1 << bits
    cb = (rng.standard_normal((M, kc, d // M)) * 0.2).astype(np.float32)
    return unit_rows(rng, n, d), cb, rng.integers(0, kc, (n, M)).astype(np.uint8), unit_rows(rng, nq, d)


# one point more than results; the edges of 32 points, of a block, of a workgroup's points; one query, the edges of a tile, of
# a stage of two tiles and of 128; every kind of subspace (1, 2, 3, 4, 5, 8, 12, 16, 24 dimensions) and number of steps, codes
# that do not fit the decoder's buffer; rows of 1 to 128 bytes
@pytest.mark.parametrize("n,d,M,bits,nq,k,R", [
    (11, 32, 16, 4, 1, 10, 0), (31, 32, 16, 4, 31, 1, 3), (33, 16, 8, 4, 32, 5, 20), (255, 48, 16, 4, 33, 10, 100),
    (257, 64, 32, 4, 63, 10, 100), (511, 80, 20, 8, 64, 10, 100), (513, 96, 12, 4, 65, 10, 50), (1025, 100, 50, 4, 127, 10, 100),
    (2049, 105, 35, 4, 129, 10, 100), (5000, 100, 25, 8, 40, 10, 200), (4097, 128, 64, 4, 96, 100, 512), (3000, 144, 6, 4, 20, 10, 100),
    (3001, 160, 10, 8, 20, 10, 100), (2500, 192, 96, 4, 70, 10, 100), (1500, 224, 224, 4, 18, 10, 60), (1300, 256, 32, 8, 17, 10, 100),
    (1400, 256, 256, 4, 33, 10, 100), (1100, 60, 60, 8, 16, 10, 100), (1200, 6, 3, 4, 50, 10, 100), (1000, 2, 1, 4, 20, 3, 10),
    (900, 25, 5, 4, 20, 10, 64), (901, 36, 9, 8, 20, 10, 64), (1800, 128, 128, 4, 20, 10, 100), (700, 15, 15, 8, 20, 10, 0),
    (40_000, 32, 16, 4, 300, 10, 100), (70_001, 64, 32, 4, 40, 10, 100), (60_000, 100, 25, 8, 33, 10, 10)])
def test_product_matches(n, d, M, bits, nq, k, R):
    # few code values against many results: ties, and more than the refinement holds, are in these draws too
    check(*draw(n, d, M, bits, nq)[:3], bits, draw(n, d, M, bits, nq)[3], k, R, None)


# The guess holds, and what it lets through fits, for data without many equal sums.
@pytest.mark.parametrize("n,d,M,bits,nq", [(30_000, 100, 50, 4, 200), (30_000, 100, 25, 8, 200), (260_000, 64, 32, 4, 64),
                                           (20_000, 160, 20, 8, 100), (20_000, 192, 96, 4, 70), (12_000, 256, 64, 4, 50)])
def test_product_answers_all(n, d, M, bits, nq):
    x, cb, codes, q = draw(n, d, M, bits, nq)
    check(x, cb, codes, bits, q, 10, 100, 0)


# Queries of zeros and copies of one point (every product the same: the plain scan answers, ties to the lower id), negative
# scores throughout, values of all magnitudes, a dictionary without a range for its 8-bit tables.
def test_product_odd_values():
    x, cb, codes, q = draw(6000, 32, 16, 4, 40)
    q[3] = 0.0
    check(x, cb, codes, 4, q, 10, 100, None)
    check(x, cb, np.repeat(codes[:1], 6000, 0), 4, q, 10, 100, None)
    check(x, cb, codes[np.random.default_rng(0).integers(0, 3, 6000)], 4, q, 10, 50, None)
    check(np.abs(x), -np.abs(cb), codes, 4, np.abs(q), 10, 100, None)
    q2 = q * np.logspace(-20, 17, 40)[:, None].astype(np.float32)
    check(x, cb, codes, 4, q2.astype(np.float32), 10, 100, None)
    check(x, (cb * 1e-20).astype(np.float32), codes, 4, q, 10, 100, None)
    check(x, (cb * 1e15).astype(np.float32), codes, 4, q, 10, 100, None)
    check(x, np.repeat(cb[:, :1], 16, 1).copy(), codes, 4, q, 10, 100, None)


# Which batches take this path: profile stage "sample" counts the sampling launch, "rescan" is one of its launches too, and
# the path over 8-bit tables or over block bounds records "merge" or "final" instead.
@pytest.mark.parametrize("n,d,M,bits,nq,k,R,mode,product", [
    (100_000, 32, 16, 4, 15, 10, 100, 0, False), (100_000, 32, 16, 4, 1000, 10, 100, 0, True), (16_000, 32, 16, 4, 2047, 10, 100, 0, False),
    (16_000, 32, 16, 4, 2048, 10, 100, 0, True), (16_000, 32, 16, 4, 2048, 10, 200, 0, False), (16_000, 32, 16, 4, 2048, 10, 20, 1, False),
    (40_000, 32, 16, 4, 1000, 10, 100, 1, False), (40_000, 32, 16, 4, 1000, 10, 10, 1, True), (20_000, 36, 9, 8, 16, 10, 100, 0, True),
    (20_000, 36, 9, 8, 15, 10, 100, 0, False), (4000, 100, 25, 8, 64, 10, 100, 0, False), (4000, 100, 25, 8, 1000, 10, 100, 1, True),
    (20_000, 64, 32, 4, 100, 10, 100, 1, True), (3000, 260, 130, 4, 500, 10, 100, 0, False)])
def test_rule_of_product(n, d, M, bits, nq, k, R, mode, product):
    x, cb, codes, q = draw(n, d, M, bits, nq)
    idx = index(x, cb, codes, bits)
    idx.profile_enable()
    qd = torch.from_numpy(q).cuda()
    ids, sc = idx.search(qd, k, R, mode)
    stages = idx.profile_read()
    assert (stages["sample"][1] > 0 and stages["finalize"][1] == 0) == product
    idx.set_tuning("scan_product", 1)
    ids1, sc1 = idx.search(qd, k, R, mode)
    assert torch.equal(ids, ids1) and torch.equal(sc, sc1)


# More queries than one part of a call takes, and a call that is captured and replayed with other queries in the same place.
def test_product_parts_and_capture():
    x, cb, codes, q = draw(20_000, 32, 16, 4, 20_000)
    idx = index(x, cb, codes, 4)
    qd = torch.from_numpy(q).cuda()
    idx.set_tuning("scan_product", 2)
    ids, sc = idx.search(qd, 10, 50, avq.LUT_F32)
    for lo in (0, 9_990, 19_900):
        a, b = idx.search(qd[lo:lo + 100], 10, 50, avq.LUT_F32)
        assert torch.equal(ids[lo:lo + 100], a) and torch.equal(sc[lo:lo + 100], b)
    buf = qd[:500].clone()
    out = (torch.empty((500, 10), dtype=torch.int32, device="cuda"), torch.empty((500, 10), device="cuda"))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        idx.search(buf, 10, 50, avq.LUT_F32, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        idx.search(buf, 10, 50, avq.LUT_F32, out=out)
    for lo in (500, 3000, 700):
        buf.copy_(qd[lo:lo + 500])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[0], ids[lo:lo + 500]) and torch.equal(out[1], sc[lo:lo + 500])


# ---- partitioned indexes ----------------------------------------------------------------

def draw_leaves(n, d, M, bits, nq, leaves, seed=0, skew=False):
    rng = np.random.default_rng(n + 7 * d + M + nq + seed)
    x, cb, codes, q = draw(n, d, M, bits, nq)
    centers = (0.5 * unit_rows(rng, leaves, d)).astype(np.float32)
    assign = rng.integers(0, leaves, n) if not skew else np.minimum(rng.geometric(0.3, n) - 1, leaves - 2)  # one leaf stays empty
    return x, cb, codes, q, centers, assign.astype(np.int32)


def leaf_index(x, cb, codes, bits, centers, assign):
    idx = avq.Index(x.shape[1], codes.shape[1], bits, n_leaves=len(centers))
    idx.set_codebooks(cb)
    idx.set_leaf_centers(centers)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(oracle.pack_codes(codes, bits)).cuda(), torch.from_numpy(assign).cuda())
    return idx


def check_leaves(x, cb, codes, bits, q, centers, assign, k, R, L, unverified=None):
    idx = leaf_index(x, cb, codes, bits, centers, assign)
    idx.set_tuning("scan_product", 2)
    qd = torch.from_numpy(q).cuda()
    for mode in (avq.LUT_F32, avq.LUT_U8):
        oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, mode, centers=centers, assign=assign, leaves_to_search=L)
        for prefilter in (0, 2):  # 2: every odd query goes to the plain scan
            idx.set_tuning("scan_prefilter", prefilter)
            ids, sc = idx.search(qd, k, R, mode, L)
            np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="tables %d prefilter %d" % (mode, prefilter))
            np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="tables %d prefilter %d" % (mode, prefilter))
            if prefilter == 2:
                assert idx.debug_unverified_queries() >= len(q) // 2
            elif unverified is not None:
                assert idx.debug_unverified_queries() == unverified


# a leaf's last block nearly empty or full, several blocks that share classes, leaves without points; fewer points than results;
# classes of 64, 16 and 4 points; one query, the edges of a tile and of the 512 queries that a workgroup takes; steps of 16
# dimensions in waves of two and of four; every kind of subspace
@pytest.mark.parametrize("n,d,M,bits,nq,leaves,L,k,R,skew", [
    (500, 32, 16, 4, 1, 20, 3, 10, 100, False), (3000, 100, 50, 4, 33, 11, 5, 10, 100, False), (5120, 64, 32, 4, 64, 20, 20, 10, 20, False),
    (9000, 32, 16, 4, 40, 6, 4, 10, 50, True), (4000, 100, 25, 8, 31, 8, 8, 10, 100, False), (6000, 105, 35, 4, 32, 12, 6, 100, 0, False),
    (2500, 192, 96, 4, 20, 5, 3, 10, 100, True), (2000, 256, 32, 8, 18, 7, 2, 10, 64, False), (3000, 160, 10, 8, 20, 9, 9, 10, 500, False),
    (20_000, 32, 16, 4, 515, 5, 2, 10, 10, True), (1500, 128, 128, 4, 20, 10, 4, 10, 0, False), (30_000, 36, 9, 8, 50, 40, 10, 10, 100, False),
    (700, 48, 16, 4, 20, 300, 40, 10, 100, False), (4000, 224, 28, 4, 20, 3, 2, 10, 300, False)])
def test_product_leaves_match(n, d, M, bits, nq, leaves, L, k, R, skew):
    check_leaves(*reorder_args(draw_leaves(n, d, M, bits, nq, leaves, skew=skew), bits), k, R, L)


# Data without many equal sums: no query is handed back. Classes of 64, 16 and 4 points in waves of two column tiles, of 32, 16 and 4 in
# waves of one; blocks that share classes; few of the leaves probed.
@pytest.mark.parametrize("n,d,M,bits,nq,leaves,L,R", [
    (6000, 100, 50, 4, 64, 12, 4, 10), (6000, 100, 50, 4, 64, 12, 4, 20), (6000, 100, 25, 8, 64, 12, 4, 100), (6000, 192, 96, 4, 40, 12, 4, 10),
    (6000, 192, 96, 4, 40, 12, 4, 40), (6000, 256, 32, 8, 40, 12, 4, 100), (20_000, 64, 32, 4, 40, 6, 4, 50), (20_000, 160, 80, 4, 40, 6, 4, 50),
    (40_000, 32, 16, 4, 40, 70, 2, 10), (40_000, 32, 16, 4, 40, 70, 4, 300)])
def test_product_leaves_answers_all(n, d, M, bits, nq, leaves, L, R):
    check_leaves(*reorder_args(draw_leaves(n, d, M, bits, nq, leaves), bits), min(R, 10), R, L, 0)


def reorder_args(drawn, bits):
    x, cb, codes, q, centers, assign = drawn
    return x, cb, codes, bits, q, centers, assign


# A query of zeros, leaves far from the origin beside tight codes, negative scores, values of all magnitudes.
def test_product_leaves_odd_values():
    x, cb, codes, q, centers, assign = draw_leaves(6000, 32, 16, 4, 40, 12)
    q[3] = 0.0
    check_leaves(x, cb, codes, 4, q, centers, assign, 10, 100, 3)
    check_leaves(x, (cb * 1e-3).astype(np.float32), codes, 4, q, centers * 100, assign, 10, 100, 4)
    check_leaves(np.abs(x), -np.abs(cb), codes, 4, np.abs(q) + 0.01, -np.abs(centers), assign, 10, 100, 5)
    q2 = (unit_rows(np.random.default_rng(1), 40, 32) * np.logspace(-15, 14, 40)[:, None]).astype(np.float32)
    check_leaves(x, cb, codes, 4, q2, centers, assign, 10, 100, 5)


# Fewer points in a query's leaves than results: id -1 and score -infinity fill up, whoever answers (a query of zeros has no
# range of 8-bit entries and is always scanned plainly).
@pytest.mark.parametrize("R", [0, 100])
def test_product_leaves_fill_up(R):
    x, cb, codes, q, centers, assign = draw_leaves(700, 48, 16, 4, 20, 300)
    q[3] = 0.0
    check_leaves(x, cb, codes, 4, q, centers, assign, 50, R, 6)


# A leaf of 1,024 blocks among 131,200: as many workgroups as the blocks and 65,536 queries allow for would be 2^32 threads, more
# than a launch takes, and the scratch several GB; the batch is taken in parts.
def test_product_leaves_parts():
    rng = np.random.default_rng(3)
    d, M, leaves, big, nq, L, k = 130, 10, 131_200, 262_144, 65_536, 128, 5
    n = big + leaves - 1
    assign = np.maximum(np.arange(n) - big + 1, 0).astype(np.int32)
    cb = (rng.standard_normal((M, 16, d // M)) * 0.2).astype(np.float32)
    idx = leaf_index(unit_rows(rng, n, d), cb, rng.integers(0, 16, (n, M)).astype(np.uint8), 4, 0.5 * unit_rows(rng, leaves, d), assign)
    qd = torch.nn.functional.normalize(torch.randn((nq, d), device="cuda", generator=torch.Generator("cuda").manual_seed(1)))
    idx.set_tuning("scan_product", 2)
    ids, sc = idx.search(qd, k, 0, avq.LUT_F32, L)
    idx.set_tuning("scan_product", 1)
    for lo in (0, nq // 2 - 20, nq - 40):
        a, b = idx.search(qd[lo:lo + 40].contiguous(), k, 0, avq.LUT_F32, L)
        assert torch.equal(ids[lo:lo + 40], a) and torch.equal(sc[lo:lo + 40], b)


# A query whose product with the center of a probed leaf is infinite has no line to compare with: it is scanned plainly, the others
# are not. (A leaf at -infinity is not probed.)
@pytest.mark.parametrize("k,R", [(50, 0), (50, 512)])
def test_product_leaves_infinite_center(k, R):
    x, cb, codes, q, centers, assign = draw_leaves(700, 32, 16, 4, 40, 3)
    centers[1] = 0.0
    centers[1, 0] = 1e20
    q[::2] *= 1e22
    handed = int((q[::2, 0] > 0).sum())
    assert 0 < handed < 20
    idx = leaf_index(x, cb, codes, 4, centers, assign)
    qd = torch.from_numpy(q).cuda()
    for mode in (avq.LUT_F32, avq.LUT_U8):
        idx.set_tuning("scan_product", 2)
        idx.set_tuning("small_batch_impl", 0)
        ids, sc = idx.search(qd, k, R, mode, 3)
        assert idx.debug_unverified_queries() == handed
        idx.set_tuning("scan_product", 1)
        idx.set_tuning("small_batch_impl", 1) # every point scored
        ids1, sc1 = idx.search(qd, k, R, mode, 3)
        assert torch.equal(ids, ids1)
        np.testing.assert_array_equal(sc.cpu().numpy(), sc1.cpu().numpy())


# Scratch for some 300 queries: the batch is taken in parts, whose handed back queries are counted together. Scratch for none: the
# other paths answer.
@pytest.mark.parametrize("leaves", [0, 12])
@pytest.mark.parametrize("bits,M", [(4, 16), (8, 8)])
def test_product_scratch_limit(leaves, bits, M):
    x, cb, codes, q, centers, assign = draw_leaves(20_000, 32, M, bits, 900, max(leaves, 1))
    idx = leaf_index(x, cb, codes, bits, centers, assign) if leaves else index(x, cb, codes, bits)
    idx.set_tuning("scan_product", 2)
    idx.profile_enable()
    qd = torch.from_numpy(q).cuda()
    for mode in (avq.LUT_F32, avq.LUT_U8):
        ids, sc = idx.search(qd, 10, 50, mode, leaves // 2)
        assert idx.profile_read()["scan"][1] == 1
        for limit, parts in ((30_000, True), (100, False)):
            idx.set_tuning("scratch_limit_kb", limit)
            idx.set_tuning("scan_prefilter", 2) # every odd query of a part is handed back
            a, b = idx.search(qd, 10, 50, mode, leaves // 2)
            stages = idx.profile_read()
            assert (stages["scan"][1] > 1) == parts and (stages["finalize"][1] == 0 or not parts)
            assert not parts or 440 <= idx.debug_unverified_queries() <= 460
            assert torch.equal(ids, a) and torch.equal(sc, b)
            idx.set_tuning("scratch_limit_kb", 0)
            idx.set_tuning("scan_prefilter", 0)


# Few of the leaves probed and many results: classes enough for a line that holds, rather than every query scanned plainly.
def test_product_leaves_few_of_large_ones():
    rng = np.random.default_rng(8)
    n, d, M, leaves, nq = 1_300_000, 16, 8, 100, 64
    cb = (rng.standard_normal((M, 16, d // M)) * 0.2).astype(np.float32)
    idx = leaf_index(unit_rows(rng, n, d), cb, rng.integers(0, 16, (n, M)).astype(np.uint8), 4, 0.5 * unit_rows(rng, leaves, d),
                     rng.integers(0, leaves, n).astype(np.int32))
    qd = torch.from_numpy(unit_rows(rng, nq, d)).cuda()
    for mode in (avq.LUT_F32, avq.LUT_U8):
        idx.set_tuning("scan_product", 2)
        ids, sc = idx.search(qd, 10, 500, mode, 2)
        assert idx.debug_unverified_queries() <= nq // 10
        idx.set_tuning("scan_product", 1)
        a, b = idx.search(qd, 10, 500, mode, 2)
        assert torch.equal(ids, a) and torch.equal(sc, b)


# too little work; enough; just too few and enough queries of a leaf
@pytest.mark.parametrize("n,leaves,nq,L,product", [(20_000, 20, 256, 100 // 10, False), (20_000, 20, 2600, 10, True), (20_000, 20, 2400, 10, False),
                                                   (1_000_000, 1000, 100, 290, False), (1_000_000, 1000, 100, 310, True)])
def test_rule_of_product_leaves(n, leaves, nq, L, product):
    x, cb, codes, q, centers, assign = draw_leaves(n, 32, 16, 4, nq, leaves)
    idx = avq.Index(32, 16, 4, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(centers)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(oracle.pack_codes(codes, 4)).cuda(), torch.from_numpy(assign).cuda())
    idx.profile_enable()
    qd = torch.from_numpy(q).cuda()
    ids, sc = idx.search(qd, 10, 100, avq.LUT_F32, L)
    stages = idx.profile_read()
    assert (stages["sample"][1] > 0 and stages["finalize"][1] == 0) == product
    idx.set_tuning("scan_product", 1)
    ids1, sc1 = idx.search(qd, 10, 100, avq.LUT_F32, L)
    assert torch.equal(ids, ids1) and torch.equal(sc, sc1)

"""A few queries on partitioned indexes of any code size against the oracle: leaf selection, and the scan of the probed
leaves by block maxima and by lists."""
import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def pack(codes, bits):
    if bits == 8:
        return codes
    n, M = codes.shape
    wide = np.zeros((n, M + M % 2), np.uint8)
    wide[:, :M] = codes
    return wide[:, 0::2] | (wide[:, 1::2] << 4)


# code bytes below, at and above four and eight of them, an odd number of subspaces, large codes, 8-bit codes with and without a
# kernel of their own, the most that those kernels' tables have room for (64) and more (65: the list scan); leaves of several blocks
@pytest.mark.parametrize("d,M,bits", [(6, 3, 4), (32, 16, 4), (64, 32, 4), (105, 35, 4), (192, 96, 4), (36, 9, 8), (50, 25, 8), (64, 32, 8),
                                      (33, 33, 8), (64, 64, 8), (65, 65, 8)])
@pytest.mark.parametrize("nq,k,R,L", [(1, 10, 100, 7), (5, 1, 0, 3), (3, 10, 512, 13)])
@pytest.mark.parametrize("mode", [avq.LUT_F32, avq.LUT_U8])
def test_few_queries_on_any_code_size(d, M, bits, nq, k, R, L, mode):
    if M >= 64 and mode == avq.LUT_U8:
        pytest.skip("8-bit tables of more than 62 KB are refused")
    rng = np.random.default_rng([d, M, nq])
    n, leaves = 6000, 13
    x, q, cen = unit_rows(rng, n, d), unit_rows(rng, nq, d), unit_rows(rng, leaves, d)
    cb = (rng.standard_normal((M, 1 << bits, d // M)) / np.sqrt(d)).astype(np.float32)
    codes = rng.integers(0, 1 << bits, (n, M), dtype=np.uint8)
    assign = rng.integers(0, leaves - 1, n).astype(np.int32)  # the last leaf is empty
    assign[: 2000] = 4                                         # and one has several blocks
    idx = avq.Index(d, M, bits, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(cen)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes, bits)).cuda(), assign)
    oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, mode, centers=cen, assign=assign, leaves_to_search=L)
    qd = torch.from_numpy(q).cuda()
    for impl in (0, 1):  # 1: the list scan
        idx.set_tuning("small_batch_impl", impl)
        ids, sc = idx.search(qd, k, R, mode, L)
        np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="small_batch_impl %d" % impl)
        np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="small_batch_impl %d" % impl)


# more blocks listed than are ranked by counting (512), and more candidates; as many codes as points, some dozens (thousands of
# points of each score, and every block's maximum the same but for a few), and one
@pytest.mark.parametrize("M,bits", [(16, 4), (35, 4), (50, 4), (25, 8), (33, 8), (64, 8)])
@pytest.mark.parametrize("distinct", [0, 40, 1])
@pytest.mark.parametrize("nq,R", [(1, 100), (3, 512)])
def test_few_queries_of_many_blocks(M, bits, distinct, nq, R):
    rng = np.random.default_rng([M, bits, distinct, R])
    n, d, k, leaves, L = 150_000, M, 10, 13, 12
    x, q, cen = unit_rows(rng, n, d), unit_rows(rng, nq, d), unit_rows(rng, leaves, d)
    cen[:] = cen[0] if distinct == 1 else cen  # (a leaf's own product is a part of its points' scores)
    cb = (rng.standard_normal((M, 1 << bits, 1)) / np.sqrt(d)).astype(np.float32)
    codes = rng.integers(0, 1 << bits, (distinct or n, M), dtype=np.uint8)
    if distinct:
        codes = codes[rng.integers(0, distinct, n)]
    assign = rng.integers(0, leaves, n).astype(np.int32)
    idx = avq.Index(d, M, bits, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(cen)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes, bits)).cuda(), assign)
    oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, avq.LUT_F32, centers=cen, assign=assign, leaves_to_search=L)
    idx.profile_enable()
    for impl in (0, 1):  # 1: the list scan, which has no second pass
        idx.set_tuning("small_batch_impl", impl)
        ids, sc = idx.search(torch.from_numpy(q).cuda(), k, R, avq.LUT_F32, L)
        np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="small_batch_impl %d" % impl)
        np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="small_batch_impl %d" % impl)
        assert (idx.profile_read()["rescan"][1] > 0) == (impl == 0)  # (reads and resets)


# one leaf, as many as threads and one more, as many as the histogram's registers hold and more; equal scores (one bin), all but one
# equal (a bin with more than there is room for), infinite ones
@pytest.mark.parametrize("leaves", [1, 2, 1024, 1025, 8192, 8193])
@pytest.mark.parametrize("law", ["unit", "equal", "one", "infinite"])
def test_leaf_selection_of_few_queries(leaves, law):
    rng = np.random.default_rng(leaves)
    d = 8
    cen, q = unit_rows(rng, leaves, d), unit_rows(rng, 2, d)
    if law == "equal":
        cen[:] = cen[0]
    elif law == "one":
        cen[:] = cen[0]
        cen[leaves // 2] = 100.0 * q[0]
    elif law == "infinite":
        cen[:: 3] = 0.0
        cen[:: 3, 0] = 3e38
        q *= np.float32(80.0)
    idx = avq.Index(d, 1, 4, n_leaves=leaves)
    idx.set_leaf_centers(cen)
    idx.set_codebooks(np.zeros((1, 16, d), np.float32))
    qd = torch.from_numpy(q).cuda()
    for L in (1, min(leaves, 100), min(leaves, 512)):
        right = [oracle.leaf_select(cen, q[qi], L) for qi in range(len(q))]
        for _ in range(8):  # (a selection that goes wrong does so now and then)
            ids, ip = idx.debug_leaf_select(qd, L)
            for qi, (oi, oip) in enumerate(right):
                np.testing.assert_array_equal(ids[qi].cpu().numpy(), oi)
                np.testing.assert_array_equal(ip[qi].cpu().numpy(), oip)


# dimensions of which a query fits the LDS of the kernel that scores leaves for a few queries, and more: the list scan's selection
@pytest.mark.parametrize("d", [15_360, 15_488])
@pytest.mark.parametrize("M,bits", [(16, 4), (32, 4), (16, 8)])
def test_few_queries_of_many_dimensions(d, M, bits):
    rng = np.random.default_rng([d, M])
    n, nq, k, R, leaves, L = 300, 2, 10, 40, 5, 3
    x, q, cen = unit_rows(rng, n, d), unit_rows(rng, nq, d), unit_rows(rng, leaves, d)
    cb = (rng.standard_normal((M, 1 << bits, d // M)) / np.sqrt(d)).astype(np.float32)
    codes = rng.integers(0, 1 << bits, (n, M), dtype=np.uint8)
    assign = rng.integers(0, leaves, n).astype(np.int32)
    idx = avq.Index(d, M, bits, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(cen)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes, bits)).cuda(), assign)
    oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, avq.LUT_F32, centers=cen, assign=assign, leaves_to_search=L)
    ids, sc = idx.search(torch.from_numpy(q).cuda(), k, R, avq.LUT_F32, L)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)


# 67 MB of scratch are asked for; where they are not to be had, the list scan answers, for a tenth of that
@pytest.mark.parametrize("bits", [4, 8])
def test_few_queries_within_a_scratch_limit(bits):
    rng = np.random.default_rng(bits)
    n, d, M, nq, k, R, leaves, L = 6000, 50, 25, 64, 10, 512, 13, 5
    x, q, cen = unit_rows(rng, n, d), unit_rows(rng, nq, d), unit_rows(rng, leaves, d)
    cb = (rng.standard_normal((M, 1 << bits, d // M)) / np.sqrt(d)).astype(np.float32)
    codes = rng.integers(0, 1 << bits, (n, M), dtype=np.uint8)
    assign = rng.integers(0, leaves, n).astype(np.int32)
    idx = avq.Index(d, M, bits, n_leaves=leaves)
    idx.set_codebooks(cb)
    idx.set_leaf_centers(cen)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes, bits)).cuda(), assign)
    oi, os_ = oracle.search(x, cb, codes, bits, q, k, R, avq.LUT_F32, centers=cen, assign=assign, leaves_to_search=L)
    qd = torch.from_numpy(q).cuda()
    idx.set_tuning("scan_product", 1)  # not the path of batches, whatever it costs
    taken = []
    for limit_kb in (1024, 0, 1024):
        idx.set_tuning("scratch_limit_kb", limit_kb)
        free = torch.cuda.mem_get_info()[0]
        ids, sc = idx.search(qd, k, R, avq.LUT_F32, L)
        taken.append(free - torch.cuda.mem_get_info()[0])
        np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="limit %d KB" % limit_kb)
        np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="limit %d KB" % limit_kb)
    assert taken[0] < 32 << 20 < 64 << 20 < taken[1], taken


# which of the two scans answers a few queries, where one takes twice as long as the other: 228 blocks of 1,300 are a query's; only
# the scan by block maxima has a second pass
@pytest.mark.parametrize("nq,R,maxima", [(1, 100, True), (60, 100, True), (12, 400, True), (60, 400, False), (80, 300, False)])
def test_form_of_a_few_queries(nq, R, maxima):
    rng = np.random.default_rng(nq)
    n, d, M, leaves, L = 300_000, 32, 32, 100, 16
    idx = avq.Index(d, M, 4, n_leaves=leaves)
    idx.set_codebooks(rng.standard_normal((M, 16, 1)).astype(np.float32))
    idx.set_leaf_centers(unit_rows(rng, leaves, d))
    x = torch.from_numpy(unit_rows(rng, 1000, d)).cuda().repeat(300, 1)
    idx.set_database(x, torch.from_numpy(rng.integers(0, 256, (n, 16), dtype=np.uint8)).cuda(), (np.arange(n) % leaves).astype(np.int32))
    idx.profile_enable()
    idx.search(torch.from_numpy(unit_rows(rng, nq, d)).cuda(), 10, R, avq.LUT_F32, L)
    assert (idx.profile_read()["rescan"][1] > 0) == maxima

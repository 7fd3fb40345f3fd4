"""Searches that one launch answers (small flat indexes, 4-bit codes, fp32 tables) against the oracle, where blocks of 256
points, rounds of sixteen blocks, code sizes and result counts meet their edges."""
import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def pack(codes):
    n, M = codes.shape
    wide = np.zeros((n, M + M % 2), np.uint8)
    wide[:, :M] = codes
    return wide[:, 0::2] | (wide[:, 1::2] << 4)


def check(x, cb, codes, q, k, R):
    idx = avq.Index(x.shape[1], codes.shape[1], 4)
    idx.set_codebooks(cb)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes)).cuda())
    oi, os_ = oracle.search(x, cb, codes, 4, q, k, R, avq.LUT_F32)
    qd = torch.from_numpy(q).cuda()
    for split in (0, 1):  # 1: the path over several launches
        idx.set_tuning("select_split", split)
        ids, sc = idx.search(qd, k, R, avq.LUT_F32)
        np.testing.assert_array_equal(ids.cpu().numpy(), oi, err_msg="select_split %d" % split)
        np.testing.assert_array_equal(sc.cpu().numpy(), os_, err_msg="select_split %d" % split)


# one point, fewer points than candidates, the last point of a block and the first of the next, a wave's second and last
# block, the largest index of the rule and one beyond; odd subspace counts, code sizes without kernels of their own,
# a query longer than the workgroup; as many floats to re-score as the rule allows, and more
@pytest.mark.parametrize("n,d,M,nq,k,R", [(1, 32, 16, 1, 1, 1), (7, 32, 16, 3, 7, 10), (256, 100, 25, 2, 10, 0), (257, 100, 50, 1, 10, 257),
                                          (4096, 128, 64, 3, 10, 100), (4097, 105, 35, 5, 100, 100), (9999, 32, 16, 40, 10, 100),
                                          (12_289, 192, 96, 1, 10, 500), (16_384, 100, 50, 2, 1, 1), (16_384, 64, 32, 9, 100, 0),
                                          (16_385, 32, 16, 2, 10, 100), (600, 1026, 513 // 3, 2, 10, 20), (3000, 6, 3, 2, 10, 50), (2000, 200, 100, 2, 10, 500),
                                          (2000, 208, 104, 1, 10, 512)])
def test_search_one_matches(n, d, M, nq, k, R):
    rng = np.random.default_rng(n + d)
    x, q = unit_rows(rng, n, d), unit_rows(rng, nq, d)
    cb = (rng.standard_normal((M, 16, d // M)) * 0.2).astype(np.float32)
    check(x, cb, rng.integers(0, 16, (n, M)).astype(np.uint8), q, k, R)


# every sum the same, and a few sums only: the lower ids win
@pytest.mark.parametrize("distinct", [1, 3])
def test_search_one_equal_sums(distinct):
    rng = np.random.default_rng(distinct)
    x, q = unit_rows(rng, 5000, 32), unit_rows(rng, 2, 32)
    cb = (rng.standard_normal((16, 16, 2)) * 0.2).astype(np.float32)
    rows = rng.integers(0, 16, (distinct, 16)).astype(np.uint8)
    codes = rows[rng.integers(0, distinct, 5000)]
    check(x, cb, codes, q, 10, 0)
    check(x, cb, codes, q, 10, 100)


# Which searches the one launch answers: all that score every block anyway (as many candidates as blocks), else up to a
# number of code bytes that its one compute unit adds up as fast as the several launches do. The selection is a launch of its own on
# the path over several, so its count tells the two apart.
@pytest.mark.parametrize("n,M,nq,k,R,one", [(16_384, 16, 1, 10, 0, True), (12_288, 50, 1, 10, 0, True), (12_545, 50, 1, 10, 0, False),
                                            (16_384, 64, 1, 10, 0, False), (16_384, 64, 1, 64, 0, False), (16_384, 64, 1, 65, 0, True),
                                            (16_384, 64, 1, 10, 100, True), (8192, 72, 1, 10, 0, True), (8193, 72, 2, 10, 10, False),
                                            (14_000, 50, 15, 30, 0, False), (14_000, 50, 16, 30, 0, True), (16_384, 64, 64, 10, 0, True),
                                            (300, 16, 511, 2, 0, True), (300, 16, 512, 2, 0, False), (300, 16, 512, 1, 3, True),
                                            (9000, 2, 1, 10, 0, False), (9000, 2, 1, 37, 0, True)])
def test_rule_of_search_one(n, M, nq, k, R, one):
    rng = np.random.default_rng(n + M)
    x, q = unit_rows(rng, n, 2 * M), unit_rows(rng, nq, 2 * M)
    cb = (rng.standard_normal((M, 16, 2)) * 0.2).astype(np.float32)
    codes = rng.integers(0, 16, (n, M)).astype(np.uint8)
    idx = avq.Index(2 * M, M, 4)
    idx.set_codebooks(cb)
    idx.set_database(torch.from_numpy(x).cuda(), torch.from_numpy(pack(codes)).cuda())
    idx.profile_enable()
    ids, sc = idx.search(torch.from_numpy(q).cuda(), k, R, avq.LUT_F32)
    assert (idx.profile_read()["merge"][1] == 0) == one
    oi, os_ = oracle.search(x, cb, codes, 4, q, k, R, avq.LUT_F32)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)

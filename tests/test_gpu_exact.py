"""Exact search on the GPU against the oracle, at the sizes where the matrix product's tiles and the block selection meet
their edges, and with values that its operands cannot hold."""
import time

import numpy as np
import pytest

import oracle
from util import unit_rows

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
avq = pytest.importorskip("paper_1908_10396_amd")


def exact_index(x, codes=None):
    n, d = x.shape
    idx = avq.Index(d, 1, 4)
    idx.set_codebooks(np.zeros((1, 16, d), np.float32))
    idx.set_database(x if isinstance(x, torch.Tensor) else torch.from_numpy(x).cuda(), torch.zeros((n, 1), dtype=torch.uint8, device="cuda"))
    return idx


def check(x, q, k):
    ids, sc = exact_index(x).brute_force(torch.from_numpy(q).cuda(), k)
    oi, os_ = oracle.brute_force(x, q, k)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)


# blocks of 64 and 32 points, workgroups of 512 and 256, query tiles of 32, every number of 16-coordinate steps and
# odd dimensions (scalar loads), the edge of the rule for small indexes; 257 dimensions take the plain kernel
@pytest.mark.parametrize("n,d,nq,k", [(1, 2, 1, 1), (256, 32, 31, 1), (2559, 33, 32, 10), (2560, 33, 32, 10), (513, 48, 33, 2),
                                      (4097, 64, 64, 16), (25_600, 65, 260, 100), (20_011, 100, 7, 64), (5000, 105, 40, 10),
                                      (2048, 128, 33, 8), (2049, 129, 20, 8), (1000, 192, 3, 1), (1025, 193, 9, 4),
                                      (70_000, 256, 17, 200), (900, 257, 5, 3)])
def test_exact_search_matches(n, d, nq, k):
    rng = np.random.default_rng(n + d)
    check(unit_rows(rng, n, d), unit_rows(rng, nq, d), k)


# 256 and 257, 512 and 513 workgroups, two and three query tiles: one and two workgroups to a compute unit
@pytest.mark.parametrize("n,nq", [(131_072, 65), (131_073, 64), (131_073, 65), (262_144, 33), (262_145, 33), (262_145, 32)])
def test_exact_search_of_one_and_two_workgroups_to_a_compute_unit(n, nq):
    rng = np.random.default_rng(n + nq)
    check(unit_rows(rng, n, 100), unit_rows(rng, nq, 100), 10)


# rows through LDS (eight tiles of queries on more than 256 workgroups): an odd and an even number of quads a row, rows that are
# no whole quads or do not start at one, a last piece of sixteen rows that is short; and an array beyond 256 MB
@pytest.mark.parametrize("n,d,nq,shift", [(131_073, 100, 225, 0), (131_090, 104, 225, 0), (131_073, 112, 226, 0), (131_600, 105, 225, 0),
                                          (131_073, 98, 225, 0), (131_075, 100, 225, 1), (671_100, 100, 3, 0), (671_203, 97, 2, 0)])
def test_exact_search_with_rows_through_lds(n, d, nq, shift):
    rng = np.random.default_rng([n, d])
    x, q = unit_rows(rng, n, d), unit_rows(rng, nq, d)
    room = torch.empty(n * d + shift, device="cuda")
    xd = room[shift:].view(n, d)
    xd.copy_(torch.from_numpy(x))
    ids, sc = exact_index(xd).brute_force(torch.from_numpy(q).cuda(), 10)
    oi, os_ = oracle.brute_force(x, q, 10)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)


# the end of a row within a load of four words, before it and at it, in every number of steps; the last row is the array's end
@pytest.mark.parametrize("d", [4, 5, 6, 7, 15, 17, 31, 34, 47, 49, 51, 63, 65, 66, 79, 81, 83, 95, 97, 99, 111, 114, 127, 130, 131, 191, 195, 253, 255])
def test_exact_search_of_rows_that_are_no_whole_quads(d):
    rng = np.random.default_rng(d)
    check(unit_rows(rng, 3001, d), unit_rows(rng, 40, d), 10)


# 65 to 112 dimensions on more than 256 workgroups, by the size of the array (200, 256, 400, 448 and 640 MB) and tiles of queries (one,
# two, eight, sixteen): two workgroups a compute unit, whose lanes read their rows or have them through LDS, past the caches or not
@pytest.mark.parametrize("n,d,nq", [(131_073, 66, 33), (131_100, 96, 40), (131_080, 97, 40), (545_001, 97, 225), (547_003, 96, 33), (671_203, 101, 33),
                                    (1_200_007, 98, 34), (1_800_003, 66, 513), (1_600_001, 80, 40), (800_003, 87, 40), (820_007, 84, 5),
                                    (800_003, 87, 70), (1_300_009, 84, 513), (1_800_001, 96, 70)])
def test_exact_search_by_the_size_of_the_array(n, d, nq):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    xd = torch.nn.functional.normalize(torch.randn((n, d), generator=gen, device="cuda"))
    q = unit_rows(np.random.default_rng(n), nq, d)
    ids, sc = exact_index(xd).brute_force(torch.from_numpy(q).cuda(), 10)
    some = [0, nq // 2, nq - 1]
    oi, os_ = oracle.brute_force(xd.cpu().numpy(), np.ascontiguousarray(q[some]), 10)
    np.testing.assert_array_equal(ids.cpu().numpy()[some], oi)
    np.testing.assert_array_equal(sc.cpu().numpy()[some], os_)


# as many results as classes of blocks can tell apart, and more; values that many blocks share
@pytest.mark.parametrize("n,nq,k", [(30_000, 20, 1), (30_000, 300, 15), (30_000, 20, 16), (30_000, 20, 17), (40_000, 20, 128),
                                    (40_000, 260, 128), (40_000, 260, 129), (80_000, 20, 257), (40_000, 20, 33), (70_000, 260, 17),
                                    (140_000, 20, 64)])
def test_exact_search_at_the_lines_of_the_selection(n, nq, k):
    rng = np.random.default_rng([n, nq, k])
    x = np.round(unit_rows(rng, n, 24) * 16).astype(np.float32)
    check(x, np.round(unit_rows(rng, nq, 24) * 16).astype(np.float32), k)


# one to four query tiles through three buffers and two accumulators: two column tiles per wave of 10 (80 dimensions), 12 (96), 14
# (112) and 16 (113) operands, and one column tile (129, 256); points beyond the last full wave
@pytest.mark.parametrize("d", [80, 96, 112, 113, 129, 256])
@pytest.mark.parametrize("nq", [32, 33, 96, 97])
def test_exact_search_of_every_number_of_query_tiles(d, nq):
    rng = np.random.default_rng(d + nq)
    check(unit_rows(rng, 4097, d), unit_rows(rng, nq, d), 10)


# two and three dimensions, on both sides of the line above which the plain kernel takes them (100,000 and 500,000 points)
@pytest.mark.parametrize("n,d", [(100_000, 2), (100_001, 2), (500_000, 3), (500_001, 3)])
def test_exact_search_of_a_few_dimensions(n, d):
    rng = np.random.default_rng(n)
    check(unit_rows(rng, n, d), unit_rows(rng, 9, d), 10)


# the rule for a few queries and many results: 48 | 49 results of one query (64 | 65 dimensions), of up to seven (200 | 201), 64 | 65
@pytest.mark.parametrize("n,d,nq,k", [(17_000, 65, 1, 48), (17_000, 65, 1, 49), (17_000, 64, 1, 64), (17_000, 201, 7, 49),
                                      (17_000, 200, 7, 64), (17_000, 201, 8, 64), (17_000, 40, 15, 65), (17_000, 40, 16, 65)])
def test_exact_search_of_a_few_queries(n, d, nq, k):
    rng = np.random.default_rng(n + d)
    check(unit_rows(rng, n, d), unit_rows(rng, nq, d), k)


# ties everywhere (copies of a few rows), norms over many magnitudes, values that vanish in squares, zero rows
@pytest.mark.parametrize("kind", ["copies", "norms", "tiny", "zero"])
def test_exact_search_of_unusual_points(kind):
    rng = np.random.default_rng(11)
    x, q = unit_rows(rng, 6000, 36), unit_rows(rng, 40, 36)
    if kind == "copies":
        x = np.ascontiguousarray(x[rng.integers(0, 7, 6000)])
    elif kind == "norms":
        x *= np.exp(rng.uniform(-20, 20, (6000, 1))).astype(np.float32)
        q *= np.exp(rng.uniform(-20, 20, (40, 1))).astype(np.float32)
    elif kind == "tiny":
        x *= np.float32(1e-21)
    else:
        x[::2] = 0
        q[3] = 0
    check(x, q, 20)


# infinities, and norms above what the product takes: every query by the plain kernel
@pytest.mark.parametrize("value", [np.inf, 3e18])
def test_exact_search_of_large_values(value):
    rng = np.random.default_rng(12)
    x, q = unit_rows(rng, 3000, 20), np.abs(unit_rows(rng, 9, 20))
    x[1234] = np.abs(x[1234])
    x[1234, 5] = value
    check(x, q, 10)


# Queries whose list of blocks is too long for the selection, alone and among others of the same tile of eight: the plain
# kernel answers those. 64- and 32-point blocks, several tiles of queries, a last tile that is not full.
@pytest.mark.parametrize("n,d", [(20_000, 24), (20_001, 33), (12_000, 200)])
@pytest.mark.parametrize("law", ["copies", "common", "some_queries", "large_query"])
@pytest.mark.parametrize("nq,k", [(1, 5), (45, 10)])
def test_exact_search_where_the_product_decides_little(n, d, law, nq, k):
    rng = np.random.default_rng(n + nq)
    x, q = unit_rows(rng, n, d), unit_rows(rng, nq, d)
    if law == "copies":
        x = np.ascontiguousarray(x[rng.integers(0, 3, n)])
    elif law == "common":
        x = (x + 300 * unit_rows(rng, 1, d)).astype(np.float32)
    else:
        q[[0, 13, 14, 44] if nq > 1 else 0] = 0 if law == "some_queries" else 3e18 * np.float32(d ** -0.5)
    check(x, q, k)


def exact_seconds(x, q, k):
    """The fastest of eight calls."""
    idx = exact_index(x)
    best = float("inf")
    for _ in range(9):
        torch.cuda.synchronize()
        t = time.perf_counter()
        idx.brute_force(q, k)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


# Measured: copies of a row 1.8 times as long as rows that differ (32 times with the list scored whatever its length), a
# query of zeros among others 2.1 times (28 times)
@pytest.mark.parametrize("law", ["copies", "zero_query"])
def test_exact_search_time_where_the_product_decides_little(law):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    x = torch.nn.functional.normalize(torch.randn((200_000, 100), generator=gen, device="cuda"))
    q = torch.nn.functional.normalize(torch.randn((16, 100), generator=gen, device="cuda"))
    usual = exact_seconds(x, q, 10)
    if law == "copies":
        x = x[:1].expand(x.shape).contiguous()
    else:
        q[5] = 0
    assert exact_seconds(x, q, 10) < 6 * usual


# Queries in several launches (96, 96 and 38 at 38,000 x 24 points, whose block maxima take 2.4 KB a query), one of them with a
# query for the plain kernel; a limit below 32 queries' scratch: the plain kernel for all
@pytest.mark.parametrize("limit_kb,bad", [(300, None), (300, 120), (300, 5), (8, None), (0, 120)])
def test_exact_search_within_limited_scratch(limit_kb, bad):
    rng = np.random.default_rng(21)
    x, q = unit_rows(rng, 38_000, 24), unit_rows(rng, 230, 24)
    if bad is not None:
        q[bad] = 3e18
    idx = exact_index(x)
    idx.set_tuning("scratch_limit_kb", limit_kb)
    ids, sc = idx.brute_force(torch.from_numpy(q).cuda(), 7)
    oi, os_ = oracle.brute_force(x, q, 7)
    np.testing.assert_array_equal(ids.cpu().numpy(), oi)
    np.testing.assert_array_equal(sc.cpu().numpy(), os_)

"""The work that a user of this framework has it do, as cases that can be timed.

An index is learned (`train`), the points are encoded under the anisotropic loss
(`encode`), and queries are answered: one at a time, a few, or in batches, over a
flat or a partitioned index, with fp32 or 8-bit tables on 4-bit or 8-bit codes
(`search`). Exact search (`exact`) supplies the ground truth for recall. The
sizes are those of `synth_inputs.CONFIGS` (`bench.py`, the tests) and, in
`draw`, anything between its smallest and its largest; the data follow the same
law as there (mixture of Gaussians, unit norm), drawn on the GPU.

Every search case installs its dictionaries and leaf centers and encodes its
points with the library, so that searches run on codes as they occur; the
dictionaries come from a few Lloyd steps in fp64 here, which the seed alone
determines.
"""
import math

import torch

import paper_1908_10396_amd as avq

GLOVE = dict(n=1_183_514, d=100)


def listed():
    return [
        # a small collection (a few thousand documents), one request: all latency
        dict(name="one_small", kind="search", n=10_000, d=32, M=16, bits=4, leaves=0, probe=0, nq=1, k=10, R=100, tables="f32"),
        # a serving process that answers one request at a time over the Glove-shaped collection
        dict(name="one_glove", kind="search", **GLOVE, M=50, bits=4, leaves=0, probe=0, nq=1, k=10, R=100, tables="f32"),
        # requests collected for a moment, 8-bit codes with 8-bit tables
        dict(name="few_glove8_u8", kind="search", **GLOVE, M=25, bits=8, leaves=0, probe=0, nq=16, k=10, R=100, tables="u8"),
        # one request on a partitioned index
        dict(name="one_glove_ivf", kind="search", **GLOVE, M=50, bits=4, leaves=2000, probe=100, nq=1, k=10, R=100, tables="f32"),
        # the headline: 10,000 queries at once on the flat index (evaluation, offline retrieval)
        dict(name="batch_glove", kind="search", **GLOVE, M=50, bits=4, leaves=0, probe=0, nq=10_000, k=10, R=100, tables="f32"),
        # the same collection with 8-bit codes; a batch that is no multiple of any tile
        dict(name="batch_glove8", kind="search", **GLOVE, M=25, bits=8, leaves=0, probe=0, nq=1999, k=10, R=100, tables="f32"),
        # 10,000 queries on the partitioned index
        dict(name="batch_glove_ivf", kind="search", **GLOVE, M=50, bits=4, leaves=2000, probe=100, nq=10_000, k=10, R=100, tables="f32"),
        # a large collection, whose codes do not fit a cache; 8-bit tables
        dict(name="batch_large4_u8", kind="search", n=10_000_000, d=128, M=64, bits=4, leaves=0, probe=0, nq=1024, k=10, R=200, tables="u8"),
        # ground truth for a recall measurement
        dict(name="exact_glove", kind="exact", **GLOVE, nq=1000, k=10),
        # dictionaries learned on a sample of the collection, as bench.py does
        dict(name="train_glove", kind="train", n=262_144, d=100, M=50, bits=4, leaves=0, iters=20),
        # the collection encoded with known dictionaries (new or changed data), the codes taken to be stored
        dict(name="encode_glove", kind="encode", **GLOVE, M=50, bits=4, leaves=0),
        # a partitioned index made from nothing: leaf centers, dictionaries of the residuals, leaf of every point, codes
        dict(name="build_glove_ivf", kind="build", **GLOVE, M=50, bits=4, leaves=2000, iters=20),
    ]


# d, M, bits: the configurations' shapes, then generic ones (16, 18, 9 and 48 code bytes; an odd number of subspaces)
SHAPES = [(32, 16, 4), (100, 50, 4), (100, 25, 4), (128, 64, 4), (100, 25, 8), (256, 32, 8),
          (64, 32, 4), (105, 35, 4), (36, 9, 8), (192, 96, 4)]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))


def draw(rng):
    kind = rng.choice(["search"] * 6 + ["exact", "train", "encode", "build"])
    d, M, bits = rng.choice(SHAPES)
    kc = 1 << bits
    if kind == "search":
        ivf = rng.random() < 0.35
        nq = _log_int(rng, 1, 10_000)
        n_max = min(1e7, 6e11 / (nq * M), 3e9 / d)     # at most the work of the largest listed searches
        if ivf:
            n_max = min(1_200_000, 6e11 / (nq * M) * 10)
        n = _log_int(rng, 2_000, n_max)
        R = rng.choice([0, 50, 100, 100, 200, 500])
        k = rng.choice([1, 10, 10, 100])
        k = k if R == 0 else min(k, R)
        leaves = max(8, min(2000, int(n ** 0.5 * rng.uniform(0.5, 2)))) if ivf else 0
        probe = max(1, int(leaves * rng.uniform(0.02, 0.1))) if ivf else 0
        return dict(kind=kind, n=n, d=d, M=M, bits=bits, leaves=leaves, probe=probe, nq=nq, k=k, R=R,
                    tables=rng.choice(["f32", "f32", "u8"]))
    if kind == "exact":
        nq = _log_int(rng, 1, 1_000)
        return dict(kind=kind, n=_log_int(rng, 2_000, min(4e6, 1.1e11 / (nq * d))), d=d, nq=nq, k=rng.choice([1, 10, 100]))
    if kind == "encode":
        # kc * d terms per point and pass: at most 2e6 points of the Glove shape
        return dict(kind=kind, n=_log_int(rng, 2_000, min(2e6, 3.2e9 / (kc * d))), d=d, M=M, bits=bits, leaves=0)
    leaves = 0
    n = _log_int(rng, 4_000, min(262_144, 4.2e8 * 20 / (20 * kc * d)))
    if kind == "build":
        leaves = rng.choice([0, max(8, min(2000, int(n ** 0.5 * rng.uniform(0.5, 2))))])
    return dict(kind=kind, n=n, d=d, M=M, bits=bits, leaves=leaves, iters=rng.choice([10, 20]))


# ---- inputs ----------------------------------------------------------------------------

N_COMP, SIGMA = 1000, 0.3


def _mixture(n, d, means, gen):
    """Unit-norm rows: a uniformly drawn mean plus SIGMA * N(0, I), as in synth_inputs."""
    out = torch.empty((n, d), dtype=torch.float32, device="cuda")
    for lo in range(0, n, 1 << 20):
        m = min(n - lo, 1 << 20)
        comp = torch.randint(N_COMP, (m,), generator=gen, device="cuda")
        v = torch.randn((m, d), generator=gen, device="cuda") * SIGMA + means[comp]
        out[lo:lo + m] = torch.nn.functional.normalize(v)
    return out


def _lloyd(x, k, steps, gen):
    """k means of each of the G sets x [G][rows][dim] (fp64) by a few Lloyd steps: ([G][k][dim], [G][rows])."""
    c = x[:, torch.randperm(x.shape[1], generator=gen, device="cuda")[:k]]
    for s in range(steps + 1):
        dist = c.pow(2).sum(-1)[:, None] - 2 * torch.bmm(x, c.transpose(1, 2).contiguous())
        near = dist.argmin(-1)
        if s == steps:
            return c, near
        member = torch.nn.functional.one_hot(near, k).double().transpose(1, 2).contiguous()
        count = member.sum(-1, keepdim=True)
        c = torch.where(count > 0, torch.bmm(member, x) / count.clamp(min=1), c)


def _index(case, x, gen):
    """An index with leaf centers and dictionaries learned on a sample."""
    d, M, leaves = case["d"], case["M"], case["leaves"]
    idx = avq.Index(d, M, case["bits"], T=0.2, n_leaves=leaves)
    sample = x[: 16_384].double()
    if leaves:
        centers, near = _lloyd(sample[None], leaves, 2, gen)
        centers = centers[0].float().contiguous()
        idx.set_leaf_centers(centers)
        sample = sample - centers.double()[near[0]]
    parts = sample.reshape(sample.shape[0], M, d // M).transpose(0, 1).contiguous()
    codebooks, _ = _lloyd(parts, idx.kc, 4, gen)
    idx.set_codebooks(codebooks.float().contiguous())
    return idx


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n, d = case["n"], case["d"]
    means = torch.nn.functional.normalize(torch.randn((N_COMP, d), generator=gen, device="cuda"))
    x = _mixture(n, d, means, gen)
    state = {"case": case, "x": x}
    kind = case["kind"]
    if kind in ("search", "exact"):
        state["queries"] = _mixture(case["nq"], d, means, gen)
    if kind == "search":
        state["index"] = _index(case, x, gen)
        state["index"].encode(x)
        shape = (case["nq"], case["k"])
        state["out"] = (torch.empty(shape, dtype=torch.int32, device="cuda"), torch.empty(shape, device="cuda"))
    elif kind == "exact":
        # exact search needs the points only; the codes that an index must have are of no account
        state["index"] = avq.Index(d, 1, 4)
        state["index"].set_codebooks(torch.zeros((1, 16, d), device="cuda"))
        state["index"].set_database(x, torch.zeros((n, 1), dtype=torch.uint8, device="cuda"))
    elif kind == "encode":
        state["index"] = _index(case, x, gen)
    elif kind == "train":
        state["index"] = avq.Index(d, case["M"], case["bits"], T=0.2, kmeans_iters=case["iters"], seed=seed)
    elif kind == "build":
        state["seed"] = seed
    return state


# ---- one pass --------------------------------------------------------------------------

def run(state):
    case, x = state["case"], state["x"]
    kind = case["kind"]
    if kind == "search":
        mode = avq.LUT_F32 if case["tables"] == "f32" else avq.LUT_U8
        return state["index"].search(state["queries"], case["k"], case["R"], mode, case["probe"], out=state["out"])
    if kind == "exact":
        return state["index"].brute_force(state["queries"], case["k"])
    if kind == "train":
        state["index"].train(x)
        return state["index"].get_codebooks()
    if kind == "encode":
        state["index"].encode(x)
        return state["index"].get_codes()
    idx = avq.Index(case["d"], case["M"], case["bits"], T=0.2, kmeans_iters=case["iters"], n_leaves=case["leaves"],
                    leaf_kmeans_iters=10, seed=state["seed"])
    idx.train(x[: 262_144])
    idx.encode(x)
    state["index"] = idx
    out = {"codebooks": idx.get_codebooks(), "codes": idx.get_codes()}
    if case["leaves"]:
        out["centers"] = idx.get_leaf_centers()
        out["leaf"] = idx.get_leaf_assign()
    return out


def work(case):
    """Bytes: inputs read once, outputs written once. Flops: the method's own multiplications and additions."""
    n, d, kind = case["n"], case["d"], case["kind"]
    if kind == "exact":
        nq, k = case["nq"], case["k"]
        return {"bytes": 4.0 * (n + nq) * d + 8.0 * nq * k, "flops": 2.0 * n * nq * d}
    M, bits, leaves = case["M"], case["bits"], case["leaves"]
    kc, nb = 1 << bits, (M * bits + 7) // 8
    if kind == "search":
        nq, k, R = case["nq"], case["k"], case["R"]
        part = case["probe"] / leaves if leaves else 1.0         # share of the points that a query scores
        read = min(1.0, part * nq)                               # share of the codes that the call reads
        nbytes = nb * n * read + 4.0 * (kc * d + leaves * d + nq * d) + 8.0 * nq * k + 4.0 * d * min(n, nq * R)
        # an addition per subspace, point and query; tables, leaf scores, exact scores
        return {"bytes": nbytes, "flops": nq * (1.0 * M * n * part + 2.0 * d * (kc + leaves + R))}
    out = 4.0 * kc * d + 4.0 * leaves * d
    # a Lloyd step of the dictionaries: <x, c> for every codeword; of the leaves: for every center, on 256 points a leaf
    learn = 2.0 * min(n, 262_144) * kc * d * case.get("iters", 0) + 2.0 * min(n, 256 * leaves, 262_144) * leaves * d * 10
    if kind == "train":
        return {"bytes": 4.0 * n * d + out, "flops": learn}
    # encoding: <x, c> and the loss of every codeword in at least two passes over the subspaces, and the nearest leaf
    code = n * (2.0 * kc * d + 2 * 4.0 * kc * M + 2.0 * leaves * d)
    return {"bytes": (4.0 * d + nb + (4 if leaves else 0)) * n + out, "flops": code + (learn if kind == "build" else 0.0)}


def tolerance(case):
    # searches and exact search have one right answer: every sum has a stated order of additions, ties go to the lower id
    if case["kind"] in ("search", "exact"):
        return "exact"
    # codes are arg-mins of fp64 losses: only near-ties may fall differently
    if case["kind"] == "encode":
        return {"rel": 0.0, "differ": 1e-6}
    # means are fp64 sums in any order, rounded to fp32. A plain fp64 Lloyd in torch gave the very same dictionaries,
    # centers, leaves and codes at the listed sizes; room is left for roundings that fall the other way (6e-8 each)
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-6}

"""The library's working range as measurable cases.

Each case is a call that a user makes through `paper_2104_06357_amd`: all-pairs distances or the fused
k-NN between the rows of two seeded random CSR matrices.  The matrices are drawn on the GPU, after the
laws of this repository's synthetic workloads (gen/synth.py):

  tiny      uniform columns at 2 % density, values Uniform(0, 1]
  skewed    Zipf row lengths (median 4, longest 2,000) and Zipf columns, values |N(0, 1)|
  words     bag of words: lognormal rows of ~230, Zipf columns, TF-IDF values in unit rows
  counts    count matrix: 7 % density, uniform columns, values normalised to sum 1 in each row
  binary    power-law rows of 1 to 50,000 ones over 2^20 columns, Zipf columns
  ngrams    rows of two or three small counts over 858,000 columns
  ratings   power-law rows of 1 to 24,000 ratings over 194,000 columns
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2104_06357_amd as spd

# columns; exponent of the column law (0: uniform); longest row
FAMILIES = {
    "tiny": (512, 0.0, 64),
    "skewed": (20_000, 1.1, 2_000),
    "words": (102_660, 1.1, 2_000),
    "counts": (26_000, 0.0, 12_000),
    "binary": (1 << 20, 1.1, 50_000),
    "ngrams": (858_000, 1.05, 51),
    "ratings": (194_000, 1.02, 24_000),
}


def listed():
    """`entry` is the call, m x n the rows of its two operands over `cols` columns.  `k` is the number of neighbours,
    `p` the degree of Minkowski's distance, and `host_rows` says whether the caller passes the host copy of the row
    pointers that it built the matrices from (the binding's default) or has them on the GPU alone."""
    base = {"cols": 0, "k": 0, "p": 2.0, "host_rows": True}

    def case(name, family, entry, metric, m, n, **more):
        c = dict(base, name=name, family=family, entry=entry, metric=metric, m=m, n=n, **more)
        c["cols"] = c["cols"] or FAMILIES[family][0]
        return c

    return [
        # a small interactive call: latency and launches
        case("tiny_l1", "tiny", "pairwise", "l1", 256, 256),
        # the ordinary call: a dense 10,000 x 10,000 matrix of distances of a mid-sized skewed data set
        case("skewed_l1", "skewed", "pairwise", "l1", 10_000, 10_000),
        case("skewed_cosine", "skewed", "pairwise", "cosine", 10_000, 10_000),
        # nearest neighbours on the same data
        case("skewed_knn_cosine", "skewed", "knn", "cosine", 10_000, 10_000, k=32),
        # sum() = max, which is completed from the unmatched columns, at ragged sizes
        case("ragged_chebyshev", "skewed", "pairwise", "chebyshev", 3_333, 7_777, cols=20_011),
        # a tile of documents against a large corpus
        case("words_cosine", "words", "pairwise", "cosine", 1_024, 300_000),
        # batches of queries against a corpus that was prepared once
        case("words_index_knn", "words", "index_knn", "hellinger", 2_048, 300_000, k=32),
        # the largest work: a tile of a self-join of long rows, a cheap and an expensive product
        case("counts_l1", "counts", "pairwise", "l1", 4_096, 65_536),
        case("counts_js", "counts", "pairwise", "jensen_shannon", 4_096, 65_536),
        # set similarity search in very many columns
        case("binary_knn_jaccard", "binary", "knn", "jaccard", 4_096, 500_000, k=32),
        # record matching: very short rows, the largest row count
        case("ngrams_knn_cosine", "ngrams", "knn", "cosine", 4_096, 663_000, k=32),
        # rows of very different lengths, odd sizes, row pointers on the GPU alone
        case("ratings_canberra", "ratings", "pairwise", "canberra", 1_531, 28_301, host_rows=False),
    ]


# sizes that draw() takes per family: rows of the first operand, rows of the second, largest product of the two
RANGES = {
    "tiny": ((16, 700), (16, 700), 500_000),
    "skewed": ((300, 12_000), (300, 12_000), 100_000_000),
    "words": ((17, 1_500), (5_000, 300_000), 200_000_000),
    "counts": ((16, 4_000), (500, 60_000), 60_000_000),
    "binary": ((40, 4_096), (8_000, 400_000), 700_000_000),
    "ngrams": ((40, 4_096), (8_000, 663_000), 2_000_000_000),
    "ratings": ((40, 4_096), (2_000, 200_000), 150_000_000),
}
DOT = ("inner_product", "cosine", "l2_expanded", "correlation", "hellinger")
UNION = ("l1", "canberra", "hamming", "kl_divergence", "jensen_shannon", "minkowski", "chebyshev")
SETS = ("jaccard", "dice", "russell_rao")


def draw(rng):
    """One more case of the same ranges, without a name."""
    family = rng.choice(sorted(FAMILIES))
    (m_lo, m_hi), (n_lo, n_hi), most = RANGES[family]

    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    m, n = size(m_lo, m_hi), size(n_lo, n_hi)
    n = max(n_lo, min(n, most // m))
    entry = rng.choice(("pairwise", "knn") if family == "tiny" else ("pairwise", "pairwise", "knn", "knn", "index_knn", "index_pairwise"))
    if family == "binary":
        metric = rng.choice(SETS + ("hamming",))
        entry = rng.choice(("knn", "knn", "index_knn"))
    elif family == "ngrams":
        metric, entry = rng.choice(("cosine", "jaccard", "l1")), rng.choice(("knn", "knn", "index_knn"))
    elif family == "words":
        metric = rng.choice(DOT + SETS)
    else:
        metric = rng.choice(DOT + UNION + UNION + SETS)
    if metric in ("minkowski", "chebyshev"):
        n = max(n_lo // 2, min(n, most // 4 // m))
    cols = FAMILIES[family][0] - (rng.randrange(1, 200) if rng.random() < 0.5 else 0)
    return {"family": family, "entry": entry, "metric": metric, "m": m, "n": n, "cols": cols,
            "k": min(n, rng.choice((1, 5, 10, 32, 64))) if "knn" in entry else 0,
            "p": rng.choice((3.0, 3.0, 1.5)) if metric == "minkowski" else 2.0,
            "host_rows": rng.random() < 0.7}


# --------------------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------------------
class _Columns:
    """The column law: uniform, or rank r with probability proportional to the integral of x**-s over
    [r, r + 1), the ranks permuted over the columns."""

    def __init__(self, cols, s, gen):
        self.cols, self.s, self.gen = cols, s, gen
        self.perm = torch.randperm(cols, generator=gen, device="cuda") if s else None

    def draw(self, count):
        if not self.s:
            return torch.randint(0, self.cols, (count,), generator=self.gen, device="cuda")
        u = torch.rand(count, generator=self.gen, device="cuda", dtype=torch.float64)
        x = (1.0 + u * ((self.cols + 1.0) ** (1.0 - self.s) - 1.0)) ** (1.0 / (1.0 - self.s))
        return self.perm[(x.long() - 1).clamp_(0, self.cols - 1)]


def _table_lengths(weights, rows, gen):
    cdf = torch.cumsum(torch.as_tensor(weights, dtype=torch.float64, device="cuda"), 0)
    u = torch.rand(rows, generator=gen, device="cuda", dtype=torch.float64)
    return torch.searchsorted(cdf / cdf[-1], u).clamp_(max=len(weights) - 1) + 1


def _lengths(family, rows, cols, gen):
    longest = min(FAMILIES[family][2], cols)
    if family == "tiny":
        chance = torch.full((rows, cols), 0.02, device="cuda")
        return torch.bernoulli(chance, generator=gen).sum(1).long().clamp_(1, longest)
    if family == "skewed":
        z = _table_lengths(np.arange(1, longest + 1, dtype=np.float64) ** -1.8, rows, gen)
        return (4 * z).clamp_(1, longest)
    if family in ("words", "counts"):
        mean, sigma, least = (230.0, 0.8, 1) if family == "words" else (0.07 * cols, 0.5, 500)
        g = torch.randn(rows, generator=gen, device="cuda", dtype=torch.float64)
        return torch.exp(math.log(mean) - 0.5 * sigma * sigma + sigma * g).round_().long().clamp_(least, longest)
    if family == "ngrams":
        u = torch.rand(rows, generator=gen, device="cuda", dtype=torch.float64).clamp_(min=1e-12)
        return torch.ceil(torch.log(u) / math.log(0.55)).long().clamp_(1, longest)
    alpha = 1.5 if family == "binary" else 1.45
    return _table_lengths(np.arange(1, longest + 1, dtype=np.float64) ** -alpha, rows, gen)


def _structure(family, rows, cols, law, gen):
    """Row of every entry, its column (ascending in each row, distinct) and the row lengths.  A row whose draws fall on
    one column more than once is drawn on a few times and stays a little shorter than asked for if that leaves a gap."""
    want = _lengths(family, rows, cols, gen)
    keys, missing = torch.empty(0, dtype=torch.int64, device="cuda"), want
    for _ in range(4):
        r = torch.repeat_interleave(torch.arange(rows, device="cuda"), missing)
        if r.numel() == 0:
            break
        keys = torch.unique(torch.cat((keys, r * cols + law.draw(r.numel()))))
        have = torch.bincount(keys // cols, minlength=rows)
        missing = want - have
    row = keys // cols
    return row, (keys - row * cols).to(torch.int32), torch.bincount(row, minlength=rows)


def _values(family, row, rows, col, frequency, gen):
    count = row.numel()
    if family == "binary":
        return torch.ones(count, device="cuda")
    if family == "skewed":
        return torch.randn(count, generator=gen, device="cuda").abs_().clamp_(min=1e-7)
    if family == "ngrams":
        return 1.0 + torch.poisson(torch.full((count,), 0.3, device="cuda"), generator=gen)
    if family == "ratings":
        return 0.5 * torch.randint(1, 11, (count,), generator=gen, device="cuda").float()
    u = torch.rand(count, generator=gen, device="cuda")
    if family == "tiny":
        return 1.0 - u
    if family == "words":
        tf = torch.ceil(torch.exp(torch.randn(count, generator=gen, device="cuda", dtype=torch.float64)))
        v = tf * (torch.log((1.0 + frequency[1]) / (1.0 + frequency[0])) + 1.0)[col.long()]
        norm = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, row, v * v).sqrt_()
        return (v / norm[row]).float()
    # negative binomial counts (the sum of two geometric ones), 0 counted as 1, in shares of the row's sum
    geometric = torch.floor(torch.log(u.clamp_(min=1e-7)) / math.log(0.6))
    u = torch.rand(count, generator=gen, device="cuda")
    v = (geometric + torch.floor(torch.log(u.clamp_(min=1e-7)) / math.log(0.6))).clamp_(min=1.0).double()
    total = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, row, v)
    return (v / total[row]).float()


def _matrix(case, rows, law, frequency, gen):
    row, col, length = _structure(case["family"], rows, case["cols"], law, gen)
    if frequency is None:
        frequency = (torch.bincount(col, minlength=case["cols"]).double(), rows)
    value = _values(case["family"], row, rows, col, frequency, gen)
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(length, 0, out=indptr[1:])
    host = indptr.cpu().numpy() if case["host_rows"] else None
    return spd.DeviceCsr(rows, case["cols"], indptr, col, value.contiguous(), host_indptr=host), frequency


def _some_rows(case, M, rows):
    """The first `rows` rows of M as a matrix of their own (a tile of a self-join)."""
    indptr = M.indptr[:rows + 1].clone()
    last = int(indptr[-1])
    host = indptr.cpu().numpy() if case["host_rows"] else None
    return spd.DeviceCsr(rows, M.n_cols, indptr, M.indices[:last].clone(), M.values[:last].clone(), host_indptr=host)


class State:
    """The matrices, the handle, the outputs' buffers and, for the prepared entry points, the index."""


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(1_000_003 * (seed + 1))
    law = _Columns(case["cols"], FAMILIES[case["family"]][1], gen)
    s = State()
    s.case = case
    s.B, frequency = _matrix(case, case["n"], law, None, gen)
    if case["family"] in ("counts", "ngrams", "ratings") and case["m"] <= case["n"]:
        s.A = _some_rows(case, s.B, case["m"])          # these are joined with themselves
    else:
        s.A, _ = _matrix(case, case["m"], law, frequency, gen)
    s.handle = spd.Handle()
    s.index = s.handle.index_create(s.B, case["metric"], p=case["p"]) if case["entry"].startswith("index") else None
    if "knn" in case["entry"]:
        s.idx = torch.zeros((case["m"], case["k"]), dtype=torch.int64, device="cuda")
        s.dist = torch.zeros((case["m"], case["k"]), dtype=torch.float32, device="cuda")
    else:
        s.out = torch.zeros((case["m"], case["n"]), dtype=torch.float32, device="cuda")
    return s


def run(s):
    c = s.case
    if c["entry"] == "pairwise":
        return s.handle.pairwise(s.A, s.B, c["metric"], p=c["p"], out=s.out)
    if c["entry"] == "index_pairwise":
        return s.index.pairwise(s.A, out=s.out)
    if c["entry"] == "knn":
        return s.handle.knn(s.A, s.B, c["metric"], c["k"], p=c["p"], out_idx=s.idx, out_dist=s.dist)
    return s.index.knn(s.A, c["k"], out_idx=s.idx, out_dist=s.dist)


# --------------------------------------------------------------------------------------
# what a pass cannot do without, and how far apart two correct results may lie
# --------------------------------------------------------------------------------------
MEAN_LENGTH = {"tiny": 10.2, "skewed": 37.0, "words": 228.0, "counts": 1_820.0, "binary": 170.0, "ngrams": 2.2,
               "ratings": 160.0}
# arithmetic per column that both rows store (divisions, roots and logarithms count as one operation each)
FLOPS_PER_MATCH = {"canberra": 5, "kl_divergence": 4, "jensen_shannon": 9, "minkowski": 8}


def _matches_per_pair(case):
    """Columns that two rows of mean length share."""
    length, cols, s = MEAN_LENGTH[case["family"]], case["cols"], FAMILIES[case["family"]][1]
    if not s:
        return length * length / cols
    edge = np.arange(1, cols + 2, dtype=np.float64) ** (1.0 - s)
    chance = -np.expm1(-length * np.diff(edge) / (edge[-1] - edge[0]))
    return float((chance * chance).sum())


def work(case):
    """Both matrices read once and the results written once; the products of the columns that two rows share."""
    pairs = case["m"] * case["n"]
    entries = (case["m"] + case["n"]) * MEAN_LENGTH[case["family"]]
    results = case["m"] * case["k"] * 12 if "knn" in case["entry"] else pairs * 4
    return {"bytes": int(8 * entries + 8 * (case["m"] + case["n"] + 2) + results),
            "flops": int(pairs * (FLOPS_PER_MATCH.get(case["metric"], 2) * _matches_per_pair(case) + 1))}


def tolerance(case):
    """Distances are single precision numbers off double precision sums: 2e-8 to 3e-8 off the same formula in 64 bits
    throughout.  Single terms of some products are single precision (quotients and logarithms: 6e-8, powers: 4e-7).
    Neighbours came out the same with the sums in another order; two rows that lie equally near within single precision
    may change places."""
    t = {"rel": {"kl_divergence": 4e-7, "jensen_shannon": 4e-7, "canberra": 4e-7, "minkowski": 2e-6}.get(case["metric"], 2e-7)}
    if "knn" in case["entry"]:
        t["differ"] = 0.0 if case["metric"] in SETS + ("hamming",) else 1e-4
    return t

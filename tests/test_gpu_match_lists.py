"""The column lists (option "match_lists"): B transposed per tile of rows, a wavefront per row of A.
Parity with the CPU oracle through the C-ABI at the sizes where tiles, lists and batches end (needs an
MI355X; run with -m gpu)."""
import numpy as np
import pytest

import oracle
from gen import synth
from test_gpu_parity import _p_of
from util import ALL_METRICS, ORACLE_NAME, assert_distances_close, assert_knn_matches

pytestmark = pytest.mark.gpu

SERVED = [m for m in ALL_METRICS if m != "chebyshev"]


@pytest.fixture(scope="module")
def spd():
    import paper_2104_06357_amd as lib
    return lib


def _np(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


def _matrix(rng, rows, cols, lengths):
    """Rows of the given lengths (in turn) with columns that every row, few rows or one row stores, a stored zero
    in some, an empty row first."""
    d = np.zeros((rows, cols))
    for r in range(1 if rows > 1 else 0, rows):
        n = min(lengths[r % len(lengths)], cols)
        d[r, rng.choice(cols, size=n, replace=False)] = rng.integers(1, 9, size=n) / 8.0
        if n and r % 3:
            d[r, 2] = rng.integers(1, 5) / 4.0          # a list of two thirds of the tile
    out = synth.from_dense(np.asarray(d.astype(np.float32), dtype=np.float64))
    zero = rng.choice(len(out["values"]), size=max(1, len(out["values"]) // 50), replace=False)
    out["values"][zero] = 0.0
    return out


def _lists(spd, **options):
    h = spd.Handle()
    h.set_option("match_lists", 2)
    h.set_option("check_plan", 1)
    for name, value in options.items():
        h.set_option(name, value)
    return h


# rows of B: one, around a wavefront, several tiles with a short last one (32 KB of LDS make tiles of 448 rows for a
# count, 192 for one fp64 sum, 128 for two and 64 for Minkowski's three; 20 KB 256, 128, 64 and 64); rows of A: fewer than
# the wavefronts of a workgroup, and more
@pytest.mark.parametrize("metric", SERVED)
@pytest.mark.parametrize("m,n,cols,budget", [(1, 1, 5, 163840), (3, 63, 70, 163840), (70, 65, 200, 163840), (18, 1300, 300, 163840),
                                             (5, 129, 140, 32768), (150, 1000, 130, 32768), (17, 257, 90, 20480)])
def test_edges(spd, metric, m, n, cols, budget):
    rng = np.random.default_rng(m * 1000 + n)
    A = _matrix(rng, m, cols, (3, 64, 65, 1, 130, 0, 17))
    B = _matrix(rng, n, cols, (2, 5, 0, 40, 9))
    print("match lists", metric, m, n, cols, budget, flush=True)
    h = _lists(spd, lds_budget=budget, profile=1)
    p = _p_of(metric)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    k = min(n, 33)
    idx, dist = h.knn(dA, dB, metric, k, p)
    assert_knn_matches(_np(idx), _np(dist), want, k, metric, metric)
    index = h.index_create(dB, metric, p)
    assert np.array_equal(_np(index.pairwise(dA)), _np(h.pairwise(dA, dB, metric, p)))
    i2, d2 = index.knn(dA, k)
    assert np.array_equal(_np(i2), _np(idx)) and np.array_equal(_np(d2), _np(dist))
    index.close()
    h.close()


@pytest.mark.parametrize("metric", ["inner_product", "l1", "hamming", "canberra"])
def test_chunks_of_a_batch(spd, metric):
    """A step is four chunks of 16 entries of any lists: rows of A whose batches of 64 entries end on, before and behind a
    chunk, a step, four steps and a group of 64 chunks, and rows of B that every list of a step holds (they meet in one sum
    there).  The values are powers of two, so every sum is exact whatever its order."""
    rng = np.random.default_rng(16)
    n, lengths = 640, (1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 127, 128, 129, 0)
    cols = 64 * len(lengths)
    B = np.zeros((n, cols))
    for c in range(cols):                                  # lists of those lengths, 64 of each; rows 0 to 9 in most of them
        L = lengths[c % len(lengths)]
        rows = np.concatenate([np.arange(min(10, L)), 10 + rng.choice(n - 10, size=max(0, L - 10), replace=False)])
        B[rows, c] = 2.0 ** rng.integers(-2, 3, size=L)
    A = []
    for count in (1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 17, 31, 32, 33, 48, 49, 63, 64, 65, 128, 130):
        for L in (1, 16, 17, 33, 129, None):               # `count` lists of one length, or of all lengths
            of = np.arange(cols) if L is None else np.flatnonzero(np.arange(cols) % len(lengths) == lengths.index(L))
            row = np.zeros(cols)
            chosen = rng.choice(of, size=min(count, len(of)), replace=False)
            row[chosen] = 2.0 ** rng.integers(-2, 3, size=len(chosen))
            A.append(row)
    A, B = synth.from_dense(np.array(A)), synth.from_dense(B)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric])
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd)
    got = _np(h.pairwise(dA, dB, metric))
    if metric in ("inner_product", "l1"):
        assert np.array_equal(got, want.astype(np.float32))
    else:
        assert_distances_close(got, want, metric)
    idx, dist = h.knn(dA, dB, metric, 20)
    assert_knn_matches(_np(idx), _np(dist), want, 20, metric, metric)
    h.close()


def test_a_sum_is_formed_in_the_order_of_the_columns(spd):
    """Products of 2^55 and 1 of either sign: a sum in 64 bits depends on the order of its terms, and is the one of ascending
    columns also where the chunks of a step hold entries of one row (lists of 1 to 16 entries, four of them to a step,
    most with the same rows), across steps and across batches of 64 entries."""
    rng = np.random.default_rng(60)
    m, n, cols = 40, 640, 400
    B = np.zeros((n, cols))
    for c in range(cols):
        rows = rng.choice(24, size=rng.integers(1, 17), replace=False)
        B[rows, c] = rng.choice([-1.0, 1.0], size=len(rows))
    B[np.arange(24, n), rng.integers(0, cols, size=n - 24)] = 1.0
    A = np.zeros((m, cols))
    for r in range(m):
        chosen = rng.choice(cols, size=(4, 16, 64, 65, 200)[r % 5], replace=False)
        A[r, chosen] = np.where(rng.random(len(chosen)) < 0.4, 2.0 ** 55, 1.0)
    want = np.zeros((m, n))
    for c in range(cols):
        want += np.outer(A[:, c], B[:, c])                 # (one column after the other)
    other = np.zeros((m, n))
    for c in reversed(range(cols)):
        other += np.outer(A[:, c], B[:, c])
    assert (want[:, :24].astype(np.float32) != other[:, :24].astype(np.float32)).mean() > 0.05
    dA, dB = (spd.DeviceCsr.from_host(synth.from_dense(M)) for M in (A, B))
    h = _lists(spd)
    for _ in range(3):
        assert np.array_equal(_np(h.pairwise(dA, dB, "inner_product")), want.astype(np.float32))
    h.close()


@pytest.mark.parametrize("metric", ["inner_product", "cosine", "l2_expanded", "correlation", "canberra", "l1"])
def test_sums_that_cancel(spd, metric):
    """Pairs that share columns and whose sum is 0 all the same count as any other pair: rows of both signs in every tile, nearer and
    farther than the rows that share nothing."""
    rng = np.random.default_rng(61)
    cols, m, n = 20_000, 1_024, 13_000
    base = np.sort(rng.choice(np.arange(50, cols), size=(n, 3)), axis=1)
    keep = np.concatenate([np.ones((n, 1), bool), np.diff(base, axis=1) > 0], axis=1)
    size = np.where(rng.random(n) < 0.3, 0.25, 2.0)        # small rows: nearer than any that shares nothing
    indices, values, indptr = [], [], [0]
    for r in range(n):
        pair = 2 * int(rng.integers(0, 25))                # (two columns below 50 of opposite sign: 0 against equal entries)
        sign = size[r] * rng.choice([-1.0, 1.0])
        indices += [pair, pair + 1] + base[r][keep[r]].tolist()
        values += [sign, -sign if r % 3 else sign] + [size[r]] * int(keep[r].sum())
        indptr.append(len(indices))
    B = {"n_rows": n, "n_cols": cols, "indptr": np.array(indptr, np.int64), "indices": np.array(indices, np.int32), "values": np.array(values, np.float32)}
    pairs = 2 * (np.arange(m) % 25)
    A = {"n_rows": m, "n_cols": cols, "indptr": np.arange(m + 1, dtype=np.int64) * 2,
         "indices": np.stack([pairs, pairs + 1], axis=1).reshape(-1).astype(np.int32), "values": np.full(2 * m, 0.5, np.float32)}
    rows = np.arange(0, m, 37)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], rows_a=rows)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd)
    assert_distances_close(_np(h.pairwise(dA, dB, metric))[rows], want, metric)
    for k in (1, 7, 40):
        idx, dist = h.knn(dA, dB, metric, k)
        assert_knn_matches(_np(idx)[rows], _np(dist)[rows], want, k, metric, "%s k=%d" % (metric, k))
    h.close()


@pytest.mark.parametrize("metric", ["l2_expanded", "l1", "hamming", "jensen_shannon", "minkowski"])
@pytest.mark.parametrize("m,n,cols,lengths_a,lengths_b", [
    (20, 1300, 1203, (1200, 257, 256, 900, 5, 0, 1203), (30, 3, 200)),           # rows that wavefronts share, one per tile and more
    (33, 21_001, 3_001, (40, 2, 300, 0, 64), (31, 0, 37, 40)),                  # tiles dealt to the XCDs: 16 or more, lists beyond an L2
])
def test_shared_rows_and_many_tiles(spd, metric, m, n, cols, lengths_a, lengths_b):
    rng = np.random.default_rng(n)

    def matrix(rows, lengths):
        indptr, indices, values = [0], [], []
        for r in range(rows):
            c = np.unique(rng.integers(0, cols, size=lengths[r % len(lengths)]))
            indices.append(c)
            values.append(rng.integers(0, 9, size=len(c)) / 8.0)                 # an eighth of them stored zeros
            indptr.append(indptr[-1] + len(c))
        return {"n_rows": rows, "n_cols": cols, "indptr": np.asarray(indptr, dtype=np.int64),
                "indices": np.concatenate(indices).astype(np.int32), "values": np.concatenate(values).astype(np.float32)}

    A, B = matrix(m, lengths_a), matrix(n, lengths_b)
    print("match lists", metric, m, n, cols, flush=True)
    h = _lists(spd)
    p = _p_of(metric)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
    idx, dist = h.knn(dA, dB, metric, 64, p)
    assert_knn_matches(_np(idx), _np(dist), want, 64, metric, metric)
    h.close()


@pytest.mark.parametrize("metric", ["cosine", "l1", "hamming", "canberra", "kl_divergence", "jensen_shannon", "minkowski"])
@pytest.mark.parametrize("mean_a,mean_b", [(600, 2), (400, 60), (2, 900), (30, 30)])
def test_operands_of_different_laws_and_the_way_they_take(spd, metric, mean_a, mean_b):
    """Long rows against short ones, either way round, wherever the lists are wanted and where the default puts them."""
    rng = np.random.default_rng(mean_a)
    cols, m, n = 5_000, 700, 2_600

    def matrix(rows, mean):
        c = [np.unique(rng.integers(0, cols, size=int(x))) for x in rng.poisson(mean, size=rows)]
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(x) for x in c])]).astype(np.int64),
                "indices": np.concatenate(c).astype(np.int32), "values": (rng.integers(1, 9, size=sum(map(len, c))) / 8.0).astype(np.float32)}

    A, B = matrix(m, mean_a), matrix(n, mean_b)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    p = _p_of(metric)
    rows = np.unique(rng.integers(0, m, size=40))
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p, rows_a=rows)
    lists, default = _lists(spd), spd.Handle()
    default.set_option("profile", 1)
    for h in (lists, default):
        for k in (0, 17):
            print("laws", metric, mean_a, mean_b, k, flush=True)
            if k == 0:
                assert_distances_close(_np(h.pairwise(dA, dB, metric, p))[rows], want, metric)
            else:
                idx, dist = h.knn(dA, dB, metric, k, p)
                assert_knn_matches(_np(idx)[rows], _np(dist)[rows], want, k, metric, metric)
            if h is default:
                plan = spd.testing.host_list_plan(m, int(A["indptr"][-1]), n, int(B["indptr"][-1]), cols, metric, p, k_neighbors=k)
                assert ({r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}) == bool(plan["wanted"])
    lists.close()
    default.close()


@pytest.mark.parametrize("metric", ["cosine", "jensen_shannon", "jaccard", "minkowski"])
def test_same_as_the_staged_scan(spd, metric):
    """Several thousand rows by the shapes of the synthetic data, rows longer than a batch, lists longer than a step."""
    A, B = synth.workload(1, scale=0.3)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    p = _p_of(metric)
    lists, staged = _lists(spd), spd.Handle()
    staged.set_option("match_lists", 0)
    got, want = _np(lists.pairwise(dA, dB, metric, p)), _np(staged.pairwise(dA, dB, metric, p))
    # two roundings to single precision of sums that differ by the order of their double precision terms
    assert np.allclose(got, want, rtol=2.5e-7, atol=1e-7)
    assert np.array_equal(got, _np(lists.pairwise(dA, dB, metric, p)))          # and the same bits every time
    gi, gd = lists.knn(dA, dB, metric, 32, p)
    wi, wd = staged.knn(dA, dB, metric, 32, p)
    assert np.allclose(_np(gd), _np(wd), rtol=2.5e-7, atol=1e-7)
    assert np.mean(_np(gi) != _np(wi)) <= 1e-3
    lists.close()
    staged.close()


@pytest.mark.parametrize("entry", ["pairwise", "knn", "index_pairwise"])
@pytest.mark.parametrize("fault", ["row longer than the column count", "pointers do not begin at 0", "pointers decrease", "last pointer"])
def test_what_the_staged_scan_refuses_is_refused(spd, entry, fault):
    """The same operands, malformed one at a time, through both ways: the same status, and where nothing is refused (the
    scan looks at the lengths of the operand it stages alone) none from either."""
    rng = np.random.default_rng(3)
    good = _matrix(rng, 40, 30, (3, 17, 0, 9))

    def malformed():
        m = {name: (value.copy() if hasattr(value, "copy") else value) for name, value in good.items()}
        if fault == "row longer than the column count":         # (a column twice: 40 entries in 30 columns)
            long_row = np.sort(np.concatenate([np.arange(30), np.arange(10)])).astype(np.int32)
            m["indices"] = np.concatenate([m["indices"], long_row])
            m["values"] = np.concatenate([m["values"], np.full(40, 0.5, dtype=np.float32)])
            m["indptr"] = np.concatenate([m["indptr"], m["indptr"][-1:] + 40])
            m["n_rows"] += 1
        elif fault == "pointers do not begin at 0":
            m["indptr"][0] = 1
        elif fault == "pointers decrease":
            m["indptr"][5] = m["indptr"][9] + 1
        else:
            m["indptr"][-1] += 1
        return m

    def status(lists, swap, A, B):
        h = spd.Handle()
        h.set_option("match_lists", lists)
        h.set_option("swap_operands", swap)
        dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
        try:
            if entry == "pairwise":
                h.pairwise(dA, dB, "l1")
            elif entry == "knn":
                h.knn(dA, dB, "l1", 3)
            else:
                ix = h.index_create(dB, "l1")
                try:
                    ix.pairwise(dA)
                finally:
                    ix.close()
            return "SPD_OK"
        except spd.SpdError as e:
            return e.status_name
        finally:
            h.close()

    for A, B in ((malformed(), good), (good, malformed())):
        for swap in (0, 2):
            print("refusals", entry, fault, swap, flush=True)
            assert status(2, swap, A, B) == status(0, swap, A, B)
    assert status(2, 0, malformed(), good) != "SPD_OK"


def test_refusals_and_documented_scratch(spd):
    import torch
    A, B = synth.workload(0)
    h = _lists(spd)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    bad = dict(A, indptr=A["indptr"].copy())
    bad["indptr"][3] = bad["indptr"][5] + 1
    for first, second in ((spd.DeviceCsr.from_host(bad), dB), (dA, spd.DeviceCsr.from_host(bad))):
        with pytest.raises(spd.SpdError) as e:
            h.pairwise(first, second, "l1")
        assert e.value.status_name == "SPD_ERR_BAD_CSR"
    want = oracle.pairwise(A, B, "manhattan")
    need = h.workspace_bytes(dA, dB, "l1")
    h.set_workspace(torch.empty(need, dtype=torch.uint8, device="cuda"))
    assert_distances_close(_np(h.pairwise(dA, dB, "l1")), want, "documented scratch")
    h.close()


def test_scratch_for_the_lists_over_all_columns_alone(spd):
    """Scratch that holds the lists over all columns and not the copy, which would be preferred: the bits of the former."""
    import torch
    rng = np.random.default_rng(83)
    m, n, cols, nnz = 133, 13_649, 328_013, 2_082_360

    def matrix(rows, entries):
        cell = np.unique(rng.integers(0, rows * cols, size=entries))
        indptr = np.concatenate([[0], np.cumsum(np.bincount(cell // cols, minlength=rows))]).astype(np.int64)
        return spd.DeviceCsr.from_host({"n_rows": rows, "n_cols": cols, "indptr": indptr, "indices": (cell % cols).astype(np.int32),
                                        "values": (rng.random(len(cell)) + 0.01).astype(np.float32)})

    dA, dB = matrix(m, 137), matrix(n, nnz)
    sizes = (m, dA.nnz, n, dB.nnz, cols, "l2_expanded")
    plans = [spd.testing.host_list_plan(*sizes, match_lists=way) for way in (1, 2)]
    assert plans[0]["way"] == 2 and plans[1]["scratch_bytes"] < plans[0]["scratch_bytes"]
    want = _lists(spd).pairwise(dA, dB, "l2_expanded")
    h = spd.Handle()
    h.set_option("check_plan", 1)
    h.set_option("profile", 1)
    h.set_workspace(torch.empty(plans[1]["scratch_bytes"] + 4_096, dtype=torch.uint8, device="cuda"))
    assert torch.equal(h.pairwise(dA, dB, "l2_expanded"), want)
    names = {r["name"] for r in h.profile_read()}
    assert "lists_b" in names and "columns" not in names
    h.set_workspace(torch.empty(plans[0]["scratch_bytes"], dtype=torch.uint8, device="cuda"))
    assert torch.allclose(h.pairwise(dA, dB, "l2_expanded"), want, rtol=2.5e-7, atol=1e-7)
    assert "columns" in {r["name"] for r in h.profile_read()}
    h.close()


def test_scratch_for_the_scan_alone(spd):
    """Scratch that holds what the staged scan needs and not the lists, lent by the caller or the static array: the same bits as
    the staged scan, and two roundings of reordered fp64 sums from the lists."""
    import torch
    A, B = synth.workload(1, scale=7.5)
    A = synth.slice_rows(A, 0, 500)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    lists, staged = _lists(spd, profile=1), spd.Handle()
    staged.set_option("match_lists", 0)
    kinds = lambda h: {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"}
    for metric in ("cosine", "jensen_shannon"):
        sizes = (A["n_rows"], int(A["indptr"][-1]), B["n_rows"], int(B["indptr"][-1]), B["n_cols"], metric)
        assert spd.testing.host_list_plan(*sizes, match_lists=2)["scratch_bytes"] > 32 << 20
        assert spd.testing.host_list_plan(*sizes)["wanted"]                 # (by default too)
        want, scan = lists.pairwise(dA, dB, metric), staged.pairwise(dA, dB, metric)
        assert kinds(lists) == {6}
        assert torch.allclose(want, scan, rtol=2.5e-7, atol=1e-7)
        got = torch.empty_like(want)
        lists.pairwise_static(dA, dB, metric, got)
        assert torch.equal(got, scan)
        lists.set_workspace(torch.empty(32 << 20, dtype=torch.uint8, device="cuda"))
        assert torch.equal(lists.pairwise(dA, dB, metric), scan) and 6 not in kinds(lists)
        lists.set_workspace(None)
    lists.close()
    staged.close()


def test_an_index_under_other_options_and_on_other_streams(spd):
    """The lists of an index serve the options it was created under; a second handle on a stream of its own reads the same ones."""
    import torch
    A, B = synth.workload(1, scale=0.3)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd, profile=1)
    kinds = lambda handle: {r["staging_kind"] for r in handle.profile_read() if r["name"] == "scan"}
    want = oracle.pairwise(A, B, "canberra")
    plain = h.pairwise(dA, dB, "canberra")
    ix = h.index_create(dB, "canberra")
    assert torch.equal(ix.pairwise(dA), plain) and kinds(h) == {6}
    for name, value, before in (("lds_budget", 98304, 163840), ("match_lists", 0, 2)):
        h.set_option(name, value)
        assert_distances_close(_np(ix.pairwise(dA)), want, name)
        assert 6 not in kinds(h)
        h.set_option(name, before)
    assert torch.equal(ix.pairwise(dA), plain) and kinds(h) == {6}
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        other = _lists(spd, profile=1)
        view = type(ix)(other, ix._ptr, dB)
        for _ in range(3):                                      # both at once
            theirs, ours = view.pairwise(dA), ix.pairwise(dA)
            torch.cuda.synchronize()
            assert torch.equal(theirs, plain) and torch.equal(ours, plain)
        assert kinds(other) == {6}
        view._ptr = None                                        # (ix owns it)
        other.close()
    ix.close()
    h.close()


def test_the_profile_has_a_record_for_every_launch(spd):
    A, B = synth.workload(0)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd, profile=1)

    def names(call):
        call()
        records = h.profile_read()
        assert all(r["ms"] > 0.0 for r in records)
        return [r["name"] for r in records]

    build = ["norms_b", "lists_b"]
    assert names(lambda: h.pairwise(dA, dB, "l1")) == build + ["norms_a", "scan"]
    assert names(lambda: h.knn(dA, dB, "l1", 5)) == build + ["norms_a", "knn_begin", "scan", "knn_merge"]
    ix = h.index_create(dB, "l1")
    assert [r["name"] for r in h.profile_read()] == ["pack_b"] + build
    assert names(lambda: ix.pairwise(dA)) == ["norms_a", "scan"]
    assert names(lambda: ix.knn(dA, 5)) == ["norms_a", "knn_begin", "scan", "knn_merge"]
    ix.close()
    h.close()


def test_the_profile_over_the_columns_of_a(spd):
    A, B = synth.workload(0)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd, match_lists=3, profile=1)
    build = ["norms_b", "columns", "lists_b", "norms_a"]
    h.pairwise(dA, dB, "l1")
    assert [r["name"] for r in h.profile_read()] == build + ["scan"]
    h.knn(dA, dB, "l1", 5)
    assert [r["name"] for r in h.profile_read()] == build + ["knn_begin", "scan", "knn_merge"]
    h.close()


@pytest.mark.parametrize("metric", ["inner_product", "cosine", "kl_divergence"])
def test_a_value_that_is_not_finite_stays_in_its_row(spd, metric):
    """Row 7 of A, shared by a workgroup's wavefronts, meets a dense column of B with an infinity: what it leaves behind the
    last tile's end must not reach the distances of the rows that the same wavefronts take next."""
    rng = np.random.default_rng(77)
    cols, m, n = 3_001, 520, 21_001                    # 18 tiles in 8 groups, 32 slices of A's rows

    def matrix(rows, lengths):
        c = [np.unique(np.concatenate([[2], rng.integers(0, cols, size=lengths[r % len(lengths)])])) for r in range(rows)]
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(x) for x in c])]).astype(np.int64),
                "indices": np.concatenate(c).astype(np.int32), "values": (rng.integers(1, 9, size=sum(map(len, c))) / 8.0).astype(np.float32)}

    A, B = matrix(m, (40,) * 7 + (1_200,) + (40,) * 512), matrix(n, (31, 29, 37, 40))
    plan = spd.testing.host_list_plan(m, int(A["indptr"][-1]), n, int(B["indptr"][-1]), cols, metric, match_lists=2)
    assert plan["groups"] < plan["tiles"] and n % plan["tile_rows"] != 0
    bad = dict(A, values=A["values"].copy())
    bad["values"][A["indptr"][7] + int(np.searchsorted(A["indices"][A["indptr"][7]:A["indptr"][8]], 2))] = np.inf
    h = _lists(spd)
    dB = spd.DeviceCsr.from_host(B)
    want, got = (_np(h.pairwise(spd.DeviceCsr.from_host(M), dB, metric)) for M in (A, bad))
    others = np.arange(m) != 7
    assert np.array_equal(got[others], want[others])
    wi, wd = h.knn(spd.DeviceCsr.from_host(A), dB, metric, 9)
    gi, gd = h.knn(spd.DeviceCsr.from_host(bad), dB, metric, 9)
    assert np.array_equal(_np(gi)[others], _np(wi)[others]) and np.array_equal(_np(gd)[others], _np(wd)[others])
    h.close()


@pytest.mark.parametrize("metric", ["l1", "l2_expanded", "hellinger", "canberra", "jensen_shannon", "hamming"])
def test_the_row_of_the_least_norm_wherever_it_lies_in_its_tile(spd, metric):
    """k-NN passes over a tile that a row meets in a few entries where the tile's row of the least norm is no nearer than the k-th
    neighbour so far: one short row per tile, at the places where the search for it goes from lane to lane, is the nearest
    of all rows that share no column with the query, the nearer the later its tile."""
    cols, m = 30_000, 1_024

    def plan(n):
        return spd.testing.host_list_plan(m, 2 * m, n, 4 * n, cols, metric, k_neighbors=2, match_lists=2)

    tile = max(plan(n)["tile_rows"] for n in (40_000, 400_000))
    places = (0, 1, 63, 64, 127, 128, 255, 256, 257, tile - 1, 17)
    n = tile * len(places) - 40
    assert plan(n)["tile_rows"] == tile and plan(n)["tiles"] == len(places) > plan(n)["groups"]
    rng = np.random.default_rng(n)
    c = np.sort(rng.integers(1_000, cols - 4, size=(n, 1)) + np.arange(4), axis=1)
    values = np.full((n, 4), 2.0)
    for t, at in enumerate(places):
        values[t * tile + at] = 0.0                        # (stored zeros are absent: one entry stays)
        values[t * tile + at, 0] = 1.0 - t / 16.0
    B = {"n_rows": n, "n_cols": cols, "indptr": np.arange(n + 1, dtype=np.int64) * 4, "indices": c.reshape(-1).astype(np.int32),
         "values": values.reshape(-1).astype(np.float32)}
    ca = np.stack([np.arange(m) % 900, 1_000 + np.arange(m) * 28], axis=1)     # (the second column meets a row here and there)
    A = {"n_rows": m, "n_cols": cols, "indptr": np.arange(m + 1, dtype=np.int64) * 2, "indices": ca.reshape(-1).astype(np.int32),
         "values": np.full(2 * m, 0.5, np.float32)}
    rows = np.arange(0, m, 17)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], rows_a=rows)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd)
    for k in (1, 2, 13):
        idx, dist = h.knn(dA, dB, metric, k)
        assert_knn_matches(_np(idx)[rows], _np(dist)[rows], want, k, metric, "%s k=%d" % (metric, k))
    h.close()


@pytest.mark.parametrize("metric", ["l1", "l2_expanded", "hellinger", "cosine", "canberra", "jensen_shannon"])
def test_a_tile_is_not_passed_over_for_a_norm_that_is_not_a_number(spd, metric):
    """A row of B that holds a NaN shares no column with the queries and lies in a late tile, behind rows that bound the k-th
    distance: the neighbours are the staged scan's, which takes a sum that is not a number for 0."""
    cols, m, most = 30_000, 1_024, 1_216
    n = 11 * most - 40
    rng = np.random.default_rng(5)
    c = np.sort(rng.integers(1_000, cols - 4, size=(n, 1)) + np.arange(4), axis=1)
    values = np.full((n, 4), 2.0)
    values[9 * most + 300, 1] = values[10 * most + 7, 3] = np.nan
    B = {"n_rows": n, "n_cols": cols, "indptr": np.arange(n + 1, dtype=np.int64) * 4, "indices": c.reshape(-1).astype(np.int32),
         "values": values.reshape(-1).astype(np.float32)}
    A = {"n_rows": m, "n_cols": cols, "indptr": np.arange(m + 1, dtype=np.int64) * 2,
         "indices": np.stack([np.arange(m) % 900, 900 + np.arange(m) % 100], axis=1).reshape(-1).astype(np.int32),
         "values": np.full(2 * m, 0.5, np.float32)}
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    plan = spd.testing.host_list_plan(m, 2 * m, n, 4 * n, cols, metric, k_neighbors=3, match_lists=2)
    assert plan["tile_rows"] == most and plan["tiles"] == 11 > plan["groups"]
    h, staged = _lists(spd), _lists(spd, match_lists=0)
    for k in (1, 5):
        for got, want in zip(h.knn(dA, dB, metric, k), staged.knn(dA, dB, metric, k)):
            assert np.array_equal(_np(got), _np(want)), (metric, k)
    staged.close()
    h.close()


@pytest.mark.parametrize("metric", ["inner_product", "cosine", "kl_divergence"])
def test_a_value_that_is_not_finite_stays_in_its_row_over_runs_of_tiles(spd, metric):
    """Every 20th row of A, each one wavefront's but the first, which the workgroup's wavefronts share, meets a dense column of B
    with an infinity.  A wavefront goes through a run of three tiles with a row: behind the last, short tile come an
    earlier, full one and another row."""
    rng = np.random.default_rng(78)
    cols, m = 3_001, 2_100

    def matrix(rows, lengths):
        c = [np.unique(np.concatenate([[2], rng.integers(0, cols, size=lengths[r % len(lengths)])])) for r in range(rows)]
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(x) for x in c])]).astype(np.int64),
                "indices": np.concatenate(c).astype(np.int32), "values": (rng.integers(1, 9, size=sum(map(len, c))) / 8.0).astype(np.float32)}

    most = max(spd.testing.host_list_plan(m, 40 * m, n, 45 * n, cols, metric, match_lists=2)["tile_rows"] for n in (40_000, 400_000))
    n = 17 * most + most * 9 // 16                     # 18 tiles in 8 groups, 32 slices of A's rows; column 2 is dense in the last tile too
    A, B = matrix(m, (40,) * 7 + (1_200,) + (40,) * (m - 8)), matrix(n, (43, 41, 49, 52))
    for k in (0, 9):
        plan = spd.testing.host_list_plan(m, int(A["indptr"][-1]), n, int(B["indptr"][-1]), cols, metric, k_neighbors=k, match_lists=2)
        assert plan["tile_rows"] == most and plan["tiles"] == 18 and plan["groups"] == 8 and plan["run"] >= 3
    assert -(-(n - 17 * most) // 256) * 256 < most     # (rows that no result is read from, and a round of 256 rows does not reach)
    bad = dict(A, values=A["values"].copy())
    rows = np.arange(7, m, 20)
    for r in rows:
        bad["values"][A["indptr"][r] + int(np.searchsorted(A["indices"][A["indptr"][r]:A["indptr"][r + 1]], 2))] = np.inf
    others = np.setdiff1d(np.arange(m), rows)
    h = _lists(spd)
    dB = spd.DeviceCsr.from_host(B)
    want, got = (_np(h.pairwise(spd.DeviceCsr.from_host(M), dB, metric))[others] for M in (A, bad))
    assert np.array_equal(got, want)
    (wi, wd), (gi, gd) = (h.knn(spd.DeviceCsr.from_host(M), dB, metric, 9) for M in (A, bad))
    assert np.array_equal(_np(gi)[others], _np(wi)[others]) and np.array_equal(_np(gd)[others], _np(wd)[others])
    h.close()


# columns: one word of 32, its end, a workgroup's 4,096 words and beyond them; entries of B: under a mask of 64, at the ends of
# masks and of a workgroup's 4,096 entries, and more than 1,024 workgroups (the sums of sums)
@pytest.mark.parametrize("metric", SERVED)
@pytest.mark.parametrize("m,n,cols,lengths_a,lengths_b", [(1, 1, 5, (3,), (4,)), (3, 63, 33, (1, 7, 0), (1, 1, 0, 2)),
                                                          (21, 1300, 131_073, (2, 65, 0, 300, 1), (5, 0, 40, 3)),
                                                          (40, 1025, 4_000, (1, 2, 3), (4,)), (9, 64, 1 << 21, (64, 700), (64, 128))])
def test_lists_over_the_columns_of_a(spd, metric, m, n, cols, lengths_a, lengths_b):
    rng = np.random.default_rng(cols + n)
    head = rng.choice(cols, size=min(cols, 60), replace=False)             # most entries lie here, the others anywhere

    def matrix(rows, lengths):
        c = [np.unique(np.concatenate([rng.choice(head, size=min(len(head), (3 * k + 3) // 4), replace=False), rng.integers(0, cols, size=k // 4)]))
             if (k := lengths[r % len(lengths)]) else np.zeros(0, np.int64) for r in range(rows)]
        values = rng.integers(0, 9, size=sum(map(len, c))) / 8.0           # (a stored zero among them)
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(x) for x in c])]).astype(np.int64),
                "indices": np.concatenate(c).astype(np.int32), "values": values.astype(np.float32)}

    A, B = matrix(m, lengths_a), matrix(n, lengths_b)
    print("lists over A's columns", metric, m, n, cols, flush=True)
    p, k = _p_of(metric), min(n, 33)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd, match_lists=3, profile=1)
    assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
    assert [r["name"] for r in h.profile_read()][:3] == ["norms_b", "columns", "lists_b"]
    idx, dist = h.knn(dA, dB, metric, k, p)
    assert_knn_matches(_np(idx), _np(dist), want, k, metric, metric)
    index = h.index_create(dB, metric, p)
    assert np.array_equal(_np(index.pairwise(dA)), _np(h.pairwise(dA, dB, metric, p)))
    i2, d2 = index.knn(dA, k)
    assert np.array_equal(_np(i2), _np(idx)) and np.array_equal(_np(d2), _np(dist))
    index.close()
    h.close()


def test_columns_of_many_entries(spd):
    """Enough entries of B for a second round of the sums of sums, values that are exact in any order."""
    rng = np.random.default_rng(3)
    cols, m, n, per = 300_000, 24, 70_000, 62                              # 4.3 M entries: 1,060 workgroups
    cb = np.sort(np.concatenate([rng.integers(0, 40, size=(n, 2)), rng.integers(0, cols, size=(n, per - 2))], axis=1), axis=1)
    keep = np.concatenate([np.ones((n, 1), bool), np.diff(cb, axis=1) > 0], axis=1)
    B = {"n_rows": n, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64),
         "indices": cb[keep].astype(np.int32), "values": rng.integers(1, 5, size=int(keep.sum())).astype(np.float32)}
    rows = [np.unique(np.concatenate([np.arange(r, 40, 3), rng.integers(0, cols, size=50 * r)])) for r in range(m)]
    A = {"n_rows": m, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64),
         "indices": np.concatenate(rows).astype(np.int32), "values": rng.integers(1, 5, size=sum(map(len, rows))).astype(np.float32)}
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    staged, h = _lists(spd, match_lists=0), _lists(spd, match_lists=3)
    for metric in ("inner_product", "l1", "jaccard"):
        assert np.array_equal(_np(h.pairwise(dA, dB, metric)), _np(staged.pairwise(dA, dB, metric)))
        for got, want in zip(h.knn(dA, dB, metric, 10), staged.knn(dA, dB, metric, 10)):
            assert np.array_equal(_np(got), _np(want))
    staged.close()
    h.close()


@pytest.fixture()
def scarce(spd):
    """Operands whose lists (a word per tile and column) take more memory than the device has left, and whose scan takes
    some megabytes."""
    import torch
    rng = np.random.default_rng(8)
    cols = 2_000_000_000

    def matrix(rows):
        c = np.sort(rng.integers(0, 40, size=(rows, 6)) + 49_999_999 * rng.integers(0, 40, size=(rows, 1)), axis=1)
        keep = np.concatenate([np.ones((rows, 1), bool), np.diff(c, axis=1) > 0], axis=1)
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64),
                "indices": c[keep].astype(np.int32), "values": rng.integers(1, 9, size=int(keep.sum())).astype(np.float32)}

    dA, dB = spd.DeviceCsr.from_host(matrix(5)), spd.DeviceCsr.from_host(matrix(2_000))
    staged = spd.Handle()
    staged.set_option("match_lists", 0)
    want = _np(staged.pairwise(dA, dB, "minkowski", 3.0))
    staged.close()
    h = _lists(spd, profile=1)
    need = h.workspace_bytes(dA, dB, "minkowski")
    assert need > 30 << 30
    filler = torch.empty(torch.cuda.mem_get_info()[0] - need // 2, dtype=torch.uint8, device="cuda")
    yield h, dA, dB, want
    h.close()
    del filler
    torch.cuda.empty_cache()


def test_a_call_without_memory_for_the_lists_takes_the_scan(scarce):
    h, dA, dB, want = scarce
    print("lists beyond the device's memory", flush=True)
    for _ in range(2):
        assert np.array_equal(_np(h.pairwise(dA, dB, "minkowski", 3.0)), want)
        assert all(r["staging_kind"] != 6 for r in h.profile_read() if r["name"] == "scan")
    idx, dist = h.knn(dA, dB, "minkowski", 4, 3.0)
    assert np.array_equal(_np(dist), np.sort(want, axis=1)[:, :4])


def test_an_index_without_memory_for_the_lists_keeps_the_packed_copy(scarce):
    h, dA, dB, want = scarce
    print("index, lists beyond the device's memory", flush=True)
    ix = h.index_create(dB, "minkowski", 3.0)
    assert np.array_equal(_np(ix.pairwise(dA)), want)
    idx, dist = ix.knn(dA, 4)
    assert np.array_equal(_np(dist), np.sort(want, axis=1)[:, :4])
    ix.close()


@pytest.mark.parametrize("metric", ["cosine", "l2_expanded", "correlation", "hellinger", "l1", "canberra"])
@pytest.mark.parametrize("n,long_every", [(640, 16), (130, 1)])           # lists, and columns that more than half of the rows store
def test_sums_in_fixed_point(spd, metric, n, long_every):
    """Rows whose values lie 2^80 apart, of one entry and of more than 4,096 that two rows share, entries 2^26 apart in a row, rows that
    equal one another.  L1 and Canberra: a term is rounded to 2^-52 of the row's largest (match_fixed in spd_match.h), so a sum of
    `terms` of them is off by terms * 2^-52 * largest at most.  The distances of a dot product, whose sums are in fp64: by terms * 2^-53 of
    what the sum has come to.  A distance is off by that and two roundings to single precision."""
    rng = np.random.default_rng(n)
    cols, m = 6_000, 20
    signed = metric in ("cosine", "l2_expanded", "correlation", "l1", "canberra")

    def matrix(rows, long_rows, exponents):
        d = np.zeros((rows, cols))
        for r in range(rows):
            size = 5_400 if r % long_rows == 0 else (1, 3, 40)[r % 3]
            c = rng.choice(cols, size=size, replace=False)
            v = rng.integers(1, 1 << 12, size=size) * 2.0 ** rng.integers(-26, 1, size=size)
            if signed:
                v *= rng.choice([-1.0, 1.0], size=size)
            d[r, c] = v * 2.0 ** exponents[r % len(exponents)]
        return d

    exponents = (0, -40, 0, 40, -1) if metric != "correlation" else (0, -20, 20)
    A, B = matrix(m, 2, exponents), matrix(n, long_every, exponents)
    B[16 if long_every > 1 else 1] = A[0]
    A, B = synth.from_dense(A), synth.from_dense(B)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric])
    h = _lists(spd)
    got = _np(h.pairwise(spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B), metric)).astype(np.float64)
    h.close()

    def rows_of(M, f):
        return np.array([f(M["values"][M["indptr"][r]:M["indptr"][r + 1]].astype(np.float64)) for r in range(M["n_rows"])])

    terms = 5_400.0
    units = 4.0 * terms * 2.0 ** -52                       # of rows' largest entries; 4: the norms' own sums, and a scale above the largest
    if metric == "canberra":
        # (a ratio is formed in single precision through a reciprocal: 2^-22 of it, on no more than the shared columns)
        bound = 2.0 ** -22 * np.abs(want) + units * 2.0
    elif metric == "l1":
        size = rows_of(A, lambda v: np.abs(v).sum())[:, None] + rows_of(B, lambda v: np.abs(v).sum())[None, :]
        bound = 2.0 ** -23 * np.abs(want) + units * size
    elif metric in ("l2_expanded", "hellinger"):
        f = (lambda v: (v * v).sum()) if metric == "l2_expanded" else (lambda v: v.sum())
        size = rows_of(A, f)[:, None] + rows_of(B, f)[None, :]
        # a root of t + e: e / root(t) at most, root(e) where t is 0
        bound = 2.0 ** -22 * np.abs(want) + np.minimum(units * size / np.maximum(want, 1e-300), np.sqrt(units * size))
    else:
        bound = 2.0 ** -23 * np.abs(want) + units * (cols if metric == "correlation" else 1.0)
    assert np.all(np.abs(got - want) <= bound), float((np.abs(got - want) / bound).max())


@pytest.mark.parametrize("m,n,cols,lengths_a,lengths_b", [
    (1, 1, 5, (3,), (4,)), (3, 63, 70, (1, 7, 0), (1, 0, 2, 40)),
    (70, 65, 200, (31, 32, 33, 64, 65, 130, 0), (31, 32, 33, 2, 100)),           # all the ranked entries of a row and one more
    (40, 2_600, 300, (40, 2, 90, 64), (5, 0, 40, 9, 33)),                        # several tiles, the last one short
    (20, 1_700, 3_003, (2_900, 1_300, 700, 5, 0), (30, 3, 900)),                 # rows that wavefronts share
])
def test_chebyshev_by_lists(spd, m, n, cols, lengths_a, lengths_b):
    """The maximum over shared columns completed from the largest entry that the other row does not store: ranks at their end, rows
    all of whose ranked entries are met (B holds rows of A, and some of them with small entries left out or added), entries that
    tie, stored zeros, either sign.  The staged scan's bits: both take maxima of the same differences."""
    rng = np.random.default_rng(cols + n)
    A, B = _matrix(rng, m, cols, lengths_a), _matrix(rng, n, cols, lengths_b)
    for M in (A, B):
        M["values"] *= rng.choice(np.array([-1.0, 1.0], np.float32), size=len(M["values"]))

    def rows_of(M):
        return [(M["indices"][M["indptr"][r]:M["indptr"][r + 1]], M["values"][M["indptr"][r]:M["indptr"][r + 1]]) for r in range(M["n_rows"])]

    rows = rows_of(B)
    for at, r in enumerate(range(0, m, 3)):                # copies of rows of A, whole, without their least entry, and with one more
        c, v = rows_of(A)[r]
        if at % 3 == 1 and len(c):
            keep = np.arange(len(c)) != np.argmin(np.abs(v))
            c, v = c[keep], v[keep]
        elif at % 3 == 2 and len(c) < cols:
            more = int(np.setdiff1d(np.arange(cols), c)[0])
            where = int(np.searchsorted(c, more))
            c, v = np.insert(c, where, more), np.insert(v, where, np.float32(1.0 / 16.0))
        rows[(at * 7 + 1) % n] = (c, v)
    B = {"n_rows": n, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum([len(c) for c, _ in rows])]).astype(np.int64),
         "indices": np.concatenate([c for c, _ in rows]).astype(np.int32), "values": np.concatenate([v for _, v in rows]).astype(np.float32)}
    print("chebyshev by lists", m, n, cols, flush=True)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h, staged = _lists(spd, profile=1), _lists(spd, match_lists=0)
    got = _np(h.pairwise(dA, dB, "chebyshev"))
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert_distances_close(got, oracle.pairwise(A, B, "chebyshev"), "chebyshev")
    assert np.array_equal(got, _np(staged.pairwise(dA, dB, "chebyshev")))
    idx, dist = h.knn(dA, dB, "chebyshev", min(n, 5))      # (by the scan)
    assert np.array_equal(_np(dist), np.sort(got, axis=1)[:, :min(n, 5)])
    h.close()
    staged.close()


@pytest.mark.parametrize("metric", ["l2_expanded", "hellinger"])
def test_equal_rows_of_two_entries_lie_at_distance_0(spd, metric):
    """The products of two single precision numbers are exact in 64 bits and their sum is rounded once, in the norms as in the inner
    product: nothing is left of |a|^2 - 2 <a, b> + |b|^2 where a and b are equal, whatever the values."""
    rng = np.random.default_rng(12)
    rows, cols = 400, 150
    c = np.sort(np.array([rng.choice(cols, size=2, replace=False) for _ in range(rows)]), axis=1)
    A = {"n_rows": rows, "n_cols": cols, "indptr": 2 * np.arange(rows + 1, dtype=np.int64), "indices": c.reshape(-1).astype(np.int32),
         "values": np.abs(rng.standard_normal(2 * rows)).astype(np.float32)}
    h = _lists(spd, profile=1)
    dA = spd.DeviceCsr.from_host(A)
    got = _np(h.pairwise(dA, dA, metric))
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert np.all(np.diag(got) == 0.0), int((np.diag(got) != 0.0).sum())
    _, dist = h.knn(dA, dA, metric, 1)
    assert np.all(_np(dist) == 0.0)
    h.close()


@pytest.mark.parametrize("n", [640, 70])                # lists, and columns that more than half of the rows store
def test_canberra_of_values_at_the_ends_of_their_range(spd, n):
    """Entries whose magnitudes add up to less than 2^-126, the reciprocal of which single precision does not hold, or to more than it
    holds, equal to their partners, near them and of the other sign: a ratio is between 0 and 1 all the same."""
    rng = np.random.default_rng(n)
    cols, m = 90, 24

    def matrix(rows, share):
        d = np.zeros((rows, cols))
        for r in range(rows):
            c = rng.choice(cols, size=60 if r % share == 0 else 7, replace=False)
            kind = rng.integers(0, 4, size=len(c))
            kind[0] = 0
            tiny, large = rng.integers(1, 1 << 9, size=len(c)) * 2.0 ** -149, rng.integers(1 << 22, 1 << 24, size=len(c)) * 2.0 ** 104
            d[r, c] = np.choose(kind, [tiny, large, 2.0 ** -140 * np.ones(len(c)), rng.integers(1, 9, size=len(c)) / 8.0]) * rng.choice([-1.0, 1.0], size=len(c))
        return d

    A, B = matrix(m, 3), matrix(n, 1 if n < 100 else 16)
    B[5] = A[0]
    A, B = synth.from_dense(A), synth.from_dense(B)
    h = _lists(spd, profile=1)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    want = oracle.pairwise(A, B, "canberra")
    assert_distances_close(_np(h.pairwise(dA, dB, "canberra")), want, "canberra")
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    idx, dist = h.knn(dA, dB, "canberra", 9)
    assert_knn_matches(_np(idx), _np(dist), want, 9, "canberra", "canberra")
    h.close()


@pytest.mark.parametrize("entry,metric,lists", [("pairwise", "chebyshev", 2)] + [
    (entry, metric, lists) for entry, metric in (("pairwise", "l1"), ("pairwise", "cosine"), ("knn", "canberra"), ("index_knn", "jaccard"))
    for lists in (2, 3)])
def test_row_pointers_on_the_gpu_alone(spd, lists, entry, metric):
    """What is launched before the row pointers are on the host: the results of the call that brings them, the same refusals, nothing
    written for a call that is refused, and a sound call after one."""
    import torch
    rng = np.random.default_rng(8)
    A, B = _matrix(rng, 40, 60, (3, 17, 0, 9)), _matrix(rng, 70, 60, (5, 1, 30))
    h = spd.Handle()
    h.set_option("match_lists", lists)
    h.set_option("profile", 1)

    def call(h, MA, MB, keep):
        dA, dB = (spd.DeviceCsr.from_host(M, keep_host_indptr=keep) for M in (MA, MB))
        if entry == "pairwise":
            out = [h.pairwise(dA, dB, metric)]
        elif entry == "knn":
            out = h.knn(dA, dB, metric, 7)
        else:
            ix = h.index_create(spd.DeviceCsr.from_host(B), metric)
            out = ix.knn(dA, 7)
        out = [_np(x) for x in out]
        if entry == "index_knn":
            ix.close()
        return out

    want = call(h, A, B, True)
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    scratch = torch.empty(1 << 22, dtype=torch.uint8, device="cuda")
    h.set_workspace(scratch)
    for fault in ("pointers do not begin at 0", "pointers decrease", "all entries in every other row", "last pointer", "row longer than the column count"):
        for which in (0, 1) if entry != "index_knn" else (0,):
            M = [{name: (value.copy() if hasattr(value, "copy") else value) for name, value in X.items()} for X in (A, B)]
            ip = M[which]["indptr"]
            if fault == "pointers do not begin at 0":
                ip[0] = 1
            elif fault == "pointers decrease":
                ip[5] = ip[9] + 1
            elif fault == "all entries in every other row":
                ip[1:-1:2] = ip[-1]
                ip[2:-1:2] = 0
            elif fault == "last pointer":
                ip[-1] += 1
            else:
                ip[1:-1] = ip[-1]                           # (the first row has them all)
            print("row pointers on the GPU alone", lists, entry, metric, fault, which, flush=True)
            scratch.fill_(0xA5)
            status = []
            for keep in (True, False):
                try:
                    call(h, M[0], M[1], keep)
                    status.append("SPD_OK")
                except spd.SpdError as e:
                    status.append(e.status_name)
            assert status[0] == status[1]
            if fault != "row longer than the column count":
                assert status[1] != "SPD_OK"
                # (over A's columns those are counted beside the row pointers)
                assert lists == 3 or bool((scratch == 0xA5).all().item())
    for got, same in zip(call(h, A, B, False), want):
        assert np.array_equal(got, same)
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    h.close()


@pytest.mark.parametrize("m,n", [(60, 70), (60, 900), (4_200, 66)])              # all rows shared, several tiles, a wavefront to the row
@pytest.mark.parametrize("size,kind", [(32, "one support"), (33, "one support"), (70, "one support"), (70, "a column less"), (150, "a column less"),
                                       (70, "ones and twos"), (140, "stored zeros"), (70, "other places")])
def test_chebyshev_of_rows_that_are_nearly_alike(spd, m, n, size, kind):
    """Rows of A whose 32 largest entries B's rows all store: what decides is among the others, in columns that only one of the two rows
    stores, at the same place in both rows, next to it or elsewhere.  The staged scan's bits."""
    rng = np.random.default_rng(size + n)
    cols = 400
    support = np.sort(rng.choice(np.arange(100, cols), size=size, replace=False))

    def matrix(rows):
        d = np.zeros((rows, cols), np.float32)
        d[:, support] = 1.0
        if kind == "a column less":
            d[np.arange(rows), rng.choice(support, size=rows)] = 0.0
        elif kind == "ones and twos":
            d[:, support[: size // 2]] = 2.0
            d[np.arange(rows), rng.choice(support[size // 2:], size=rows)] = rng.integers(0, 3, size=rows)
        elif kind == "other places":
            for r in range(rows):                          # (entries in front of the shared ones: these lie at other places in the two rows)
                d[r, rng.choice(100, size=r % 5, replace=False)] = 0.5
        return d

    dense = [matrix(m), matrix(n)]
    A, B = (synth.from_dense(d.astype(np.float64)) for d in dense)
    if kind == "stored zeros":
        for M in (A, B):
            M["values"][rng.choice(len(M["values"]), size=len(M["values"]) // 100, replace=False)] = 0.0
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h, staged = _lists(spd, profile=1), _lists(spd, match_lists=0)
    got = _np(h.pairwise(dA, dB, "chebyshev"))
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert np.array_equal(got, _np(staged.pairwise(dA, dB, "chebyshev")))
    assert_distances_close(got[:40], oracle.pairwise(synth.slice_rows(A, 0, 40), B, "chebyshev"), "chebyshev")
    h.close()
    staged.close()


@pytest.mark.parametrize("metric", ["cosine", "correlation", "canberra", "kl_divergence", "jensen_shannon", "minkowski"])
@pytest.mark.parametrize("n,mean_b", [(1_500, 30), (22_000, 30)])                # few tiles, and tiles that are dealt to the XCDs
def test_long_rows_go_to_the_workgroups_as_they_come(spd, metric, n, mean_b):
    """Most of A's rows are shared by the wavefronts of a workgroup, and which workgroup takes one depends on the schedule: the same bits
    every time, and the oracle's distances."""
    rng = np.random.default_rng(n)
    cols, m = 3_001, 90

    def matrix(rows, mean):
        lengths = np.minimum(cols, np.maximum(1, (mean * rng.exponential(size=rows)).astype(int)))
        c = [np.sort(rng.choice(cols, size=k, replace=False)) for k in lengths]
        return {"n_rows": rows, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64),
                "indices": np.concatenate(c).astype(np.int32), "values": rng.integers(1, 1 << 20, size=int(lengths.sum())).astype(np.float32) / (1 << 20)}

    A, B = matrix(m, 900), matrix(n, mean_b)
    h = _lists(spd)
    p = _p_of(metric)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    first = _np(h.pairwise(dA, dB, metric, p)).copy()
    assert_distances_close(first, want, metric)
    idx, dist = (_np(x).copy() for x in h.knn(dA, dB, metric, 20, p))
    assert_knn_matches(idx, dist, want, 20, metric, metric)
    for _ in range(4):
        assert np.array_equal(first, _np(h.pairwise(dA, dB, metric, p)))
        i2, d2 = h.knn(dA, dB, metric, 20, p)
        assert np.array_equal(idx, _np(i2)) and np.array_equal(dist, _np(d2))
    h.close()


# Columns that so many rows store (in turn): around the 16 entries from which on a list begins at a line, with short lists between them; all of them
# lists whose gaps would take more than their block's room, so that it has none; and such that nearly all of its room is gaps.
@pytest.mark.parametrize("metric", ["l1", "cosine", "jaccard", "chebyshev"])
@pytest.mark.parametrize("stored", [(15, 16, 17, 1, 31, 32, 33, 3, 0, 48), (17,), (49, 2, 50, 1, 1, 47)])
def test_lists_that_begin_at_lines(spd, metric, stored):
    rng = np.random.default_rng(len(stored))
    n, cols = 700, 260
    d = np.zeros((n, cols))
    for c in range(cols):
        d[rng.choice(n, size=stored[c % len(stored)], replace=False), c] = rng.integers(1, 9, size=stored[c % len(stored)]) / 8.0
    B = synth.from_dense(d)
    A = _matrix(rng, 40, cols, (3, 64, 65, 1, 130, 0, 17, 260))
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    print("lists at lines", metric, stored, flush=True)
    h = _lists(spd, profile=1)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric])
    assert_distances_close(_np(h.pairwise(dA, dB, metric)), want, metric)
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    if metric != "chebyshev":
        idx, dist = h.knn(dA, dB, metric, 9)
        assert_knn_matches(_np(idx), _np(dist), want, 9, metric, metric)
    h.close()


# Blocks of the build: one that stores far more entries than a workgroup's lanes hold (nearly all rows store the same 70 columns of
# thousands), rows whose stretch of a block is most of it, in all no more entries than are looked at together, in one block and on both sides of
# blocks' ends; with tiles of up to three rows to a lane, ("long tile") of up to five and ("short tile") of one.
@pytest.mark.parametrize("metric", ["l1", "cosine", "hellinger", "jaccard", "hamming", "minkowski", "chebyshev"])
@pytest.mark.parametrize("kind", ["full block", "long tile", "short tile", "long rows", "few entries", "few entries of several blocks"])
def test_blocks_of_the_build(spd, metric, kind):
    rng = np.random.default_rng(3)
    n, cols = {"full block": (2_600, 9_000), "long tile": (2_400, 9_000), "short tile": (900, 9_000), "long rows": (1_100, 12_000), "few entries": (3, 40),
               "few entries of several blocks": (3, 9_000)}[kind]
    budget = 40_000 if kind == "short tile" else 163_840
    cut = spd.testing.host_list_plan(30, 2_000, n, {"few entries": 7, "few entries of several blocks": 7, "long rows": 26_000}.get(kind, 62 * n), cols, metric,
                                     _p_of(metric), match_lists=2, lds_budget=budget)
    width = cut["block_columns"]
    assert kind != "long tile" or metric not in ("jaccard", "hamming") or cut["tile_rows"] > 3 * 512
    assert kind != "short tile" or cut["tile_rows"] <= 512
    assert (width < cols) == (kind != "few entries")
    rows = []
    for r in range(n):
        if kind in ("full block", "long tile", "short tile"):
            c = np.concatenate([100 + rng.choice(70, size=60, replace=False), rng.integers(0, cols, size=2)])
        elif kind == "long rows":
            c = rng.choice(cols, size=11_000, replace=False) if r in (3, 700) else rng.integers(0, cols, size=4)
        elif kind == "few entries":
            c = rng.integers(0, cols, size=(2, 0, 3)[r])
        else:
            c = ((0, width - 1, width, cols - 1), (), (width - 1, width + 1, 2 * width))[r]
        rows.append(np.unique(np.asarray(c, dtype=np.int64)))
    indptr = np.concatenate([[0], np.cumsum([len(c) for c in rows])]).astype(np.int64)
    B = {"n_rows": n, "n_cols": cols, "indptr": indptr, "indices": np.concatenate(rows).astype(np.int32),
         "values": (rng.integers(0, 17, size=int(indptr[-1])) / 8.0).astype(np.float32)}
    if kind == "few entries of several blocks":
        assert 0 < len(B["values"]) < 8
        B["values"] = 1.0 + np.arange(len(B["values"]), dtype=np.float32) / 8.0
    A = _matrix(rng, 30, cols, (3, 64, 65, 1, 130, 0, 17, cols if kind == "few entries of several blocks" else 2_000))
    print("blocks of the build", metric, kind, flush=True)
    h = _lists(spd, profile=1, lds_budget=budget)
    p = _p_of(metric)
    got = _np(h.pairwise(spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B), metric, p))
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert_distances_close(got, oracle.pairwise(A, B, ORACLE_NAME[metric], p), metric)
    h.close()


# Blocks as wide as what lanes hold fits: nine tenths full and, of a few thousand, some beyond (which are gone through twice), with the 16 entries of a lane
# and, where that doubles the width, 24.
@pytest.mark.parametrize("metric", ["kl_divergence", "jensen_shannon", "chebyshev", "cosine"])
def test_full_blocks_of_the_build(spd, metric):
    rng = np.random.default_rng(71)
    n, cols = 12_200, 6_600
    share = np.exp(0.35 * rng.standard_normal(cols)).clip(0.5, 2.0)
    share *= 0.0695 / share.mean()
    rows, indices = np.nonzero(rng.random((n, cols), dtype=np.float32) < share)
    B = {"n_rows": n, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64),
         "indices": indices.astype(np.int32), "values": (rng.integers(1, 17, size=len(indices)) / 8.0).astype(np.float32)}
    A = _matrix(rng, 30, cols, (3, 64, 65, 1, 130, 0, 17, 2_000))
    cut = spd.testing.host_list_plan(30, int(A["indptr"][-1]), n, len(indices), cols, metric, match_lists=2)
    entries = len(indices) / cols * cut["tile_rows"] / n * cut["block_columns"]
    held = (16 if metric in ("kl_divergence", "chebyshev") else 24) * 512
    assert cut["block_columns"] == 128 and held / 1.25 < entries < held / 1.08, (cut, entries)
    print("full blocks", metric, flush=True)
    h = _lists(spd, profile=1)
    got = _np(h.pairwise(spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B), metric))
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert_distances_close(got, oracle.pairwise(A, B, ORACLE_NAME[metric]), metric)
    h.close()


# Many rows, several of which a wavefront sums one after the other: of 4,096 entries and more among those of one wavefront, at its ends and at the ends of a
# workgroup's and of all, with short and empty ones between.  As B's rows, and as A's, whose scales are found with the norms.
@pytest.mark.parametrize("metric", ["cosine", "correlation", "l2_expanded", "l1", "canberra", "jensen_shannon", "minkowski"])
def test_norms_of_many_rows_with_long_ones_among_them(spd, metric):
    rng = np.random.default_rng(29)
    n, cols = 65_600, 9_000
    lengths = rng.integers(0, 36, size=n)
    lengths[[0, 3, 4, 7, 8, 31, 32, 40_000, 40_001, n - 9, n - 1]] = (4_096, 4_097, 9_000, 5_000, 4_097, 8_000, 4_100, 6_000, 4_095, 7_000, 4_500)
    parts = [np.unique(rng.integers(0, cols, size=L)) if L < 4_000 else np.sort(rng.choice(cols, size=L, replace=False)) for L in lengths]
    indptr = np.concatenate([[0], np.cumsum([len(c) for c in parts])]).astype(np.int64)
    assert 16 * n <= indptr[-1] <= 256 * n                     # (a wavefront to the row; eight rows of so many)
    B = {"n_rows": n, "n_cols": cols, "indptr": indptr, "indices": np.concatenate(parts).astype(np.int32),
         "values": (rng.integers(1, 17, size=int(indptr[-1])) / 8.0).astype(np.float32)}
    A = _matrix(rng, 12, cols, (3, 64, 65, 1, 130, 0, 17, 4_500))
    p = _p_of(metric)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = _lists(spd, profile=1)
    print("norms of many rows", metric, flush=True)
    assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
    assert {r["staging_kind"] for r in h.profile_read() if r["name"] == "scan"} == {6}
    assert_distances_close(_np(h.pairwise(dB, dA, metric, p)), want.T, metric + ", the long operand first")
    h.close()


# An index whose lists would take more than it may keep if they began at lines of memory, and do not without the gaps: such lists are kept, and calls that
# lay theirs out with gaps go by them.
@pytest.mark.parametrize("metric,nnz", [("cosine", 240_000), ("l1", 200_000), ("canberra", 200_000), ("jensen_shannon", 200_000), ("hamming", 152_000),
                                        ("kl_divergence", 230_000), ("minkowski", 286_000)])
def test_an_index_that_keeps_its_lists_without_gaps(spd, metric, nnz):
    rng = np.random.default_rng(35)
    n, cols = 3_500, 160_000
    heavy = np.concatenate([c + cols * rng.choice(n, size=15 + 16 * c, replace=False) for c in range(80)])          # 15 to 1,279 rows store these columns
    light = np.setdiff1d(np.unique(rng.integers(0, n * cols, size=nnz)), heavy)
    cell = np.sort(np.concatenate([heavy, rng.choice(light, size=nnz - len(heavy), replace=False)]))
    B = {"n_rows": n, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(np.bincount(cell // cols, minlength=n))]).astype(np.int64),
         "indices": (cell % cols).astype(np.int32), "values": (rng.integers(1, 17, size=nnz) / 8.0).astype(np.float32)}
    cell = np.unique(np.concatenate([r * cols + np.unique(np.concatenate([rng.integers(0, 90, size=30), rng.integers(0, cols, size=12)])) for r in range(60)]))
    A = {"n_rows": 60, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(np.bincount(cell // cols, minlength=60))]).astype(np.int64),
         "indices": (cell % cols).astype(np.int32), "values": (rng.integers(1, 17, size=len(cell)) / 8.0).astype(np.float32)}
    p = _p_of(metric)
    plan = spd.testing.host_list_plan(60, len(cell), n, nnz, cols, metric, p, with_index=True)
    assert plan["index_bytes"] > 0 and not plan["index_aligned"] and plan["aligned"], plan
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = spd.Handle()
    h.set_option("check_plan", 1)
    h.set_option("profile", 1)
    index = h.index_create(dB, metric, p)
    h.set_option("match_lists", 2)
    print("index without gaps", metric, flush=True)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    got = index.pairwise(dA)
    names = [(r["name"], r["staging_kind"]) for r in h.profile_read()]
    assert ("scan", 6) in names and "lists_b" not in [name for name, _ in names], names
    assert_distances_close(_np(got), want, metric)
    idx, dist = index.knn(dA, 20)
    assert ("scan", 6) in [(r["name"], r["staging_kind"]) for r in h.profile_read()]
    assert_knn_matches(_np(idx), _np(dist), want, 20, metric, metric)
    if metric in ("l1", "canberra", "hamming"):                # (sums that no order changes)
        assert np.array_equal(_np(got), _np(h.pairwise(dA, dB, metric, p)))
    index.close()
    h.close()

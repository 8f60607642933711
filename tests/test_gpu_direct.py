"""Small calls in one launch (option "direct"): parity with the CPU oracle where strips, workgroups and batches of
entries end, and the refusals of the other ways (needs an MI355X; run with -m gpu)."""
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
    d = np.zeros((rows, cols))
    for r in range(rows):
        k = min(lengths[r % len(lengths)], cols)
        d[r, rng.choice(cols, size=k, replace=False)] = rng.integers(1, 9, size=k) / 8.0
    out = synth.from_dense(np.asarray(d.astype(np.float32), dtype=np.float64))
    out["values"][::17] = 0.0                              # stored zeros are absent
    return out


def _kinds(h):
    return [(r["name"], r["staging_kind"]) for r in h.profile_read()]


# rows of A: around the four of a workgroup; rows of B: around a wavefront, the 256 of a workgroup and the 1,024 of k-NN; columns:
# one, and as many as a strip has; rows of 0 to all entries, around the four that are in flight
@pytest.mark.parametrize("metric", SERVED)
@pytest.mark.parametrize("m,n,cols,lengths", [(1, 1, 1, (1,)), (3, 63, 40, (0, 1, 4, 5, 40)), (4, 65, 512, (10, 8, 3)),
                                              (5, 257, 2048, (7, 64, 0, 9)), (9, 1024, 300, (2, 3, 4)), (700, 700, 512, (10, 12, 9))])
def test_parity(spd, metric, m, n, cols, lengths):
    rng = np.random.default_rng(m + 10 * n)
    A, B, p = _matrix(rng, m, cols, lengths), _matrix(rng, n, cols, lengths[::-1]), _p_of(metric)
    print("direct", metric, m, n, cols, flush=True)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    h = spd.Handle()
    h.set_option("profile", 1)
    k = min(n, 64)
    for host in (True, False):                             # (row pointers on the GPU alone are read back)
        dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
        if not host:
            dA, dB = (spd.DeviceCsr(x.n_rows, x.n_cols, x.indptr, x.indices, x.values, host_indptr=None) for x in (dA, dB))
        got = _np(h.pairwise(dA, dB, metric, p))
        assert _kinds(h) == [("scan", 7)]
        assert_distances_close(got, want, metric)
        idx, dist = h.knn(dA, dB, metric, k, p)
        assert _kinds(h) == [("scan", 7)]
        assert_knn_matches(_np(idx), _np(dist), want, k, metric, metric)
    out = h.pairwise(dA, dB, metric, p)
    index = h.index_create(dB, metric, p)
    assert np.array_equal(_np(index.pairwise(dA)), _np(out))
    i2, d2 = index.knn(dA, k)
    assert np.array_equal(_np(i2), _np(idx)) and np.array_equal(_np(d2), _np(dist))
    index.close()
    h.set_option("direct", 0)                              # the general path over the same operands
    assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
    assert ("scan", 7) not in _kinds(h)
    h.close()


# four lanes to a row of B: rows around the 4 entries that they hold together, the 16 in flight and several rounds of them; rows of B
# around the 256 of a workgroup, k-NN's strides of them and its 1,024; fewer rows of A than a workgroup's four
@pytest.mark.parametrize("metric", SERVED)
@pytest.mark.parametrize("m,n,cols,lengths", [(1, 1, 70, (17,)), (3, 255, 200, (16, 3, 0, 15, 33, 4)), (6, 257, 100, (31, 32, 33, 1, 5)),
                                              (2, 1024, 64, (2, 9, 8, 3, 1)), (9, 40, 128, (64, 65, 0, 47))])
def test_four_lanes_to_a_row(spd, metric, m, n, cols, lengths):
    rng = np.random.default_rng(m + 10 * n + cols)
    A, B, p = _matrix(rng, m, cols, (7, 64, 0, 20)), _matrix(rng, n, cols, lengths), _p_of(metric)
    print("direct, four lanes", metric, m, n, cols, flush=True)
    want = oracle.pairwise(A, B, ORACLE_NAME[metric], p)
    dA, dB = spd.DeviceCsr.from_host(A), spd.DeviceCsr.from_host(B)
    h = spd.Handle()
    h.set_option("profile", 1)
    for k in (0, min(n, 33)):
        lanes = spd.testing.host_direct_lanes(B["indptr"], m, len(A["values"]), cols, metric, p, k)
        assert lanes == (4 if k or max(lengths) >= 16 else 1)
        if k == 0:
            assert_distances_close(_np(h.pairwise(dA, dB, metric, p)), want, metric)
        else:
            idx, dist = h.knn(dA, dB, metric, k, p)
            assert_knn_matches(_np(idx), _np(dist), want, k, metric, metric)
        assert [(r["staging_kind"], r["block"]) for r in h.profile_read()] == [(7, 256 * lanes)]
    h.close()


@pytest.mark.parametrize("law", ["all long", "one long"])
def test_long_rows_run_by_the_other_ways(spd, law):
    """A lane, or four, would go through 2,048 entries one after the other while the other lanes are idle."""
    rng = np.random.default_rng(8)
    n, cols, k = 32 if law == "all long" else 700, 2048, 5
    lengths = np.full(n, 2048 if law == "all long" else 3)
    lengths[n // 2] = 2048
    idx = [np.sort(rng.choice(cols, size=c, replace=False)) for c in lengths]
    B = {"n_rows": n, "n_cols": cols, "indptr": np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64),
         "indices": np.concatenate(idx).astype(np.int32), "values": (rng.integers(1, 9, size=int(lengths.sum())) / 8.0).astype(np.float32)}
    A = _matrix(rng, 32, cols, (5, 60, 0))
    want = oracle.pairwise(A, B, "manhattan")
    h = spd.Handle()
    h.set_option("profile", 1)
    for host in (True, False):
        dA, dB = (spd.DeviceCsr.from_host(M, keep_host_indptr=host) for M in (A, B))
        assert_distances_close(_np(h.pairwise(dA, dB, "l1")), want, law)
        assert not {kind for _, kind in _kinds(h)} & {7}
        i, d = h.knn(dA, dB, "l1", k)
        assert not {kind for _, kind in _kinds(h)} & {7}
        assert_knn_matches(_np(i), _np(d), want, k, "l1", law)
        index = h.index_create(dB, "l1")
        i, d = index.knn(dA, k)
        assert not {kind for _, kind in _kinds(h)} & {7}
        assert_knn_matches(_np(i), _np(d), want, k, "l1", law)
        index.close()
    h.close()


def test_where_it_ends(spd):
    """One row, column, pair or entry more than it takes, k-NN over too many rows, products and knobs it does not have."""
    rng = np.random.default_rng(4)
    h = spd.Handle()
    h.set_option("profile", 1)

    def kinds(m, n, cols, metric="l1", k=0, per=1):
        A, B = (spd.DeviceCsr.from_host({"n_rows": r, "n_cols": cols, "indptr": np.arange(r + 1, dtype=np.int64) * per,
                                         "indices": np.concatenate([np.sort(rng.choice(cols, size=per, replace=False)) for _ in range(r)]).astype(np.int32),
                                         "values": np.ones(r * per, np.float32)}) for r in (m, n))
        h.knn(A, B, metric, k) if k else h.pairwise(A, B, metric)
        return {kind for name, kind in _kinds(h) if name == "scan"}

    assert kinds(512, 1024, 2048) == {7} and 7 not in kinds(512, 1025, 2048) and 7 not in kinds(512, 1024, 2049)
    assert kinds(8, 1024, 64, k=3) == {7} and 7 not in kinds(8, 1025, 64, k=3)
    assert kinds(8, 1024, 100, per=64) == {7} and 7 not in kinds(8, 1025, 100, per=64)
    assert 7 not in kinds(8, 64, 64, "chebyshev")
    h.set_option("max_rows", 4)
    assert 7 not in kinds(8, 64, 64)
    h.close()


def test_what_is_refused(spd):
    import torch
    h, staged = spd.Handle(), spd.Handle()
    staged.set_option("direct", 0)

    def matrix(indptr, cols, host):
        ip = np.asarray(indptr, dtype=np.int64)
        nnz = int(ip[-1])
        t = lambda a: torch.as_tensor(a, device="cuda")
        return spd.DeviceCsr(len(ip) - 1, cols, t(ip), t(np.arange(max(nnz, 1), dtype=np.int32) % cols)[:nnz],
                             torch.ones(nnz, device="cuda"), host_indptr=ip if host else None)

    good = lambda host: matrix([0, 2, 4], 4, host)
    for host in (True, False):
        for bad in ([0, 3, 2], [1, 2, 3], [0, 7, 8]):      # decreasing, not from 0, longer than the column count
            for call in (lambda x, A, B: x.pairwise(A, B, "l1"), lambda x, A, B: x.knn(A, B, "cosine", 1)):
                for A, B in ((matrix(bad, 4, host), good(host)), (good(host), matrix(bad, 4, host))):
                    got = []
                    for x in (h, staged):
                        try:
                            call(x, A, B)
                            torch.cuda.synchronize()
                            got.append("taken")
                        except spd.SpdError as e:
                            got.append(e.status_name)
                    assert got[0] == got[1], (bad, host, got)
    h.close()
    staged.close()


def test_static_staging_is_asked_for_as_by_the_other_ways(spd):
    """The entry point that allocates nothing refuses operands whose plans its staging memory does not hold, also where one
    launch would need no plan."""
    import torch
    h, staged = spd.Handle(), spd.Handle()
    staged.set_option("direct", 0)
    for m, taken in ((1_000, True), (80_000, True), (100_000, False)):
        A, B = (spd.DeviceCsr.from_host({"n_rows": r, "n_cols": 64, "indptr": np.minimum(np.arange(r + 1), 50_000).astype(np.int64),
                                         "indices": (np.arange(min(r, 50_000)) % 64).astype(np.int32),
                                         "values": np.ones(min(r, 50_000), np.float32)}) for r in (m, 2))
        out = [torch.full((m, 2), -1.0, device="cuda") for _ in range(2)]
        for x, o in zip((h, staged), out):
            if taken:
                x.pairwise_static(A, B, "l1", o)
            else:
                with pytest.raises(spd.SpdError) as e:
                    x.pairwise_static(A, B, "l1", o)
                assert e.value.status_name == "SPD_ERR_WORKSPACE"
        assert np.array_equal(_np(out[0]), _np(out[1]))
    h.close()
    staged.close()

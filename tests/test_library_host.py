"""The C-ABI library without a GPU: it loads, exports what include/*.h declares, rejects
bad arguments, and its host logic (planner; shared per-visit arithmetic) is consistent."""
import ctypes
import os
import re

import numpy as np
import pytest

import oracle
import paper_2104_06357_amd as spd
from gen import synth
from util import ALL_METRICS, NONNEGATIVE_ONLY, ORACLE_NAME, assert_distances_close, quotient_cases

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    names = set()
    for header in os.listdir(os.path.join(ROOT, "include")):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names.update(re.findall(r"\b(spd_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_library_loads_and_exports_every_declared_symbol():
    L = spd.lib()
    declared = _declared_functions()
    assert {"spd_create", "spd_destroy", "spd_pairwise", "spd_knn", "spd_workspace_bytes", "spd_set_workspace",
            "spd_csr_validate", "spd_set_option", "spd_last_error", "spd_metric_name", "spd_version",
            "spd_host_pair_value", "spd_host_plan_summary"} <= set(declared)
    for name in declared:
        assert hasattr(L, name), name
    assert b"gfx950" in L.spd_version()
    for i, name in enumerate(spd.METRICS):
        assert L.spd_metric_name(i).decode() == name


def test_null_handle_and_missing_gpu_fail_loudly():
    L = spd.lib()
    assert L.spd_pairwise(None, None, None, 0, 2.0, None) == 1          # SPD_ERR_NULL
    assert L.spd_knn(None, None, None, 0, 2.0, 1, None, None) == 1
    assert L.spd_destroy(None) == 1
    import torch
    if not torch.cuda.is_available():
        h = ctypes.c_void_p()
        assert L.spd_create(ctypes.byref(h), None) == 8                   # SPD_ERR_HIP: no CPU fallback
        assert not h
        with pytest.raises(RuntimeError):
            spd.Handle()


def test_host_pair_value_argument_checks():
    c = np.array([1], dtype=np.int32); v = np.array([1.0], dtype=np.float32)
    with pytest.raises(spd.SpdError) as e:
        spd.testing.host_pair_value("minkowski", 0.0, 4, c, v, c, v)
    assert e.value.status_name == "SPD_ERR_BAD_P"
    with pytest.raises(spd.SpdError) as e:
        spd.testing.host_pair_value(99, 2.0, 4, c, v, c, v)
    assert e.value.status_name == "SPD_ERR_BAD_METRIC"


@pytest.mark.parametrize("metric", ALL_METRICS)
def test_single_sweep_arithmetic_matches_the_oracle(metric):
    """The products g(a, b), norms and expansion functions the kernels run, evaluated on
    the host for single pairs: the union family's one-sweep form (norms plus corrections on
    the intersection) and the expanded forms equal the oracle's plain definitions."""
    A, B = synth.workload(0)
    ra, rb = np.arange(0, 256, 7), np.arange(0, 256, 5)
    for p in ((0.5, 1.0, 3.0) if metric == "minkowski" else (2.0,)):
        want = oracle.pairwise(A, B, ORACLE_NAME[metric], p, rows_a=ra, rows_b=rb)
        got = np.empty_like(want)
        for x, i in enumerate(ra):
            a0, a1 = A["indptr"][i], A["indptr"][i + 1]
            for y, j in enumerate(rb):
                b0, b1 = B["indptr"][j], B["indptr"][j + 1]
                got[x, y] = spd.testing.host_pair_value(metric, p, A["n_cols"], A["indices"][a0:a1], A["values"][a0:a1],
                                                B["indices"][b0:b1], B["values"][b0:b1])
        assert_distances_close(got, want, "%s p=%g" % (metric, p))


@pytest.mark.parametrize("metric", ALL_METRICS)
def test_single_sweep_arithmetic_identical_and_signed_rows(metric):
    rng = np.random.default_rng(5)
    signed = metric not in NONNEGATIVE_ONLY
    k = 300
    rows = []
    for _ in range(6):
        cols = np.sort(rng.choice(k, size=rng.integers(1, 120), replace=False)).astype(np.int32)
        vals = (rng.standard_normal(cols.size) if signed else rng.random(cols.size) + 0.01) * 40.0
        rows.append((cols, vals.astype(np.float32)))
    rows.append((np.empty(0, np.int32), np.empty(0, np.float32)))            # an empty row
    rows.append((rows[0][0].copy(), rows[0][1].copy()))                      # a duplicate of row 0
    half = rows[1][1].copy(); half[::2] = rows[1][1][::2] * np.float32(1.0000001)
    rows.append((rows[1][0].copy(), half))                                   # a near duplicate of row 1
    dense = np.zeros((len(rows), k))
    for r, (c, v) in enumerate(rows):
        dense[r, c] = v
    M = synth.from_dense(dense)
    want = oracle.pairwise(M, M, ORACLE_NAME[metric], 3.0)
    got = np.array([[spd.testing.host_pair_value(metric, 3.0, k, ca, va, cb, vb) for cb, vb in rows] for ca, va in rows])
    assert_distances_close(got, want, metric)


def test_planner_paths_and_thresholds():
    A, B = synth.workload(1, 0.2)
    auto = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine")
    assert all(c["kind"] == 2 for c in auto["classes"])                      # 20,000 columns: slot strip
    assert auto["packed_entries"] == B["indptr"][-1] and auto["spilled_rows"] == 0
    for kind in (1, 3, 5):
        s = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine", force_kind=kind)
        assert all(c["kind"] == kind for c in s["classes"])
    small, _ = synth.workload(0)
    s = spd.testing.host_plan_summary(small["indptr"], small["indptr"], small["n_cols"], "l1")
    assert [c["kind"] for c in s["classes"]] == [1] and s["classes"][0]["R"] == 8
    # a tight LDS budget forces slices (partitions) of the long rows
    s = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "l1", force_kind=3, lds_budget=16384)
    assert s["spilled_rows"] > 0 and s["partial_slots"] >= 2 * s["spilled_rows"]
    assert all(c["lds_bytes"] + 4096 <= 16384 for c in s["classes"])
    # rows at the split threshold (256 for a small B, or the option): one below stays whole
    for length, split in ((255, 0), (256, 1), (257, 1)):
        ip = np.array([0, length], dtype=np.int64)
        s = spd.testing.host_plan_summary(ip, ip, 4096, "l1", force_kind=3)
        assert s["split_rows"] == split, (length, s)
    for length, split in ((127, 0), (128, 1), (129, 1)):
        ip = np.array([0, length], dtype=np.int64)
        s = spd.testing.host_plan_summary(ip, ip, 4096, "l1", force_kind=3, split_len=128)
        assert s["split_rows"] == split, (length, s)
    # a B of 2^22 stored entries or more is cut at 512
    ip = np.arange(0, 511 * 8300, 511, dtype=np.int64)
    assert spd.testing.host_plan_summary(ip[:2], ip, 4096, "l1", force_kind=3)["split_rows"] == 0
    ip = np.arange(0, 512 * 8300, 512, dtype=np.int64)
    assert spd.testing.host_plan_summary(ip[:2], ip, 4096, "l1", force_kind=3)["split_rows"] == 8299
    # Jensen-Shannon keeps at most 8 rows per group
    s = spd.testing.host_plan_summary(small["indptr"], small["indptr"], small["n_cols"], "jensen_shannon")
    assert max(c["R"] for c in s["classes"]) == 8
    # the fused k-NN keeps a list and a queue of 64 keys per staged row beside the tables
    s = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine", k_neighbors=64)
    p = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine")
    assert max(c["lds_bytes"] for c in s["classes"]) <= 160 * 1024 - 4096
    light = [c for c in s["classes"] if c["R"] == 8 and c["groups"] > 100]
    assert light and all(c["lds_bytes"] >= 20001 * 2 + 8 * 1024 for c in light)
    assert sum(c["R"] * c["groups"] for c in s["classes"]) >= A["n_rows"] and p["classes"]


def test_planner_rejects_bad_row_pointers():
    good = np.array([0, 2, 5], dtype=np.int64)
    bad = np.array([0, 3, 2], dtype=np.int64)
    with pytest.raises(spd.SpdError):
        spd.testing.host_plan_summary(bad, good, 16, "l1")
    with pytest.raises(spd.SpdError):
        spd.testing.host_plan_summary(good, bad, 16, "l1")
    with pytest.raises(spd.SpdError):
        spd.testing.host_plan_summary(np.array([0, 40], dtype=np.int64), good, 16, "l1")   # row longer than k


@pytest.mark.parametrize("config,scale", [(2, 0.02), (3, 0.01), (4, 0.02)])
def test_planner_on_the_large_shapes(config, scale):
    A, B = synth.workload(config, scale)
    metric = {2: "cosine", 3: "jensen_shannon", 4: "jaccard"}[config]
    s = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], metric, k_neighbors=32 if config == 4 else 0)
    assert s["packed_entries"] == B["indptr"][-1]
    expected_kind = {2: 5, 3: 2, 4: 3}[config]                               # bitmap / slot strip / hash
    assert all(c["kind"] == expected_kind for c in s["classes"]), s
    if config == 3:
        # the 16-bit column-slot strip leaves room for a whole 12,000-entry row; a hash table does not
        assert s["spilled_rows"] == 0
        h = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], metric, force_kind=3)
        assert h["spilled_rows"] >= 1 and h["partial_slots"] >= 2


def test_planner_sort_key_small_classes_and_bloom_rows():
    A, B = synth.workload(1)
    # sorting B's rows by whole blocks of four steps costs no step, and keeps equal rows in row order
    exact = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine", sort_slack=0)
    blocks = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine", sort_slack=1)
    assert blocks["total_slab_steps"] == exact["total_slab_steps"] and blocks["slabs"] == exact["slabs"]
    # a class of a few groups joins the class of the same R that needs more LDS, and the longest rows go
    # three to a group of four rather than two to a group of two: three launches, not five
    assert sorted((c["R"], c["groups"]) for c in blocks["classes"]) == [(4, 43), (8, 29), (8, 1202)]
    halved = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "cosine", partial_groups=0)
    assert sorted((c["R"], c["groups"]) for c in halved["classes"]) == [(2, 28), (4, 24), (8, 29), (8, 1202)]
    # Chebyshev keeps full groups: an idle place there still ranks its column
    ch = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "chebyshev")
    ch0 = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "chebyshev", partial_groups=0)
    assert [(c["R"], c["groups"]) for c in ch["classes"]] == [(c["R"], c["groups"]) for c in ch0["classes"]]
    js = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "jensen_shannon")
    js0 = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "jensen_shannon", partial_groups=0)
    assert sum(c["groups"] for c in js["classes"]) < sum(c["groups"] for c in js0["classes"])
    assert sum(c["R"] * c["groups"] for c in blocks["classes"]) >= A["n_rows"]
    # the cost model's estimates: the large launch far above the small ones, a few groups of long rows get 2 chunks
    by_groups = sorted(blocks["classes"], key=lambda c: c["groups"])
    assert by_groups[-1]["cost"] > 3 * max(c["cost"] for c in by_groups[:-1]) > 0
    assert all(c["chunks"] <= 2 for c in by_groups[:-1])
    # Bloom staging: every row alone, or only the rows that would have been cut into slices
    s = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "l1", force_kind=4)
    assert [(c["kind"], c["R"], c["groups"]) for c in s["classes"]] == [(4, 1, A["n_rows"])]
    assert all(c["lds_bytes"] <= 65536 for c in s["classes"])
    with pytest.raises(spd.SpdError):
        spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "chebyshev", force_kind=4)
    tight = dict(force_kind=3, lds_budget=8192 + 65536)
    long_rows = int((np.diff(A["indptr"]) > 2048).sum())
    sliced = spd.testing.host_plan_summary(A["indptr"], B["indptr"], A["n_cols"], "l1", **tight)
    assert sliced["spilled_rows"] == long_rows == 0 or sliced["spilled_rows"] == long_rows
    ip = np.array([0, 5, 3005, 3010, 9010], dtype=np.int64)                  # rows of 5, 3000, 5, 6000 entries
    sliced = spd.testing.host_plan_summary(ip, ip, 10000, "l1", **tight)
    filtered = spd.testing.host_plan_summary(ip, ip, 10000, "l1", bloom_long_rows=1, **tight)
    assert sliced["spilled_rows"] == 2 and filtered["spilled_rows"] == 0
    assert sorted(c["kind"] for c in filtered["classes"]) == [3, 4]


@pytest.mark.parametrize("metric", ["jensen_shannon", "kl_divergence", "kl_divergence_strict"])
def test_quotients_inside_the_logarithms_on_the_host(metric):
    """A quotient that rounds to 1, or underflows, must not leave log(0) behind: a column whose
    two entries differ by a factor of 1e8 adds what the formula says, not minus infinity."""
    for a, b in quotient_cases():
        A, B = synth.from_dense(a[None, :]), synth.from_dense(b[None, :])
        want = oracle.pairwise(A, B, ORACLE_NAME[metric], mode="full")
        got = spd.testing.host_pair_value(metric, 2.0, 16, A["indices"], A["values"], B["indices"], B["values"])
        assert_distances_close(np.array([[got]]), want, "%s on %s" % (metric, (a[3], b[3])))
    # the case the advisor gave: a = {1, 0.5}, b = {1e-8, 0.5}
    A = synth.from_dense(np.array([[1.0, 0.5]])); B = synth.from_dense(np.array([[1e-8, 0.5]]))
    got = spd.testing.host_pair_value("jensen_shannon", 2.0, 2, A["indices"], A["values"], B["indices"], B["values"])
    assert abs(got - 0.5887) < 1e-4


def _wanted(m, mean_a, n, mean_b, cols, metric, **more):
    return bool(spd.testing.host_list_plan(m, m * mean_a, n, n * mean_b, cols, metric, **more)["wanted"])


@pytest.mark.parametrize("metric", ["l1", "cosine", "hamming", "canberra", "kl_divergence", "jensen_shannon", "minkowski"])
def test_column_lists_are_left_alone_where_a_is_long_against_b(metric):
    """The lists cost a step per entry of A and tile, the staged scan a visit per staged row and streamed entry: for a given
    B, long enough rows of A turn the choice, once, whatever else the call is."""
    for with_index, k in ((False, 32), (True, 0), (True, 32)):
        choice = [_wanted(2_000, mean_a, 10_000, 20, 20_000, metric, k_neighbors=k, with_index=with_index)
                  for mean_a in (1, 3, 10, 30, 100, 300, 1_000, 3_000)]
        assert choice[1] and not choice[-2] and not choice[-1], (with_index, k, choice)
        assert choice[1:] == sorted(choice[1:], reverse=True), choice


def test_column_lists_against_the_scan_that_would_run():
    # both ways measured, staged / lists in ms: 0.14 / 0.70, 0.14 / 0.90, 0.15 / 1.03, 2.18 / 6.52
    assert not _wanted(1_000, 1_360, 10_000, 20, 20_000, "l1")
    assert not _wanted(1_000, 1_346, 10_000, 20, 20_000, "l1", k_neighbors=32)
    assert not _wanted(766, 1_468, 3_599, 35, 20_000, "minkowski", p=3.0, k_neighbors=32, with_index=True)
    assert not _wanted(436, 2_548, 217_842, 50, 200_000, "hamming")
    # a pairwise call that would stage B and stream the long rows of A: 36.7 / 1.49
    assert _wanted(8_934, 598, 10_816, 9, 60_000, "jensen_shannon")
    # operands of one law: 0.65 / 0.41, 11.4 / 6.7, 17.1 / 10.2, 87 / 36, 349 / 59, 2.67 / 1.16
    assert _wanted(10_000, 37, 10_000, 37, 20_000, "l1") and _wanted(10_000, 37, 10_000, 37, 20_000, "cosine")
    assert _wanted(1_024, 228, 300_000, 228, 102_660, "cosine")
    assert _wanted(2_048, 228, 300_000, 228, 102_660, "hellinger", k_neighbors=32, with_index=True)
    assert _wanted(4_096, 1_820, 65_536, 1_820, 26_000, "l1") and _wanted(4_096, 1_820, 65_536, 1_820, 26_000, "jensen_shannon")
    assert _wanted(1_531, 160, 28_301, 160, 194_000, "canberra")
    # and the option decides where it is asked to
    assert not _wanted(10_000, 37, 10_000, 37, 20_000, "l1", match_lists=0)
    assert _wanted(766, 1_468, 3_599, 35, 20_000, "minkowski", match_lists=2)


def test_column_lists_where_either_way_was_measured_the_faster():
    def way(m, nnz_a, n, nnz_b, cols, metric, k=0, with_index=False):
        return spd.testing.host_list_plan(m, nnz_a, n, nnz_b, cols, metric, p=3.0, k_neighbors=k, with_index=with_index)["way"]

    # staged / lists in us
    for call in ((593, 1_098_834, 12_826, 23_146_901, 25_801, "kl_divergence", 10, True),                # 5,537 / 1,725
                 (284, 508_523, 32_451, 58_624_655, 25_871, "kl_divergence", 1),                         # 7,534 / 3,568
                 (3_523, 6_436_960, 939, 1_723_471, 25_977, "kl_divergence", 5),                         # 2,846 / 844
                 (3_365, 6_104_649, 606, 1_122_609, 25_803, "hamming"),                                  # 1,143 / 464
                 (166, 80_710, 63_912, 30_733_557, 9_590, "kl_divergence", 0, True),                     # 1,582 / 479
                 (303, 18_008, 15_994, 700_407, 26_578, "kl_divergence"),                                # 420 / 110
                 (4_192, 9_815, 15_752, 36_404, 5_716, "minkowski"),                                     # 578 / 217
                 (2_628, 1_644_603, 38_556, 18_370_748, 2_656, "canberra")):                             # 14,985 / 8,086
        assert way(*call) == 1, call
    for call in ((99, 200, 386_927, 860_302, 858_000, "cosine", 10, True),                               # 192 / 259 over A's columns
                 (225, 16_379, 3_387, 257_241, 4_996, "l1", 64, True),                                   # 56 / 100
                 (285, 16_409, 2_183, 121_792, 5_120, "hamming", 1, True)):                              # 61 / 107
        assert way(*call) == 0, call


def test_correlation_goes_the_way_of_the_other_dot_products():
    """It reads a second norm a pair, and its lists and visits are cosine's: both ways take the same times by either metric."""
    def way(m, nnz_a, n, nnz_b, cols, metric):
        return spd.testing.host_list_plan(m, nnz_a, n, nnz_b, cols, metric)["way"]

    # by correlation, staged / lists in us
    for call in ((307, 40_824, 3_449, 517_333, 193_879),                                                 # 312 / 124
                 (72, 141_200, 35_647, 65_078_019, 26_000),                                              # 3,055 / 1,357
                 (106, 195_719, 12_282, 22_371_889, 25_958),                                             # 1,166 / 520
                 (212, 360_947, 4_950, 9_034_151, 25_864),                                               # 589 / 376
                 (91, 5_303, 3_171, 391_568, 193_823),                                                   # 147 / 91
                 (573, 185_212, 3_605, 1_255_751, 60_000),                                               # 314 / 128, rows of one length 158 / 160
                 (573, 182_658, 3_605, 1_203_924, 25_248)):                                              # 207 / 131, rows of one length 138 / 160
        assert way(*call, "correlation") == 1, call
    rng = np.random.default_rng(41)
    apart = lists = 0
    for _ in range(3_000):                                 # words, counts and ratings
        cols, mean, least, most = ((102_660, 228, 5_000, 300_000), (26_000, 1_820, 500, 60_000), (194_000, 160, 2_000, 200_000))[rng.integers(3)]
        m, n = int(np.exp(rng.uniform(np.log(17), np.log(4_000)))), int(np.exp(rng.uniform(np.log(least), np.log(most))))
        ways = [way(m, m * mean, n, n * mean, cols, metric) for metric in ("cosine", "correlation")]
        lists += ways[0] != 0
        apart += ways[0] != ways[1]
    assert lists > 1_500 and apart < 30, (lists, apart)


@pytest.mark.parametrize("m,n,metric,k", [(89, 8_333, "l1", 64), (1_514, 20_515, "cosine", 10), (1_783, 12_134, "cosine", 10)])
def test_column_lists_count_their_bounds(m, n, metric, k):
    """A word per tile and column: few rows of two entries over very many columns, staged / lists in us 99 / 137, 200 / 235,
    166 / 191."""
    assert not _wanted(m, 2, n, 2, 858_000, metric, k_neighbors=k)


def test_column_lists_only_where_a_workgroup_can_number_its_work():
    """A workgroup's (tile, row)s are numbered in 32 bits: 6.25 million rows of a slice in 2,056 tiles are more."""
    def plan(m):
        return spd.testing.host_list_plan(m, 2 * m, 20_000_000, 200_000_000, 100_000, "l1", k_neighbors=4, match_lists=2)

    for m in (10_000, 1_000_000, 16_000_000, 200_000_000, 2_000_000_000):
        p = plan(m)
        items = -(-m // p["slices"]) * -(-p["tiles"] // p["groups"])
        assert bool(p["wanted"]) == (items < 1 << 30), p
    assert plan(16_000_000)["wanted"] and not plan(200_000_000)["wanted"]


def test_column_lists_only_where_their_launches_fit_a_grid():
    """A launch has fewer than 2^32 work-items: over A's columns one for every stored entry of A, a wavefront for the norm of every
    row of A, 1,024 threads for a tile."""
    def way(m, mean_a, n, mean_b, cols, metric, **more):
        return spd.testing.host_list_plan(m, m * mean_a, n, n * mean_b, cols, metric, **more)["way"]

    assert way(4_096, 160, 500_000, 150, 1 << 20, "jaccard", k_neighbors=32) == 2
    assert way(1 << 24, 255, 2_000, 40_000, 1 << 20, "jaccard", match_lists=3) == 2
    assert way(1 << 24, 256, 2_000, 40_000, 1 << 20, "jaccard", match_lists=3) == 0
    assert way(1 << 24, 256, 2_000, 40_000, 1 << 20, "jaccard", match_lists=2) == 1
    for m in ((1 << 26) - 1_024, 1 << 26):
        for lists in (2, 3):
            assert (way(m, 16, 100, 200, 10_000, "l1", match_lists=lists) > 0) == (m < 1 << 26)
            assert way(m, 15, 100, 200, 10_000, "l1", match_lists=lists) > 0
    assert way(1_000, 10, 200_000_000, 1, 50, "l1", match_lists=2, lds_budget=163_840) == 1
    for n in (268_000_000, 269_000_000):                   # (tiles of 64 rows: 2^22 of them are too many)
        plan = spd.testing.host_list_plan(1_000, 10_000, n, n, 50, "l1", match_lists=2, lds_budget=16_000)
        assert plan["consistent"] and (plan["way"] == 1) == (plan["tiles"] < 1 << 22)
    for tiles in ((1 << 22) - 16, (1 << 22) - 5):           # (... and whole rounds of eight of them)
        assert (way(1_000, 10, 64 * tiles, 1, 50, "l1", match_lists=2, lds_budget=16_000) == 1) == (tiles == (1 << 22) - 16)
    for rows in ((1 << 26) - 24, (1 << 26) - 3):            # (a wavefront to the row that is ranked)
        assert (way(rows - 100, 2, 100, 20, 1_000, "chebyshev", match_lists=2) == 1) == (rows == (1 << 26) - 24)


def test_inner_products_of_as_many_entries_as_other_products_take_the_lists():
    """Dense columns of a dot product begin at fewer rows and need more room; positions of list entries end at 2^29 for all products."""
    for n, nnz, cols in ((380_421, 331_064_897, 20_521), (380_421, 360_000_000, 20_521), (300_000, 440_000_000, 102_660)):
        plans = [spd.testing.host_list_plan(12, 3_500, n, nnz, cols, metric, match_lists=2) for metric in ("inner_product", "cosine", "l1", "canberra")]
        assert len({p["way"] for p in plans}) == 1 and all(p["consistent"] == p["wanted"] for p in plans), (n, nnz, cols)


def test_the_cut_of_the_column_lists_is_consistent():
    """What check_plan verifies, over random sizes, with the lists wanted wherever a product has them."""
    rng = np.random.default_rng(23)
    wanted = 0
    for _ in range(4_000):
        m, n, cols = (int(2 ** rng.uniform(0, e)) for e in (24, 24, 31))
        mean_a, mean_b = (min(2 ** rng.uniform(-2, 12), cols) for _ in range(2))
        metric = ALL_METRICS[rng.integers(len(ALL_METRICS))]
        plan = spd.testing.host_list_plan(m, int(m * mean_a), n, int(n * mean_b), cols, metric, k_neighbors=int(rng.integers(0, 2)) * min(n, 64),
                                          match_lists=2, lds_budget=int(rng.choice([8192, 20000, 65536, 163840])))
        wanted += plan["wanted"]
        assert plan["consistent"] or not plan["wanted"], (m, n, cols, metric, plan)
    assert wanted > 1_000


def test_the_cut_over_the_columns_of_a_is_consistent():
    """The same of the lists over the columns that A stores, which may be fewer than B's rows are long, and of the default choice."""
    rng = np.random.default_rng(29)
    ways = [0, 0, 0]
    for i in range(6_000):
        m, n, cols = (int(2 ** rng.uniform(0, e)) for e in (20, 22, 30))
        mean_a, mean_b = (min(2 ** rng.uniform(-2, 12), cols) for _ in range(2))
        metric = ALL_METRICS[rng.integers(len(ALL_METRICS))]
        k, with_index = int(rng.integers(0, 2)) * min(n, 64), bool(rng.integers(0, 2))
        plan = spd.testing.host_list_plan(m, int(m * mean_a), n, int(n * mean_b), cols, metric, k_neighbors=k, with_index=with_index,
                                          match_lists=3 if i % 2 else 1)
        assert plan["consistent"] or not plan["way"], (m, n, cols, metric, plan)
        if i % 2:
            assert plan["way"] in (0, 2)
        if plan["way"] == 2:
            assert 1 <= plan["columns"] <= min(cols, int(m * mean_a))
            # both operands' copies, the bits of the columns, the lists and their bounds
            assert plan["scratch_bytes"] >= 4 * int(m * mean_a) + 16 * int(n * mean_b) + 4 * plan["tiles"] * plan["columns"] + cols // 4
        ways[plan["way"]] += 1 if i % 2 == 0 or plan["way"] == 2 else 0
    assert min(ways) > 100, ways


def test_lists_over_the_columns_of_a_where_they_were_measured_the_faster():
    def way(m, nnz_a, n, nnz_b, cols, metric, k, with_index=False):
        return spd.testing.host_list_plan(m, nnz_a, n, nnz_b, cols, metric, k_neighbors=k, with_index=with_index)["way"]

    # staged / lists over A's columns in us
    for call in ((46, 1_181, 56_760, 7_850_605, 1 << 20, "russell_rao", 10),                             # 729 / 296
                 (304, 18_179, 47_031, 6_320_193, 1_048_489, "jaccard", 1),                              # 928 / 415
                 (322, 43_735, 235_775, 32_212_992, 1 << 20, "hamming", 5, True),                        # 3,254 / 2,043
                 (2_852, 331_584, 45_723, 5_793_187, 1_048_432, "dice", 32),                             # 2,636 / 1,194
                 (55, 105, 31_228, 69_773, 858_000, "l1", 32),                                           # 165 / 115
                 (73, 175, 392_314, 873_637, 857_938, "l1", 32),                                         # 2,131 / 622
                 (2_580, 5_713, 589_528, 1_311_120, 858_000, "l1", 1, True)):                            # 2,747 / 1,043
        assert way(*call) == 2, call
    for call in ((45, 6_537, 132_700, 18_125_390, 1 << 20, "hamming", 64, True),                         # 653 / 733
                 (53, 107, 139_569, 309_837, 857_836, "jaccard", 1, True),                               # 74 / 126
                 (161, 349, 106_492, 236_060, 857_888, "cosine", 32, True)):                             # 110 / 176
        assert way(*call) == 0, call


def test_blocks_of_the_build_are_as_wide_as_their_entries_fit():
    def columns(n, mean, cols, metric):
        return spd.testing.host_list_plan(32, 32 * mean, n, n * mean, cols, metric, match_lists=2)["block_columns"]

    # the build in us, narrower / so
    assert columns(60_000, 1_824, 26_000, "kl_divergence") == 128                                        # 1,671 / 1,042
    assert columns(60_000, 1_824, 26_000, "chebyshev") == 128                                            # 2,009 / 1,250
    assert columns(60_000, 1_824, 26_000, "jensen_shannon") == 128                                       # 1,551 / 1,105
    assert columns(300_000, 228, 102_660, "kl_divergence") == 4_096                                      # 899 / 701
    # two workgroups to a compute unit come first: 31.7 / 43.8 with the wider
    assert columns(8_000, 228, 102_660, "kl_divergence") == 2_048


def test_long_rows_are_shared_where_the_wavefronts_have_few_between_them():
    def shared(m, mean_a, n, mean, cols, metric, k=0):
        return spd.testing.host_list_plan(m, m * mean_a, n, n * mean, cols, metric, p=3.0, k_neighbors=k, match_lists=2)["shared_len"] < 2 * mean_a

    counts, words = (1_824, 26_000), (256, 102_660)
    # rows from 256 entries or a third of a share on in parts / from twice the mean length on, the walk in us
    for m, n, (mean, cols), metric in ((32, 60_000, counts, "kl_divergence"),                            # 571 / 678
                                       (64, 60_000, counts, "cosine"),                                   # 835 / 920
                                       (130, 60_000, counts, "kl_divergence"),                           # 1,442 / 1,603
                                       (32, 20_000, counts, "cosine"),                                   # 307 / 384
                                       (130, 20_000, counts, "minkowski"),                               # 1,141 / 1,470
                                       (300, 4_000, counts, "minkowski")):                               # 580 / 736
        assert shared(m, mean, n, mean, cols, metric), (m, n, metric)
    for m, n, (mean, cols), metric, k in ((1_500, 6_000, words, "cosine", 0),                            # 205 / 173
                                          (1_500, 6_000, words, "cosine", 10),                           # 322 / 242
                                          (700, 6_000, words, "kl_divergence", 0),                       # 232 / 210
                                          (64, 60_000, counts, "cosine", 10),                            # 1,105 / 942
                                          (3_000, 20_000, counts, "kl_divergence", 0)):
        assert not shared(m, mean, n, mean, cols, metric, k), (m, n, metric, k)
    # sums that need no order go to one strip
    assert shared(32, 1_824, 60_000, 1_824, 26_000, "l1")


def test_many_short_rows_over_few_columns_take_the_copy():
    """The bounds of the lists over all columns, a word per tile and column, have no room beside so many short rows."""
    # staged / lists over A's columns in us
    for m, n, mean, cols, metric, k in ((200, 1_000_000, 5, 32_768, "cosine", 0),                        # 3,392 / 748
                                        (200, 1_000_000, 5, 32_768, "l1", 10),                           # 3,337 / 780
                                        (1_000, 1_000_000, 5, 32_768, "l1", 10),                         # 5,111 / 1,121
                                        (1_000, 700_000, 4, 32_000, "cosine", 10),                       # 3,225 / 655
                                        (100, 1_200_000, 6, 30_000, "canberra", 0),                      # 4,311 / 849
                                        (3_000, 900_000, 3, 32_768, "canberra", 10),                     # 9,013 / 1,503
                                        (4_096, 2_000_000, 2, 16_384, "l1", 10)):                        # 19,735 / 5,611
        plan = spd.testing.host_list_plan(m, m * mean, n, n * mean, cols, metric, k_neighbors=k)
        assert plan["way"] == 2 and plan["consistent"], (m, n, mean, cols, metric, plan)


def test_calls_that_estimates_without_maps_and_launches_sent_the_slower_way():
    def plan(m, nnz_a, n, nnz_b, cols, metric, k, with_index):
        return spd.testing.host_list_plan(m, nnz_a, n, nnz_b, cols, metric, p=3.0, k_neighbors=k, with_index=with_index)

    # staged / lists over all columns / over A's in us
    for want, call in ((2, (10, 17_433, 653_968, 19_871_029, 801_333, "minkowski", 0, False)),           # 5,231 / 6,300 / 771
                       (2, (48, 16_506, 16_102, 1_135_587, 1_953_194, "kl_divergence", 0, False)),       # 469 / 318 / 102
                       (2, (275, 46_199, 256_474, 34_595_634, 1_048_576, "dice", 1, False)),             # 3,838 / - / 1,176
                       (2, (417, 117_487, 72_252, 9_886_247, 1_048_447, "russell_rao", 5, False)),       # 1,650 / - / 468
                       (2, (773, 259_693, 81_326, 14_935_108, 1_324_059, "russell_rao", 32, True)),      # 1,854 / - / 614
                       (2, (79, 1_347, 66_155, 699_988, 548_212, "jensen_shannon", 0, True)),            # 321 / - / 104
                       (0, (3_035, 2_460_418, 251, 546, 1_558_033, "l1", 0, True)),                      # 63 / - / 247
                       (0, (245, 114_662, 2_392, 12_094, 17_153, "l2_unexpanded", 32, False)),           # 61 / 192 / 233
                       (0, (222, 95_908, 4_494, 1_493_679, 121_762, "hamming", 0, False)),               # 135 / 408 / 460
                       (0, (148, 164_243, 11_371, 7_706_568, 10_950, "inner_product", 0, True)),         # 204 / 567 / 777
                       # words, whose rows store many columns that most rows store
                       (0, (184, 40_638, 9_756, 2_111_019, 102_602, "jaccard", 1, False)),               # 184 / 313 / -
                       (0, (62, 14_856, 36_208, 7_871_693, 102_571, "jaccard", 10, False)),              # 270 / 446 / -
                       (0, (1_073, 228_568, 22_501, 4_881_044, 102_482, "dice", 32, True)),              # 572 / 859 / -
                       (1, (378, 86_000, 251_417, 54_600_000, 102_660, "dice", 10, False)),              # 3,790 / 2,752 / 3,101
                       # few long rows against many: most of the scan's time goes into making B ready, the more the longer B's rows are
                       (1, (88, 138_589, 26_958, 49_192_777, 25_946, "hellinger", 10, False)),           # 1,973 / 1,069 / -
                       (1, (31, 66_323, 19_632, 35_679_941, 26_000, "canberra", 0, False)),              # 1,086 / 762 / -
                       (1, (36, 61_070, 33_011, 59_949_140, 25_987, "l1", 0, False)),                    # 1,694 / 942 / -
                       (1, (23, 37_526, 9_196, 16_915_257, 26_000, "hamming", 0, False)),                # 458 / 311 / -
                       (1, (19, 31_920, 25_736, 46_613_550, 26_000, "dice", 5, False)),                  # 1,031 / 705 / -
                       (1, (54, 95_458, 7_022, 12_689_675, 25_848, "minkowski", 1, False))):             # 1,005 / 651 / -
        assert plan(*call)["way"] == want, call
    # the scan's maps: a strip of few columns, slots, a bitmap, a table, and fewer rows of them the longer they are
    kinds = [plan(1_000, 40_000, 20_000, 800_000, cols, "l1", 0, False)["staged_kind"] for cols in (2_000, 20_000, 100_000, 400_000)]
    assert kinds == [1, 2, 5, 3]
    rows = [plan(1_000, 1_000 * mean, 20_000, 800_000, 100_000, "l1", 0, False)["staged_rows"] for mean in (40, 2_000, 8_000, 30_000)]
    assert rows == sorted(rows, reverse=True) and rows[0] == 8 and rows[-1] == 1, rows


def test_scratch_for_the_lists_over_all_columns_alone():
    """Where the copy over A's columns is preferred and takes more scratch than there is, the lists over all columns serve the call."""
    for call, k in (((133, 137, 13_649, 2_082_360, 328_013, "l2_expanded"), 0), ((39, 131, 78_887, 2_049_022, 69_229, "inner_product"), 10)):
        plan = lambda **more: spd.testing.host_list_plan(*call, k_neighbors=k, **more)
        free, all_columns = plan(), plan(match_lists=2)
        assert free["way"] == 2 and all_columns["scratch_bytes"] < free["scratch_bytes"]
        for scratch, way in ((free["scratch_bytes"], 2), (free["scratch_bytes"] - 1, 1), (all_columns["scratch_bytes"], 1), (all_columns["scratch_bytes"] - 1, 0)):
            assert plan(scratch=scratch)["way"] == way, (call, scratch, way)


def test_an_index_keeps_lists_that_calls_may_want_within_the_stated_memory():
    def kept(n, mean, cols, metric, **more):
        plan = spd.testing.host_list_plan(1_000, 30_000, n, int(n * mean), cols, metric, with_index=True, **more)
        assert more.get("match_lists") == 2 or plan["index_bytes"] <= 20 * int(n * mean) + 16 * n + (1 << 20)
        return plan["index_bytes"]

    rng = np.random.default_rng(17)
    for _ in range(2_000):
        cols = int(2 ** rng.uniform(4, 30))
        kept(int(2 ** rng.uniform(0, 22)), min(2 ** rng.uniform(-2, 12), cols), cols, ALL_METRICS[rng.integers(len(ALL_METRICS))])
    # more list bounds than entries (24 MB of them for 17,600 entries); a cell in six stored; set metrics; scan knobs turned
    assert kept(8_000, 2.2, 858_000, "cosine") == 0 and kept(100, 10, 1_000_000, "l1") == 0
    assert kept(20_000, 50, 300, "l1") == 0 and kept(20_000, 50, 300, "jensen_shannon") > 0
    assert kept(20_000, 50, 20_000, "jaccard") == 0
    assert kept(20_000, 50, 20_000, "l1") > 0 and kept(20_000, 50, 20_000, "l1", force_kind=3) == 0
    assert kept(20_000, 50, 20_000, "l1", match_lists=0) == 0 and kept(8_000, 2.2, 858_000, "cosine", match_lists=2) > 0
    # near the limit: wide column blocks, many blocks of few entries, tiles of products of 12 bytes a pair.  Calls by the scan / by lists in
    # us: 4,897 / 800, 596 / 238, 2,961 / 268
    for n, nnz, cols, metric in ((56_257, 5_172_942, 236_097, "hellinger"), (12_970, 77_804, 10_261, "jensen_shannon"),
                                 (10_772, 4_546_630, 728_767, "kl_divergence")):
        assert kept(n, nnz / n, cols, metric) > 0, (n, cols, metric)
    # ... and with an entry of six bytes, and six to what a dense column may need: sizes whose lists eight left out
    for n, nnz, cols, metric in ((94_601, 70_971, 2_890, "jensen_shannon"), (172_261, 19_812, 862, "cosine"), (3_570, 1_759, 42_690, "l1"),
                                 (15_919, 8_254, 20_697, "hamming"), (185_974, 572_974, 10_395, "hamming")):
        assert kept(n, nnz / n, cols, metric) > 0, (n, cols, metric)
    # the working range
    for n, mean, cols in ((300, 37, 20_000), (12_000, 37, 20_000), (5_000, 228, 102_660), (300_000, 228, 102_660), (500, 1_820, 26_000),
                          (60_000, 1_820, 26_000), (2_000, 160, 194_000), (200_000, 160, 194_000)):
        # (Minkowski's tiles are half as long: over 194,000 columns their bounds outgrow rows of 160)
        for metric in ("cosine", "l1", "canberra", "jensen_shannon") + (("minkowski",) if cols < 194_000 else ()):
            assert kept(n, mean, cols, metric) > 0, (n, mean, cols, metric)


def test_small_calls_are_one_launch_where_no_row_of_b_is_long():
    def lanes(m, mean_a, lengths, cols, metric, **more):
        return spd.testing.host_direct_lanes(np.concatenate([[0], np.cumsum(lengths)]), m, m * mean_a, cols, metric, **more)

    def one_long(n, short, longest):
        return [longest] + [short] * (n - 1)

    # both ways measured, others / one launch in us: 27 / 8.5, 52 / 30
    assert lanes(256, 10, [10] * 256, 512, "l1") == 1
    assert lanes(7, 1, [337] * 194, 512, "l1") == 4
    # 59 / 3,140 with a lane to the row, 73 / 3,546, 31 / 1,616, 41 / 1,510, 40 / 1,309
    assert lanes(10_633, 6, one_long(47, 700, 2_048), 2_048, "jensen_shannon") == 0
    assert lanes(16, 17, one_long(1_024, 52, 1_000), 1_000, "minkowski", p=3.0, k_neighbors=10) == 0
    assert lanes(3, 2, one_long(9, 400, 2_048), 2_048, "minkowski", p=3.0) == 0
    assert lanes(16, 1, one_long(3, 10, 1_868), 2_048, "minkowski", p=3.0, k_neighbors=3) == 0
    assert lanes(1, 3, one_long(7, 2, 1_653), 2_048, "minkowski", p=3.0, k_neighbors=7) == 0
    # longer rows turn the choice once, sooner with an index, which leaves less for one launch to save
    for metric in ("l1", "hamming", "jensen_shannon", "minkowski"):
        for k in (0, 5):
            plain, index = ([lanes(64, 10, [c] * 30, 2_048, metric, k_neighbors=k, with_index=ix) > 0 for c in (1, 4, 16, 64, 256, 1_024, 2_048)]
                            for ix in (False, True))
            assert plain[0] and not plain[-1] and plain == sorted(plain, reverse=True) and index == sorted(index, reverse=True)
            assert sum(index) <= sum(plain)
    # one entry, column, pair or row more than it takes
    assert lanes(8, 1, [1] * 1_024, 2_048, "l1") > 0 and lanes(8, 1, [1] * 1_024, 2_049, "l1") == 0
    assert lanes(1, 1, [1] * 32_768, 64, "l1") > 0 and lanes(1, 1, [1] * 32_769, 64, "l1") == 0
    assert lanes(8, 1, [1] * 1_024, 64, "l1", k_neighbors=3) > 0 and lanes(8, 1, [1] * 1_025, 64, "l1", k_neighbors=3) == 0
    assert lanes(8, 1, [1] * 64, 64, "chebyshev") == 0

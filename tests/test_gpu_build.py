"""GPU parity of tree growth (Alg. 1 / Alg. 2, median split): every split value (bit for
bit in binary64), split index, chosen direction, leaf order and leaf membership of every
tree equals the oracle's on the same data and directions."""

import numpy as np
import pytest
import torch

import oracle
from tests.helpers import problem

pytestmark = pytest.mark.gpu

CASES = [
    # name, n, d, T, n0, n_try, kind, dup
    ("mixture_10k_d16", 10_000, 16, 4, 50, 1, "mixture", 0),      # one multi-block level
    ("aniso_20k_d128", 20_000, 128, 3, 256, 1, "aniso", 0),
    ("d1", 3000, 1, 2, 20, 1, "mixture", 0),
    ("d33_scalar_path", 5000, 33, 2, 40, 1, "mixture", 0),
    ("ntry3_small", 3000, 12, 2, 30, 3, "aniso", 0),
    ("ntry4_large", 12_000, 20, 2, 64, 4, "aniso", 0),
    ("duplicates", 9000, 8, 3, 30, 1, "mixture", 7),
    ("wide_exponents", 6000, 24, 2, 50, 1, "wide", 0),
    ("quantized_d784", 5000, 784, 2, 512, 1, "quant", 0),
    ("single_leaf", 300, 5, 2, 300, 1, "mixture", 0),
    ("n0_plus_1", 51, 5, 2, 50, 1, "mixture", 0),
    ("tiny_n0_1", 37, 3, 2, 1, 1, "mixture", 0),
]


def _gpu_forest(x, R, T, n0, n_try):
    from paper_1812_11689_amd import rpf
    X = torch.from_numpy(x).cuda()
    Rd = torch.from_numpy(np.ascontiguousarray(R[:T])).cuda()
    return rpf.build(X, T, n0, Rd, n_try=n_try)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_build_matches_oracle(case):
    name, n, d, T, n0, n_try, kind, dup = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0} nTry={n_try}", flush=True)
    x, R = problem(n, d, T, n0, n_try, seed=len(name), kind=kind, dup_every=dup)
    ref = oracle.build_forest(x, R, T, n0, n_try)
    f = _gpu_forest(x, R, T, n0, n_try)
    info = f.info()  # synchronises and surfaces device-side invariant failures
    assert info["depth"] == ref.L
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        np.testing.assert_array_equal(g["leaf_of"], ref.leaf_of[t])
        assert np.array_equal(g["split"].view(np.uint64), ref.split[t].view(np.uint64)) or \
            np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
        np.testing.assert_array_equal(g["chosen"], ref.chosen[t])
    f.free()


SELECT_CASES = [
    # the median of multi-block nodes: read whole up to 16 384 members, bracketed from a sample
    # of 2 048 above; more than 1 024 chunks
    # name, n, d, T, n0, n_try, what
    ("one_over_a_workgroup", 4097, 6, 3, 2000, 1, "mixture"),
    ("read_whole_16384", 16_384, 4, 2, 9000, 1, "mixture"),
    ("bracketed_16385", 16_385, 4, 2, 9000, 1, "mixture"),
    ("bracketed_tries", 66_000, 6, 2, 20_000, 3, "mixture"),
    ("ties_at_the_median", 70_000, 3, 2, 9000, 1, "ties"),
    ("bracket_read_again", 300_000, 3, 2, 90_000, 1, "mixture"),  # more listed than registers hold
    ("two_values", 40_000, 1, 2, 6000, 1, "two"),
    ("sample_misses", 70_000, 1, 2, 20_000, 1, "misses"),
    ("spread_overflows", 9_000, 1, 2, 3000, 1, "huge"),
    ("chunks_past_1024", 4_300_000, 2, 1, 1_100_000, 1, "mixture"),
    ("chunks_past_1024_sample_misses", 4_300_000, 1, 1, 2_200_000, 1, "misses"),
]


@pytest.mark.parametrize("case", SELECT_CASES, ids=[c[0] for c in SELECT_CASES])
def test_median_select_matches_oracle(case):
    name, n, d, T, n0, n_try, what = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0}", flush=True)
    x, R = problem(n, d, T, n0, n_try, seed=len(name) + 60)
    if what == "ties":
        x[: 2 * n // 3] = x[n - 1]  # two thirds of the rows are one point
    elif what == "two":
        x[:] = (np.arange(n) % 3 == 0).astype(np.float32)[:, None]
    elif what == "huge":  # differences of projections reach 1e38 beside values near 1e-38
        x *= np.float32(10.0) ** np.linspace(-38, 37, n, dtype=np.float32)[:, None]
    elif what == "misses":  # the evenly spaced sample holds only the largest values
        at = (np.arange(2048, dtype=np.int64) * n + n // 2) // 2048
        x[at] += np.float32(1000.0)
    ref = oracle.build_forest(x, R, T, n0, n_try)
    f = _gpu_forest(x, R, T, n0, n_try)
    f.info()  # surfaces device-side invariant failures
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        np.testing.assert_array_equal(g["leaf_of"], ref.leaf_of[t])
        assert np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
    f.free()


EQUAL_CASES = [
    # medians among many equal keys: at either end of the bracket or between, in any chunk
    # name, n, d, T, n0, distinct rows, share of the first (rows in runs: whole chunks of one key)
    ("two_thirds_one_row", 70_000, 3, 2, 5000, 0, 0.67, False),
    ("a_fifth_one_row", 100_000, 4, 3, 5000, 0, 0.2, False),
    ("five_rows", 100_000, 4, 3, 5000, 5, 0.0, False),
    ("five_rows_in_runs", 100_000, 4, 3, 5000, 5, 0.0, True),
    ("twelve_rows_many_nodes", 20_000, 3, 130, 4200, 12, 0.0, False),
    ("one_row", 40_000, 2, 2, 5000, 1, 0.0, False),
    ("chunks_past_1024", 4_300_000, 2, 1, 1_100_000, 3, 0.0, False),
]


@pytest.mark.parametrize("case", EQUAL_CASES, ids=[c[0] for c in EQUAL_CASES])
def test_median_among_equal_keys(case):
    name, n, d, T, n0, rows, share, runs = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0}", flush=True)
    rng = np.random.default_rng(len(name) + 75)
    x, R = problem(n, d, T, n0, 1, seed=len(name) + 75)
    if rows:
        pick = rng.integers(0, rows, n)
        x = x[np.sort(pick) if runs else pick]
    if share:
        x[rng.random(n) < share] = x[0]
    x = np.ascontiguousarray(x)
    ref = oracle.build_forest(x, R, T, n0, 1)
    f = _gpu_forest(x, R, T, n0, 1)
    f.info()
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        assert np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
    f.free()


WIDE_CASES = [
    # levels of at most 256 workgroups: 1024 threads each, from 512 members on
    # name, n, d, T, n0, n_try, kind, dup
    ("wide_511", 511, 6, 1, 100, 1, "mixture", 0),
    ("wide_512", 512, 7, 1, 100, 1, "aniso", 0),
    ("wide_1025_fed", 1025, 33, 2, 200, 1, "mixture", 0),
    ("wide_4096", 4096, 20, 1, 30, 1, "aniso", 0),
    ("wide_4097_chunks", 4097, 20, 3, 30, 1, "aniso", 0),
    ("wide_256_workgroups", 2048, 8, 128, 500, 1, "aniso", 0),   # 256 at the second level
    ("wide_258_workgroups", 2048, 8, 129, 500, 1, "aniso", 0),   # 258: 256 threads
    ("wide_ties", 3000, 4, 2, 40, 1, "mixture", 5),
    ("wide_d1500", 5000, 1500, 1, 600, 1, "mixture", 0),         # directions past the staged length
]


@pytest.mark.parametrize("case", WIDE_CASES, ids=[c[0] for c in WIDE_CASES])
def test_wide_levels_match_oracle(case):
    test_build_matches_oracle(case)


@pytest.mark.parametrize("d", [48, 50])
def test_wide_levels_of_a_grid_forest(d):
    from paper_1812_11689_amd import rpf
    x = (np.random.default_rng(70).integers(0, 256, (9000, d)) / 255).astype(np.float32)
    R = np.random.default_rng(71).standard_normal((2, 2 ** rpf.depth(9000, 300) - 1, 1, d)).astype(np.float32)
    ref = oracle.build_forest(x, R, 2, 300, 1)
    f = rpf.build(torch.from_numpy(x).cuda(), 2, 300, torch.from_numpy(R).cuda(), dist_prec="u8grid")
    for t in range(2):
        np.testing.assert_array_equal(f.tree_dump(t)["perm"].cpu().numpy(), ref.perm[t])
    f.free()


DIGIT_CASES = [
    # grid forests of long rows: keys by digits, exact ones around the median
    # name, n, d, T, n0, what
    ("d512_chunks", 9000, 512, 2, 300, "images"),
    ("d513_scalar", 5000, 513, 2, 60, "images"),
    ("d1024", 4097, 1024, 1, 100, "images"),
    ("d1023_small_nodes", 700, 1023, 3, 20, "images"),
    ("nodes_of_128", 512, 600, 2, 30, "images"),
    ("two_values_ties", 6000, 512, 2, 100, "binary"),       # members in the band by the hundred
    ("few_distinct_rows", 9000, 520, 2, 100, "copies"),
    ("one_row", 5000, 512, 1, 600, "one"),                  # every member in the band
    ("zero_directions", 3000, 512, 2, 100, "zero"),
    ("wide_directions", 9000, 700, 2, 100, "wide"),         # 1e30 beside 1e-30: a band of many
]


@pytest.mark.parametrize("case", DIGIT_CASES, ids=[c[0] for c in DIGIT_CASES])
def test_digit_projections_match_oracle(case):
    from paper_1812_11689_amd import rpf
    name, n, d, T, n0, what = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0}", flush=True)
    rng = np.random.default_rng(len(name) + 72)
    k = rng.integers(0, 256, (n, d))
    if what == "binary":
        k = 255 * (k[:, :1] < 128) * (np.arange(d) < 4)[None] + 0 * k
    elif what == "copies":
        k = k[rng.integers(0, 5, n)]
    elif what == "one":
        k = np.broadcast_to(k[:1], (n, d))
    x = (np.ascontiguousarray(k).astype(np.float32) / np.float32(255)).astype(np.float32)
    R = rng.standard_normal((T, 2 ** rpf.depth(n, n0) - 1, 1, d)).astype(np.float32)
    if what == "zero":
        R[:, ::2] = 0
    elif what == "wide":
        R *= (np.float32(10.0) ** rng.uniform(-30, 30, R.shape)).astype(np.float32)
    ref = oracle.build_forest(x, R, T, n0, 1)
    f = rpf.build(torch.from_numpy(x).cuda(), T, n0, torch.from_numpy(R).cuda(), dist_prec="u8grid")
    f.info()
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        assert np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
    f.free()


BAND_CASES = [
    # most members near their node's median: the pairs of levels below the first project exactly
    # name, n, d, T, n0, what
    ("half_blank_chunks", 70_000, 512, 1, 900, "blank"),      # four multi-block levels
    ("half_blank_scalar", 70_000, 513, 1, 900, "blank"),
    ("half_blank_one_workgroup", 6000, 600, 3, 40, "blank"),
    ("blank_then_not", 40_000, 512, 2, 200, "part"),          # some nodes full of copies, some with none
    ("directions_of_zeros", 40_000, 512, 2, 300, "zeros"),    # every third node
]


@pytest.mark.parametrize("case", BAND_CASES, ids=[c[0] for c in BAND_CASES])
def test_digit_bands_of_many_members_match_oracle(case):
    from paper_1812_11689_amd import rpf
    name, n, d, T, n0, what = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0}", flush=True)
    rng = np.random.default_rng(len(name) + 76)
    k = rng.integers(0, 256, (n, d), dtype=np.uint8)
    if what == "blank":
        k[::2] = 0
    elif what == "part":
        k[: n // 4] = k[0]
    x = (np.arange(256, dtype=np.float32) / np.float32(255))[k]
    R = rng.standard_normal((T, 2 ** rpf.depth(n, n0) - 1, 1, d)).astype(np.float32)
    if what == "zeros":
        R[:, ::3] = 0
    ref = oracle.build_forest(x, R, T, n0, 1)
    f = rpf.build(torch.from_numpy(x).cuda(), T, n0, torch.from_numpy(R).cuda(), dist_prec="u8grid")
    f.info()
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        assert np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
    f.free()


TRY_CASES = [
    # several tries per node: sums over pieces of 256 members, nodes scored in one workgroup
    # (up to 512 members) or over many blocks, 2 to 5 tries per read, more than 16 tries
    # name, n, d, T, n0, n_try, kind, dup
    ("try2_513_over_the_workgroup", 513, 7, 3, 40, 2, "aniso", 0),
    ("try10_512_one_workgroup", 512, 49, 3, 20, 10, "aniso", 0),
    ("try7_257_members", 257, 166, 2, 16, 7, "mixture", 0),
    ("try3_pieces_at_the_root", 70_000, 5, 2, 64, 3, "aniso", 0),  # 274 pieces of 256
    ("try19_two_groups", 9000, 18, 2, 30, 19, "mixture", 0),
    ("try4_duplicates", 3000, 8, 2, 25, 4, "mixture", 7),
    ("try2_d1100_long_rows", 1500, 1100, 1, 100, 2, "mixture", 0),
    ("try5_n0_1", 61, 3, 2, 1, 5, "mixture", 0),
]


@pytest.mark.parametrize("case", TRY_CASES, ids=[c[0] for c in TRY_CASES])
def test_tries_match_oracle(case):
    test_build_matches_oracle(case)


def test_tries_within_a_tight_memory_budget():
    """A budget that leaves no room for the tries' projections still grows the same forest."""
    from paper_1812_11689_amd import rpf
    n, d, T, n0, n_try = 1500, 12, 2, 20, 4
    x, R = problem(n, d, T, n0, n_try, seed=23, kind="aniso")
    ref = oracle.build_forest(x, R, T, n0, n_try)
    Xd, Rd = torch.from_numpy(x).cuda(), torch.from_numpy(np.ascontiguousarray(R[:T])).cuda()
    f = rpf.build(Xd, T, n0, Rd, n_try=n_try)
    budget = f.info()["device_bytes"] + T * n * 16 * 4  # and the query copies (rows padded to 16)
    f.free()
    f = rpf.build(Xd, T, n0, Rd, n_try=n_try, mem_budget_bytes=budget)
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        np.testing.assert_array_equal(g["chosen"], ref.chosen[t])
    f.free()


GRID_CASES = [
    # points on the 1/255 grid, built with RPF_DIST_U8GRID: the projections read each row from
    # the int8 copy (k - 128) instead of X and must give the same splits bit for bit
    # name, n, d, T, n0, n_try
    ("grid_d784", 5000, 784, 2, 512, 1),
    ("grid_d50_multiblock", 40_000, 50, 3, 64, 1),
    ("grid_d7_ntry3", 6000, 7, 2, 30, 3),
]


@pytest.mark.parametrize("case", GRID_CASES, ids=[c[0] for c in GRID_CASES])
def test_grid_build_matches_oracle(case):
    from paper_1812_11689_amd import rpf
    name, n, d, T, n0, n_try = case
    print(f"[build] {name} n={n} d={d} T={T} n0={n0} nTry={n_try} (int8 grid rows)", flush=True)
    x, R = problem(n, d, T, n0, n_try, seed=len(name) + 50, kind="quant")
    ref = oracle.build_forest(x, R, T, n0, n_try)
    f = rpf.build(torch.from_numpy(x).cuda(), T, n0, torch.from_numpy(np.ascontiguousarray(R[:T])).cuda(),
                  n_try=n_try, dist_prec="u8grid")
    f.info()
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        np.testing.assert_array_equal(g["leaf_of"], ref.leaf_of[t])
        assert np.array_equal(g["split"].view(np.uint64), ref.split[t].view(np.uint64))
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
        np.testing.assert_array_equal(g["chosen"], ref.chosen[t])
    f.free()


SUBTREE_CASES = [c for c in CASES if c[5] == 1 and c[0] not in ("single_leaf", "n0_plus_1")] + [
    # every level one-block from the root; levels of mixed leaf and internal nodes
    ("all_small_levels", 3000, 6, 3, 10, 1, "mixture", 0),
    ("n0_3_deep", 4000, 9, 2, 3, 1, "aniso", 0),
]


@pytest.mark.parametrize("case", SUBTREE_CASES, ids=[c[0] for c in SUBTREE_CASES])
def test_subtree_schedule_matches_oracle(case):
    # RPF_BUILD_SUBTREES: the one-block levels run as one persistent launch; the forest must be
    # the same, bit for bit
    from paper_1812_11689_amd import rpf
    name, n, d, T, n0, n_try, kind, dup = case
    print(f"[subtree] {name} n={n} d={d} T={T} n0={n0}", flush=True)
    x, R = problem(n, d, T, n0, n_try, seed=len(name) + 50, kind=kind, dup_every=dup)
    ref = oracle.build_forest(x, R, T, n0, n_try)
    rpf.profile_reset()
    rpf.profile_enable(True)
    f = rpf.build(torch.from_numpy(x).cuda(), T, n0, torch.from_numpy(np.ascontiguousarray(R[:T])).cuda(),
                  n_try=n_try, subtrees=True)
    info = f.info()
    rpf.profile_enable(False)
    prof = rpf.profile_read()
    if ref.L >= 2:
        assert "subtree_levels" in prof, "the persistent launch did not run"
    for t in range(T):
        g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
        np.testing.assert_array_equal(g["perm"], ref.perm[t])
        np.testing.assert_array_equal(g["leaf_of"], ref.leaf_of[t])
        assert np.array_equal(g["split"].view(np.uint64), ref.split[t].view(np.uint64)) or \
            np.array_equal(g["split"], ref.split[t], equal_nan=True)
        np.testing.assert_array_equal(g["split_idx"], ref.split_idx[t])
    assert info["depth"] == ref.L
    f.free()


def test_build_twice_bit_identical():
    x, R = problem(8000, 32, 3, 40, seed=5)
    a = _gpu_forest(x, R, 3, 40, 1)
    b = _gpu_forest(x, R, 3, 40, 1)
    for t in range(3):
        da, db = a.tree_dump(t), b.tree_dump(t)
        for k in da:
            assert torch.equal(da[k].view(torch.int64) if da[k].dtype == torch.float64 else da[k],
                               db[k].view(torch.int64) if db[k].dtype == torch.float64 else db[k]), k


def test_routing_matches_oracle():
    x, R = problem(12_000, 24, 4, 60, seed=9)
    q, _ = problem(3000, 24, 1, 60, seed=19)
    ref = oracle.build_forest(x, R, 4, 60)
    f = _gpu_forest(x, R, 4, 60, 1)
    got = f.route(torch.from_numpy(q).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got, oracle.route(ref, q))
    # data points fall into their own leaves
    got_self = f.route(torch.from_numpy(x).cuda()).cpu().numpy()
    np.testing.assert_array_equal(got_self, ref.leaf_of)


def test_nonfinite_input_rejected():
    from paper_1812_11689_amd import rpf
    x, R = problem(500, 4, 2, 20, seed=3)
    x[17, 2] = np.nan
    with pytest.raises(rpf.RpfError) as e:
        _gpu_forest(x, R, 2, 20, 1)
    assert e.value.status == rpf.RPF_EINVAL


@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "unaligned"])
def test_input_copy_check_edges(shift):
    """The input copy and its non-finite check, on 16-byte aligned and unaligned inputs whose
    length is not a multiple of four: a NaN or an infinity anywhere (first value, middle, the
    last value) is rejected, and a finite input grows the same forest as the oracle."""
    from paper_1812_11689_amd import rpf
    n, d, T, n0 = 333, 3, 2, 20
    x, R = problem(n, d, T, n0, 1, seed=11)
    print(f"[build] input copy check shift={shift} n={n} d={d}", flush=True)
    Rd = torch.from_numpy(np.ascontiguousarray(R[:T])).cuda()

    def as_dev(a):
        buf = torch.zeros(n * d + 4, dtype=torch.float32, device="cuda")
        buf[shift:shift + n * d] = torch.from_numpy(a.reshape(-1)).cuda()
        return buf[shift:shift + n * d].view(n, d)

    for pos, bad in [(0, np.nan), (n * d // 2, np.inf), (n * d - 1, np.nan), (n * d - 2, -np.inf)]:
        xb = x.copy().reshape(-1)
        xb[pos] = bad
        with pytest.raises(rpf.RpfError) as e:
            rpf.build(as_dev(xb.reshape(n, d)), T, n0, Rd)
        assert e.value.status == rpf.RPF_EINVAL
    ref = oracle.build_forest(x, R, T, n0, 1)
    f = rpf.build(as_dev(x), T, n0, Rd)
    try:
        for t in range(T):
            g = {k: v.cpu().numpy() for k, v in f.tree_dump(t).items()}
            np.testing.assert_array_equal(g["perm"], ref.perm[t])
            np.testing.assert_array_equal(g["leaf_of"], ref.leaf_of[t])
            assert np.array_equal(g["split"].view(np.uint64), ref.split[t].view(np.uint64)) or \
                np.array_equal(g["split"], ref.split[t], equal_nan=True)
    finally:
        f.free()

"""The ways a batch is grouped and its rows reduced, at the sizes where each can go wrong.  Integer work
(the grouping) must equal the oracle's; updates run on exact inputs (small integers, powers of two), so the
touched rows must be equal too, whatever the order of the sums."""
import numpy as np
import pytest
import torch

import paper_1906_00091_amd as hot
from oracle import oracle
from workloads import gen

from hotpath_util import DEV, SCALE_FLOOR, Compact, partition_bits, table_to_numpy, widen_host
from test_gpu_exact_counts import _assert_only_touched_rows_changed, _integer_dS, _integer_tables, _max_run, _pow2_weights, _run_update

pytestmark = pytest.mark.gpu


def _batch(lengths, rows, seed, d=4):
    """A batch of the given bag lengths [K][B], uniform row ids."""
    rng = np.random.default_rng([9, seed])
    bags = [[rng.integers(0, rows[k], size=n).tolist() for n in lengths[k]] for k in range(len(lengths))]
    return gen.batch_from_lists(rows, bags, d=d, seed=seed)


# name, lookups of every table (in bags of about `bag`), rows: partition digits 1, 4 and more (2: see below); no tile, one
# tile and more tiles than a round of the column scan takes; more tables than lookups
GROUPINGS = [
    ("tables-without-lookups-between", [0, 1, 0, 1023, 1024, 1025, 0], 7, 3000),
    ("more-tables-than-lookups", [1 if k % 7 == 0 else 0 for k in range(600)], 1, 50),
    ("many-tables-few-digits", [(k * 37) % 300 for k in range(700)], 5, 4),
    ("column-scan-255-256-257-tiles", [255 * 1024, 256 * 1024, 256 * 1024 + 1], 64, 1 << 20),
    ("column-scan-ragged-tables", [700 * 1024 - 3, 5, 0, 1024], 33, 70000),
    # bag starts of a tile: 1024 of 1024 (1024 digits too), tables whose later bags are empty, 1365 of 4096
    ("one-hot-1024-digits", [200000], 1, 5000),
    ("one-hot-then-empty-bags", [70000, 3, 0, 69999, 1024], 1, 100000),
    ("large-tiles-short-bags", [1200001, 5000], 3, 3000),
]


@pytest.mark.parametrize("case", GROUPINGS, ids=[c[0] for c in GROUPINGS])
def test_grouping_equals_the_oracle_at_partition_edges(case):
    name, per_table, bag, m = case
    print("[case] grouping " + name, flush=True)
    B = max(1, max(per_table) // bag)
    lengths = [[n // B + (1 if b < n % B else 0) for b in range(B)] for n in per_table]
    K = len(per_table)
    b = _batch(lengths, [m] * K, seed=1)
    t = torch.zeros((m, 4), dtype=torch.float32, device=DEV)
    sb = hot.SparseBatch([t] * K, gen.F32, torch.from_numpy(b.indices).to(DEV), torch.from_numpy(b.offsets).to(DEV),
                         torch.from_numpy(b.tbl_off).to(DEV), b.nnz)
    out = [torch.zeros(b.nnz, dtype=torch.int64, device=DEV) for _ in range(2)]
    sbag = torch.zeros(b.nnz, dtype=torch.int32, device=DEV)
    nu = torch.zeros(K, dtype=torch.int64, device=DEV)
    hot.dlrm_emb_bag_bwd_export_groups(sb, hot.alloc_workspace(sb), out[0], out[1], sbag, nu)
    torch.cuda.synchronize()
    uniq, seg, sbag, nu = out[0].cpu().numpy(), out[1].cpu().numpy(), sbag.cpu().numpy(), nu.cpu().numpy()
    want = oracle.group_rows(b.indices, b.offsets, b.tbl_off)
    for k in range(K):
        a0, a1 = int(b.tbl_off[k]), int(b.tbl_off[k + 1])
        wu, wseg, _, wbag = want[k]
        assert int(nu[k]) == len(wu)
        assert np.array_equal(uniq[a0:a0 + len(wu)], wu) and np.array_equal(seg[a0:a0 + len(wu)], wseg)
        assert np.array_equal(sbag[a0:a1], wbag)


# the bits of the partition digit that those cases have, and one of two digits, which no case above has any more
GROUPING_BITS = {"tables-without-lookups-between": 2, "more-tables-than-lookups": 0, "many-tables-few-digits": 0,
                 "column-scan-255-256-257-tiles": 9, "column-scan-ragged-tables": 9, "one-hot-1024-digits": 10,
                 "one-hot-then-empty-bags": 8, "large-tiles-short-bags": 10}


def test_groupings_cover_the_partition_digits():
    for name, per_table, _, m in GROUPINGS:
        assert partition_bits(sum(per_table), len(per_table), 4, m) == GROUPING_BITS[name], name


def test_grouping_of_many_tables_with_two_digits_equals_the_oracle():
    per_table = [(k * 37) % 600 for k in range(700)]
    assert partition_bits(sum(per_table), 700, 4, 4) == 1
    test_grouping_equals_the_oracle_at_partition_edges(("many-tables-two-digits", per_table, 5, 4))


# around the limits of the one-launch form (65536 lengths, 4096 tables), a scan round (4096 bags) and a wavefront
@pytest.mark.parametrize("K,B", [(1, 1), (3, 63), (1, 4096), (2, 4097), (1, 65536), (1, 65537), (16, 4096), (17, 4096),
                                 (4096, 16), (4097, 3), (4096, 1)])
def test_lengths_to_offsets_is_exact_around_its_launch_limits(K, B):
    print("[case] lengths K=%d B=%d" % (K, B), flush=True)
    lengths = np.random.default_rng([K, B]).integers(0, 200, size=(K, B)).astype(np.int32)
    off = torch.full((K, B + 1), -7, dtype=torch.int64, device=DEV)
    tbl = torch.full((K + 1,), -7, dtype=torch.int64, device=DEV)
    hot.dlrm_lengths_to_offsets(torch.from_numpy(lengths).to(DEV), off, tbl)
    torch.cuda.synchronize()
    want_off, want_tbl = oracle.lengths_to_offsets(lengths)
    assert np.array_equal(off.cpu().numpy(), want_off) and np.array_equal(tbl.cpu().numpy(), want_tbl)


@pytest.mark.parametrize("B", [2 ** 31 - 4095, 2 ** 31 - 2])
def test_lengths_to_offsets_up_to_the_largest_batch(B):
    """K * (B + 1) up to DLRM_MAX_NNZ: a scan round of 4096 bags ends beyond 2^31."""
    print("[case] lengths K=1 B=%d" % B, flush=True)
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 26 GB of device memory for lengths and offsets")
    g = torch.Generator(device=DEV).manual_seed(1)
    lengths = torch.randint(0, 3, (1, B), generator=g, device=DEV, dtype=torch.int32)
    off = torch.full((1, B + 1), -7, dtype=torch.int64, device=DEV)
    tbl = torch.full((2,), -7, dtype=torch.int64, device=DEV)
    hot.dlrm_lengths_to_offsets(lengths, off, tbl)
    assert off[0, 0].item() == 0 and tbl.tolist() == [0, off[0, B].item()]
    for b0 in range(0, B, 1 << 28):
        n = min(1 << 28, B - b0)
        assert torch.equal(off[0, b0 + 1:b0 + n + 1] - off[0, b0:b0 + n], lengths[0, b0:b0 + n].long())
    del lengths, off
    torch.cuda.empty_cache()


def _assert_exact_update(b, dtype, weighted, modes):
    """The update of batch b on exactly representable numbers equals the oracle's; returns the routes of the last mode."""
    w = b.workload
    wts = _pow2_weights(b) if weighted else None
    dS = _integer_dS(w.B, w.K, w.d, max(_max_run(b), 1), 2.0 if weighted else 1.0)
    lr = 0.5 if dtype == gen.F32 else 2.0 ** -8
    start = _integer_tables(b.rows, w.d, dtype, seed=5)
    comp = Compact(b, host_rows_of=lambda k, u: table_to_numpy(
        start[k].index_select(0, torch.from_numpy(u).to(DEV)), dtype))
    ref = [t.copy() for t in comp.tables]
    if weighted:
        oracle.emb_bag_bwd_weighted(ref, dtype, comp.indices, b.offsets, b.tbl_off, wts, dS, lr)
    else:
        oracle.emb_bag_bwd_sgd(ref, dtype, comp.indices, b.offsets, b.tbl_off, dS, lr)
    dT = torch.zeros((w.B, w.K + 1, w.d), dtype=torch.float32, device=DEV)
    dT[:, 1:, :] = torch.from_numpy(dS).to(DEV)
    for mode in modes:
        tables = [t.clone() for t in start]
        counts = _run_update(b, tables, dT, lr, mode, weights=wts)
        for k in range(w.K):
            got = table_to_numpy(tables[k].index_select(0, torch.from_numpy(comp.uniq[k]).to(DEV)), dtype)
            assert np.array_equal(got.view(np.uint8), ref[k].view(np.uint8)), (mode, k)
            _assert_only_touched_rows_changed(start[k], tables[k], comp.uniq[k])
    return counts


# name, tables, bags, d, type, rows, lookups per bag: 1 .. 7 hot rows are gathered and 8 go to the matrix cores; bag
# groups (256 bags and up) one short of full, full plus one, and many; one, two and four 64-column pieces; more than
# 64 tables (whose hot lists' starts are summed by 64 lanes)
HOT = [
    ("one-row-255-bags", 1, 255, 4, gen.F32, 1, 300),
    ("seven-rows-257-bags", 2, 257, 64, gen.F16, 7, 300),
    ("eight-rows-257-bags", 2, 257, 64, gen.F16, 8, 300),
    ("five-rows-two-pieces", 1, 1025, 136, gen.BF16, 5, 70),
    ("three-rows-wide", 1, 4097, 256, gen.F32, 3, 40),
    ("seventy-tables", 70, 513, 12, gen.F32, 2, 9),
]


@pytest.mark.parametrize("weighted", [False, True], ids=["sum", "pow2-weights"])
@pytest.mark.parametrize("case", HOT, ids=[c[0] for c in HOT])
def test_hot_rows_at_the_edges_of_bag_groups(case, weighted):
    name, K, B, d, dtype, rows, bag = case
    print("[case] hot rows %s weighted=%s" % (name, weighted), flush=True)
    b = gen.make_batch(gen.custom_workload(name, K=K, B=B, d=d, dtype=dtype, rows=rows, bag=("fixed", bag), dist=("uniform",),
                                           seed=31))
    counts = _assert_exact_update(b, dtype, weighted, ("sort",))
    assert counts["hot_rows"] == K * rows


# rows narrower than a 64-column piece; dT fills whole 2 MiB pages, the last row of the last table ends with them
@pytest.mark.parametrize("B,d", [(262144, 4), (65536, 32), (131072, 36)])
def test_dense_hot_rows_read_nothing_behind_the_gradients(B, d):
    """Nothing is mapped behind an allocation of whole pages: a lane that read past the last row would fault."""
    print("[case] dense hot rows, narrow B=%d d=%d" % (B, d), flush=True)
    K = 2
    assert B * (K + 1) * d * 4 % (2 << 20) == 0 and B * (K + 1) * d * 4 >= 10 << 20
    torch.cuda.empty_cache()
    b = gen.make_batch(gen.custom_workload("narrow", K=K, B=B, d=d, dtype=gen.F32, rows=9, bag=("fixed", 1), dist=("uniform",),
                                           seed=8))
    counts = _assert_exact_update(b, gen.F32, False, ("sort",))
    assert counts["hot_rows"] == 9 * K and counts["dense_hot_tables"] == K


# one and two tables with hot rows among others: their bag groups are cut by the number of such tables (batch 5000:
# ten groups of 512 bags for one among 128 tables, whose share of the machine would be six), 3 rows gathered, 9 dense
@pytest.mark.parametrize("d", [4, 132])
@pytest.mark.parametrize("hot_at", [(77,), (0, 127)])
@pytest.mark.parametrize("rows", [3, 9])
def test_hot_rows_in_few_of_many_tables(rows, hot_at, d):
    print("[case] hot rows in few tables rows=%d at=%s d=%d" % (rows, hot_at, d), flush=True)
    B, K = 5000, 128
    lengths = [[5] * B if k in hot_at else [1 if (b + k) % 9 == 0 else 0 for b in range(B)] for k in range(K)]
    b = _batch(lengths, [rows if k in hot_at else 400 + k for k in range(K)], seed=rows, d=d)
    assert _assert_exact_update(b, gen.F32, False, ("sort", "prepared"))["hot_rows"] == rows * len(hot_at)


def test_hot_rows_with_little_room_for_partial_sums():
    """One table with three hot rows among 300 tables of ten lookups: the arrays left over after the grouping hold
    fewer bag groups than the array laid out for partial sums, which is then used."""
    print("[case] hot rows, little room", flush=True)
    B, K, d = 3000, 301, 256
    lengths = [[28] * B] + [[1] * 10 + [0] * (B - 10)] * (K - 1)
    b = _batch(lengths, [3] + [40] * (K - 1), seed=4, d=d)
    # groups of 8 LDS tiles of 64 bags laid out; bytes of the leftover arrays: 8 a lookup, or (weighted) 1024 counts a tile
    laid_out, sums = -(-B // 512), (b.nnz // 2048 + K) * d * 4
    assert b.nnz * 8 // sums < laid_out and 1024 * 4 * ((b.nnz >> 10) + K) // sums < laid_out
    for weighted in (False, True):
        assert _assert_exact_update(b, gen.F32, weighted, ("sort",))["hot_rows"] == 3


# one table whose last bag group (2^31 - 65536) and whose bag search too (2^31 - 2) end beyond 2^31: 3 rows are
# gathered, 9 go to the matrix cores
@pytest.mark.parametrize("weighted", [False, True], ids=["sum", "weighted"])
@pytest.mark.parametrize("rows", [3, 9])
@pytest.mark.parametrize("B", [2 ** 31 - 65536, 2 ** 31 - 2])
def test_hot_rows_of_a_batch_close_to_the_largest(B, rows, weighted):
    """Lookups spread evenly over the bags, every bag with the same gradient: each row moves by its count."""
    nnz = 10000 * 9
    print("[case] hot rows B=%d rows=%d weighted=%s" % (B, rows, weighted), flush=True)
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 17 GB of device memory for the offsets")
    off = torch.empty((1, B + 1), dtype=torch.int64, device=DEV)
    for b0 in range(0, B + 1, 1 << 27):
        n = min(1 << 27, B + 1 - b0)
        off[0, b0:b0 + n] = torch.arange(b0, b0 + n, device=DEV) * nnz // B
    t = torch.zeros((rows, 4), dtype=torch.float32, device=DEV)
    sb = hot.SparseBatch([t], gen.F32, torch.arange(nnz, device=DEV) % rows, off,
                         torch.tensor([0, nnz], dtype=torch.int64, device=DEV), nnz,
                         weights=torch.ones(nnz, device=DEV) if weighted else None)
    g = torch.tensor([[1.0, -2.0, 3.0, 4.0]], device=DEV)
    hot.dlrm_emb_bag_bwd_sgd(sb, g, 0, 4, 1.0, hot.alloc_workspace(sb), algo=hot.BWD_SORT)
    assert torch.equal(t, -(nnz // rows) * g.expand(rows, 4))
    del off, sb
    torch.cuda.empty_cache()


def test_an_infinite_gradient_stays_with_the_hot_rows_it_belongs_to():
    """Three hot rows, each in every bag but one: the gradient of a bag that does not name a row never meets it."""
    print("[case] hot rows, infinite gradient", flush=True)
    B, per = 3000, 30
    bags = [[0] * per + [1] * per if i == 17 else [0] * per + [2] * per for i in range(B)]
    b = gen.batch_from_lists([3], [bags], d=16, seed=2)
    t = torch.zeros((3, 16), dtype=torch.float32, device=DEV)
    dT = torch.ones((B, 2, 16), dtype=torch.float32, device=DEV)
    dT[17, 1, 3] = float("inf")
    counts = _run_update(b, [t], dT, 1.0, "sort")
    assert counts["hot_rows"] == 2
    want = -np.array([[per * B] * 16, [per] * 16, [per * (B - 1)] * 16], dtype=np.float32)
    want[0, 3] = want[1, 3] = -np.inf
    assert np.array_equal(t.cpu().numpy(), want)


def _assert_as_partitioned(b, m, weighted):
    """Exact inputs: the oracle's rows and the routes of the partitioned path.  Any inputs: its bits, with both index
    types and both optimizers.  Tables of m rows; returns the routes."""
    K, B, d = b.workload.K, b.workload.B, b.workload.d
    routes = [_assert_exact_update(b, gen.F32, weighted, (mode,)) for mode in ("prepared", "sort")]
    assert routes[0] == routes[1]

    g = torch.Generator(device=DEV).manual_seed(B)
    wts = torch.rand(b.nnz, generator=g, device=DEV) if weighted else None
    dS = torch.randn((B, K, d), generator=g, device=DEV)
    for dtype, tdt in ((gen.F32, torch.float32), (gen.BF16, torch.bfloat16)):
        start = torch.randn((K, m, d), generator=g, device=DEV).to(tdt)
        h0 = torch.rand((K, m, d), generator=g, device=DEV)
        for itype in (np.int32, np.int64):
            for adagrad in (False, True):
                got = []
                for prepared in (True, False):
                    t, h = start.clone(), h0.clone()
                    sb = hot.SparseBatch([t[k] for k in range(K)], dtype, torch.from_numpy(b.indices.astype(itype)).to(DEV),
                                         torch.from_numpy(b.offsets).to(DEV), torch.from_numpy(b.tbl_off).to(DEV), b.nnz,
                                         weights=wts)
                    ws = hot.alloc_workspace(sb)
                    ws.fill_(0xFF)   # nothing in the workspace is assumed to be zero
                    if prepared:
                        hot.dlrm_emb_bag_bwd_prepare(sb, ws)
                    algo = hot.BWD_SORT_PREPARED if prepared else hot.BWD_SORT
                    if adagrad:
                        hot.dlrm_emb_bag_bwd_adagrad(sb, hot.state_pointers([h[k] for k in range(K)]), dS, K * d, d, 0.1, 1e-8,
                                                     ws, algo=algo)
                    else:
                        hot.dlrm_emb_bag_bwd_sgd(sb, dS, K * d, d, 0.1, ws, algo=algo)
                    got.append((t, h))
                assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), (dtype, itype, adagrad)
    return routes[0]


# Batches of at most 65536 lookups, whose buckets pick their pairs out of the table's lookups.
# name, lookups of every table, bags, rows: chunks of 2048 lookups one short, full and one over; bags of one length
# (1, 3) and ragged ones with empty ones among them, fewer and more of them than the 256 sampled offsets; single-row
# tables, whose buckets outgrow the LDS sort, and tables of three rows; one table with all but a few of 65536 lookups
# (buckets beyond LDS), one with 30000 (buckets within it)
DIRECT = [
    ("chunk-edges-ragged", [2047, 0, 2048, 2049, 1, 4097, 6143], 700, 5000),
    ("one-lookup", [1], 1, 1),
    ("one-hot", [2048] * 3, 2048, 1 << 20),
    ("three-each", [3 * 1025] * 2, 1025, 3000),
    ("one-bag", [2500, 7], 1, 90),
    ("256-bags", [4096, 2048, 5], 256, 300),
    ("257-bags-few-rows", [5000, 2100, 300], 257, 3),
    ("one-row-tables", [3000, 2048, 0, 2049], 2000, 1),
    ("mostly-empty-bags", [500, 40, 0, 2600], 9000, 777),
    ("65536-mostly-in-one-table", [1] * 7 + [65521] + [1] * 8, 900, 5000),
    ("long-table-within-lds", [30000] + [300] * 7, 700, 4000),
]


@pytest.mark.parametrize("weighted", [False, True], ids=["sum", "pow2-weights"])
@pytest.mark.parametrize("case", DIRECT, ids=[c[0] for c in DIRECT])
def test_small_batches_update_as_the_partitioned_path_does(case, weighted):
    name, per_table, B, m = case
    print("[case] direct %s weighted=%s" % (name, weighted), flush=True)
    rng = np.random.default_rng([B, m])
    lengths = [[n // B] * B if n % B == 0 else np.bincount(rng.integers(0, B, size=n), minlength=B).tolist() for n in per_table]
    _assert_as_partitioned(_batch(lengths, [m] * len(per_table), seed=6, d=24), m, weighted)


# One long table (its share of the rows' range a digit of 128 rows) among short ones.  name, its lookups by row (or by
# range of rows) and the route counters of its buckets: rows that dominate their buckets and are split off, beside fewer
# and more others than the LDS sort takes; ranges without such rows, sorted through global memory; both
SKEWED = [
    ("dominant-rows", [(700, 701, 5000), (701, 702, 3000), (2500, 2501, 2500), (640, 768, 900), (0, 4000, 3000)],
     {"oversized_ranges": 2, "dominant_row_splits": 2, "global_sorts": 0, "huge_runs_in_place": 3}),
    ("dominant-row-and-long-rest", [(1300, 1301, 6000), (1280, 1408, 4000), (3900, 4000, 4500), (0, 4000, 2000)],
     {"oversized_ranges": 2, "dominant_row_splits": 1, "global_sorts": 2, "huge_runs_in_place": 1}),
    ("no-dominant-row", [(1280, 1408, 9000), (2560, 2688, 8000), (3968, 4000, 2700), (0, 128, 2049)],
     {"oversized_ranges": 4, "dominant_row_splits": 0, "global_sorts": 4, "huge_runs_in_place": 0}),
]


@pytest.mark.parametrize("weighted", [False, True], ids=["sum", "pow2-weights"])
@pytest.mark.parametrize("case", SKEWED, ids=[c[0] for c in SKEWED])
def test_small_batches_with_one_long_table(case, weighted):
    name, parts, want = case
    print("[case] direct, skewed %s weighted=%s" % (name, weighted), flush=True)
    rng = np.random.default_rng(len(name))
    B, m, K = 600, 4000, 8
    ids = rng.permutation(np.concatenate([rng.integers(lo, hi, size=n) for lo, hi, n in parts]))
    long = [x.tolist() for x in np.split(ids, np.sort(rng.integers(0, len(ids) + 1, size=B - 1)))]
    short = [[[int(i) for i in rng.integers(0, m, size=n)] for n in rng.integers(0, 3, size=B)] for _ in range(K - 1)]
    b = gen.batch_from_lists([m] * K, short[:2] + [long] + short[2:], d=24, seed=6)
    counts = _assert_as_partitioned(b, m, weighted)
    assert {n: counts[n] for n in want} == want


def _assert_adagrad_update(b, dtype, weighted, modes):
    """The Adagrad update of batch b with exact gradient sums g: h + g * g is rounded once on both sides and must be equal; the step
    lr * g / (sqrt(h) + eps) takes a square root, a sum, a quotient, a product and a difference in fp32, half a unit each, and one
    rounding to the storage type.  Rows without lookups (g = 0, none of them touched) keep their bits."""
    w = b.workload
    wts = _pow2_weights(b) if weighted else None
    dS = _integer_dS(w.B, w.K, w.d, max(_max_run(b), 1), 2.0 if weighted else 1.0)
    lr, eps = float(np.float32(0.05)), float(np.float32(1e-8))
    g = [np.zeros((int(m), w.d), dtype=np.float32) for m in b.rows]
    if weighted:
        oracle.emb_bag_bwd_weighted(g, gen.F32, b.indices, b.offsets, b.tbl_off, wts, dS, -1.0)
    else:
        oracle.emb_bag_bwd_sgd(g, gen.F32, b.indices, b.offsets, b.tbl_off, dS, -1.0)
    dT = torch.zeros((w.B, w.K + 1, w.d), dtype=torch.float32, device=DEV)
    dT[:, 1:, :] = torch.from_numpy(dS).to(DEV)
    start = _integer_tables(b.rows, w.d, dtype, seed=5)
    bound = 5 * 2.0 ** -24 + {gen.F32: 0.0, gen.F16: 2.0 ** -11, gen.BF16: 2.0 ** -8}[dtype]
    for mode in modes:
        tables = [t.clone() for t in start]
        state = [torch.full((int(m), w.d), 3.0, device=DEV) for m in b.rows]
        _run_update(b, tables, dT, lr, mode, weights=wts, state=state, eps=eps)
        for k in range(w.K):
            h = (3.0 + g[k].astype(np.float64) ** 2).astype(np.float32)
            assert np.array_equal(state[k].cpu().numpy(), h), (mode, k)
            before = widen_host(table_to_numpy(start[k], dtype), dtype).astype(np.float64)
            after = widen_host(table_to_numpy(tables[k], dtype), dtype).astype(np.float64)
            step = lr * g[k].astype(np.float64) / (np.sqrt(h.astype(np.float64)) + eps)
            scale = np.abs(before) + np.abs(step)
            assert (np.abs(after - (before - step)) <= bound * np.maximum(scale, SCALE_FLOOR[dtype])).all(), (mode, k)
            a0, a1 = int(b.tbl_off[k]), int(b.tbl_off[k + 1])
            _assert_only_touched_rows_changed(start[k], tables[k], np.unique(b.indices[a0:a1]))


# rows on either side of the widths up to which the update keeps rows that share 64-byte sectors in the caches (fp32: SGD
# below 160 bytes, Adagrad below 256; 16-bit: 128 and 96), and whole sectors; buckets of neighbouring rows
@pytest.mark.parametrize("dtype,d", [(gen.F32, 4), (gen.F32, 36), (gen.F32, 44), (gen.F32, 60), (gen.F32, 64), (gen.F16, 8),
                                     (gen.BF16, 40), (gen.F16, 56), (gen.BF16, 72)])
def test_updates_of_rows_that_share_sectors(dtype, d):
    print("[case] shared sectors dtype=%s d=%d" % (dtype, d), flush=True)
    B, m = 900, 700
    for longest in (8, 160):   # 3600 and 72000 lookups a table: without and with a partition
        b = gen.make_batch(gen.custom_workload("sectors", K=2, B=B, d=d, dtype=dtype, rows=m, bag=("uniform", 0, longest),
                                               dist=("uniform",), seed=d))
        for weighted in (False, True):
            _assert_exact_update(b, dtype, weighted, ("sort", "prepared"))
        for weighted in (False, True):
            _assert_adagrad_update(b, dtype, weighted, ("sort", "prepared"))


# row blocks, columns and batches on either side of where the forward takes W wavefronts a sample; the last sample of the large
# batch alone in a call of its own too
@pytest.mark.parametrize("F,d,B", [(34, 28, 513), (34, 60, 1025), (49, 64, 1025), (50, 32, 1025), (50, 64, 8191), (65, 132, 4095),
                                   (66, 4, 1025), (66, 36, 4097), (81, 64, 4097), (90, 28, 1025), (101, 32, 1025), (113, 20, 1025),
                                   (114, 68, 513), (128, 256, 600)])
def test_interaction_forward_gives_the_same_bits_at_any_batch_size(F, d, B):
    print("[case] interaction forward F=%d d=%d B=%d" % (F, d, B), flush=True)
    g = torch.Generator(device=DEV).manual_seed(F)
    T = torch.randn((B, F, d), generator=g, device=DEV)
    n = d + F * (F - 1) // 2
    R = torch.full((B, n), float("nan"), device=DEV)
    hot.dlrm_interact_dot_fwd(T, R)
    parts = torch.full((B, n), float("nan"), device=DEV)
    for b0 in list(range(0, B - 1, 512)) + [B - 1]:
        b1 = min(b0 + 512, B - 1) if b0 < B - 1 else B
        hot.dlrm_interact_dot_fwd(T[b0:b1].contiguous(), parts[b0:b1])
    assert torch.equal(R, parts)
    ref = oracle.interact_dot_fwd(T[-2:].cpu().numpy())
    scale = oracle.interact_dot_fwd(T[-2:].abs().cpu().numpy())
    assert np.max(np.abs(R[-2:].cpu().numpy() - ref) / np.maximum(scale, 1e-30)) <= d * 2.0 ** -24   # fp32 sums of d terms


# ... and from 102 rows on, where it takes them for every batch, with eight row blocks of rows of one stage and of more, and with three
# row blocks on either side of batches that it leaves out
@pytest.mark.parametrize("F,d,B", [(101, 20, 1025), (102, 20, 1025), (113, 4, 2049), (114, 4, 1025), (128, 64, 513), (121, 68, 513),
                                   (47, 80, 2432), (47, 80, 2433), (47, 92, 4096), (47, 92, 4097), (49, 140, 3072), (49, 140, 3456),
                                   (36, 80, 7168), (36, 80, 7169), (34, 144, 4096), (34, 144, 4481)])
def test_interaction_forward_gives_the_same_bits_on_its_other_lines_too(F, d, B):
    test_interaction_forward_gives_the_same_bits_at_any_batch_size(F, d, B)


def test_interaction_forward_beyond_one_launch():
    """2^23 samples and more of 34 rows, a workgroup each: as many as one launch is given.  The samples repeat, so the results must
    too."""
    print("[case] interaction forward F=34 B=2^23+64", flush=True)
    F, d, n = 34, 64, 64
    m, B = d + F * (F - 1) // 2, (1 << 23) + n
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < B * (F * d + m) * 4 + (8 << 30):
        pytest.skip("needs 102 GB of device memory")
    g = torch.Generator(device=DEV).manual_seed(F)
    T, R, want = torch.empty((B, F, d), device=DEV), torch.full((B, m), -5.0, device=DEV), torch.empty((n, m), device=DEV)
    T.view(-1, n, F, d).copy_(torch.randn((n, F, d), generator=g, device=DEV).expand(B // n, n, F, d))
    hot.dlrm_interact_dot_fwd(T[:n], want)
    hot.dlrm_interact_dot_fwd(T, R)
    for part in R.view(-1, n, m).split(1 << 14):
        assert (part == want).all()
    del T, R, part
    torch.cuda.empty_cache()


# two to five row blocks on either side of the batch size up to which wavefronts share a sample; rows of dR at
# every alignment (d + P odd) and at one
@pytest.mark.parametrize("F,d,below", [(18, 20, 1024), (33, 128, 1024), (34, 36, 1024), (50, 72, 1024), (65, 16, 1024),
                                       (65, 68, 1024), (66, 4, 4096), (70, 64, 4096), (81, 68, 12288)])
def test_interaction_backward_gives_the_same_bits_at_any_batch_size(F, d, below):
    print("[case] interaction backward F=%d d=%d" % (F, d), flush=True)
    g = torch.Generator(device=DEV).manual_seed(F)
    B, P = below + 1, F * (F - 1) // 2
    T = torch.randn((B, F, d), generator=g, device=DEV)
    dR = torch.randn((B, d + P), generator=g, device=DEV)
    whole, parts = torch.full_like(T, -5.0), torch.full_like(T, -5.0)
    hot.dlrm_interact_dot_bwd(T, dR, whole)
    for b0, b1 in ((0, below), (below, B)):
        hot.dlrm_interact_dot_bwd(T[b0:b1], dR[b0:b1], parts[b0:b1])
    assert torch.equal(whole, parts)
    Z = torch.zeros((3, F, F), dtype=torch.float64)
    i, j = torch.tril_indices(F, F, -1)
    Z[:, i, j] = dR[:3, d:].double().cpu()
    want = (Z + Z.transpose(1, 2)) @ T[:3].double().cpu()
    want[:, 0] += dR[:3, :d].double().cpu()
    scale = (Z.abs() + Z.abs().transpose(1, 2)) @ T[:3].double().cpu().abs() + 1.0
    # F + 1 terms, each rounded a few times in fp32: far below 1e-5 of the sum of magnitudes
    assert ((whole[:3].double().cpu() - want).abs() / scale).max() <= 1e-5


# one, two and four columns a lane, every storage type, one to four row blocks; bags of no row, one and more
@pytest.mark.parametrize("dtype", [gen.F32, gen.F16, gen.BF16])
@pytest.mark.parametrize("K,d", [(7, 8), (16, 16), (17, 24), (26, 32), (26, 40), (40, 16), (64, 8), (64, 24)])
def test_backward_without_T_of_narrow_rows(K, d, dtype):
    print("[case] backward without T K=%d d=%d dtype=%s" % (K, d, dtype), flush=True)
    b = gen.make_batch(gen.custom_workload("narrow", K=K, B=77, d=d, dtype=dtype, rows=50, bag=("uniform", 0, 3), dist=("uniform",), seed=K))
    g = torch.Generator(device=DEV).manual_seed(d)
    tables = [(torch.randn((50, d), generator=g, device=DEV)).to({gen.F32: torch.float32, gen.F16: torch.float16}.get(dtype, torch.bfloat16))
              for _ in range(K)]
    sb = hot.SparseBatch(tables, dtype, torch.from_numpy(b.indices).to(DEV), torch.from_numpy(b.offsets).to(DEV),
                         torch.from_numpy(b.tbl_off).to(DEV), b.nnz)
    F, n = K + 1, d + (K + 1) * K // 2
    x, dR = torch.randn((77, d), generator=g, device=DEV), torch.randn((77, n), generator=g, device=DEV)
    T, R = torch.full((77, F, d), -5.0, device=DEV), torch.empty((77, n), device=DEV)
    hot.dlrm_emb_interact_fwd(sb, x, T, R, algo=hot.FWD_FUSED)
    want, got = torch.full_like(T, -5.0), torch.full_like(T, -7.0)
    hot.dlrm_interact_dot_bwd(T, dR, want)
    hot.dlrm_emb_interact_bwd(sb, x, dR, got)
    assert torch.equal(got, want)


def test_interaction_backward_beyond_one_launch():
    """2^24 samples of 82 rows, a workgroup of 256 threads each: more threads than one launch holds.  The samples repeat,
    so the gradients must too."""
    print("[case] interaction backward F=82 B=2^24+64", flush=True)
    F, d, n = 82, 4, 64
    P, B = F * (F - 1) // 2, (1 << 24) + n
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < B * (2 * F * d + d + P) * 4 + (8 << 30):
        pytest.skip("needs 275 GB of device memory")
    g = torch.Generator(device=DEV).manual_seed(F)
    T, dR = torch.empty((B, F, d), device=DEV), torch.empty((B, d + P), device=DEV)
    dT = torch.full((B, F, d), -5.0, device=DEV)
    T.view(-1, n, F, d).copy_(torch.randn((n, F, d), generator=g, device=DEV).expand(B // n, n, F, d))
    dR.view(-1, n, d + P).copy_(torch.randn((n, d + P), generator=g, device=DEV).expand(B // n, n, d + P))
    want = torch.empty((n, F, d), device=DEV)
    hot.dlrm_interact_dot_bwd(T[:n], dR[:n], want)
    hot.dlrm_interact_dot_bwd(T, dR, dT)
    for part in dT.view(-1, n, F, d).split(1 << 14):
        assert (part == want).all()
    del T, dR, dT, part
    torch.cuda.empty_cache()


# buckets of n lookups on either side of a wavefront, two and the workgroup (one item of the ranking a lane, then two), from one
# row to rows of 24 and 25 unsorted bits; repeated rows, their bags in order
@pytest.mark.parametrize("m,sizes", [(2, (1, 64, 257)), (600, (1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257)),
                                     (1 << 25, (65, 256, 257)), (1 << 26, (65, 256, 257))])
def test_small_buckets_on_either_side_of_a_wavefront_and_of_the_workgroup(m, sizes):
    print("[case] small buckets m=%d" % m, flush=True)
    rng = np.random.default_rng(m)
    B = 40
    bags = []
    for n in sizes:
        rows = rng.integers(0, (m + 1) // 2, size=max(n // 3, 1))   # one bucket: at most two of them (one digit bit)
        ids = rng.choice(rows, size=n)
        bags.append([x.tolist() for x in np.split(ids, np.sort(rng.integers(0, n + 1, size=B - 1)))])
    b = gen.batch_from_lists([m] * len(sizes), bags, d=4, seed=3)
    for weighted in (False, True):
        _assert_exact_update(b, gen.F32, weighted, ("sort", "prepared"))


# rows split off an oversized bucket: more of them than fit LDS together, the most there can be, one of the largest size that is
# not queued beside small ones; with and without other rows
@pytest.mark.parametrize("weighted", [False, True], ids=["sum", "pow2-weights"])
@pytest.mark.parametrize("dtype,d", [(gen.F32, 24), (gen.F16, 128), (gen.BF16, 8)])
@pytest.mark.parametrize("runs,others", [([400] * 9, 1500), ([160] * 15, 0), ([2048, 300, 2047, 290], 70)])
def test_rows_split_off_oversized_buckets_fill_lds_piecewise(runs, others, dtype, d, weighted):
    print("[case] split rows %s others=%d dtype=%s d=%d weighted=%s" % (runs, others, dtype, d, weighted), flush=True)
    rng = np.random.default_rng(others)
    B, m, K = 500, 4000, 8
    parts = [np.full(n, 700 + i) for i, n in enumerate(runs)] + [rng.integers(640, 768, size=others), rng.integers(0, 600, size=2000)]
    ids = rng.permutation(np.concatenate(parts))
    long = [x.tolist() for x in np.split(ids, np.sort(rng.integers(0, len(ids) + 1, size=B - 1)))]
    short = [[[int(i) for i in rng.integers(0, m, size=n)] for n in rng.integers(0, 3, size=B)] for _ in range(K - 1)]
    b = gen.batch_from_lists([m] * K, short[:3] + [long] + short[3:], d=d, dtype=dtype, seed=6)
    assert _assert_exact_update(b, dtype, weighted, ("sort", "prepared"))["dominant_row_splits"] >= 1


# the partition digit by the lanes of a row (4 and less, 8, 16, 32, 64) at the smallest batches it depends on: tables x lookups a
# table, tables of fewer rows than digits among larger ones and one such table alone
@pytest.mark.parametrize("K,per", [(8, 8194), (13, 5043), (16, 7200), (1, 120000)])
@pytest.mark.parametrize("d", [4, 16, 28, 64, 100, 132])
def test_partition_digits_by_row_width(K, per, d):
    print("[case] digits by width K=%d per=%d d=%d" % (K, per, d), flush=True)
    rng = np.random.default_rng([K, d])
    B = 900
    rows = [20000 if k % 3 else 37 for k in range(K)]
    cuts = np.sort(rng.integers(0, per + 1, size=(K, B - 1)), axis=1)
    b = _batch([np.diff(c, prepend=0, append=per).tolist() for c in cuts], rows, seed=d, d=d)
    for weighted in (False, True):
        _assert_exact_update(b, gen.F32, weighted, ("sort", "prepared"))


# the lines of that rule: tables, lookups a table, rows, columns, bits.  Both sides of a step of every class, few rows; 1024 digits
# by narrow and by wide rows, with and without the column scan (more than 512 tiles); tables of fewer rows than digits among larger
# ones, and alone
@pytest.mark.parametrize("K,per,m,d,bits", [
    (40, 3584, 20000, 4, 4), (40, 3585, 20000, 16, 5), (40, 3072, 20000, 28, 4), (40, 3073, 20000, 28, 5), (24, 4097, 20000, 28, 6), (12, 7168, 20000, 16, 5),
    (12, 8193, 20000, 16, 7), (97, 3840, 20000, 28, 5), (97, 3839, 20000, 28, 4), (1, 114688, 20000, 4, 9),
    (13, 5043, 20000, 64, 6), (13, 5119, 20000, 100, 6), (13, 7168, 20000, 100, 7), (8, 8194, 20000, 132, 7), (13, 7168, 7168, 100, 7),
    (13, 7168, 7167, 100, 6), (8, 8194, 20000, 100, 7), (8, 8194, 37, 100, 6), (1, 120000, 20000, 4, 10), (1, 120000, 20000, 100, 10),
    (1, 120000, 37, 28, 6), (4, 114688, 30000, 132, 10), (4, 114687, 30000, 132, 9), (2, 57344, 60000, 132, 10), (2, 57343, 60000, 132, 9), (4, 164000, 30000, 132, 10)])
def test_partition_digits_on_either_side_of_a_line(K, per, m, d, bits):
    print("[case] digits at a line K=%d per=%d m=%d d=%d" % (K, per, m, d), flush=True)
    assert partition_bits(K * per, K, d, m) == bits
    rng = np.random.default_rng([K, d])
    B = 900
    rows = [37 if k % 3 == 1 else m for k in range(K)]
    cuts = np.sort(rng.integers(0, per + 1, size=(K, B - 1)), axis=1)
    b = _batch([np.diff(c, prepend=0, append=per).tolist() for c in cuts], rows, seed=d, d=d)
    for weighted in (False, True):
        _assert_exact_update(b, gen.F32, weighted, ("sort", "prepared"))


@pytest.mark.parametrize("dtype,d", [(gen.F32, 4), (gen.F32, 256), (gen.F16, 512)])
def test_one_launch_forward_without_lookups(dtype, d):
    """No index to read: every pooled vector is zero, the dense part of the result a copy (rows up to the widest)."""
    print("[case] forward without lookups dtype=%s d=%d" % (dtype, d), flush=True)
    K, B = 20, 70
    t = torch.ones((5, d), dtype=torch.float32 if dtype == gen.F32 else torch.float16, device=DEV)
    sb = hot.SparseBatch([t] * K, dtype, torch.empty(0, dtype=torch.int64, device=DEV),
                         torch.zeros((K, B + 1), dtype=torch.int64, device=DEV), torch.zeros(K + 1, dtype=torch.int64, device=DEV), 0)
    x = torch.randn((B, d), device=DEV)
    T, R = torch.full((B, K + 1, d), 7.0, device=DEV), torch.full((B, d + K * (K + 1) // 2), 7.0, device=DEV)
    hot.dlrm_emb_interact_fwd(sb, x, T, R, algo=hot.FWD_FUSED)
    assert torch.equal(R[:, :d], x) and not R[:, d:].any() and torch.equal(T[:, 0], x) and not T[:, 1:].any()

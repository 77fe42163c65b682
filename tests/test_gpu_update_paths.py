"""The ways a batch is grouped and its rows reduced, at the sizes where each can go wrong.  Integer work
(the grouping) must equal the oracle's; updates run on exact inputs (small integers, powers of two), so the
touched rows must be equal too, whatever the order of the sums."""
import numpy as np
import pytest
import torch

import paper_1906_00091_amd as hot
from oracle import oracle
from workloads import gen

from hotpath_util import DEV

pytestmark = pytest.mark.gpu


def _batch(lengths, rows, seed, d=4):
    """A batch of the given bag lengths [K][B], uniform row ids."""
    rng = np.random.default_rng([9, seed])
    bags = [[rng.integers(0, rows[k], size=n).tolist() for n in lengths[k]] for k in range(len(lengths))]
    return gen.batch_from_lists(rows, bags, d=d, seed=seed)


# name, tables, lookups of every table (in bags of about `bag`), rows: partition digits 1, 2, 4 and more; no tile, one
# tile and more tiles than a round of the column scan takes; more tables than lookups
GROUPINGS = [
    ("tables-without-lookups-between", [0, 1, 0, 1023, 1024, 1025, 0], 7, 3000),
    ("more-tables-than-lookups", [1 if k % 7 == 0 else 0 for k in range(600)], 1, 50),
    ("many-tables-few-digits", [(k * 37) % 300 for k in range(700)], 5, 4),
    ("column-scan-255-256-257-tiles", [255 * 1024, 256 * 1024, 256 * 1024 + 1], 64, 1 << 20),
    ("column-scan-ragged-tables", [700 * 1024 - 3, 5, 0, 1024], 33, 70000),
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

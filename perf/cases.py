"""Performance cases of the DLRM sparse hot path: what its users have it do, through its public calls.

Three kinds of program are covered ("mode"):
  train : one training step of the sparse side -- forward (dlrm_emb_interact_fwd), interaction backward, and the
          embedding backward fused with the row update.  Short bags with a T of 16 MiB or more take the pair that
          never writes T, as bench.py does.
  pool  : a model that uses the pooled lookup alone (it concatenates, or has an interaction of its own): the lookup
          and the backward with the row update from a given upstream gradient.  This pair is the headline metric.
  serve : scoring, forward only.
Sizes are those of workloads/gen.py (the five workloads), of the tests' shapes and generic ones between them.

Tables of one case lie in one allocation, and buffers and the backward's workspace are kept from step to step, as a
training loop keeps them.  Tables (and Adagrad state) are updated in place by every pass."""
import math

import numpy as np
import torch

import paper_1906_00091_amd as hot
from workloads import gen

DEV = "cuda:0"
DTYPES = {"f32": (hot.F32, torch.float32, 4), "f16": (hot.F16, torch.float16, 2), "bf16": (hot.BF16, torch.bfloat16, 2)}
FUSED_BAG = 4                   # dlrm_emb_interact_fwd(DLRM_FWD_AUTO) can do without T up to this mean bag, K <= 64, no weights
NO_T_FROM_BYTES = 16 << 20      # a training step leaves T out from this size of T on (bench.py)
HEAD = 4096                     # ranks of a Zipf law with exact probabilities (the tail: its integral)


def _case(name, mode, K, B, d, dtype, rows, bag, alpha=0.0, weighted=False, index32=False, optimizer="sgd", lengths=False):
    """rows: one size, or (lo, hi, cap on the sum) for log-uniform sizes; bag: one length, or (lo, hi) for uniform ones;
    alpha: 0 = uniform indices, else Zipf; lengths: the batch arrives as bag lengths and run() makes the offsets."""
    lo, hi, cap = rows if isinstance(rows, tuple) else (rows, rows, 0)
    b0, b1 = bag if isinstance(bag, tuple) else (bag, bag)
    c = {"name": name, "mode": mode, "K": K, "B": B, "d": d, "dtype": dtype, "rows_lo": lo, "rows_hi": hi, "rows_cap": cap,
         "bag_lo": b0, "bag_hi": b1, "alpha": alpha, "weighted": weighted, "index32": index32, "optimizer": optimizer,
         "lengths": lengths}
    if not name:
        del c["name"]
    return c


def listed():
    return [
        # one request batch of a click-through model being scored: latency of a handful of microseconds
        _case("serve_clicklog_b64", "serve", 26, 64, 16, "f32", (3, 10_000_000, 0), 1, alpha=1.05),
        # scoring of few-hot requests that arrive as lengths, weighted, on 16-bit tables
        _case("serve_weighted_bf16", "serve", 26, 500, 64, "bf16", 1_000_000, (1, 40), alpha=1.05, weighted=True,
              index32=True, lengths=True),
        # the smallest training step (workload 1)
        _case("train_tiny", "train", 8, 128, 16, "f32", 1000, (1, 4)),
        # a click log's one-hot features (workload 2)
        _case("train_clicklog", "train", 26, 2048, 16, "f32", (3, 10_000_000, 0), 1, alpha=1.05),
        # multi-hot pooling and its update (workload 3)
        _case("pool_multihot", "pool", 8, 2048, 64, "f32", 1_000_000, (1, 200)),
        # the profiled model of the paper (8 x 1M x 64, batch 2048, 1..100 lookups, int32), weighted, Adagrad
        _case("train_multihot_adagrad", "train", 8, 2048, 64, "f32", 1_000_000, (1, 100), weighted=True, index32=True,
              optimizer="adagrad"),
        # one-hot features over tens of millions of rows (workload 4)
        _case("train_large_onehot", "train", 26, 8192, 128, "f32", (1000, 40_000_000, 180_000_000), 1, alpha=1.05),
        # many lookups of few rows, 64 fp16 tables (workload 5): the largest
        _case("train_hotrow_f16", "train", 64, 16384, 128, "f16", 2_000_000, 32, alpha=1.2),
        # an ordinary few-hot model on bf16 tables of very different sizes, empty bags among the others
        _case("train_fewhot_bf16", "train", 26, 4096, 64, "bf16", (100, 10_000_000, 0), (0, 20), alpha=1.05, index32=True),
        # odd sizes everywhere, ragged bags with empty ones, lengths in, Adagrad
        _case("pool_ragged_odd", "pool", 13, 1999, 36, "f32", 50_021, (0, 37), optimizer="adagrad", lengths=True),
        # the widest rows the backward takes
        _case("pool_wide", "pool", 4, 8192, 256, "f32", 2_000_000, 20),
        # more tables than the one-launch forward takes, small fp16 tables, short bags
        _case("train_many_tables_f16", "train", 100, 1024, 32, "f16", (3, 100_000, 0), (1, 7), alpha=1.1, optimizer="adagrad"),
    ]


def draw(rng):
    """Another case of the same ranges: any mode, table count, batch, width, storage type, table size, bag mix,
    skew, weights, index type and optimizer, with the lookups, gradients and tables of the largest listed case
    as the limit."""
    logu = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))
    while True:
        mode = rng.choice(["train", "train", "pool", "pool", "serve"])
        dtype = rng.choice(["f32", "f32", "f16", "bf16"])
        d = 4 * logu(1, 64) if dtype == "f32" else 8 * logu(1, 32)
        K, B = logu(1, 100), logu(16, 16384)
        hi = logu(1, 200)
        bag = hi if rng.random() < 0.4 else (rng.choice([0, 1]), hi)
        lo_r = logu(3, 2_000_000)
        rows = lo_r if rng.random() < 0.4 else (lo_r, logu(lo_r, 40_000_000), 180_000_000)
        alpha = rng.choice([0.0, round(rng.uniform(1.05, 1.2), 3)])
        c = _case("", mode, K, B, d, dtype, rows, bag, alpha=alpha, weighted=rng.random() < 0.3, index32=rng.random() < 0.5,
                  optimizer=rng.choice(["sgd", "sgd", "adagrad"]) if mode != "serve" else "sgd", lengths=rng.random() < 0.3)
        nnz, F, tables = K * B * _mean_bag(c), K + 1, int(_table_rows(c).sum()) * d
        if (nnz <= 8e6 and nnz * d <= 4e8 and B * F * d <= 1.4e8 and B * F * F / 2 <= 34e6
                and tables * (DTYPES[dtype][2] + (4 if c["optimizer"] == "adagrad" else 0)) <= 24e9):
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _mean_bag(c):
    return (c["bag_lo"] + c["bag_hi"]) / 2.0


def _without_t(c):
    fused = c["bag_hi"] <= FUSED_BAG and c["K"] <= 64 and not c["weighted"]
    return fused and (c["mode"] == "serve" or c["B"] * (c["K"] + 1) * c["d"] * 4 >= NO_T_FROM_BYTES)


def _table_rows(c):
    spec = ("fixed", c["rows_lo"]) if c["rows_lo"] == c["rows_hi"] else (
        "loguniform", c["rows_lo"], c["rows_hi"], c["rows_cap"] or None, c["rows_lo"])
    return gen.table_rows(gen.Workload("case", K=c["K"], B=c["B"], d=c["d"], dtype=gen.F32, rows=spec,
                                       bag=("fixed", 1), dist=("uniform",)))


def _zipf_head(m, alpha):
    """p(r) ~ r^-alpha over ranks 1..m: cumulative weights of the first ranks, and the weight of the rest."""
    n = min(m, HEAD)
    head = np.cumsum(np.arange(1, n + 1, dtype=np.float64) ** -alpha)
    tail = ((n + 0.5) ** (1 - alpha) - (m + 0.5) ** (1 - alpha)) / (alpha - 1) if m > n else 0.0
    return head, tail


def _draw_rows(g, rng, n, m, alpha):
    """n row ids of a table of m rows.  Zipf: by inverse CDF, popular ranks scattered over the table by an affine map."""
    if alpha == 0.0:
        return torch.randint(0, m, (n,), generator=g, device=DEV)
    head, tail = _zipf_head(m, alpha)
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * (head[-1] + tail)
    rank = torch.searchsorted(torch.from_numpy(head).to(DEV), u)
    if tail > 0.0:
        k = len(head) + 0.5
        x = (k ** (1 - alpha) - (u - head[-1]).clamp_min(0.0) * (alpha - 1)) ** (1.0 / (1 - alpha))
        rank = torch.where(u > head[-1], (x - 0.5).long(), rank)
    rank = rank.clamp(0, m - 1)
    a = int(rng.integers(1, m)) if m > 1 else 1
    while math.gcd(a, m) != 1:
        a += 1
    return (rank * a + int(rng.integers(0, m))) % m


def _step_size(c):
    """(size of the upstream gradient, learning rate).  train: the gradient of a mean loss, and a rate at which the
    linear map that a step with fixed gradients is on the tables stays close to 1, so that tables stay finite over
    thousands of passes.  pool: the gradient does not depend on the tables, which then move by a constant."""
    if c["mode"] == "pool":
        return c["B"] ** -0.5, 0.01
    gain = 2.0 * max(_mean_bag(c), 1.0) * math.sqrt(c["K"] + 1) / c["B"] * (math.sqrt(c["B"]) if c["alpha"] else 1.0)
    return 1.0 / c["B"], 1e-3 if c["optimizer"] == "adagrad" else 1e-3 / gain


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    g = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng([seed, 0])
    K, B, d, F = c["K"], c["B"], c["d"], c["K"] + 1
    code, tdt, eb = DTYPES[c["dtype"]]
    rows = [int(m) for m in _table_rows(c)]
    # the sparse batch: bag lengths -> offsets, then the row ids table by table
    lens = torch.randint(c["bag_lo"], c["bag_hi"] + 1, (K, B), generator=g, device=DEV, dtype=torch.int32)
    offsets = torch.zeros((K, B + 1), dtype=torch.int64, device=DEV)
    offsets[:, 1:] = torch.cumsum(lens, 1, dtype=torch.int64)
    per_table = [int(n) for n in offsets[:, B].cpu()]
    tbl_off = torch.tensor([0] + per_table, dtype=torch.int64).cumsum(0).to(DEV)
    nnz = sum(per_table)
    indices = torch.empty(nnz, dtype=torch.int32 if c["index32"] else torch.int64, device=DEV)
    at = 0
    for k in range(K):
        indices[at:at + per_table[k]] = _draw_rows(g, rng, per_table[k], rows[k], c["alpha"])
        at += per_table[k]
    weights = torch.rand(nnz, generator=g, device=DEV) + 0.5 if c["weighted"] else None
    # the model: tables U(-1/sqrt(m), 1/sqrt(m)), Adagrad state as after some training
    s.tables = torch.empty((sum(rows), d), dtype=tdt, device=DEV)
    views = list(torch.split(s.tables, rows))
    for k in range(K):
        hot.dlrm_table_init_hash(views[k], code, gen.table_key(seed, k), float(gen.table_scale(rows[k])))
    s.batch = hot.SparseBatch(views, code, indices, offsets, tbl_off, nnz, weights=weights)
    s.lens = lens if c["lengths"] else None
    s.mode, s.adagrad, s.d, s.F = c["mode"], c["optimizer"] == "adagrad", d, F
    grad, s.lr = _step_size(c)
    s.no_t = _without_t(c)
    if s.mode == "pool":
        s.S = torch.empty((B, K, d), dtype=torch.float32, device=DEV)
        s.dS = torch.randn((B, K, d), generator=g, device=DEV) * grad
    else:
        P = F * (F - 1) // 2
        s.x = torch.randn((B, d), generator=g, device=DEV)
        s.T = None if s.no_t else torch.empty((B, F, d), dtype=torch.float32, device=DEV)
        s.R = torch.empty((B, d + P), dtype=torch.float32, device=DEV)
    if s.mode == "train":
        s.dR = torch.randn((B, d + P), generator=g, device=DEV) * grad
        s.dT = torch.empty((B, F, d), dtype=torch.float32, device=DEV)
    if s.mode != "serve":
        s.ws = hot.alloc_workspace(s.batch)
        if s.adagrad:
            # squares of gradients of the size this model sees
            size = grad if s.mode == "pool" else grad * math.sqrt(F * max(_mean_bag(c), 1.0) / max(rows))
            s.h = (torch.rand((sum(rows), d), generator=g, device=DEV) + 0.5) * size ** 2
            s.h_ptrs = hot.state_pointers(list(torch.split(s.h, rows)))
    return s


def run(s):
    batch, d, F = s.batch, s.d, s.F
    if s.lens is not None:
        hot.dlrm_lengths_to_offsets(s.lens, batch.offsets, batch.tbl_off)
    if s.mode == "serve":
        hot.dlrm_emb_interact_fwd(batch, s.x, s.T, s.R)
        return {"R": s.R, "T": s.T}
    if s.mode == "pool":
        out = {"S": s.S, "tables": s.tables}
        stride, dS, off = (F - 1) * d, s.dS, 0
        hot.dlrm_emb_bag_fwd(batch, s.S, stride, d)
    else:
        out = {"R": s.R, "T": s.T, "dT": s.dT, "tables": s.tables}
        stride, dS, off = F * d, s.dT, d
        hot.dlrm_emb_interact_fwd(batch, s.x, s.T, s.R)
        if s.no_t:
            hot.dlrm_emb_interact_bwd(batch, s.x, s.dR, s.dT)
        else:
            hot.dlrm_interact_dot_bwd(s.T, s.dR, s.dT)
    if s.adagrad:
        out["h"] = s.h
        hot.dlrm_emb_bag_bwd_adagrad(batch, s.h_ptrs, dS, stride, d, s.lr, 1e-8, s.ws, dS_offset=off)
    else:
        hot.dlrm_emb_bag_bwd_sgd(batch, dS, stride, d, s.lr, s.ws, dS_offset=off)
    return out


# ---------------------------------------------------------------------------------------------- what it takes
def _distinct(m, n, alpha):
    """Expected distinct rows among n lookups of a table of m rows."""
    if alpha == 0.0:
        return m * -math.expm1(n * math.log1p(-1.0 / m)) if m > 1 else min(n, 1)
    head, tail = _zipf_head(m, alpha)
    total = head[-1] + tail
    seen = float(np.sum(-np.expm1(-n * np.diff(head, prepend=0.0) / total)))
    if tail > 0.0:
        edge = np.exp(np.linspace(math.log(len(head) + 0.5), math.log(m + 0.5), 400))
        mid = np.sqrt(edge[1:] * edge[:-1])
        seen += float(np.sum(np.diff(edge) * -np.expm1(-n * mid ** -alpha / total)))
    return seen


def work(case):
    """Bytes: every touched row, index, weight and offset, the dense vectors and the upstream gradient read once, every
    result written once; T counts where the call writes it.  Flops: pooling, interaction and update."""
    c = case
    K, B, d, F = c["K"], c["B"], c["d"], c["K"] + 1
    P = F * (F - 1) // 2
    eb = DTYPES[c["dtype"]][2]
    per_table = B * _mean_bag(c)
    nnz = K * per_table
    U = sum(_distinct(int(m), per_table, c["alpha"]) for m in _table_rows(c))
    update = c["mode"] != "serve"
    nbytes = U * d * eb + nnz * ((4 if c["index32"] else 8) + (4 if c["weighted"] else 0))
    nbytes += K * B * (4 + 8) if c["lengths"] else K * B * 8
    flops = nnz * d * (2 if c["weighted"] else 1)
    if update:
        nbytes += U * d * (eb + (8 if c["optimizer"] == "adagrad" else 0))
        flops += nnz * d * (2 if c["weighted"] else 1) + U * d * (6 if c["optimizer"] == "adagrad" else 2)
    if c["mode"] == "pool":
        nbytes += 2 * B * K * d * 4                                          # S written, dS read
    else:
        nbytes += B * d * 4 + B * (d + P) * 4 + (0 if _without_t(c) else B * F * d * 4)    # x read, R and T written
        flops += 2 * B * P * d
        if update:
            nbytes += B * (d + P) * 4 + B * F * d * 4                         # dR read, dT written
            flops += 4 * B * P * d
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    """About four times the largest error of the listed and 40 drawn cases against the same pass in 64-bit arithmetic
    (its table rows rounded once to the storage type).  fp32: 2-norm 1e-6 (Adagrad state; the rest 2e-7), single
    elements 7e-5 (an Adagrad step whose gradient nearly cancels; the rest 6e-6).  16-bit tables: a sum near a tie
    rounds the other way, one unit in the last place of single elements (fp16 1e-3, bf16 4e-3 of the value), 7e-6 in
    the 2-norm; tables of a few hundred elements have to allow for one such element."""
    ulp = {"f32": 0.0, "f16": 1e-3, "bf16": 8e-3}[case["dtype"]]
    if case["mode"] == "serve" or not ulp:
        return {"rel": 4e-6, "max": 3e-4}
    elements = float(_table_rows(case).sum()) * case["d"]
    return {"rel": max(3e-5, 2 * ulp / math.sqrt(elements)), "max": 2 * ulp}

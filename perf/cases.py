"""The work that a user of this library has it do, as cases to be measured.

Every case is one pass through the public calls of `paper_2211_05239_amd.recd.Context` on a session-structured batch
(the samples of a session lie side by side and mostly repeat the same lists):

  step       a training step: builder, pooled lookup, expand, planned backward with row-wise Adagrad
  forward    builder, pooled lookup (sum or mean) and expand, as two calls or in one pass; serving, evaluation
  kjt        the pooled lookup without deduplication
  seq        builder, unpooled lookup on the unique lists and jagged expand (sequence features)
  seq_bwd    gradients of the sequence path for a given IKJT, no optimizer
  weighted   a training step with one weight per id
  maxpool    a training step with max pooling
  grouped    grouped builder, lookup, element-wise sum over every group on the unique rows, one expand per group

Sizes: those of the repository's benchmark configurations, of its tests, and odd ones between them.
Inputs are drawn on the GPU from the seed alone.  `exact` is the same result in 64 bits from the batch itself.
"""
import math

import numpy as np
import torch

from paper_2211_05239_amd import recd

DEV = "cuda"
LR, EPS = 0.01, 1e-8
DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}


def _case(name, kind, F, B, S, len_law, len_max, len_a, id_law, id_a, rows, D, dtype, pool="sum", one_pass=False,
          redraw=0.0, group=1):
    return {"name": name, "kind": kind, "F": F, "B": B, "S": S, "len_law": len_law, "len_max": len_max,
            "len_a": len_a, "id_law": id_law, "id_a": id_a, "rows": rows, "D": D, "dtype": dtype, "pool": pool,
            "one_pass": one_pass, "redraw": redraw, "group": group}


def listed():
    return [
        # the smallest call: one request of a few dozen samples to be scored, where launches count
        _case("request_f16", "forward", 7, 37, 4, "uniform", 20, 0.0, "uniform", 0.0, 100_000, 32, "f16",
              one_pass=True),
        # a training step on a small batch (benchmark configuration 1 with the backward pass)
        _case("step_small", "step", 4, 512, 4, "uniform", 20, 0.0, "uniform", 0.0, 100_000, 64, "f32", one_pass=True),
        # an ordinary training step: skewed lengths and ids, a tenth of the samples redrawn (configuration 2)
        _case("step_mid", "step", 16, 4096, 8, "zipf", 100, 1.2, "zipf", 1.05, 1_000_000, 128, "f32", redraw=0.1),
        # the largest: the headline training step (configuration 5)
        _case("step_large", "step", 64, 16384, 16, "zipf", 256, 1.1, "zipf", 1.05, 1_000_000, 128, "f32"),
        # evaluation of a large batch on 16-bit tables (configuration 3)
        _case("forward_f16", "forward", 64, 16384, 16, "zipf", 256, 1.1, "zipf", 1.05, 1_000_000, 128, "f16",
              one_pass=True),
        # odd sizes throughout: features not a multiple of 8, rows of twelve 16-byte pieces, average pooling
        _case("forward_ragged", "forward", 26, 5003, 6, "zipf", 100, 1.2, "zipf", 1.05, 300_007, 96, "bf16",
              pool="mean"),
        # the comparison path: a batch that is not deduplicated (configuration 4)
        _case("kjt_f32", "kjt", 32, 8192, 8, "uniform", 128, 0.0, "uniform", 0.0, 1_000_000, 128, "f32"),
        # sequence features, forward, on 16-bit tables
        _case("sequence_bf16", "seq", 16, 4096, 8, "zipf", 100, 1.2, "zipf", 1.05, 1_000_000, 128, "bf16"),
        # sequence features, gradients only: the caller has an optimizer of its own
        _case("sequence_grad", "seq_bwd", 12, 2500, 8, "uniform", 64, 0.0, "zipf", 1.05, 500_000, 64, "f32"),
        # per-id weights, training
        _case("weighted_step", "weighted", 16, 4096, 8, "zipf", 100, 1.2, "zipf", 1.05, 500_000, 128, "f32"),
        # max pooling, training
        _case("max_step", "maxpool", 24, 3000, 6, "uniform", 50, 0.0, "zipf", 1.05, 300_000, 128, "f32"),
        # feature groups that share one inverse index, with a module run on the unique rows
        _case("grouped_forward", "grouped", 32, 8192, 8, "zipf", 100, 1.2, "zipf", 1.05, 500_000, 64, "f32", group=4),
    ]


def draw(rng):
    """One more case of the same ranges; at most about half the ids and rows of the largest listed case."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "forward", "forward", "kjt", "seq", "seq_bwd", "weighted", "maxpool", "grouped"])
    F = rng.choice([1, 3, 8, log(2, 64), log(2, 64), log(2, 96)])
    B = log(16, 16384)
    S = rng.choice([1, 2, 4, 8, 16, 32])
    D = rng.choice([16, 32, 64, 64, 96, 128, 128, 128, 192, 256])
    len_law = rng.choice(["uniform", "zipf"])
    len_max = log(8, 128 if len_law == "uniform" else 256)
    dtype = "f32"
    if kind in ("forward", "kjt", "seq", "grouped"):
        dtype = rng.choice(["f32", "f16", "bf16"])
    mean = len_max / 2 if len_law == "uniform" else 0.35 * len_max
    # below step_large in output elements, in ids, in ids of unique lists, and in rows written per id
    most = [5e7 / (F * D), 1.2e7 / (F * mean), 2e6 * S / (F * mean)]
    if kind in ("kjt", "seq", "seq_bwd"):
        most.append(5e8 / (F * mean * D))
    if kind == "maxpool":
        most.append(1e8 * S / (F * mean * D))
    B = max(16, min([B] + [int(x) for x in most]))
    rows = min(log(1000, 1_000_000), max(1000, int(6e9 / (F * D * 4))))
    return {"kind": kind, "F": F, "B": B, "S": S, "len_law": len_law,
            "len_max": len_max, "len_a": rng.choice([1.1, 1.2]) if len_law == "zipf" else 0.0,
            "id_law": (id_law := rng.choice(["uniform", "zipf"])), "id_a": 1.05 if id_law == "zipf" else 0.0,
            "rows": rows, "D": D, "dtype": dtype,
            "pool": rng.choice(["sum", "sum", "mean"]) if kind in ("forward", "kjt") else "sum",
            "one_pass": F * B <= 16384 or dtype != "f32", "redraw": rng.choice([0.0, 0.0, 0.1]),
            "group": rng.choice([2, 4, 5]) if kind == "grouped" else 1}


# ---- inputs --------------------------------------------------------------------------------------------------

def _zipf_pdf(n, a):
    p = np.arange(1, n + 1, dtype=np.float64) ** (-a)
    return p / p.sum()


def _ranks(gen, shape, n, a):
    """Ranks 1..n with P(k) proportional to k**-a."""
    k = torch.arange(1, n + 1, dtype=torch.float64, device=DEV)
    cdf = torch.cumsum(k.pow_(-a), 0)
    u = torch.rand(shape, dtype=torch.float64, device=DEV, generator=gen) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=n - 1) + 1


def _batch(c, seed):
    """A KJT batch (values, offsets) on the GPU."""
    rng = np.random.default_rng(1_000_003 * seed + 17)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1_000_003 * seed + 29)
    F, B, S = c["F"], c["B"], c["S"]
    sizes = np.ones(B, dtype=np.int64) if S <= 1 else rng.geometric(1.0 / S, size=B)
    starts = np.concatenate([[0], np.cumsum(sizes)])
    first_of = np.repeat(starts[:-1], sizes)[:B]
    src = first_of.copy()
    if c["redraw"] > 0:
        changed = (rng.random(B) < c["redraw"]) & (np.arange(B) != first_of)
        src[changed] = np.arange(B)[changed]
    uniq, which = np.unique(src, return_inverse=True)  # the draws, and the draw that each sample carries
    K = len(uniq)
    which = torch.from_numpy(which.astype(np.int64)).to(DEV)
    if c["len_law"] == "uniform":
        dl = torch.randint(0, c["len_max"] + 1, (F, K), device=DEV, generator=gen)
    else:
        dl = _ranks(gen, (F, K), c["len_max"], c["len_a"])
    flat = dl.reshape(-1)
    doff = torch.cumsum(flat, 0) - flat
    drawn = int(flat.sum())  # a bound of the unique ids
    if c["id_law"] == "uniform":
        ids = torch.randint(0, c["rows"], (drawn,), device=DEV, generator=gen)
    else:
        ids = _ranks(gen, (drawn,), c["rows"], c["id_a"]) - 1
    sl = dl[:, which].reshape(-1)
    offsets = torch.zeros(F * B + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(sl, 0, out=offsets[1:])
    begin = doff.reshape(F, K)[:, which].reshape(-1)
    N = int(offsets[-1])
    pos = torch.repeat_interleave(begin - offsets[:-1], sl, output_size=N) + torch.arange(N, device=DEV)
    n_cap, m_cap = _capacity(c)
    assert N <= n_cap and drawn <= m_cap, (N, n_cap, drawn, m_cap)
    return ids[pos].contiguous(), offsets


def _capacity(c):
    """(ids of a batch, ids of its unique lists) that buffers are allocated for, whatever the seed: the expected
    number and eight standard deviations (lists of a session have one length, sessions have geometric sizes)."""
    F, B, S = c["F"], c["B"], c["S"]
    n = c["len_max"]
    mean = _mean_length(c)
    if c["len_law"] == "uniform":
        square = n * (2 * n + 1) / 6
    else:
        square = float((np.arange(1, n + 1, dtype=np.float64) ** 2 * _zipf_pdf(n, c["len_a"])).sum())
    lists = F * (B / S * (1 + c["redraw"] * (S - 1)) + 8 * math.sqrt(B) + 8)
    n_cap = F * B * mean + 8 * math.sqrt(F * B * 2 * S * square) + 8 * n
    m_cap = lists * mean + 8 * math.sqrt(lists * square) + 8 * n
    n_cap = int(min(n_cap, F * B * n))
    return n_cap, int(min(m_cap, n_cap))


def _normal(seed, tag, shape, dtype=torch.float32):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1_000_003 * seed + tag)
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, 0.01, generator=gen)


def _tables(c, seed):
    return _normal(seed, 41, (c["F"], c["rows"], c["D"]), DTYPE[c["dtype"]])


def _weights(values, offsets):
    """One of eight levels by id and position, so that equal lists carry equal weights."""
    lens = offsets[1:] - offsets[:-1]
    at = torch.arange(values.numel(), device=DEV) - torch.repeat_interleave(offsets[:-1], lens,
                                                                             output_size=values.numel())
    return (((values * 2654435761 + at * 40503) % 8) + 1).to(torch.float32) * 0.25


def _group_off(c):
    return list(range(0, c["F"], c["group"])) + [c["F"]]


def _zeros(*shape, dtype=torch.int64):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def prepare(case, seed):
    c = case
    F, B, D, kind = c["F"], c["B"], c["D"], c["kind"]
    dt = DTYPE[c["dtype"]]
    values, offsets = _batch(c, seed)
    N = values.numel()
    n_cap, m_cap = _capacity(c)
    s = {"case": c, "values": values, "offsets": offsets, "rows": [c["rows"]] * F, "u_hint": F * B}
    if kind != "seq_bwd":
        s["tables"] = _tables(c, seed)
        s["table_list"] = list(s["tables"].unbind(0))
    s["ctx"] = ctx = recd.Context(0, workspace_hint_bytes=recd.workspace_bytes(F, B, m_cap, D))
    if kind == "kjt":
        s["out"] = _zeros(F, B, D, dtype=dt)
        return s
    s.update(u_values=_zeros(n_cap), u_offsets=_zeros(F * B + 1), inverse=_zeros(F * B, dtype=torch.int32),
             feat_uoff=_zeros(F + 1))
    if c["one_pass"]:
        s["run_index"] = _zeros(3 * (F * B + 2))
    if kind in ("step", "forward", "weighted", "maxpool", "grouped"):
        s["pooled"] = _zeros(F * B, D, dtype=dt)
        s["out"] = _zeros(len(_group_off(c)) - 1 if kind == "grouped" else F, B, D, dtype=dt)
    if kind in ("step", "weighted", "maxpool"):
        s["grad_out"] = _normal(seed, 53, (F, B, D))
        s["state"] = _zeros(F, c["rows"], dtype=torch.float32)
        s["state_list"] = list(s["state"].unbind(0))
    if kind in ("step", "weighted", "maxpool", "seq_bwd"):
        s["touched"], s["feat_roff"] = _zeros(m_cap), _zeros(F + 1)
    if kind == "weighted":
        s["weights"] = _weights(values, offsets)
        s["u_weights"] = _zeros(n_cap, dtype=torch.float32)
    if kind == "grouped":
        G = len(_group_off(c)) - 1
        s.update(group_off=_group_off(c), inverse_g=_zeros(G * B, dtype=torch.int32), group_uoff=_zeros(G + 1),
                 combined=_zeros(G * B, D, dtype=dt))
    if kind == "seq":
        s["emb"], s["out"] = _zeros(m_cap, D, dtype=dt), _zeros(n_cap, D, dtype=dt)
    if kind == "seq_bwd":
        # the IKJT and the upstream gradient are what the forward pass left
        s["U"], s["M"] = ctx.build_ikjt(F, B, values, offsets, s["u_values"], s["u_offsets"], s["inverse"],
                                        s["feat_uoff"], want_counts=True)
        s["grad_out"] = _normal(seed, 53, (N, D))
        s["grad_emb"] = _zeros(m_cap, D, dtype=torch.float32)
        s["grad_rows"] = _zeros(m_cap, D, dtype=torch.float32)
    return s


# ---- one pass ------------------------------------------------------------------------------------------------

def _build(s, c):
    ctx = s["ctx"]
    ikjt = (s["u_values"], s["u_offsets"], s["inverse"], s["feat_uoff"])
    if c["one_pass"]:
        ctx.build_ikjt_runs(c["F"], c["B"], s["values"], s["offsets"], *ikjt, s["run_index"])
    else:
        ctx.build_ikjt(c["F"], c["B"], s["values"], s["offsets"], *ikjt)


def _forward(s, c):
    ctx, U = s["ctx"], s["u_hint"]
    if c["one_pass"] and c["pool"] == "sum":
        ctx.pooled_lookup_expand(s["table_list"], c["B"], s["u_values"], s["run_index"],
                                 min(U + U // 16, c["F"] * c["B"]), s["pooled"], s["out"])
    else:
        ctx.pooled_lookup_unique(s["table_list"], s["u_values"], s["u_offsets"], s["feat_uoff"], U, s["pooled"],
                                 mode=None if c["pool"] == "sum" else c["pool"])
        ctx.expand_inverse(c["F"], c["B"], s["pooled"], s["feat_uoff"], s["inverse"], s["out"])


def run(state):
    s = state
    c, ctx = s["case"], s["ctx"]
    F, B, D, kind = c["F"], c["B"], c["D"], c["kind"]
    if kind == "kjt":
        ctx.kjt_pooled_lookup(s["table_list"], B, s["values"], s["offsets"], s["out"],
                              mode=None if c["pool"] == "sum" else c["pool"])
        return {"out": s["out"]}
    if kind == "forward":
        _build(s, c)
        _forward(s, c)
        return {"out": s["out"], "inverse": s["inverse"], "feat_uoff": s["feat_uoff"], "u_values": s["u_values"],
                "u_offsets": s["u_offsets"]}
    if kind == "step":
        # the lookup needs no count on the host: it is enqueued behind the build, and the counts that bound the
        # backward come back meanwhile
        _build(s, c)
        _forward(s, c)
        U, M = ctx.last_ikjt_counts()
        s["u_hint"] = max(U, 1)
        ctx.backward_plan(F, B, D, s["inverse"], s["feat_uoff"], s["u_values"], s["u_offsets"], s["rows"], U, M,
                          s["touched"], s["feat_roff"])
        ctx.backward_apply(s["grad_out"], None, tables=s["table_list"], adagrad_state=s["state_list"], lr=LR, eps=EPS)
        return {"out": s["out"], "tables": s["tables"], "state": s["state"], "touched": s["touched"],
                "feat_roff": s["feat_roff"]}
    if kind == "seq":
        _build(s, c)
        ctx.sequence_lookup_unique(s["table_list"], s["u_values"], s["u_offsets"], s["feat_uoff"], F * B, s["emb"])
        ctx.jagged_expand_inverse(F, B, s["emb"], s["u_offsets"], s["feat_uoff"], s["inverse"], s["offsets"],
                                  s["out"][:s["values"].numel()])
        return {"out": s["out"], "inverse": s["inverse"], "feat_uoff": s["feat_uoff"], "u_values": s["u_values"]}
    if kind == "seq_bwd":
        ctx.backward_sequence_dedup(F, B, s["grad_out"], s["offsets"], s["inverse"], s["feat_uoff"], s["u_values"],
                                    s["u_offsets"], s["rows"], s["U"], s["M"], s["grad_emb"], s["touched"],
                                    s["feat_roff"], s["grad_rows"])
        return {"grad_rows": s["grad_rows"], "grad_emb": s["grad_emb"], "touched": s["touched"],
                "feat_roff": s["feat_roff"]}
    if kind == "weighted":
        ctx.build_ikjt_weighted(F, B, s["values"], s["weights"], s["offsets"], s["u_values"], s["u_weights"],
                                s["u_offsets"], s["inverse"], s["feat_uoff"])
        ctx.pooled_lookup_unique_weighted(s["table_list"], s["u_values"], s["u_weights"], s["u_offsets"],
                                          s["feat_uoff"], s["u_hint"], s["pooled"])
        ctx.expand_inverse(F, B, s["pooled"], s["feat_uoff"], s["inverse"], s["out"])
        U, M = ctx.last_ikjt_counts()
        s["u_hint"] = max(U, 1)
        ctx.backward_dedup_weighted(F, B, s["grad_out"], s["inverse"], s["feat_uoff"], s["u_values"], s["u_weights"],
                                    s["u_offsets"], s["rows"], U, M, s["touched"], s["feat_roff"], None,
                                    tables=s["table_list"], adagrad_state=s["state_list"], lr=LR, eps=EPS)
        return {"out": s["out"], "tables": s["tables"], "state": s["state"], "touched": s["touched"],
                "feat_roff": s["feat_roff"]}
    if kind == "maxpool":
        _build(s, c)
        ctx.pooled_lookup_unique(s["table_list"], s["u_values"], s["u_offsets"], s["feat_uoff"], s["u_hint"],
                                 s["pooled"], mode="max")
        ctx.expand_inverse(F, B, s["pooled"], s["feat_uoff"], s["inverse"], s["out"])
        U, M = ctx.last_ikjt_counts()
        s["u_hint"] = max(U, 1)
        ctx.backward_dedup_max(F, B, s["grad_out"], s["inverse"], s["feat_uoff"], s["u_values"], s["u_offsets"],
                               s["rows"], U, M, s["table_list"], s["touched"], s["feat_roff"], None,
                               tables=s["table_list"], adagrad_state=s["state_list"], lr=LR, eps=EPS)
        return {"out": s["out"], "tables": s["tables"], "state": s["state"], "touched": s["touched"],
                "feat_roff": s["feat_roff"]}
    assert kind == "grouped", kind
    ctx.build_ikjt_grouped(F, B, s["group_off"], s["values"], s["offsets"], s["u_values"], s["u_offsets"],
                           s["inverse_g"], s["group_uoff"], s["feat_uoff"])
    ctx.pooled_lookup_unique(s["table_list"], s["u_values"], s["u_offsets"], s["feat_uoff"], F * B, s["pooled"])
    ctx.group_sum_unique(F, s["group_off"], s["pooled"], s["feat_uoff"], s["group_uoff"], s["combined"])
    ctx.expand_inverse(len(s["group_off"]) - 1, B, s["combined"], s["group_uoff"], s["inverse_g"], s["out"])
    return {"out": s["out"], "inverse_g": s["inverse_g"], "group_uoff": s["group_uoff"], "feat_uoff": s["feat_uoff"],
            "u_values": s["u_values"]}


# ---- what a pass cannot do without ---------------------------------------------------------------------------

def _mean_length(c):
    if c["len_law"] == "uniform":
        return c["len_max"] / 2
    return float((np.arange(1, c["len_max"] + 1) * _zipf_pdf(c["len_max"], c["len_a"])).sum())


def _sizes(c):
    """Expected ids N, unique lists U, their ids M and distinct (feature, row) pairs R (of all N ids: the same)."""
    F, B, S = c["F"], c["B"], c["S"]
    mean = _mean_length(c)
    sessions = max(1.0, B / S)
    K = min(B, sessions + c["redraw"] * (B - sessions))
    m_f = K * mean
    if c["id_law"] == "uniform":
        r_f = c["rows"] * -math.expm1(m_f * math.log1p(-1.0 / c["rows"]))
    else:
        p = _zipf_pdf(c["rows"], c["id_a"])
        r_f = float(-np.expm1(m_f * np.log1p(-p)).sum()) if c["rows"] > 1 else 1.0
    return F * B * mean, F * K, F * m_f, F * r_f


def work(case):
    c = case
    F, B, D, kind = c["F"], c["B"], c["D"], c["kind"]
    e = SIZE[c["dtype"]]
    N, U, M, R = _sizes(c)
    kjt = N * 8 + (F * B + 1) * 8                       # the batch, read once
    ikjt = M * 8 + U * 8 + F * B * 4                     # the deduplicated batch, written once
    table, out = R * D * e, F * B * D * e               # every distinct row read once, every output row written
    update = R * (2 * D * 4 + 2 * 4 + 8)                 # table row and accumulator read and written, row id
    grad = F * B * D * 4
    if kind == "kjt":
        return {"bytes": kjt + table + out, "flops": N * D}
    if kind == "forward":
        return {"bytes": kjt + ikjt + table + out, "flops": M * D}
    if kind == "step":
        return {"bytes": kjt + ikjt + out + grad + update, "flops": 2 * M * D + F * B * D + 5 * R * D}
    if kind == "weighted":
        return {"bytes": kjt + N * 4 + ikjt + M * 4 + out + grad + update,
                "flops": 4 * M * D + F * B * D + 5 * R * D}
    if kind == "maxpool":
        return {"bytes": kjt + ikjt + out + grad + update, "flops": 3 * M * D + F * B * D + 5 * R * D}
    if kind == "seq":
        return {"bytes": kjt + ikjt + table + N * D * e, "flops": 0}
    if kind == "seq_bwd":
        return {"bytes": ikjt + (F * B + 1) * 8 + N * D * 4 + M * D * 4 + R * (D * 4 + 8), "flops": (N + M) * D}
    G = len(_group_off(c)) - 1
    return {"bytes": kjt + M * 8 + U * 8 + G * B * 4 + table + G * B * D * e, "flops": (M + U) * D}


def tolerance(case):
    if case["kind"] == "seq":
        return "exact"                                   # copies
    # Against 64 bits the sums are off by 0.5e-7 to 1.4e-7 (f32), 2.8e-4 (f16) and 1.4e-3 (bf16, both one rounding of
    # the output): about four times that between two orders of the additions, and at single values an ulp or two.
    return {"f32": {"rel": 8e-7, "max": 2e-5}, "f16": {"rel": 1e-3, "max": 2e-3},
            "bf16": {"rel": 5e-3, "max": 1.6e-2}}[case["dtype"]]


# ---- the same in 64 bits -------------------------------------------------------------------------------------

def exact(case, seed):
    c = case
    F, B, D, kind, rows = c["F"], c["B"], c["D"], c["kind"], c["rows"]
    values, offsets = _batch(c, seed)
    n_cap, m_cap = _capacity(c)
    f64 = torch.float64
    none = dict.fromkeys(("inverse", "feat_uoff", "u_values", "u_offsets", "touched", "feat_roff", "inverse_g",
                          "group_uoff"))
    bounds = offsets[::B].tolist()

    def lists(f):
        """(ids, row within the feature of every id) of feature f."""
        lens = (offsets[1:] - offsets[:-1])[f * B:(f + 1) * B]
        return values[bounds[f]:bounds[f + 1]], torch.repeat_interleave(torch.arange(B, device=DEV), lens), lens

    if kind == "seq":
        tables = _tables(c, seed)
        out = _zeros(n_cap, D, dtype=f64)
        for f in range(F):
            out[bounds[f]:bounds[f + 1]] = tables[f][lists(f)[0]].to(f64)
        return {**none, "out": out}
    if kind == "seq_bwd":
        # positions of the deduplicated lists in order of first occurrence, from the batch alone
        g = _normal(seed, 53, (values.numel(), D))
        grad_rows, grad_emb = _zeros(m_cap, D, dtype=f64), _zeros(m_cap, D, dtype=f64)
        at_r = at_m = 0
        for f in range(F):
            ids, row, lens = lists(f)
            gf = g[bounds[f]:bounds[f + 1]].to(f64)
            u, back = torch.unique(ids, return_inverse=True)  # ascending, as the touched rows are
            grad_rows[at_r:at_r + u.numel()].index_add_(0, back, gf)
            at_r += u.numel()
            host, off, seen, slot_off = ids.cpu().numpy(), np.concatenate([[0], np.cumsum(lens.cpu().numpy())]), {}, []
            total = 0
            for b in range(B):
                key = host[off[b]:off[b + 1]].tobytes()
                if key not in seen:
                    seen[key] = total
                    total += int(off[b + 1] - off[b])
                slot_off.append(seen[key])
            start = torch.tensor(slot_off, device=DEV)
            pos = start[row] + torch.arange(ids.numel(), device=DEV) - torch.from_numpy(off[:-1]).to(DEV)[row]
            grad_emb[at_m:at_m + total].index_add_(0, pos, gf)
            at_m += total
        return {**none, "grad_rows": grad_rows, "grad_emb": grad_emb}
    tables = _tables(c, seed)
    train = kind in ("step", "weighted", "maxpool")
    grad_out = _normal(seed, 53, (F, B, D)) if train else None
    weights = _weights(values, offsets) if kind == "weighted" else None
    G = len(_group_off(c)) - 1
    out = _zeros(G if kind == "grouped" else F, B, D, dtype=f64)
    new = tables.to(f64) if train else None
    state = _zeros(F, rows, dtype=f64) if train else None
    for f in range(F):
        ids, row, lens = lists(f)
        o = out[f // c["group"]]
        grad = _zeros(rows, D, dtype=f64) if train else None
        step = max(1, int(2.5e8 / D))                    # at most 2 GB of gathered rows at a time
        if kind != "maxpool":
            for i in range(0, ids.numel(), step):
                part, to = ids[i:i + step], row[i:i + step]
                w = weights[bounds[f] + i:bounds[f] + i + part.numel()].to(f64)[:, None] if weights is not None else 1.0
                o.index_add_(0, to, tables[f][part].to(f64) * w)
                if train:
                    grad.index_add_(0, part, grad_out[f].to(f64)[to] * w)
            if c["pool"] == "mean":
                o /= lens.clamp(min=1).to(f64)[:, None]
        else:
            x = tables[f][ids].to(f64)
            to = row[:, None].expand(-1, D)
            best = torch.full((B, D), -math.inf, dtype=f64, device=DEV).scatter_reduce_(0, to, x, "amax")
            at = torch.arange(ids.numel(), device=DEV)[:, None].expand(-1, D)
            won = torch.where(x == best[row], at, ids.numel())
            first = torch.full((B, D), ids.numel(), device=DEV).scatter_reduce_(0, to, won, "amin")
            o.copy_(torch.where(lens[:, None] > 0, best, torch.zeros_like(best)))
            grad.index_add_(0, ids, torch.where(first[row] == at, grad_out[f].to(f64)[row], 0.0))
        if train:
            m = grad.square().mean(1)
            hit = torch.zeros(rows, dtype=torch.bool, device=DEV)
            hit[ids] = True
            state[f] = m
            new[f] -= torch.where(hit, LR / (m.sqrt() + EPS), 0.0)[:, None] * grad
    if train:
        return {**none, "out": out, "tables": new, "state": state}
    return {**none, "out": out}

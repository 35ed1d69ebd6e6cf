"""The work that a user of this package has it do, as cases that can be timed.

Kinds of case and the public entry points they go through:

* ``step``    one decode token through ``layers`` layers of Double-P attention, each layer with a clustered cache
              of its own (``BoundDecodeStep``: a serving loop's call; ``dp_decode_attention`` where ``plain`` is set)
* ``budget``  the same with a fixed budget of clusters instead of the two thresholds (``dp_budget_decode_attention``)
* ``dense``   full attention over every token of the cache (``dp_dense_decode``)
* ``fit``     prefill: k-means over the keys, strided start, a few rounds (``dp_kmeans_fit``)
* ``build``   prefill: the cluster-contiguous cache and its metadata from token-order K / V (``dp_build_cluster_cache``)

The shapes are those of this repository's workloads (``workloads/synth.py``, ``bench.py``): head_dim 128, bf16 K / V,
4k to 128k tokens, clusters of 16 or 32 tokens on average, batch 1 to 16, GQA groups of 1 to 8.  The inputs follow
the same recipe (keys = 2 z_c + 0.5 eps around their cluster's centre, queries = a Dirichlet mix of four centres of
their own segment times a scale + N(0, I)) drawn on the GPU; the scale of a query decides whether its head is peaked
(one or two clusters hold the mass) or flat (hundreds of clusters are retained).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2602_05191_amd as dp

DIM = 128
ROW = 2 * DIM                      # bytes of one bf16 row
MOST_ROWS = 4 * 8 * 131072         # rows of the largest listed cache
MOST_FIT = 8 * 131072 * 8192 * 3   # tokens x centroids x rounds of the largest listed clustering

STEP = dict(kind="step", batch=1, kv_heads=8, group=4, context=32768, ragged=False, mean=16, sizes="poisson",
            layers=1, heads="peaked", pinned=False, p1=0.95, p2=0.9, out="bf16", plain=False)
PREFILL = dict(batch=1, kv_heads=8, context=32768, ragged=False, mean=16, sizes="poisson")


def listed():
    return [
        # the smallest call: one short sequence, one KV head; what a step costs when there is next to nothing to read
        dict(STEP, name="step_4k", kv_heads=1, context=4096, out="f32"),
        # an ordinary decode token: 32 layers of the 8B shape at 32k context, outputs in the model's bf16
        dict(STEP, name="step_32k", layers=32),
        # long context, peaked heads of every sharpness: the repository's headline workload, 16 layers so that
        # successive layers come from HBM
        dict(STEP, name="step_128k", context=131072, layers=16, heads="spread", out="f32"),
        # the same shape in a layer whose heads spread their attention (hundreds of clusters retained per head)
        dict(STEP, name="step_128k_flat", context=131072, layers=2, heads="flat"),
        # continuous batching: 16 sequences of different lengths, 512 heads in one call
        dict(STEP, name="step_batch16", batch=16, context=65536, ragged=True, mean=32, p1=0.98, p2=0.95),
        # wide GQA, skewed cluster sizes, half of the heads flat, four long sequences: the largest step
        dict(STEP, name="step_gqa8_128k", batch=4, group=8, context=131072, sizes="pareto", heads="alternate"),
        # the deployed form of the method: sink and window tokens pinned, odd lengths, some heads flat
        dict(STEP, name="step_pinned", batch=3, context=37777, ragged=True, layers=4, heads="mixed", pinned=True,
             p2=0.7, plain=True),
        # the fixed-budget rule at long context
        dict(STEP, name="budget_128k", kind="budget", context=131072, heads="spread", keep=0.25, exact=0.018),
        # layers that stay dense, and the baseline of every comparison
        dict(STEP, name="dense_128k", kind="dense", context=131072),
        # prefill of one long sequence: the clustering, and the cache it leads to
        dict(PREFILL, name="fit_128k", kind="fit", context=131072, rounds=3),
        dict(PREFILL, name="build_128k", kind="build", context=131072, sums=False),
        # prefill of a few short sequences of odd lengths together
        dict(PREFILL, name="fit_short", kind="fit", batch=3, context=5003, ragged=True, rounds=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "budget", "dense", "fit", "build"])
    while True:
        case = dict(batch=rng.choice([1, 1, 1, 2, 3, 5, 8, 16]), kv_heads=rng.choice([1, 2, 4, 8, 8]),
                    context=_log_int(rng, 2048, 131072), ragged=rng.random() < 0.5, mean=rng.choice([16, 16, 32]),
                    sizes=rng.choice(["poisson", "poisson", "pareto"]))
        if case["batch"] == 1:
            case["ragged"] = False
        if kind in ("fit", "build"):
            case["kind"] = kind
            if kind == "fit":
                case["rounds"] = rng.randint(1, 5)
            else:
                case["sums"] = rng.random() < 0.3
        else:
            p1, p2 = rng.choice([(0.95, 0.9), (0.95, 0.7), (0.98, 0.95), (0.99, 0.8)])
            case = dict(STEP, **case)
            case.update(kind=kind, group=rng.choice([1, 2, 4, 4, 8]), layers=rng.choice([1, 1, 2, 4]),
                        heads=rng.choice(["peaked", "spread", "mixed", "flat", "alternate"]),
                        pinned=kind == "step" and rng.random() < 0.3, p1=p1, p2=p2,
                        out=rng.choice(["bf16", "f32"]), plain=rng.random() < 0.3)
            if kind == "budget":
                case.update(keep=round(rng.uniform(0.05, 0.3), 3), exact=round(rng.uniform(0.005, 0.03), 4))
            if kind == "dense":
                case["layers"] = 1
        rows = sum(_contexts(case)) * case["kv_heads"]
        if rows * case.get("layers", 1) > MOST_ROWS:
            continue
        # full attention and budgets read much of what is cached: half the rows
        if kind in ("dense", "budget") and rows * case["layers"] > MOST_ROWS // 2:
            continue
        if kind == "fit" and sum(n * k for n, k in zip(_contexts(case), _clusters(case))) * case["kv_heads"] * case["rounds"] > MOST_FIT:
            continue
        return case


def _contexts(case):
    """Tokens of each sequence: the context, or from a quarter of it upwards where the batch is ragged."""
    if not case["ragged"]:
        return [case["context"]] * case["batch"]
    return [max(1, int(case["context"] * (0.25 + 0.75 * ((b + 1) * 0.6180339887 % 1.0)))) for b in range(case["batch"])]


def _clusters(case):
    return [max(1, n // case["mean"]) for n in _contexts(case)]


def _scales(case, rng):
    """Query scale of each head of one KV group."""
    flat, peaked = 0.4, 3.0
    return {"peaked": lambda h: peaked, "flat": lambda h: flat, "spread": lambda h: rng.uniform(1.0, 5.0),
            "mixed": lambda h: flat if h % 8 == 0 else peaked, "alternate": lambda h: 5.0 if h % 2 else 0.5}[case["heads"]]


def _sizes(rng, n_clusters, total, mean, dist):
    """Cluster sizes that sum to ``total``: Poisson, or Pareto (a few clusters hold many tokens), at least one each."""
    if dist == "pareto":
        raw = np.clip(np.rint(mean / 3.0 * (1.0 + rng.pareto(1.5, n_clusters))), 1, 512)
    else:
        raw = np.clip(rng.poisson(mean, n_clusters), 1, 4 * mean)
    s = raw.astype(np.int64)
    diff = total - int(s.sum())
    while diff:
        movable = np.nonzero(s > 1)[0] if diff < 0 else np.arange(n_clusters)
        take = movable[: abs(diff)]
        s[take] += 1 if diff > 0 else -1
        diff += len(take) if diff < 0 else -len(take)
    return s


class _Draws:
    """The random streams of one state: everything is a function of the seed."""

    def __init__(self, seed):
        self.np = np.random.default_rng(np.random.SeedSequence([seed, 77]))
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.gen, device="cuda")


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()


def _layer(case, d):
    """One layer's clustered cache and queries on the GPU."""
    ctx, ncl = _contexts(case), _clusters(case)
    kvh, group, batch = case["kv_heads"], case["group"], case["batch"]
    rows, total = sum(ctx) * kvh, sum(ncl) * kvh
    kw = dict(device="cuda", dtype=torch.bfloat16)
    k, v = torch.empty(rows, DIM, **kw), torch.empty(rows, DIM, **kw)
    kc, vc = torch.empty(total, DIM, **kw), torch.empty(total, DIM, **kw)
    q = torch.empty(batch, kvh * group, DIM, **kw)
    sizes, offsets, base, ptr = [], [], [], [0]
    row = 0
    for b in range(batch):
        for g in range(kvh):
            n, m = ctx[b], ncl[b]
            s = _sizes(d.np, m, n, case["mean"], case["sizes"])
            sizes.append(s)
            offsets.append(np.concatenate([[0], np.cumsum(s)[:-1]]))
            base.append(row)
            c0 = ptr[-1]
            lengths = torch.from_numpy(s).cuda()
            centres = 2.0 * d.normal(m, DIM)
            k[row:row + n] = torch.repeat_interleave(centres, lengths, dim=0, output_size=n) + 0.5 * d.normal(n, DIM)
            v[row:row + n] = d.normal(n, DIM)
            for src, dst in ((k, kc), (v, vc)):
                dst[c0:c0 + m] = torch.segment_reduce(src[row:row + n].double(), "mean", lengths=lengths, axis=0, unsafe=True)
            scale = _scales(case, d.np)
            for j in range(group):
                h = g * group + j
                mix = d.np.dirichlet(np.ones(4)) * scale(h)
                picks = torch.from_numpy(d.np.integers(0, m, 4)).cuda()
                aim = (torch.from_numpy(mix).float().cuda()[:, None] * centres[picks]).sum(0)
                q[b, h] = aim + d.normal(DIM)
            row += n
            ptr.append(c0 + m)
    flags = None
    if case["pinned"]:  # the first cluster (sink tokens) and the last four (the sliding window) of every segment
        f = np.zeros(total, dtype=np.uint8)
        for a, e in zip(ptr[:-1], ptr[1:]):
            f[a:a + 1] = dp.DP_CLUSTER_PINNED
            f[max(a, e - 4):e] = dp.DP_CLUSTER_PINNED
        flags = torch.from_numpy(f).cuda()
    return dp.DeviceCache(
        batch=batch, n_kv_heads=kvh, n_q_heads=kvh * group, head_dim=DIM, q=q, k_cache=k, v_cache=v,
        seg_row_base=torch.tensor(base, dtype=torch.int64, device="cuda"), seg_cluster_ptr=_i32(ptr),
        cluster_offsets=_i32(np.concatenate(offsets)), cluster_sizes=_i32(np.concatenate(sizes)), k_centroids=kc,
        v_centroids=vc, total_clusters=total, max_clusters_per_seg=max(ncl), max_rows_per_seg=max(ctx),
        cluster_flags=flags)


def _prepare_decode(case, seed):
    d = _Draws(seed)
    nh = case["batch"] * case["kv_heads"] * case["group"]
    dtype = torch.bfloat16 if case["out"] == "bf16" else torch.float32
    out = torch.empty(case["layers"], nh, DIM, device="cuda", dtype=dtype)
    lse = torch.empty(case["layers"], nh, device="cuda")
    calls, workspace = [], None
    for i in range(case["layers"]):
        problem = dp.Problem(_layer(case, d))
        if workspace is None:  # the layers run one after the other: one workspace serves them all
            workspace = torch.empty(dp.dp_workspace_bytes(problem), dtype=torch.uint8, device="cuda")
        o, l = out[i], lse[i]
        if case["kind"] == "budget":
            kept, exact = (max(1, int(case[k] * max(_clusters(case)))) for k in ("keep", "exact"))
            calls.append((dp.dp_budget_decode_attention, (problem, kept, exact, o, l, workspace)))
        elif case["kind"] == "dense":
            rows = _i32([n for n in _contexts(case) for _ in range(case["kv_heads"])])
            calls.append((dp.dp_dense_decode, (problem, rows, o, l, workspace)))
        elif case["plain"]:
            calls.append((dp.dp_decode_attention, (problem, case["p1"], case["p2"], o, l, workspace)))
        else:
            calls.append((dp.BoundDecodeStep(problem, case["p1"], case["p2"], o, l, workspace), ()))
    return {"calls": calls, "result": (out, lse)}


def _prepare_prefill(case, seed):
    d = _Draws(seed)
    ctx, ncl, kvh = _contexts(case), _clusters(case), case["kv_heads"]
    rows, total = sum(ctx) * kvh, sum(ncl) * kvh
    build = case["kind"] == "build"
    kw = dict(device="cuda", dtype=torch.bfloat16)
    k = torch.empty(rows, DIM, **kw)
    v = torch.empty(rows if build else 1, DIM, **kw)
    owner = torch.zeros(rows if build else 1, dtype=torch.int32, device="cuda")
    base, seg_rows, ptr, row = [], [], [0], 0
    for b in range(case["batch"]):
        for _ in range(kvh):
            n, m = ctx[b], ncl[b]
            lengths = torch.from_numpy(_sizes(d.np, m, n, case["mean"], case["sizes"])).cuda()
            own = torch.repeat_interleave(torch.arange(m, device="cuda"), lengths, output_size=n)
            own = own[torch.randperm(n, generator=d.gen, device="cuda")]  # token order
            k[row:row + n] = (2.0 * d.normal(m, DIM))[own] + 0.5 * d.normal(n, DIM)
            if build:
                v[row:row + n] = d.normal(n, DIM)
                owner[row:row + n] = own.int()
            base.append(row)
            seg_rows.append(n)
            ptr.append(ptr[-1] + m)
            row += n
    prefill = dp.Prefill(k, v, owner, torch.tensor(base, dtype=torch.int64, device="cuda"), _i32(seg_rows), _i32(ptr),
                         total, max(ncl), max(ctx))
    if build:
        ws = torch.empty(dp.dp_build_workspace_bytes(prefill), dtype=torch.uint8, device="cuda")
        out = dict(k_cache=torch.empty(rows, DIM, **kw), v_cache=torch.empty(rows, DIM, **kw),
                   cluster_offsets=torch.empty(total, dtype=torch.int32, device="cuda"),
                   cluster_sizes=torch.empty(total, dtype=torch.int32, device="cuda"),
                   k_centroids=torch.empty(total, DIM, **kw), v_centroids=torch.empty(total, DIM, **kw))
        if case["sums"]:
            out["v_sums"] = torch.empty(total, DIM, device="cuda")
            out["token_row"] = torch.empty(rows, dtype=torch.int32, device="cuda")
        return {"prefill": prefill, "workspace": ws, "out": out}
    ws = torch.empty(dp.dp_kmeans_fit_workspace_bytes(prefill), dtype=torch.uint8, device="cuda")
    return {"prefill": prefill, "workspace": ws, "rounds": case["rounds"],
            "centroids": torch.empty(total, DIM, **kw),
            "assignment": torch.empty(rows, dtype=torch.int32, device="cuda")}


def prepare(case, seed):
    state = (_prepare_prefill if case["kind"] in ("fit", "build") else _prepare_decode)(case, seed)
    state["kind"] = case["kind"]
    return state


def run(state):
    if state["kind"] == "build":
        dp.dp_build_cluster_cache(state["prefill"], workspace=state["workspace"], **state["out"])
        return state["out"]
    if state["kind"] == "fit":
        dp.dp_kmeans_fit(state["prefill"], state["centroids"], state["rounds"], dp.DP_KMEANS_INIT_STRIDED,
                         state["assignment"], state["workspace"])
        return state["centroids"], state["assignment"]
    for call, args in state["calls"]:
        call(*args)
    return state["result"]


def _selected(case, n, mean):
    """The segments of a sequence with ``n`` clusters, drawn again on the host by the recipe of the inputs: (clusters
    that some head of a group takes exactly, clusters that heads only approximate, rows summed over the heads), of
    all its KV heads together."""
    rng = np.random.default_rng(5)
    n_exact = n_approx = n_rows = 0
    for g in range(case["kv_heads"]):
        centres = 2.0 * rng.standard_normal((n, DIM), dtype=np.float32)
        scale = _scales(case, rng)
        exact, kept = np.zeros(n, bool), np.zeros(n, bool)
        for h in range(g * case["group"], (g + 1) * case["group"]):
            aim = (rng.dirichlet(np.ones(4))[:, None] * scale(h) * centres[rng.integers(0, n, 4)]).sum(0)
            x = centres @ (aim + rng.standard_normal(DIM)).astype(np.float32) / math.sqrt(DIM)
            order = np.argsort(-x)
            w = np.exp(x[order] - x.max())
            mass = np.cumsum(w) / w.sum()
            if case["kind"] == "budget":
                n1, n2 = max(1, int(case["keep"] * n)), max(1, int(case["exact"] * n))
            else:
                n1 = int(np.searchsorted(mass, case["p1"])) + 1
                n2 = int(np.searchsorted(mass, case["p2"] * mass[min(n1, n) - 1])) + 1
            exact[order[:n2]] = True
            kept[order[:n1]] = True
            n_rows += n2 * mean + n1 - n2
        n_exact += int(exact.sum())
        n_approx += int((kept & ~exact).sum())
    return n_exact, n_approx, n_rows


def work(case):
    ctx, ncl, kvh = _contexts(case), _clusters(case), case["kv_heads"]
    tokens, total = sum(ctx) * kvh, sum(ncl) * kvh
    if case["kind"] == "fit":
        pairs = sum(n * k for n, k in zip(ctx, ncl)) * kvh
        # every round reads the keys and the centroids and leaves new centroids; the last one also the assignment
        return {"bytes": case["rounds"] * (tokens * ROW + 2 * total * ROW) + 4 * tokens,
                "flops": case["rounds"] * 2.0 * DIM * pairs}
    if case["kind"] == "build":
        more = total * DIM * 4 + tokens * 4 if case["sums"] else 0
        return {"bytes": tokens * (4 * ROW + 4) + total * (2 * ROW + 8) + more, "flops": 2.0 * DIM * tokens}
    nh = case["batch"] * kvh * case["group"]
    ends = nh * (ROW + DIM * (2 if case["out"] == "bf16" else 4) + 4)
    if case["kind"] == "dense":
        return {"bytes": tokens * 2 * ROW + ends, "flops": 4.0 * DIM * tokens * case["group"]}
    nbytes = flops = 0.0
    seen = {}
    for n, m in zip(ctx, ncl):
        if m not in seen:
            seen[m] = _selected(case, m, n / m)
        exact, approx, rows = seen[m]
        if case["pinned"]:
            exact, rows = exact + 5 * kvh, rows + 5 * kvh * case["group"] * n / m
        nbytes += kvh * m * (ROW + 4) + (exact * n / m + approx) * 2 * ROW
        flops += kvh * 2.0 * DIM * m * case["group"] + 4.0 * DIM * rows
    return {"bytes": case["layers"] * (nbytes + ends), "flops": case["layers"] * flops}


def tolerance(case):
    if case["kind"] == "build":
        return "exact"  # rows are moved; means are double-precision sums rounded once
    # Below: about four times what the same inputs with their 128 dimensions permuted (the sums in another order) gave.
    if case["kind"] == "fit":
        # scores are 32-bit sums of 128 products: a token whose two best centroids differ by less than their rounding
        # may go to either, and its two clusters' means follow (seen: rel 4e-4, max 0.23, 7e-6 of the tokens)
        return {"rel": 2e-3, "max": 0.9, "differ": 1e-4}
    if case["out"] == "bf16":  # the last bit of a rounded output (seen: rel 2e-4, max 8e-3)
        return {"rel": 8e-4, "max": 3e-2}
    if case["kind"] == "dense" or (case["kind"] == "step" and case["heads"] in ("peaked", "spread")):
        return {"rel": 3e-5, "max": 3e-4}  # rows summed in another order (seen: rel 6e-6, max 5e-5)
    # a flat head has clusters whose cumulative mass, or rank, lies within 32-bit rounding of a threshold or budget:
    # one of them may fall on the other side of it (seen: rel 1.6e-4, max 7e-3)
    return {"rel": 6e-4, "max": 3e-2}

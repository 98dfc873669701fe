"""Performance cases of the mini-batch data-preparation path, through the package's public entry points.

A case is a dict of plain values.  `do` names the calls one pass makes:

  step     sample_khop + gather_features of one mini-batch (what a training loop does per step)
  sample   sample_khop alone (the sampler on a stream of its own, as the inter-batch pipeline runs it)
  server   sample_khop + build_blocks + gather_features (the whole sampling server)
  blocks   build_blocks alone (the graph constructor beside another batch's extraction)
  gather   gather_features alone, of a list of ids with a popularity skew (the extractor on its own stream)
  hotness  build_hotness of a tablet + get_hotness (pre-sampling, once per job)
  extract  sample_extract (the pipeline inside one batch)

Graphs are directed power-law graphs made on the GPU: out-degrees and in-edge popularity both fall as
1 / (rank + i0) with the largest expected degree sqrt(E), the two rankings scattered over the ids
independently of each other.  Feature values are standard normal draws.  Every result is a list of whole
numbers or a byte-for-byte copy of feature rows, so every comparison is exact.
"""
import math

import numpy as np
import torch

import paper_2305_16588_amd as lgp

# do, V, deg (mean degree), fanouts, batch, index64, topo (share of the topology that is cached), dim, fp16,
# feat (share of the feature rows that is cached), host (graph and features in pinned CPU memory, read over
# PCIe where they are not cached; otherwise everything is resident in HBM to begin with), n_ids (gather: draws
# before duplicates are dropped), n_batches (hotness)
_DEFAULTS = dict(do="step", V=10_000, deg=20.0, fanouts="10,5", batch=1024, index64=False, topo=1.0, dim=0, fp16=False,
                 feat=0.0, host=False, n_ids=0, n_batches=1)


def listed():
    return [
        # The smallest training set-up: 10 k vertices, both caches hold a fifth, the rest crosses PCIe.
        dict(_DEFAULTS, name="tiny_step", do="step", topo=0.2, dim=128, feat=0.2, host=True),
        # A small request against a resident graph (evaluation or serving of a few dozen vertices): latency.
        dict(_DEFAULTS, name="small_step", do="step", V=2_400_000, deg=25.8, fanouts="15,10,5", batch=64, dim=100,
             feat=1.0),
        # Sampling of a products-shaped graph with half of the topology cached, the rest read over PCIe.
        dict(_DEFAULTS, name="mid_sample", do="sample", V=2_400_000, deg=25.8, fanouts="15,10,5", batch=8192, topo=0.5,
             host=True),
        # The whole sampling server on that graph with everything cached: an ordinary step on one MI355X.
        dict(_DEFAULTS, name="mid_server", do="server", V=2_400_000, deg=25.8, fanouts="15,10,5", batch=8192, dim=100,
             feat=1.0),
        # Three hops over a papers-shaped graph, topology cached, 64-bit offsets.
        dict(_DEFAULTS, name="large_sample", do="sample", V=111_000_000, deg=14.4, fanouts="15,10,5", batch=8192,
             index64=True),
        # Two wide hops over one GPU's share of a billion-scale graph, resident in HBM (8 G edges): the largest graph.
        dict(_DEFAULTS, name="share_sample", do="sample", V=250_000_000, deg=32.0, fanouts="25,10", batch=8192,
             index64=True, topo=0.0),
        # Relabelling a three-hop sample of the papers-shaped graph into bipartite blocks.
        dict(_DEFAULTS, name="large_blocks", do="blocks", V=111_000_000, deg=14.4, fanouts="15,10,5", batch=8192,
             index64=True),
        # Feature extraction with every row cached, rows of whole cache lines (fp16 x 128).
        dict(_DEFAULTS, name="gather_cached", do="gather", V=30_000_000, n_ids=600_000, dim=128, fp16=True, feat=1.0),
        # The same with rows of an odd number of fp16 values (no alignment beyond two bytes).
        dict(_DEFAULTS, name="gather_ragged", do="gather", V=10_000_000, n_ids=600_000, dim=75, fp16=True, feat=1.0),
        # 400-byte rows, 30 % of them cached: most of the time goes to the rows that cross PCIe.
        dict(_DEFAULTS, name="gather_mixed", do="gather", V=2_400_000, n_ids=2_000_000, dim=100, feat=0.3, host=True),
        # Pre-sampling: 16 mini-batches with all topology in CPU memory, hotness vectors handed to the host.
        dict(_DEFAULTS, name="mid_hotness", do="hotness", V=2_400_000, deg=25.8, fanouts="15,10,5", batch=8192, topo=0.0,
             host=True, n_batches=16),
        # One mini-batch through the pipeline that overlaps a batch's sampling with its own extraction.
        dict(_DEFAULTS, name="mid_extract", do="extract", V=2_400_000, deg=25.8, fanouts="15,10,5", batch=8192, dim=100,
             feat=1.0),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    do = rng.choice(["step", "sample", "server", "blocks", "gather", "hotness", "extract"])
    c = dict(_DEFAULTS, do=do)
    c["host"] = do == "hotness" or (do in ("step", "sample", "gather", "extract") and rng.random() < 0.4)
    c["dim"] = 0 if do in ("sample", "blocks", "hotness") else log_int(16, 512)
    c["fp16"] = rng.random() < 0.5
    row = c["dim"] * (2 if c["fp16"] else 4)
    top = {"sample": 100e6, "blocks": 100e6, "hotness": 4e6}.get(do, 30e6)
    if c["host"]:
        top = min(top, 4e6)
    if row:
        top = min(top, (1.5e9 if c["host"] else 6e9) / row)
    c["V"] = log_int(10_000, top)
    c["deg"] = round(min(rng.uniform(6.0, 40.0), 1.6e9 / c["V"]), 2)
    c["index64"] = rng.random() < 0.5
    fan = [rng.randint(2, 25) for _ in range(rng.randint(1, 3))]
    c["batch"] = min(log_int(40, 8192), c["V"] // 4)
    while c["batch"] * math.prod(fan) > 8192 * 750:
        fan[fan.index(max(fan))] -= 1
    c["fanouts"] = ",".join(str(f) for f in fan)
    if c["host"]:
        c["topo"] = 0.0 if do == "hotness" else round(rng.uniform(0.2, 1.0), 3)
        c["feat"] = round(rng.uniform(0.1, 0.95), 3) if row else 0.0
    else:
        c["topo"] = 0.0 if do == "hotness" else 1.0
        c["feat"] = 1.0 if row else 0.0
    if do == "gather":
        c["n_ids"] = min(log_int(2_000, 1_000_000), c["V"])
    if do == "hotness":
        c["n_batches"] = rng.randint(2, 8)
        c["batch"] = min(c["batch"], c["V"] // (4 * c["n_batches"]))
    return c


# ---- inputs -----------------------------------------------------------------
def _law(V, E):
    """(i0, L): popularity of rank i falls as 1 / (i + i0), L = ln(1 + V / i0), and i0 = sqrt(E) / L makes the
    largest of E expected degrees sqrt(E)."""
    i0 = max(1.0, math.sqrt(E) / 8)
    for _ in range(60):
        i0 = max(1.0, math.sqrt(max(E, 1.0)) / math.log1p(V / i0))
    return i0, math.log1p(V / i0)


class _Scatter:
    """A bijection of 0 .. V-1 with no locality: x -> (x * mult + add) mod V."""

    def __init__(self, V, seed):
        r = np.random.default_rng(seed)
        self.V, self.add = V, int(r.integers(V))
        self.mult = int(V * 0.6180339887) - int(r.integers(max(1, V // 16)))
        self.mult = max(1, self.mult)
        while math.gcd(self.mult, V) != 1:
            self.mult += 1

    def __call__(self, x):
        return x.mul_(self.mult).add_(self.add).remainder_(self.V)


def _popular_ranks(n, V, i0, L, gen):
    u = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
    return u.mul_(L).expm1_().mul_(i0).to(torch.int64).clamp_(max=V - 1)


def _graph(case, seed, gen):
    """CSR arrays on the GPU: indptr [V + 1], indices [E] int32."""
    V, E = case["V"], case["V"] * case["deg"]
    i0, L = _law(V, E)
    src, dst = _Scatter(V, seed * 3 + 1), _Scatter(V, seed * 3 + 2)
    indptr = torch.zeros(V + 1, dtype=torch.int64, device="cuda")
    step = 1 << 26
    for lo in range(0, V, step):
        n = min(step, V - lo)
        rank = src(torch.arange(lo, lo + n, device="cuda")).to(torch.float64)
        d = rank.add_(i0).reciprocal_().mul_(E / L)
        d += torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
        indptr[lo + 1:lo + n + 1] = d.to(torch.int64)
        del rank, d
    torch.cumsum(indptr, 0, out=indptr)
    n_edges = int(indptr[-1])
    indices = torch.empty(n_edges, dtype=torch.int32, device="cuda")
    for lo in range(0, n_edges, step):
        n = min(step, n_edges - lo)
        indices[lo:lo + n] = dst(_popular_ranks(n, V, i0, L, gen))
    if not case["index64"] and n_edges < 2 ** 31:
        indptr = indptr.to(torch.int32)
    return indptr, indices


def _features(case, seed):
    """The feature table on the GPU, from `seed` alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 5)
    t = torch.empty((case["V"], case["dim"]), dtype=torch.float16 if case["fp16"] else torch.float32, device="cuda")
    return t.normal_(generator=gen)


def _gather_ids(case, seed):
    """(ids, n): an ascending list of distinct ids drawn with the popularity law, in a buffer of n_ids entries."""
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 6)
    V = case["V"]
    i0, L = _law(V, V * case["deg"])
    found = torch.unique(_Scatter(V, seed * 3 + 2)(_popular_ranks(case["n_ids"], V, i0, L, gen))).to(torch.int32)
    ids = torch.zeros(case["n_ids"], dtype=torch.int32, device="cuda")
    ids[:found.numel()] = found
    return ids, found.numel()


def _placed(t, host):
    """The array where the graph lives: pinned CPU memory, or where it is."""
    if not host:
        return t
    a = lgp.pinned_empty(tuple(t.shape), {torch.int32: np.int32, torch.int64: np.int64, torch.float16: np.float16,
                                          torch.float32: np.float32}[t.dtype])
    torch.from_numpy(a).copy_(t)
    return a


def _row_bytes(case):
    return case["dim"] * (2 if case["fp16"] else 4)


def prepare(case, seed):
    do, V, host = case["do"], case["V"], case["host"]
    fanouts = [int(f) for f in case["fanouts"].split(",")]
    batch = case["batch"]
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 4)
    feats = _features(case, seed) if case["dim"] else None
    st = dict(do=do, fanouts=fanouts, batch=batch, rng=seed * 1000 + 17)
    if do == "gather":
        # the extractor alone needs no topology; the cache is ranked by counts of earlier draws of the same law
        indptr, indices = torch.zeros(V + 1, dtype=torch.int32, device="cuda"), np.empty(0, np.int32)
        ctx = lgp.Context(indptr, indices, _placed(feats, host))
        hot = np.zeros(V, np.int32)
        if case["feat"] < 1.0:
            i0, L = _law(V, V * case["deg"])
            drawn = _Scatter(V, seed * 3 + 2)(_popular_ranks(4 * case["n_ids"], V, i0, L, gen))
            hot = torch.bincount(drawn, minlength=V).to(torch.int32).cpu().numpy()
        ctx.set_hotness(np.zeros(V, np.uint32), hot.view(np.uint32))
        ctx.build_cache(0, int(case["feat"] * V) * _row_bytes(case))
        ids, n = _gather_ids(case, seed)
        st.update(ctx=ctx, ids=ids, n_dev=torch.tensor([n], dtype=torch.int32, device="cuda"),
                  rows=torch.zeros((case["n_ids"], case["dim"]), dtype=feats.dtype, device="cuda"),
                  stats=torch.zeros(2, dtype=torch.int32, device="cuda"))
        return st

    indptr, indices = _graph(case, seed, gen)
    n_edges = indices.numel()
    ctx = lgp.Context(_placed(indptr, host), _placed(indices, host), None if feats is None else _placed(feats, host))
    del indptr, indices, feats
    tablet = _Scatter(V, seed * 3 + 3)(torch.arange(case["n_batches"] * batch, device="cuda")).to(torch.int32)
    st.update(ctx=ctx, tablet=tablet)
    if do == "hotness":
        return st
    if case["topo"] > 0 or case["feat"] > 0:
        ranked_on = _Scatter(V, seed * 3 + 4)(torch.arange(min(V, 2 * batch), device="cuda")).to(torch.int32)
        ctx.build_hotness(ranked_on, batch, fanouts, seed)
        ctx.build_cache(int(case["topo"] * (4 * n_edges + 8 * V)), int(case["feat"] * V) * _row_bytes(case))
    if do == "step":
        ctx.reserve(batch, fanouts)
    buf = lgp.SampleBuffers(V, batch, fanouts, last_frontier=do in ("server", "blocks"))
    for t in [*buf.frontier[1:], *buf.nbr, *buf.cnt, buf.gather_ids]:
        t.fill_(-1)                                  # entries past the counts are left untouched
    st["buf"] = buf
    if do in ("server", "blocks"):
        blk = lgp.BlockBuffers(buf)
        for t in [*blk.blk_indptr, *blk.blk_src, *blk.feat_row]:
            t.fill_(-1)
        st["blk"] = blk
    if do == "blocks":
        ctx.sample_khop(tablet, fanouts, st["rng"], out=buf)
    if do in ("step", "server", "extract"):
        st["rows"] = torch.zeros((buf.gather_cap, case["dim"]), dtype=ctx.feat_torch_dtype, device="cuda")
        st["stats"] = torch.zeros(2, dtype=torch.int32, device="cuda")
        st["groups"] = torch.zeros(len(fanouts) + 2, dtype=torch.int32, device="cuda")
    return st


# ---- one pass ---------------------------------------------------------------
def _sampled(buf):
    return {"frontier": buf.frontier[1:], "nbr": buf.nbr, "cnt": buf.cnt, "n_frontier": buf.n_frontier,
            "gather_ids": buf.gather_ids, "n_gather": buf.n_gather}


def _blocks(blk):
    return {"blk_indptr": blk.blk_indptr, "blk_src": blk.blk_src, "feat_row": blk.feat_row}


def run(st):
    do, ctx, fanouts = st["do"], st["ctx"], st["fanouts"]
    if do == "gather":
        ctx.gather_features(st["ids"], n_dev=st["n_dev"], out=st["rows"], stats=st["stats"])
        return {"rows": st["rows"], "stats": st["stats"]}
    seeds = st["tablet"]
    if do == "hotness":
        ctx.build_hotness(seeds, st["batch"], fanouts, st["rng"])
        topo, feat = ctx.get_hotness()
        return {"topo": topo.view(np.int32), "feat": feat.view(np.int32)}
    buf = st["buf"]
    if do == "blocks":
        ctx.build_blocks(seeds, fanouts, buf, out=st["blk"])
        return _blocks(st["blk"])
    if do == "extract":
        ctx.sample_extract(seeds, fanouts, st["rng"], buf, st["rows"], st["groups"], st["stats"])
        return {**_sampled(buf), "rows": st["rows"], "groups": st["groups"], "stats": st["stats"]}
    ctx.sample_khop(seeds, fanouts, st["rng"], out=buf)
    if do == "sample":
        return _sampled(buf)
    got = _sampled(buf)
    if do == "server":
        ctx.build_blocks(seeds, fanouts, buf, out=st["blk"])
        got.update(_blocks(st["blk"]))
    ctx.gather_features(buf.gather_ids, n_dev=buf.n_gather, out=st["rows"], stats=st["stats"])
    return {**got, "rows": st["rows"], "stats": st["stats"]}


# ---- what a pass cannot do without --------------------------------------------
def _expected(case):
    """Expected sizes of one mini-batch: (frontier sizes, sampled edges per hop, extracted ids)."""
    V, E = case["V"], case["V"] * case["deg"]
    i0, L = _law(V, E)
    r = np.expm1(np.linspace(0.0, L, 4001)) * i0                  # ranks, evenly spaced in the law's own measure
    mid, width = (r[1:] + r[:-1]) / 2, np.diff(r)
    degree, p = E / L / (mid + i0), 1.0 / (L * (mid + i0))

    def distinct(m):
        return float((width * -np.expm1(-m * p)).sum())

    fanouts = [int(f) for f in case["fanouts"].split(",")]
    n, edges = [float(case["batch"])], []
    for f in fanouts:
        per = float((width * np.minimum(degree, f)).sum()) / V     # sources are independent of the target ranking
        edges.append(n[-1] * per)
        n.append(distinct(edges[-1]))
    return fanouts, n, edges, min(float(V), case["batch"] + distinct(sum(edges)))


def work(case):
    """Bytes of one pass: every id, row-table entry, sampled column id and feature row read once, every result
    written once.  The path does no floating-point arithmetic."""
    do, row = case["do"], _row_bytes(case)
    if do == "gather":
        V = case["V"]
        i0, L = _law(V, V * case["deg"])
        r = np.expm1(np.linspace(0.0, L, 4001)) * i0
        p = 1.0 / (L * ((r[1:] + r[:-1]) / 2 + i0))
        n = float((np.diff(r) * -np.expm1(-case["n_ids"] * p)).sum())
        return {"bytes": n * (4 + 2 * row), "flops": 0}
    fanouts, n, edges, ids = _expected(case)
    hops = range(len(fanouts))
    if do == "hotness":
        per = sum(n[h] * (4 + 8) + edges[h] * 4 for h in hops) + ids * 8
        return {"bytes": case["n_batches"] * per + 2 * 8 * case["V"], "flops": 0}
    sampling = sum(n[h] * (4 + 8 + 4 + 4 * fanouts[h]) + edges[h] * 4 for h in hops) + 4 * (sum(n[1:-1]) + ids)
    blocks = sum(n[h] * (4 * fanouts[h] + 4 + 8) + edges[h] * 4 for h in hops) + sum(n) * 8 + 4 * ids
    gather = ids * (4 + 2 * row)
    return {"bytes": {"step": sampling + gather, "sample": sampling, "server": sampling + blocks + gather,
                      "blocks": blocks, "extract": sampling + gather}[do], "flops": 0}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The extracted rows by plain indexing.  Where the ids come out of the sampler there is nothing to round: all
    results are whole numbers and copies of feature rows."""
    if case["do"] != "gather":
        return None
    feats = _features(case, seed)
    ids, n = _gather_ids(case, seed)
    rows = torch.zeros((case["n_ids"], case["dim"]), dtype=torch.float64, device="cuda")
    rows[:n] = feats[ids[:n].long()].double()
    return {"rows": rows, "stats": None}

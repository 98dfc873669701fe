"""lgp_sample_extract -- sampling with the feature extraction overlapped hop by hop (the intra-batch pipeline of
Sec. 5) -- against the oracle: same frontiers / samples / counts as lgp_sample_khop, the listing in first-reach
order, its group bounds, the extracted bytes and the hit / miss counts, bit for bit."""
import numpy as np
import pytest
import torch

import datagen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def W():
    from gpu_common import Workload
    w = Workload(datagen.TINY)
    w.ctx.build_hotness(w.tablet_dev, w.spec.batch, w.spec.fanouts, w.spec.base_seed)
    rt, rf, _ = w.orc.build_hotness(w.tablet, w.spec.batch, w.spec.fanouts, w.spec.base_seed)
    w.qf = w.orc.rank_by_hotness(rf)
    return w


def _run_and_check(W, seeds, seeds_dev, fanouts, rng_seed, n_feat, tag, last_frontier=False, blocks=False):
    import paper_2305_16588_amd as lgp
    L = len(fanouts)
    buf = lgp.SampleBuffers(W.V, max(int(seeds_dev.numel()), 1), fanouts, last_frontier=last_frontier or blocks)
    rows = torch.full((max(buf.gather_cap, 1), W.spec.feat_dim), -3.0, dtype=W.ctx.feat_torch_dtype, device="cuda")
    groups = torch.full((L + 2,), -1, dtype=torch.int32, device="cuda")
    stats = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    W.ctx.sample_extract(seeds_dev, fanouts, rng_seed, buf, rows, groups, stats)
    blk = W.ctx.build_blocks(seeds_dev, fanouts, buf) if blocks else None
    torch.cuda.synchronize()
    ref = W.orc.sample_khop(seeds, fanouts, rng_seed, blocks=blocks)
    fr, nbr, cnt, listing = buf.to_host(seeds_dev)
    for h in range(L):
        assert fr[h].shape == ref.frontier[h].shape and (fr[h] == ref.frontier[h]).all(), f"{tag} frontier[{h}]"
        assert (nbr[h] == ref.nbr[h]).all() and (cnt[h] == ref.cnt[h]).all(), f"{tag} hop {h}"
    if last_frontier or blocks:
        assert (fr[L] == ref.frontier[L]).all(), f"{tag} last frontier"
    assert listing.tolist() == ref.hop_order.tolist(), f"{tag} listing"
    assert groups.tolist() == ref.hop_seg.tolist(), f"{tag} groups"
    n = ref.hop_order.size
    assert rows[:n].cpu().numpy().tobytes() == W.orc.gather(ref.hop_order).tobytes(), f"{tag} rows"
    n_hit = W.orc.count_hits(ref.hop_order, W.qf, n_feat) if n else 0
    assert stats.tolist() == [n_hit, n - n_hit], f"{tag} stats"
    if blocks:
        indptr, src, feat_row = blk.to_host()
        where = {int(v): i for i, v in enumerate(ref.hop_order.tolist())}
        for h in range(L):
            assert (indptr[h] == ref.blk_indptr[h]).all() and (src[h] == ref.blk_src[h]).all(), f"{tag} block {h}"
        for h in range(L + 1):
            assert feat_row[h].tolist() == [where[int(v)] for v in ref.frontier[h].tolist()], f"{tag} feat_row[{h}]"
    W.ctx.check()
    return ref


def test_every_batch_of_the_epoch(W):
    spec = W.spec
    plan = W.ctx.build_cache(*datagen.budgets(spec, W.E))
    assert 0 < plan.n_feat < W.V
    n_batches = (W.tablet.size + spec.batch - 1) // spec.batch
    for b in range(n_batches):
        seeds, seeds_dev = W.batch(b)
        _run_and_check(W, seeds, seeds_dev, spec.fanouts, spec.base_seed + b, plan.n_feat, f"batch {b}")
    # the ordinary calls still work afterwards (the pipeline leaves the dedup bitmaps clean)
    from gpu_common import assert_batch_equal
    seeds, seeds_dev = W.batch(1)
    buf = W.ctx.sample_khop(seeds_dev, spec.fanouts, 5)
    assert_batch_equal(W.orc.sample_khop(seeds, spec.fanouts, 5), buf.to_host(seeds_dev), "sample_khop afterwards")


@pytest.mark.parametrize("fanouts", [(25,), (3, 3, 3), (64, 2), (2, 2, 2, 2, 2, 2, 2, 2), (1, 1)])
def test_fanout_shapes_and_blocks(W, fanouts):
    plan = W.ctx.build_cache(*datagen.budgets(W.spec, W.E))
    seeds, seeds_dev = W.tablet[:700], W.tablet_dev[:700].contiguous()
    _run_and_check(W, seeds, seeds_dev, fanouts, 4242, plan.n_feat, str(fanouts), blocks=True)


@pytest.mark.parametrize("overlap", [False, True])
@pytest.mark.parametrize("feat_rows", [0, 2000, None])
def test_cache_ratios_and_overlap_mode(W, feat_rows, overlap):
    spec = W.spec
    topo_b, _ = datagen.budgets(spec, W.E)
    n_f = W.V if feat_rows is None else feat_rows
    plan = W.ctx.build_cache(topo_b, n_f * W.orc.row_bytes)
    assert plan.n_feat == n_f
    W.ctx.set_overlap(overlap)
    for b in (0, 9, 0):                                   # the short last batch, and a batch twice
        seeds, seeds_dev = W.batch(b)
        _run_and_check(W, seeds, seeds_dev, spec.fanouts, 77 + b, n_f, f"{n_f} cached rows, batch {b}")
    W.ctx.set_overlap(False)


def test_degenerate_seed_lists(W):
    plan = W.ctx.build_cache(*datagen.budgets(W.spec, W.E))
    deg = np.diff(W.indptr)
    isolated = np.flatnonzero(deg == 0)[:5].astype(np.int32)
    hub = np.array([int(np.argmax(deg))], dtype=np.int32)
    twice = np.concatenate([W.tablet[:40], W.tablet[:40], W.tablet[30:60]]).astype(np.int32)   # repeated seeds stay listed
    for name, seeds in (("no seeds", np.empty(0, np.int32)), ("isolated", isolated), ("hub", hub), ("repeated", twice)):
        dev = torch.from_numpy(seeds).cuda()
        _run_and_check(W, seeds, dev, (10, 5), 9, plan.n_feat, name, last_frontier=True)


def test_mid_workload_full_size():
    from gpu_common import Workload
    spec = datagen.WORKLOADS["mid"]
    M = Workload(spec, device_gen="cuda")
    M.ctx.build_hotness(M.tablet_dev, spec.batch, spec.fanouts, spec.base_seed)
    _, rf, _ = M.orc.build_hotness(M.tablet, spec.batch, spec.fanouts, spec.base_seed, max_batches=-1)
    M.qf = M.orc.rank_by_hotness(rf)
    plan = M.ctx.build_cache(*datagen.budgets(spec, M.E))
    last = (M.tablet.size - 1) // spec.batch
    for b in (0, last):
        seeds, seeds_dev = M.batch(b)
        ref = _run_and_check(M, seeds, seeds_dev, spec.fanouts, spec.base_seed + 100 + b, plan.n_feat, f"mid batch {b}",
                             blocks=(b == 0))
    assert ref.hop_seg[-1] == ref.gather_ids.size


@pytest.mark.parametrize("V,dim,dtype", [(3000, 7, np.float16), (3000, 25, np.float32), (3000, 260, np.float32),
                                         (600_000, 10, np.float32), (1_200_000, 75, np.float16), ((1 << 23) + 5, 8, np.float16)])
def test_rows_beside_a_hop(V, dim, dtype):
    """Every chunk width and dedup-map layout that a hop shares a launch with, and rows too narrow for it: nothing, half and
    everything cached, groups of one row up to many passes, hits and misses timed apart."""
    import types

    import oracle
    import paper_2305_16588_amd as lgp
    rng = np.random.default_rng(V + dim)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(0, 7, V))]).astype(np.int32)
    indices = rng.integers(0, V, int(indptr[-1])).astype(np.int32)
    feats = lgp.pinned_empty((V, dim), dtype)
    feats[:] = rng.integers(-2000, 2000, (V, dim), dtype=np.int16)
    hot = rng.integers(0, 9, V).astype(np.uint32)
    orc = oracle.Oracle(indptr, indices, feats)
    w = types.SimpleNamespace(ctx=lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices), feats), orc=orc, V=V,
                              qf=orc.rank_by_hotness(hot), spec=types.SimpleNamespace(feat_dim=dim))
    w.ctx.set_hotness(np.zeros(V, np.uint32), hot)
    for n_feat in (0, V // 2, V):
        w.ctx.build_cache(0, n_feat * orc.row_bytes)
        for n_seeds, fanouts in ((1, (1, 1)), (700, (5, 3, 2)), (2900, (4,))):
            seeds = rng.permutation(V)[:n_seeds].astype(np.int32)
            for mode in (0, 1) if n_seeds == 700 else (0,):
                w.ctx.set_profiling(mode)
                _run_and_check(w, seeds, torch.from_numpy(seeds).cuda(), fanouts, 31 + n_seeds, n_feat, f"{n_feat} {fanouts} {mode}")
    w.ctx.set_profiling(0)

"""Sampling at the sizes where the library changes how it marks and compacts the sampled vertices, bit for bit against
the oracle: the largest graph of each dedup-map layout and the smallest of the next one."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _workload(V, deg, seed):
    """Ragged rows of up to `deg` ids over V vertices, ids spread over the whole range with both ends present."""
    import oracle
    import paper_2305_16588_amd as lgp
    rng = np.random.default_rng(seed)
    d = rng.integers(0, deg + 1, V)
    d[[0, V // 2, V - 1]] = deg
    indptr = np.zeros(V + 1, np.int32)
    np.cumsum(d, out=indptr[1:])
    indices = rng.integers(0, V, int(indptr[-1]), dtype=np.int32)
    indices[:3] = [V - 1, 0, V // 2]
    p_indptr, p_indices = lgp.pinned_copy(indptr), lgp.pinned_copy(indices)
    return lgp.Context(p_indptr, p_indices), oracle.Oracle(indptr, indices, None), rng


@pytest.mark.parametrize("V", [1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 1, 1 << 23, (1 << 23) + 1])
def test_sampling_on_both_sides_of_a_map_layout(V):
    from gpu_common import assert_batch_equal
    import paper_2305_16588_amd as lgp
    ctx, orc, rng = _workload(V, 6, V)
    seeds = np.unique(np.concatenate([[0, V // 2, V - 1], rng.integers(0, V, 3000)])).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    for fanouts in ((4, 3), (5,), (2, 2, 8)):
        for last in (False, True):
            buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=last)
            for rep in range(2):                                   # the maps have to be clear again after a call
                ctx.sample_khop(seeds_dev, fanouts, 40 + rep, out=buf)
                assert_batch_equal(orc.sample_khop(seeds, fanouts, 40 + rep), buf.to_host(seeds_dev), f"{V} {fanouts}")
    ctx.check()


@pytest.mark.parametrize("cap", [(1 << 31) - 1, 1 << 31, (1 << 32) - 1, 1 << 32, (1 << 32) + 5, 1 << 40])
@pytest.mark.parametrize("V", [5000, (1 << 23) + 1])
def test_capacities_beyond_32_bits(V, cap):
    """A caller may state any capacity at or above the worst case, such as that of a large arena it cuts its lists
    from: the lists are those of exactly sized buffers, through all three kinds of compaction."""
    from gpu_common import assert_batch_equal
    import paper_2305_16588_amd as lgp
    ctx, orc, rng = _workload(V, 6, V + 1)
    seeds = np.unique(rng.integers(0, V, 300)).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    fanouts = (4, 3)
    ref = orc.sample_khop(seeds, fanouts, 11)
    for last in (False, True):
        buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=last)
        for t in [*buf.frontier[1:], buf.gather_ids]:
            t.fill_(-1)
        buf.c_struct.cap[1] = buf.c_struct.cap[2] = buf.c_struct.gather_cap = cap
        ctx.sample_khop(seeds_dev, fanouts, 11, out=buf)
        assert_batch_equal(ref, buf.to_host(seeds_dev), f"{V} {cap} {last}")
    ctx.check()
    # the intra-batch pipeline takes any frontier capacity; it gathers rows for its listing, of fewer than 2^31 ids
    feats = lgp.pinned_empty((V, 2), np.float16)
    feats.view(np.uint16)[...] = rng.integers(0, 1 << 16, (V, 2), dtype=np.uint16)
    ctx = lgp.Context(*ctx._keep[:2], feats)
    buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=True)
    rows = torch.empty((buf.gather_cap, 2), dtype=torch.float16, device="cuda")
    for t in buf.frontier[1:]:
        t.fill_(-1)
    buf.c_struct.cap[1] = buf.c_struct.cap[2] = cap
    ctx.sample_extract(seeds_dev, fanouts, 11, buf, rows)
    fr, nbr, cnt, listing = buf.to_host(seeds_dev)
    assert all((fr[h] == ref.frontier[h]).all() for h in (1, 2)) and listing.tolist() == ref.hop_order.tolist()
    assert rows[:listing.size].cpu().numpy().tobytes() == feats[listing].tobytes()
    ctx.check()


@pytest.mark.parametrize("V", [(1 << 26) + 3, (1 << 27) + 3, (1 << 28) + 3])
def test_compaction_of_large_maps(V):
    """The compaction's wider shares: four and eight words per thread, and several passes.  Only every 61st vertex has
    neighbours, so that the host side stays small."""
    from gpu_common import assert_batch_equal
    import oracle
    import paper_2305_16588_amd as lgp
    rng = np.random.default_rng(V)
    d = np.zeros(V, np.int32)
    d[::61] = 5
    indptr = lgp.pinned_empty(V + 1, np.int32)
    indptr[0] = 0
    np.cumsum(d, out=indptr[1:])
    del d
    indices = lgp.pinned_copy((rng.integers(0, (V + 60) // 61, int(indptr[-1])) * 61).astype(np.int32))
    indices[::7] = V - 1 - np.arange(indices[::7].size, dtype=np.int32) % V       # leaves, up to the last vertex
    feats = lgp.pinned_empty((V, 1), np.float16)
    feats[:, 0] = np.arange(V, dtype=np.uint32).astype(np.uint16).view(np.float16)
    ctx, orc = lgp.Context(indptr, indices, feats), oracle.Oracle(indptr, indices, feats)
    seeds = (np.unique(rng.integers(0, (V + 60) // 61, 20_000)) * 61).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    fanouts = (4, 3)
    buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=True)
    plain = lgp.SampleBuffers(V, seeds.size, fanouts)
    rows = torch.empty((buf.gather_cap, 1), dtype=torch.float16, device="cuda")
    for rep in range(2):
        ref = orc.sample_khop(seeds, fanouts, 70 + rep)
        ctx.sample_khop(seeds_dev, fanouts, 70 + rep, out=plain)
        assert_batch_equal(ref, plain.to_host(seeds_dev), f"{V}")
        ctx.sample_khop(seeds_dev, fanouts, 70 + rep, out=buf)
        assert_batch_equal(ref, buf.to_host(seeds_dev), f"{V} with the last frontier")
        ctx.sample_extract(seeds_dev, fanouts, 70 + rep, buf, rows)
        fr, _, _, listing = buf.to_host(seeds_dev)
        assert (fr[2] == ref.frontier[2]).all() and listing.tolist() == ref.hop_order.tolist()
        assert rows[:listing.size].cpu().numpy().tobytes() == orc.gather(listing).tobytes()
    ctx.check()


@pytest.mark.parametrize("row_bytes", [2, 4, 6, 10, 12, 14, 18, 30, 34, 62, 66, 126, 130, 150, 254, 258, 386, 510, 514,
                                       1022, 1030, 2050, 4100, 8190])
@pytest.mark.parametrize("shift", [0, 1, 2])
def test_rows_of_any_even_width_and_alignment(row_bytes, shift):
    """Rows copied in chunks that do not divide them, into an output that starts `shift` fp16 values off: every byte
    of every row, and not one byte beside them, through both direct paths and the partitioned one."""
    import paper_2305_16588_amd as lgp
    V, D = 700, row_bytes // 2
    rng = np.random.default_rng(row_bytes)
    feats = lgp.pinned_empty((V, D), np.float16)
    feats.view(np.uint16)[...] = rng.integers(0, 1 << 16, (V, D), dtype=np.uint16)
    ctx = lgp.Context(lgp.pinned_copy(np.zeros(V + 1, np.int32)), lgp.pinned_empty(1, np.int32)[:0], feats)
    ids = rng.integers(0, V, 611).astype(np.int32)
    dev = torch.from_numpy(ids).cuda()
    want = feats.view(np.uint16)[ids].reshape(-1)
    ctx.set_hotness(np.zeros(V, np.uint32), rng.integers(0, 9, V).astype(np.uint32))
    for n_cached in (0, 300, V):
        ctx.build_cache(0, n_cached * row_bytes)
        flat = torch.full((ids.size * D + 16,), 21845, dtype=torch.int16, device="cuda")
        out = flat[shift:shift + ids.size * D].view(torch.float16).view(ids.size, D)
        ctx.gather_features(dev, out=out)
        got = flat.cpu().numpy().view(np.uint16)
        assert (got[shift:shift + want.size] == want).all(), f"{n_cached} rows cached"
        assert (got[:shift] == 21845).all() and (got[shift + want.size:] == 21845).all()
    ctx.check()


@pytest.mark.parametrize("row_bytes,shift,ok", [(8192, 1, True), (8194, 0, False), (8194, 1, False), (8196, 0, True), (8196, 1, False),
                                                (8196, 2, True), (16384, 2, True), (16388, 0, False), (16392, 0, True),
                                                (16392, 2, False), (32768, 4, True), (32776, 0, False), (65536, 0, True)])
def test_widest_rows_of_each_alignment(row_bytes, shift, ok):
    """A row may have 4096 of the widest chunks that divide it and its output address (2, 4, 8 or 16 bytes); wider ones
    are refused, when the context is made if no output could do, else by the call."""
    import paper_2305_16588_amd as lgp
    V, D = 9, row_bytes // 2
    rng = np.random.default_rng(row_bytes)
    feats = lgp.pinned_empty((V, D), np.float16)
    feats.view(np.uint16)[...] = rng.integers(0, 1 << 16, (V, D), dtype=np.uint16)
    graph = lgp.pinned_copy(np.zeros(V + 1, np.int32)), lgp.pinned_empty(1, np.int32)[:0]
    if not ok and row_bytes in (8194, 16388, 32776):
        with pytest.raises(lgp.LegionPrepError) as e:
            lgp.Context(*graph, feats)
        assert e.value.status == -4
        return
    ctx = lgp.Context(*graph, feats)
    ids = np.array([8, 0, 3, 3, 7], np.int32)
    dev = torch.from_numpy(ids).cuda()
    ctx.set_hotness(np.zeros(V, np.uint32), np.arange(V, dtype=np.uint32))
    for n_cached in (0, 4, V):
        ctx.build_cache(0, n_cached * row_bytes)
        flat = torch.full((ids.size * D + 16,), 21845, dtype=torch.int16, device="cuda")
        out = flat[shift:shift + ids.size * D].view(torch.float16).view(ids.size, D)
        if not ok:
            with pytest.raises(lgp.LegionPrepError) as e:
                ctx.gather_features(dev, out=out)
            assert e.value.status == -4
            continue
        ctx.gather_features(dev, out=out)
        got = flat.cpu().numpy().view(np.uint16)
        assert (got[shift:shift + ids.size * D] == feats.view(np.uint16)[ids].reshape(-1)).all()
        assert (got[:shift] == 21845).all() and (got[shift + ids.size * D:] == 21845).all()
    ctx.check()


@pytest.mark.parametrize("row_bytes", [250, 258, 262, 264, 334, 338, 344, 502, 506, 516, 520, 776, 872, 1016, 1030, 1032, 1048,
                                       2040, 2046, 2056, 2558, 2562, 2568, 32760])
@pytest.mark.parametrize("list_len", [1, 63, 65, 3000])
def test_cached_rows_on_both_sides_of_a_kernel_choice(row_bytes, list_len):
    """Ragged rows around the chunk counts at which another gather kernel takes them (16, 21, 32, 64, 128 and 160 chunks),
    all cached and half cached, lists that do and do not fill the kernels' passes."""
    import paper_2305_16588_amd as lgp
    V, D = 500, row_bytes // 2
    rng = np.random.default_rng(row_bytes + list_len)
    feats = lgp.pinned_empty((V, D), np.float16)
    feats.view(np.uint16)[...] = rng.integers(0, 1 << 16, (V, D), dtype=np.uint16)
    ctx = lgp.Context(lgp.pinned_copy(np.zeros(V + 1, np.int32)), lgp.pinned_empty(1, np.int32)[:0], feats)
    ids = rng.integers(0, V, list_len).astype(np.int32)
    want = feats.view(np.uint16)[ids].reshape(-1)
    ctx.set_hotness(np.zeros(V, np.uint32), rng.integers(0, 9, V).astype(np.uint32))
    for n_cached in (V, V // 2):
        ctx.build_cache(0, n_cached * row_bytes)
        flat = torch.full((ids.size * D + 16,), 21845, dtype=torch.int16, device="cuda")
        ctx.gather_features(torch.from_numpy(ids).cuda(), out=flat[:ids.size * D].view(torch.float16).view(ids.size, D))
        got = flat.cpu().numpy().view(np.uint16)
        assert (got[:want.size] == want).all() and (got[want.size:] == 21845).all(), f"{n_cached} rows cached"
    ctx.check()


@pytest.mark.parametrize("V,fanouts,n_seeds", [(1, (2,), 1), (2, (2, 2), 2), (3, (1, 64), 3), (65, (5, 4), 9), (1500, (64, 3), 40),
                                               (200_000, (3, 2), 700), (200_000, (1, 1, 1), 256), (200_000, (25, 10), 1025)])
@pytest.mark.parametrize("span", [1.0, 0.02])
def test_blocks_of_dense_sparse_and_clustered_frontiers(V, fanouts, n_seeds, span):
    """The frontiers' index: more and fewer ids than vertices to spread them over, ids in one corner of the
    range (long empty stretches, full blocks), hops whose destinations are and are not whole tiles."""
    from gpu_common import assert_batch_equal, assert_blocks_equal
    import oracle
    import paper_2305_16588_amd as lgp
    rng = np.random.default_rng(V + n_seeds)
    d = rng.integers(0, 12, V)
    indptr = np.zeros(V + 1, np.int32)
    np.cumsum(d, out=indptr[1:])
    lo = int(V * (1 - span) * 0.7)
    indices = (lo + rng.integers(0, max(1, int(V * span)), int(indptr[-1]))).astype(np.int32)
    indices = np.minimum(indices, V - 1)
    ctx = lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices))
    orc = oracle.Oracle(indptr, indices, None)
    seeds = np.sort(rng.permutation(V)[:n_seeds]).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    buf = lgp.SampleBuffers(V, n_seeds, fanouts, last_frontier=True)
    blk = lgp.BlockBuffers(buf)
    for rep in range(2):
        ctx.sample_khop(seeds_dev, fanouts, 90 + rep, out=buf)
        ctx.build_blocks(seeds_dev, fanouts, buf, out=blk)
        ref = orc.sample_khop(seeds, fanouts, 90 + rep, blocks=True)
        assert_batch_equal(ref, buf.to_host(seeds_dev), f"{V} {fanouts}")
        assert_blocks_equal(ref, blk.to_host(), f"{V} {fanouts}")
    ctx.check()


@pytest.mark.parametrize("V,n_seeds,fanouts", [(3, 3, (2, 2)), (500, 60, (3, 64)), (60_000, 300, (5, 4, 3)),
                                               (2_000_000, 1025, (7, 3))])
@pytest.mark.parametrize("how", ["reversed", "shuffled", "two ids swapped"])
def test_blocks_of_reordered_frontiers(V, n_seeds, fanouts, how):
    """The graph constructor takes the frontiers in any order (their rows of samples in the same order): positions are
    those in the lists as they stand.  Ascending lists again afterwards, on the same context."""
    from gpu_common import assert_blocks_equal
    import paper_2305_16588_amd as lgp
    ctx, orc, rng = _workload(V, 9, V + n_seeds)
    seeds = np.sort(rng.permutation(V)[:n_seeds]).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    buf = lgp.SampleBuffers(V, n_seeds, fanouts, last_frontier=True)
    blk = lgp.BlockBuffers(buf)
    L = len(fanouts)
    for reordered in ((1,), (L,), tuple(range(1, L + 1)), ()):
        ctx.sample_khop(seeds_dev, fanouts, 21, out=buf)
        fr, nbr, cnt, gids = buf.to_host(seeds_dev)
        fr, nbr, cnt = list(fr), list(nbr), list(cnt)
        for h in reordered:
            n = fr[h].size
            perm = np.arange(n)
            if how == "reversed":
                perm = perm[::-1].copy()
            elif how == "shuffled":
                perm = rng.permutation(n)
            elif n > 1:
                perm[[n // 2 - 1, n - 1]] = perm[[n - 1, n // 2 - 1]]
            fr[h] = fr[h][perm]
            buf.frontier[h][:n] = torch.from_numpy(fr[h]).cuda()
            if h < L:
                nbr[h], cnt[h] = nbr[h][perm], cnt[h][perm]
                buf.nbr[h][:n] = torch.from_numpy(nbr[h]).cuda()
                buf.cnt[h][:n] = torch.from_numpy(cnt[h]).cuda()
        ctx.build_blocks(seeds_dev, fanouts, buf, out=blk)
        indptr, src, rows = blk.to_host()
        place = np.full(V, -1, np.int32)
        for h in range(L):
            place[fr[h + 1]] = np.arange(fr[h + 1].size, dtype=np.int32)
            assert (np.diff(indptr[h]) == cnt[h]).all() and indptr[h][0] == 0, f"{how} {reordered} indptr[{h}]"
            assert (src[h] == place[nbr[h][nbr[h] >= 0]]).all(), f"{how} {reordered} blk_src[{h}]"
        for h in range(L + 1):
            assert (gids[rows[h]] == fr[h]).all(), f"{how} {reordered} feat_row[{h}]"
    assert_blocks_equal(orc.sample_khop(seeds, fanouts, 21, blocks=True), (indptr, src, rows), "ascending")
    ctx.check()


@pytest.mark.parametrize("V", [1, 2, 70, 100_000, 3_000_000])
@pytest.mark.parametrize("where", ["first id", "last id", "both ends", "one run", "three runs", "all over"])
def test_blocks_of_frontiers_in_parts_of_the_range(V, where):
    """The frontiers' index covers the span of the list and leaves the blocks of its gaps unset."""
    from gpu_common import assert_batch_equal, assert_blocks_equal
    import oracle
    import paper_2305_16588_amd as lgp
    rng = np.random.default_rng(V)
    parts = {"first id": [(0, 1)], "last id": [(V - 1, V)], "both ends": [(0, 40), (V - 40, V)],
             "one run": [(V // 3, V // 3 + 900)], "three runs": [(V // 9, V // 9 + 5), (V // 2, V // 2 + 300), (V - 7, V)],
             "all over": [(0, V)]}[where]
    pool = np.unique(np.concatenate([np.arange(max(lo, 0), min(hi, V)) for lo, hi in parts]))
    d = rng.integers(0, 12, V)
    indptr = np.zeros(V + 1, np.int32)
    np.cumsum(d, out=indptr[1:])
    indices = pool[rng.integers(0, pool.size, int(indptr[-1]))].astype(np.int32)
    ctx = lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices))
    orc = oracle.Oracle(indptr, indices, None)
    seeds = np.sort(rng.permutation(V)[:700]).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    fanouts = (6, 3)
    buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=True)
    blk = lgp.BlockBuffers(buf)
    for rep in range(2):
        ctx.sample_khop(seeds_dev, fanouts, 50 + rep, out=buf)
        ctx.build_blocks(seeds_dev, fanouts, buf, out=blk)
        ref = orc.sample_khop(seeds, fanouts, 50 + rep, blocks=True)
        assert_batch_equal(ref, buf.to_host(seeds_dev), f"{V} {where}")
        assert_blocks_equal(ref, blk.to_host(), f"{V} {where}")
    ctx.check()


@pytest.mark.parametrize("V", [1 << 20, (1 << 23) + 1, (1 << 26) + 3, (1 << 28) + 3])
def test_compaction_that_counts_for_others(V):
    """With no polls a workgroup counts every share before its own whose status is not there yet: all three kinds of
    compaction, over byte maps, bit maps, wider shares and several passes, give the same lists."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    rng = np.random.default_rng(V + 2)
    gap = max(1, V // 2_000_000)
    sources = (V + gap - 1) // gap
    indptr = lgp.pinned_empty(V + 1, np.int32)
    d = np.zeros(V, np.int32)
    d[::gap] = 4
    indptr[0] = 0
    np.cumsum(d, out=indptr[1:])
    del d
    indices = lgp.pinned_copy((rng.integers(0, sources, int(indptr[-1])) * gap).astype(np.int32))
    indices[::5] = rng.integers(0, V, indices[::5].size)
    feats = lgp.pinned_empty((V, 1), np.float16)
    feats[:, 0] = np.arange(V, dtype=np.uint32).astype(np.uint16).view(np.float16)
    ctx, orc = lgp.Context(indptr, indices, feats), oracle.Oracle(indptr, indices, feats)
    seeds = (np.unique(rng.integers(0, sources, 9000)) * gap).astype(np.int32)
    seeds_dev = torch.from_numpy(seeds).cuda()
    fanouts = (3, 4)
    both = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=True)
    plain = lgp.SampleBuffers(V, seeds.size, fanouts)
    rows = torch.empty((both.gather_cap, 1), dtype=torch.float16, device="cuda")
    ref = orc.sample_khop(seeds, fanouts, 31)
    for polls in (0, 0, 1, 4096):
        ctx.set_wait_polls(polls)
        ctx.sample_khop(seeds_dev, fanouts, 31, out=plain)
        assert_batch_equal(ref, plain.to_host(seeds_dev), f"{V} {polls}")
        ctx.sample_khop(seeds_dev, fanouts, 31, out=both)
        assert_batch_equal(ref, both.to_host(seeds_dev), f"{V} {polls} with the last frontier")
        ctx.sample_extract(seeds_dev, fanouts, 31, both, rows)
        fr, _, _, listing = both.to_host(seeds_dev)
        assert (fr[2] == ref.frontier[2]).all() and listing.tolist() == ref.hop_order.tolist(), f"{V} {polls} listing"
        assert rows[:listing.size].cpu().numpy().tobytes() == orc.gather(listing).tobytes()
    with pytest.raises(lgp.LegionPrepError):
        ctx.set_wait_polls(-1)
    ctx.check()


def test_two_contexts_sample_side_by_side():
    """Compactions of two contexts wait for their own workgroups while both share the chip."""
    from gpu_common import assert_batch_equal
    import paper_2305_16588_amd as lgp
    V, fanouts = 1 << 20, (5, 4)
    sides = []
    for k in range(2):
        ctx, orc, rng = _workload(V, 6, 77 + k)
        seeds = np.unique(rng.integers(0, V, 6000)).astype(np.int32)
        sides.append((ctx, orc, seeds, torch.from_numpy(seeds).cuda(), torch.cuda.Stream(),
                      [lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=True) for _ in range(8)]))
    torch.cuda.synchronize()
    for i in range(8):
        for ctx, _, _, dev, stream, bufs in sides:
            ctx.sample_khop(dev, fanouts, 60 + i, out=bufs[i], stream=stream)
    torch.cuda.synchronize()
    for ctx, orc, seeds, dev, _, bufs in sides:
        for i in range(8):
            assert_batch_equal(orc.sample_khop(seeds, fanouts, 60 + i), bufs[i].to_host(dev), f"pass {i}")
        ctx.check()


@pytest.mark.parametrize("skip,V,n_edges,batch", [(0, 30_000, 240_000, 512), (1, 30_000, 240_001, 512),
                                                  (2, 30_000, 240_003, 512), (3, 30_000, 240_002, 512),
                                                  (1, 1_000_000, 6, 4096), (3, 1_000_000, 1, 4096), (0, 5000, 0, 64)])
def test_pre_sampling_with_staged_topology(skip, V, n_edges, batch):
    """Many mini-batches on a small graph, whose column ids are copied to HBM after the first one: arrays that begin at any
    multiple of four bytes and end inside a 16-byte chunk, arrays shorter than a chunk; and calls that read in place (few
    batches, no edges, after lgp_reserve)."""
    import oracle
    import paper_2305_16588_amd as lgp
    fanouts = (10, 10, 2)
    rng = np.random.default_rng(skip * 100_003 + n_edges)
    indptr = lgp.pinned_copy(np.concatenate([[0], np.sort(rng.integers(0, n_edges + 1, V - 1)), [n_edges]]).astype(np.int32))
    indices = lgp.pinned_empty(n_edges + 8, np.int32)[skip:skip + n_edges]
    indices[:] = rng.integers(0, V, n_edges)
    ctx, orc = lgp.Context(indptr, indices), oracle.Oracle(indptr, indices, None)
    tablet = rng.permutation(V).astype(np.int32)
    dev = torch.from_numpy(tablet).cuda()
    for max_batches in (-1, 2, 1, -1):
        ctx.build_hotness(dev, batch, fanouts, 5, max_batches=max_batches)
        rt, rf, _ = orc.build_hotness(tablet, batch, fanouts, 5, max_batches=max_batches)
        topo, feat = ctx.get_hotness()
        assert (topo == rt).all() and (feat == rf).all(), f"{max_batches} batches"
    ctx.reserve(batch, fanouts)                                  # nothing may be allocated now: rows are read in place
    ctx.build_hotness(dev, batch, fanouts, 5)
    topo, feat = ctx.get_hotness()
    assert (topo == rt).all() and (feat == rf).all()
    ctx.check()


@pytest.mark.parametrize("dim,dtype", [(7, np.float16), (8, np.float16), (9, np.float16), (25, np.float32), (50, np.float32),
                                       (75, np.float16), (100, np.float32), (128, np.float32), (131, np.float16),
                                       (260, np.float32)])
def test_hits_and_misses_side_by_side(dim, dtype):
    """Rows from both sources in one launch: every chunk width and lane-group size it is built for and the narrower rows it
    leaves to two launches, with one row cached, half of them and all but one, at list lengths around a workgroup pass and
    on both sides of the partition with one workgroup; timed apart (two launches) the bytes are the same."""
    import oracle
    import paper_2305_16588_amd as lgp
    V = 6000
    rng = np.random.default_rng(dim)
    indptr = lgp.pinned_copy(np.zeros(V + 1, np.int32))
    feats = lgp.pinned_empty((V, dim), dtype)
    feats[:] = rng.integers(-2000, 2000, (V, dim))
    ctx, orc = lgp.Context(indptr, np.empty(0, np.int32), feats), oracle.Oracle(indptr, np.empty(0, np.int32), feats)
    ctx.set_hotness(np.zeros(V, np.uint32), rng.permutation(V).astype(np.uint32))
    row = dim * np.dtype(dtype).itemsize
    for n_cached in (1, V // 2, V - 1):
        ctx.build_cache(0, n_cached * row)
        cached = np.zeros(V, bool)
        cached[ctx.get_cache(contents=False)[3]] = True
        assert cached.sum() == n_cached
        for n in (0, 1, 3, 64, 257, 4096, 4097, 12_000):
            ids = np.sort(rng.integers(0, V, n)).astype(np.int32) if n % 2 else rng.integers(0, V, n).astype(np.int32)
            dev = torch.from_numpy(ids).cuda()
            want = orc.gather(ids).tobytes()
            for mode in (0, 1):
                ctx.set_profiling(mode)
                out = torch.full((n + 1, dim), 7.0, dtype=ctx.feat_torch_dtype, device="cuda")
                stats = torch.full((2,), -1, dtype=torch.int32, device="cuda")
                ctx.gather_features(dev, out=out[:n], stats=stats)
                assert out[:n].cpu().numpy().tobytes() == want, f"{n_cached} cached, {n} ids, mode {mode}"
                assert (out[n] == 7.0).all() and stats.tolist() == [int(cached[ids].sum()), int((~cached[ids]).sum())]
    ctx.set_profiling(0)
    ctx.check()


@pytest.mark.parametrize("f", [1, 2, 3, 5, 7, 9, 15, 16, 17, 21, 22, 31, 32, 33, 63, 64])
def test_samples_of_rows_hardly_longer_than_the_fanout(f):
    """Rows of f - 1 to 2 f ids in turn, where most draws collide and chains of moved slots are long, at fan-outs around
    every number of vertices a wave takes; list lengths around a wave and a workgroup pass, and several passes."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    V = 9000
    d = (f - 1 + np.arange(V) % (f + 2)).astype(np.int64)
    indptr = np.concatenate([[0], np.cumsum(d)]).astype(np.int32)
    rng = np.random.default_rng(f)
    indices = rng.integers(0, V, int(indptr[-1])).astype(np.int32)
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices)), oracle.Oracle(indptr, indices, None)
    per_wave = 64 // f
    order = rng.permutation(V).astype(np.int32)
    for n in (1, per_wave, per_wave + 1, 4 * per_wave - 1, 4 * per_wave + 1, V):
        seeds = order[:n]
        dev = torch.from_numpy(seeds).cuda()
        buf = lgp.SampleBuffers(V, n, (f,))
        ctx.sample_khop(dev, (f,), 70 + n, out=buf)
        assert_batch_equal(orc.sample_khop(seeds, (f,), 70 + n), buf.to_host(dev), f"{n} seeds")
    ctx.check()


@pytest.mark.parametrize("gap", [1, 2, 31, 32, 33, 63, 64, 65, 66, 129])
@pytest.mark.parametrize("n", [1, 33, 64, 65, 96, 97, 1000])
def test_blocks_of_evenly_spaced_frontiers(gap, n):
    """Frontiers of n ids `gap` vertices apart: both kinds of index entries and the gap where they change over, blocks of 32
    vertices whose ids lie in one wave and in two; a second list has gaps in it."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_blocks_equal
    f, V = 8, max((n - 1) * gap + 1, 400)
    pool = V - 1 - np.arange(n)[::-1] * gap
    n_seeds = (n + f - 1) // f
    indptr = np.zeros(V + 1, np.int64)
    indptr[1:n_seeds + 1] = np.minimum(np.arange(1, n_seeds + 1) * f, n)
    indptr[n_seeds + 1:] = n
    for ids in (pool, np.where(np.arange(n) % 3 == 2, pool[0], pool)):
        indices = ids.astype(np.int32)
        ctx = lgp.Context(lgp.pinned_copy(indptr.astype(np.int32)), lgp.pinned_copy(indices))
        orc = oracle.Oracle(indptr.astype(np.int32), indices, None)
        seeds = np.arange(n_seeds, dtype=np.int32)
        dev = torch.from_numpy(seeds).cuda()
        buf = lgp.SampleBuffers(V, n_seeds, (f,), last_frontier=True)
        blk = lgp.BlockBuffers(buf)
        ctx.sample_khop(dev, (f,), 3, out=buf)
        ctx.build_blocks(dev, (f,), buf, out=blk)
        assert_blocks_equal(orc.sample_khop(seeds, (f,), 3, blocks=True), blk.to_host(), f"{gap} {n}")
        ctx.check()


@pytest.mark.parametrize("V", [(1 << 23) + 1, 1 << 24, (1 << 24) + 1])
def test_maps_laid_out_per_call(V):
    """Calls of many marks and of few in turn on graphs around the limits between which maps have room for both layouts, few of
    whose vertices have edges: every kind of compaction, and pre-sampling."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    rng = np.random.default_rng(V)
    sources = 20_000                                               # rows of 64 ids, the others are empty
    few = sources * 64
    indptr = np.zeros(V + 1, np.int32)
    indptr[1:sources + 1] = np.arange(1, sources + 1) * 64
    indptr[sources + 1:] = few
    indices = rng.integers(0, V, few).astype(np.int32)
    indices[::4] = rng.integers(0, sources, indices[::4].size)
    indices[:2] = [0, V - 1]
    # pretend edges behind the rows raise the mean degree, but not the marks to be expected
    more = lgp.pinned_empty(7 * V, np.int32)
    more[:few] = indices
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), more), oracle.Oracle(indptr, indices, None)
    order = np.concatenate([[0], 1 + rng.permutation(sources - 1)]).astype(np.int32)
    for n_seeds, fanouts in ((20_000, (8, 8, 8)), (300, (5, 3)), (20_000, (8, 8, 8)), (20_000, (2,))):
        seeds = order[:n_seeds]
        dev = torch.from_numpy(seeds).cuda()
        ref = orc.sample_khop(seeds, fanouts, 17)
        for last in (False, True):
            buf = lgp.SampleBuffers(V, n_seeds, fanouts, last_frontier=last)
            ctx.sample_khop(dev, fanouts, 17, out=buf)
            assert_batch_equal(ref, buf.to_host(dev), f"{n_seeds} {fanouts} {last}")
    tablet = torch.from_numpy(order).cuda()
    for fanouts in ((8, 8, 8), (3,)):
        ctx.build_hotness(tablet, 10_000, fanouts, 5)
        rt, rf, _ = orc.build_hotness(order, 10_000, fanouts, 5)
        topo, feat = ctx.get_hotness()
        assert (topo == rt).all() and (feat == rf).all()
    ctx.check()


@pytest.mark.parametrize("sources,reserve,copied", [(100_000, False, True), (2000, False, False), (100_000, True, False)])
def test_topology_is_copied_only_where_batches_read_it(sources, reserve, copied):
    """HBM that pre-sampling takes: all column ids where the first batch's reads say that a copy pays, and nothing where a
    few vertices own all edges, so that batches read far fewer rows than the mean degree suggests, or after lgp_reserve."""
    import ctypes
    import oracle
    import paper_2305_16588_amd as lgp
    V, batch, fanouts, degree = 100_000, 256, (8, 8), 4_000_000 // sources
    rng = np.random.default_rng(sources)
    order = rng.permutation(V)
    d = np.zeros(V, np.int64)
    d[order[:sources]] = degree
    indptr = np.concatenate([[0], np.cumsum(d)]).astype(np.int32)
    indices = order[rng.integers(sources, V, 4_000_000) if sources < V else rng.integers(0, V, 4_000_000)].astype(np.int32)
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices)), oracle.Oracle(indptr, indices, None)
    if reserve:
        ctx.reserve(batch, fanouts)
    hip = lgp.load_library()                                       # symbols of the runtime that the library is linked to
    used_high, pool, value = 8, ctypes.c_void_p(), ctypes.c_uint64(0)           # hipMemPoolAttrUsedMemHigh
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    tablet = rng.permutation(V).astype(np.int32)
    dev = torch.from_numpy(tablet).cuda()
    torch.cuda.synchronize()
    assert hip.hipMemPoolSetAttribute(pool, used_high, ctypes.byref(value)) == 0
    ctx.build_hotness(dev, batch, fanouts, 5)
    topo, feat = ctx.get_hotness()
    assert hip.hipMemPoolGetAttribute(pool, used_high, ctypes.byref(value)) == 0
    assert (value.value >= 4 * indices.size) if copied else value.value == 0, f"{value.value} bytes taken"
    rt, rf, _ = orc.build_hotness(tablet, batch, fanouts, 5)
    assert (topo == rt).all() and (feat == rf).all()
    ctx.check()


@pytest.mark.parametrize("f", [1, 3, 5, 8, 9, 16, 17, 21, 22, 32, 33, 64])
def test_samples_of_resident_and_host_topology(f):
    """Lanes of a vertex: as many as samples where all rows are in HBM (arrays there to begin with, or all cached), a power
    of two of them where some are read over PCIe."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    V, n = 5000, 700
    rng = np.random.default_rng(f)
    indptr = np.concatenate([[0], np.cumsum(rng.integers(0, 2 * f + 2, V))]).astype(np.int32)
    indices = rng.integers(0, V, int(indptr[-1])).astype(np.int32)
    orc = oracle.Oracle(indptr, indices, None)
    seeds = rng.permutation(V)[:n].astype(np.int32)
    dev = torch.from_numpy(seeds).cuda()
    hot = rng.integers(0, 9, V).astype(np.uint32)
    ref = orc.sample_khop(seeds, (f, 2), 41)
    for resident, budget in ((True, 0), (False, 0), (False, 2 * indices.size), (False, 1 << 40)):
        arrays = [torch.from_numpy(a).cuda() if resident else lgp.pinned_copy(a) for a in (indptr, indices)]
        ctx = lgp.Context(*arrays)
        ctx.set_hotness(hot, hot)
        ctx.build_cache(budget, 0)
        buf = lgp.SampleBuffers(V, n, (f, 2))
        ctx.sample_khop(dev, (f, 2), 41, out=buf)
        assert_batch_equal(ref, buf.to_host(dev), f"{resident} {budget}")
        ctx.check()


@pytest.mark.parametrize("row_bytes", [74, 500, 700, 2056])
def test_cached_rows_by_lane_groups_of_small_and_large_calls(row_bytes):
    """Calls on both sides of the size from which a narrower grid takes the rows (224 MiB of them), counts below the length
    of the list included."""
    import paper_2305_16588_amd as lgp
    V, most = 9000, (224 << 20) // row_bytes
    feats = torch.randint(-9, 9, (V, row_bytes // 2), dtype=torch.int16, device="cuda").view(torch.float16)
    ctx = lgp.Context(torch.zeros(V + 1, dtype=torch.int32, device="cuda"), np.empty(0, np.int32), feats)
    ctx.set_hotness(np.zeros(V, np.uint32), np.zeros(V, np.uint32))
    ctx.build_cache(0, V * row_bytes)
    ids = torch.randint(0, V, (most + 1500,), dtype=torch.int32, device="cuda")
    out = torch.empty((ids.numel(), row_bytes // 2), dtype=torch.float16, device="cuda")
    want = feats.view(torch.int16)
    for n in (ids.numel(), most + 1, most, 900, 0):
        out.view(torch.int16).fill_(99)
        ctx.gather_features(ids, n_dev=torch.tensor([n], dtype=torch.int32, device="cuda"), out=out)
        got = out.view(torch.int16)
        for lo in range(0, n, 1 << 18):                            # by parts: the reference is as large as the result
            hi = min(n, lo + (1 << 18))
            assert torch.equal(got[lo:hi], want[ids[lo:hi].long()]), f"{n} rows"
        assert bool((got[n:] == 99).all())
    ctx.check()


@pytest.mark.parametrize("V,n_seeds", [(146_000_000, 230_000), (146_000_000, 200_000), (100_000_000, 230_000)])
def test_blocks_of_sparse_frontiers_of_millions_of_ids(V, n_seeds):
    """More and fewer ids than the number from which blocks hold half as many, and a list whose blocks have bits: each
    position has to lead back to the id that was looked up."""
    import paper_2305_16588_amd as lgp
    f, gen = 10, torch.Generator(device="cuda").manual_seed(n_seeds)
    indptr = torch.full((V + 1,), n_seeds * f, dtype=torch.int32, device="cuda")
    indptr[:n_seeds + 1] = torch.arange(n_seeds + 1, dtype=torch.int32, device="cuda") * f
    indices = torch.randint(0, V, (n_seeds * f,), device="cuda", generator=gen, dtype=torch.int32)
    ctx = lgp.Context(indptr, indices)
    seeds = torch.arange(n_seeds, dtype=torch.int32, device="cuda")
    buf = lgp.SampleBuffers(V, n_seeds, (f,), last_frontier=True)
    blk = lgp.BlockBuffers(buf)
    ctx.sample_khop(seeds, (f,), 3, out=buf)
    ctx.build_blocks(seeds, (f,), buf, out=blk)
    ctx.check()
    n, sources = buf.n_frontier.tolist()
    assert n == n_seeds and sources == torch.unique(indices).numel()
    assert torch.equal(blk.blk_indptr[0], torch.arange(n + 1, dtype=torch.int64, device="cuda") * f)
    assert torch.equal(buf.frontier[1][blk.blk_src[0].long()], buf.nbr[0].flatten())
    rows = blk.feat_row[1][:sources].long()
    assert torch.equal(buf.gather_ids[rows], buf.frontier[1][:sources]) and torch.equal(buf.gather_ids[blk.feat_row[0].long()], seeds)


@pytest.mark.parametrize("row_bytes,skew", [(2046, 0), (2048, 0), (2048, 2), (2050, 2), (2570, 0), (4096, 4), (16_384, 0)])
def test_wide_rows_from_both_sources(row_bytes, skew):
    """Rows around the width from which hits beside misses are walked as runs of chunks, of whole lines and ragged, written
    to any even address; few misses, for which fewer workgroups take the hits, many, none and only misses, in lists of
    hardly any rows and of several passes."""
    import paper_2305_16588_amd as lgp
    V, dim = 40_000 if row_bytes < 4096 else 10_000, row_bytes // 2
    rng = np.random.default_rng(row_bytes + skew)
    feats = lgp.pinned_empty((V, dim), np.float16)
    feats.view(np.int16)[:] = np.arange(dim, dtype=np.int16) * np.int16(3) + np.arange(V, dtype=np.int32)[:, None].astype(np.int16)
    want = torch.from_numpy(feats.view(np.int16)).cuda()
    ctx = lgp.Context(lgp.pinned_copy(np.zeros(V + 1, np.int32)), np.empty(0, np.int32), feats)
    ctx.set_hotness(np.zeros(V, np.uint32), rng.permutation(V).astype(np.uint32))
    room = torch.empty(V * dim + 8, dtype=torch.int16, device="cuda")
    for n_cached in (1, V // 2, V - 60, V - 1):
        ctx.build_cache(0, n_cached * row_bytes)
        cached = np.zeros(V, bool)
        cached[ctx.get_cache(contents=False)[3]] = True
        everything = rng.permutation(V).astype(np.int32)
        for ids in (everything if n_cached > V // 2 else everything[:3000], everything[:5], everything[:0],
                    np.flatnonzero(cached)[:700].astype(np.int32), np.flatnonzero(~cached)[:700].astype(np.int32)):
            room.fill_(99)
            out = room[skew // 2:skew // 2 + ids.size * dim].view(ids.size, dim)
            stats = torch.full((2,), -1, dtype=torch.int32, device="cuda")
            ctx.gather_features(torch.from_numpy(ids).cuda(), out=out.view(torch.float16), stats=stats)
            assert torch.equal(out, want[torch.from_numpy(ids).cuda().long()]), f"{n_cached} cached, {ids.size} ids"
            assert bool((room[skew // 2 + ids.size * dim:] == 99).all()) and bool((room[:skew // 2] == 99).all())
            assert stats.tolist() == [int(cached[ids].sum()), int((~cached[ids]).sum())]
    ctx.check()


@pytest.mark.parametrize("V,share", [((1 << 23) + 1, 1.0), (1 << 24, 1.0), ((1 << 24) + 1, 1.0), ((1 << 23) + 1, 0.3)])
def test_maps_of_calls_with_many_marks_and_few(V, share):
    """Edges at all vertices or at a part of them, degrees below, at and beyond the fan-outs: calls that mark bytes between the
    limits and calls that mark bits in turn on one context, the pipeline inside a batch (always bits) between them."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    rng = np.random.default_rng(V + int(10 * share))
    degrees = rng.integers(1, 8, V, dtype=np.int32)
    degrees[rng.random(V) >= share] = 0
    indptr = np.concatenate([[0], np.cumsum(degrees)]).astype(np.int32)
    indices = rng.integers(0, V, int(indptr[-1]), dtype=np.int32)
    indices[:2] = [0, V - 1]
    feats = lgp.pinned_empty((V, 8), np.float16)
    feats.view(np.int16)[:] = np.arange(V, dtype=np.int32)[:, None].astype(np.int16)
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), lgp.pinned_copy(indices), feats), oracle.Oracle(indptr, indices, feats)
    order = np.concatenate([[0, V - 1], 1 + rng.permutation(V - 2)[:120_000]]).astype(np.int32)
    for n_seeds, fanouts in ((120_000, (6, 5)), (300, (5, 3)), (120_000, (6, 5)), (2000, (7,))):
        seeds = order[:n_seeds]
        dev = torch.from_numpy(seeds).cuda()
        ref = orc.sample_khop(seeds, fanouts, 19)
        for last in (False, True):
            buf = lgp.SampleBuffers(V, n_seeds, fanouts, last_frontier=last)
            ctx.sample_khop(dev, fanouts, 19, out=buf)
            assert_batch_equal(ref, buf.to_host(dev), f"{n_seeds} {fanouts} {last}")
            rows = torch.empty((buf.gather_cap, 8), dtype=torch.float16, device="cuda")
            ctx.sample_extract(dev, fanouts, 19, buf, rows)
            n = int(buf.n_gather)
            listed = buf.gather_ids[:n].cpu().numpy()
            assert np.array_equal(np.sort(listed), np.sort(ref.gather_ids)), f"{n_seeds} {fanouts} {last}"
            assert np.array_equal(rows[:n].cpu().numpy().view(np.int16), feats.view(np.int16)[listed])
    tablet = torch.from_numpy(order).cuda()
    ctx.build_hotness(tablet, 60_000, (6, 5), 5)
    rt, rf, _ = orc.build_hotness(order, 60_000, (6, 5), 5)
    topo, feat = ctx.get_hotness()
    assert (topo == rt).all() and (feat == rf).all()
    ctx.check()


@pytest.mark.parametrize("V,deg", [((9 << 20) + 1, 8), (1 << 24, 8), ((1 << 24) + 1, 8), (1 << 25, 8), ((1 << 25) + 1, 8), ((1 << 26) + 1, 4), ((1 << 27) + 1, 2), (1 << 28, 0)])
def test_samples_sorted_into_bins(V, deg):
    """Calls with many samples on a large graph sort them by ranges of vertices into segments of limited room.  Samples spread over the
    graph, at the edges of the ranges, in one range and on one vertex (segments overflow), with polls and without, with more seeds and
    more inner frontiers than the kernel loads ahead, and calls that mark maps between them; a caller who uses one buffer for two
    frontiers gets the marks in maps, and so does a graph that is crowded all over, where the others are so around the seeds only."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    rng = np.random.default_rng(V)
    gen = torch.Generator(device="cuda").manual_seed(V)
    gap = 1 if deg else 61                                     # every vertex has `deg` edges, or every 61st has 7
    deg = deg or 7
    indptr = lgp.pinned_empty(V + 1, np.int32)
    rows = (V + gap - 1) // gap
    np.multiply((np.arange(V + 1, dtype=np.int64) + gap - 1) // gap, deg, out=indptr, casting="unsafe")
    step = 1 << 17
    edges = torch.arange(0, V, step, device="cuda")
    edges = torch.unique(torch.cat([edges, edges[1:] - 1, torch.tensor([V - 1], device="cuda")]))

    def draw(kind, n):
        r = torch.randint(0, V, (n,), generator=gen, device="cuda")
        if kind == "spread":
            return r // gap * gap
        if kind == "edges":
            return edges[r % edges.numel()]
        return r % step // gap * gap if kind == "crowd" else torch.full((n,), V - 1, device="cuda")

    indices = lgp.pinned_empty(rows * deg, np.int32)
    all_lists = (("spread", "edges", "crowd", "one"), ("crowd",), ("one",)) if V <= 1 << 25 else (("spread", "edges", "spread", "one"),)
    for lists, crowded in [(lists, rows // 32) for lists in all_lists] + [(("crowd",), rows)] * (V <= 1 << 25):
        part = 1 << 24
        for lo in range(0, indices.size, part):
            n = min(part, indices.size - lo)
            pick = torch.randint(0, len(lists), (n,), generator=gen, device="cuda")
            got = torch.zeros(n, dtype=torch.int64, device="cuda")
            for k, kind in enumerate(lists):
                got = torch.where(pick == k, draw(kind, n), got)
            if lo + n > crowded * deg:
                at = max(crowded * deg - lo, 0)
                got[at:] = draw("spread", n - at)
            torch.from_numpy(indices[lo:lo + n]).copy_(got.to(torch.int32))
        ctx, orc = lgp.Context(indptr, torch.from_numpy(indices).cuda()), oracle.Oracle(indptr, indices, None)
        order = (rng.permutation(min(crowded, 1 << 20))[:140_000] * gap).astype(np.int32)
        for n_seeds, fanouts in ((30_000, (7, 6, 3)), (1, (9, 9, 2)), (60_001, (2, 2, 2, 2, 2)), (8192, (5,)), (131_073, (3, 2))):
            seeds = order[:n_seeds]
            dev = torch.from_numpy(seeds).cuda()
            ref = orc.sample_khop(seeds, fanouts, 23)
            for last in (False, True):
                buf = lgp.SampleBuffers(V, seeds.size, fanouts, last_frontier=last)
                for polls in (4096, 0, 4096):
                    ctx.set_wait_polls(polls)
                    ctx.sample_khop(dev, fanouts, 23, out=buf)
                    assert (ctx.sample_marks() == 0) == (crowded < rows and (n_seeds in (30_000, 60_001) or (V == 1 << 28 and n_seeds < 131_073)))
                    assert_batch_equal(ref, buf.to_host(dev), f"{V} {lists} {n_seeds} {fanouts} {polls} {last}")
        seeds = order[:40_000]
        dev = torch.from_numpy(seeds).cuda()
        ref = orc.sample_khop(seeds, (4, 4, 4), 29)
        buf = lgp.SampleBuffers(V, seeds.size, (4, 4, 4))
        buf.c_struct.frontier[1] = buf.frontier[2].data_ptr()
        ctx.sample_khop(dev, (4, 4, 4), 29, out=buf)
        assert ctx.sample_marks() in (1, 8)
        fr, nbr, _, ids = buf.to_host(dev)
        assert (ids == ref.gather_ids).all() and (fr[2] == ref.frontier[2]).all()
        assert all((nbr[h] == ref.nbr[h]).all() for h in range(3))
        ctx.check()
        bad = seeds.copy()
        bad[[3, 77]] = [-1, V]
        ctx.sample_khop(torch.from_numpy(bad).cuda(), (4, 4, 4), 29)
        with pytest.raises(lgp.LegionPrepError):
            ctx.check()
        ctx.sample_khop(dev, (4, 4, 4), 29, out=buf)
        assert (buf.to_host(dev)[3] == ref.gather_ids).all()
        ctx.check()
        del ctx, orc


@pytest.mark.parametrize("V", [(9 << 20) + 1, (5 << 25) + 1, 1 << 28])
def test_no_seeds_on_a_large_graph(V):
    """An empty batch is valid on every graph, with null inner frontiers as empty buffers have them: every size is written as 0.  From
    5 * 2^25 vertices on no call has too few samples for the bins, so there this one would be the only one that they hold nothing of."""
    import paper_2305_16588_amd as lgp
    gap = 61                                                   # every 61st vertex has 7 edges
    indptr = torch.arange(gap - 1, V + gap, device="cuda").div_(gap, rounding_mode="floor").mul_(7).to(torch.int32)
    gen = torch.Generator(device="cuda").manual_seed(V)
    ctx = lgp.Context(indptr, torch.randint(0, V, (int(indptr[-1]),), generator=gen, device="cuda", dtype=torch.int32))
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    some = torch.arange(0, 61 * 8192, 61, device="cuda", dtype=torch.int32)
    for fanouts in ((25, 10), (5,), (3, 2, 2, 4)):
        for last in (False, True):
            buf = lgp.SampleBuffers(V, 0, fanouts, last_frontier=last)
            assert all(f.data_ptr() == 0 for f in buf.frontier[1:])
            buf.n_frontier.fill_(77)
            buf.n_gather.fill_(77)
            ctx.sample_khop(none, fanouts, 3, out=buf)
            assert ctx.sample_marks() in (1, 8)
            assert buf.n_gather.item() == 0 and buf.n_frontier.tolist() == [0] * len(fanouts) + [77]
            # maps and segments are in order for the calls around it
            got, again = (ctx.sample_khop(some, fanouts, 3) for _ in range(2))
            assert (ctx.sample_marks() == 0) == (V > 5 << 25)
            assert got.n_gather.item() == again.n_gather.item() > 8192
            n = int(got.n_gather)
            assert torch.equal(got.gather_ids[:n], again.gather_ids[:n]) and torch.equal(got.gather_ids[:n], got.gather_ids[:n].unique())
    # one sample per seed is in no bin from 2^16 seeds on
    many = torch.arange(0, 61 * (1 << 16), 61, device="cuda", dtype=torch.int32)
    for seeds, fanouts, binned in ((many, (1,), False), (many[1:], (1,), True), (many, (2,), True), (many, (1, 1), True)):
        got = ctx.sample_khop(seeds, fanouts, 5)
        assert (ctx.sample_marks() == 0) == (binned and V > 5 << 25)
        rows = [got.nbr[h][:int(got.n_frontier[h])].flatten() for h in range(len(fanouts))]
        ids = torch.cat([seeds, *rows])
        assert torch.equal(got.gather_ids[:int(got.n_gather)], ids[ids >= 0].unique())
    ctx.check()


def test_invalid_seeds_of_binned_calls():
    """Seeds without a row, or with one that makes no sense, are no members of the batch; a row of 2^24 vertices and more, whose degree
    the row table does not hold, is like any other.  Which seeds count does not depend on the context's error word: while batches
    run, a gather of invalid ids on another stream sets it and a check there clears it."""
    import oracle
    import paper_2305_16588_amd as lgp
    V, deg, odd, long_row, more = (9 << 20) + 1, 8, 4_000_000, 6_000_000, 17_000_000
    indptr = np.arange(V + 1, dtype=np.int32) * deg
    indptr[long_row + 1:] += more
    indptr[odd + 1] -= deg + 5                                 # of `odd` the offsets descend
    gen = torch.Generator(device="cuda").manual_seed(3)
    indices = torch.randint(0, V, (int(indptr[-1]),), generator=gen, device="cuda", dtype=torch.int32)
    indices[(indices == odd)] = 7
    features = torch.zeros((V, 1), dtype=torch.float16, device="cuda")
    ctx = lgp.Context(lgp.pinned_copy(indptr), indices, features)
    rng = np.random.default_rng(5)
    fanouts = (7, 6, 3)
    good = rng.permutation(V)[:12_001].astype(np.int32)
    good = good[good != odd]
    good[[17, 11_000]] = [long_row, odd + 1]
    good = good[np.sort(np.unique(good, return_index=True)[1])]
    ref = oracle.Oracle(indptr, indices.cpu().numpy(), None).sample_khop(good, fanouts, 31)
    at = np.array([0, 5, 6, 4099, 9_000, good.size])
    mixed = np.insert(good, at, np.array([-1, V, odd, odd, -(2 ** 31), 2 ** 31 - 1], dtype=np.int32))
    valid = (mixed >= 0) & (mixed < V) & (mixed != odd)
    assert (mixed[valid] == good).all()

    def check(buf, dev, rows):
        fr, nbr, cnt, ids = buf.to_host(dev)
        assert ids.shape == ref.gather_ids.shape and (ids == ref.gather_ids).all()
        assert all(fr[h].shape == ref.frontier[h].shape and (fr[h] == ref.frontier[h]).all() for h in (1, 2))
        assert (nbr[0][rows] == ref.nbr[0]).all() and (nbr[0][~rows] == -1).all() and (cnt[0][~rows] == 0).all()
        assert all((nbr[h] == ref.nbr[h]).all() and (cnt[h] == ref.cnt[h]).all() for h in (1, 2))

    torch.cuda.synchronize()
    beside, sampler = torch.cuda.Stream(), torch.cuda.Stream()
    invalid = torch.full((1000,), -1, dtype=torch.int32, device="cuda")
    out = torch.empty((1000, 1), dtype=torch.float16, device="cuda")
    for seeds, rows in ((mixed, valid), (good, np.ones(good.size, bool))):
        dev = torch.from_numpy(seeds).cuda()
        for polls in (4096, 0):
            ctx.set_wait_polls(polls)
            buf = ctx.sample_khop(dev, fanouts, 31)
            assert ctx.sample_marks() == 0
            check(buf, dev, rows)
            if not rows.all():
                with pytest.raises(lgp.LegionPrepError):
                    ctx.check()
            ctx.check()
        ctx.set_wait_polls(4096)
        bufs = [lgp.SampleBuffers(V, seeds.size, fanouts) for _ in range(12)]
        torch.cuda.synchronize()
        for buf in bufs:
            ctx.sample_khop(dev, fanouts, 31, out=buf, stream=sampler)
        for _ in range(12):
            ctx.gather_features(invalid, out=out, stream=beside)
            with pytest.raises(lgp.LegionPrepError):
                ctx.check(beside)
        torch.cuda.synchronize()
        for buf in bufs:
            check(buf, dev, rows)
        try:
            ctx.check()
        except lgp.LegionPrepError:
            assert not rows.all()


def test_bins_while_their_segments_hold_a_call():
    """Up to 2^24 vertices: a hop that promises more than the segments of one workgroup per CU hold takes two per CU, and a call with
    one that promises more than those hold marks bytes, as does a single hop."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    V, deg = (9 << 20) + 1, 16
    gen = torch.Generator(device="cuda").manual_seed(9)
    indptr = np.arange(V + 1, dtype=np.int32) * deg
    indices = torch.randint(0, V, (V * deg,), generator=gen, device="cuda", dtype=torch.int32)
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), indices), oracle.Oracle(indptr, indices.cpu().numpy(), None)
    seeds = np.random.default_rng(1).permutation(V)[:60_000].astype(np.int32)
    # samples of the last hop over the room of two workgroups per CU (145 bins * 512 * 127): 0.7, 0.9, 1.1, 1.9, 0.7
    for n_seeds, fanouts, marks in ((30_000, (8, 8, 4), 0), (30_000, (8, 8, 5), 0), (40_000, (8, 8, 5), 0), (40_000, (8, 8, 8), 8),
                                    (60_000, (16,), 8), (30_000, (8, 8, 4), 0)):
        dev = torch.from_numpy(seeds[:n_seeds]).cuda()
        buf = ctx.sample_khop(dev, fanouts, 37)
        assert ctx.sample_marks() == marks, f"{n_seeds} {fanouts}"
        assert_batch_equal(orc.sample_khop(seeds[:n_seeds], fanouts, 37), buf.to_host(dev), f"{n_seeds} {fanouts}")
    ctx.check()


def test_segments_are_held_where_calls_use_them():
    """The room for binned samples is taken when no row crosses PCIe any more, and never on a graph without edges or with crowded column
    ids; the figure for the caller's budget has it in either case."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    V, deg = (9 << 20) + 1, 8
    words = 145 * 512 * 128 + 256 + 8 * 257 + 1                # 145 bins of 512 segments; flags, bounds of eight hops, one word
    gen = torch.Generator(device="cuda").manual_seed(2)
    indptr = lgp.pinned_copy(np.arange(V + 1, dtype=np.int32) * deg)
    spread = torch.randint(0, V, (V * deg,), generator=gen, device="cuda", dtype=torch.int32)
    host = lgp.pinned_copy(spread.cpu().numpy())
    none = lgp.pinned_copy(np.zeros(V + 1, np.int32))
    fanouts = (7, 6, 3)

    def made(*graph):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx = lgp.Context(*graph)
        return ctx, before - torch.cuda.mem_get_info()[0], ctx.workspace_bytes(1, fanouts)[0]

    keep, _, _ = made(indptr, spread)                          # what the first context of a process takes beside its own
    ctx_none, used_none, fixed_none = made(none, host[:0])
    ctx_crowd, used_crowd, fixed_crowd = made(indptr, spread % (1 << 16))
    ctx_dev, used_dev, fixed_dev = made(indptr, spread)
    ctx, used, fixed = made(indptr, host)
    assert fixed_none == fixed_crowd == fixed - words * 4 and fixed_dev == fixed
    assert abs(used_none - used) <= 4 << 20 and abs(used_crowd - used) <= 4 << 20
    assert abs(used_dev - used - words * 4) <= 4 << 20
    seeds = np.random.default_rng(1).permutation(V)[:20_000].astype(np.int32)
    dev = torch.from_numpy(seeds).cuda()
    ref = oracle.Oracle(indptr, host, None).sample_khop(seeds, fanouts, 41)
    ctx.set_hotness(np.ones(V, np.uint32), np.ones(V, np.uint32))
    half = V // 2 * (4 * deg + 8)
    for budget, binned in ((0, False), (half, False), (4 * half, True), (half, False), (4 * half, True)):
        assert (ctx.build_cache(budget, 0).n_topo == V) == binned
        assert_batch_equal(ref, ctx.sample_khop(dev, fanouts, 41).to_host(dev), f"{budget}")
        assert (ctx.sample_marks() == 0) == binned
    assert_batch_equal(ref, ctx_dev.sample_khop(dev, fanouts, 41).to_host(dev), "in HBM")
    assert ctx_dev.sample_marks() == 0
    hot = torch.ones((2, V), dtype=torch.int32, device="cuda")
    other, _, _ = made(indptr, host)
    assert sum(p.n_topo for p in other.build_clique_cache(hot, hot, 4 * half, 0)) == V
    assert_batch_equal(ref, other.sample_khop(dev, fanouts, 41).to_host(dev), "clique")
    assert other.sample_marks() == 0
    for c in (keep, ctx_none, ctx_crowd, ctx_dev, ctx, other):
        c.check()


@pytest.mark.parametrize("V", [(9 << 20) + 1, (1 << 25) + 1])
def test_binned_calls_from_a_graph_and_from_any_address(V):
    """Binned calls captured once and replayed on other seeds, invalid ones among them, with calls made directly between the replays; and
    seed lists that begin at any multiple of four bytes and end at any remainder of four seeds."""
    import oracle
    import paper_2305_16588_amd as lgp
    from gpu_common import assert_batch_equal
    deg, fanouts = 8, (7, 6, 3)
    gen = torch.Generator(device="cuda").manual_seed(V)
    indptr = np.arange(V + 1, dtype=np.int32) * deg
    indices = torch.randint(0, V, (V * deg,), generator=gen, device="cuda", dtype=torch.int32)
    ctx, orc = lgp.Context(lgp.pinned_copy(indptr), indices), oracle.Oracle(indptr, indices.cpu().numpy(), None)
    perm = np.random.default_rng(V).permutation(V)[:40_000].astype(np.int32)
    room = torch.from_numpy(perm).cuda()
    for shift, n in ((0, 20_001), (1, 20_002), (2, 20_003), (3, 20_000), (1, 8191), (3, 8194)):
        buf = ctx.sample_khop(room[shift:shift + n], (7, 6, 6), 43)
        assert ctx.sample_marks() == 0
        assert_batch_equal(orc.sample_khop(perm[shift:shift + n], (7, 6, 6), 43), buf.to_host(room[shift:shift + n]), f"{shift} {n}")

    n = 20_000
    bad = perm[n:].copy()
    bad[[0, 7777, n - 1]] = [-1, V, -7]
    lists = [perm[:n], perm[n:], bad]
    refs = [orc.sample_khop(ids[(ids >= 0) & (ids < V)], fanouts, 47) for ids in lists]
    devs = [torch.from_numpy(ids).cuda() for ids in lists]
    hold = devs[0].clone()
    out = lgp.SampleBuffers(V, n, fanouts, last_frontier=True)
    direct = lgp.SampleBuffers(V, n, fanouts)
    ctx.sample_khop(hold, fanouts, 47, out=out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.sample_khop(hold, fanouts, 47, out=out)
    assert ctx.sample_marks() == 0

    def check(buf, k):
        fr, nbr, cnt, ids = buf.to_host(devs[k])
        rows = (lists[k] >= 0) & (lists[k] < V)
        assert ids.shape == refs[k].gather_ids.shape and (ids == refs[k].gather_ids).all(), f"list {k}"
        for h in range(1, len(fr)):
            assert fr[h].shape == refs[k].frontier[h].shape and (fr[h] == refs[k].frontier[h]).all(), f"list {k}, frontier {h}"
        assert (nbr[0][rows] == refs[k].nbr[0]).all() and (cnt[0][rows] == refs[k].cnt[0]).all(), f"list {k}"
        assert all((nbr[h] == refs[k].nbr[h]).all() and (cnt[h] == refs[k].cnt[h]).all() for h in (1, 2)), f"list {k}"

    for k, other in ((1, 0), (0, 1), (2, 0), (1, 2), (2, 2), (0, 0)):
        hold.copy_(devs[k])
        graph.replay()
        torch.cuda.synchronize()
        ctx.sample_khop(devs[other], fanouts, 47, out=direct)
        torch.cuda.synchronize()
        check(out, k)
        check(direct, other)
        try:
            ctx.check()
        except lgp.LegionPrepError:
            assert 2 in (k, other)
        else:
            assert 2 not in (k, other)

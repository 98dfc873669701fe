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

"""GPU parity: the HIP library, called through the C ABI, against the CPU oracle.

Integer outputs (cache list, bitmap, draw count, block CSRs, src lists,
eligible counts, gathered rows) must be bit-exact; fp32 weights within 1e-5
relative; aggregates within 1e-5 of (1/n_v) * sum |w_e x_e| per element.
"""
import functools

import numpy as np
import pytest
import torch

import oracle
from conftest import random_symmetric_csr
from paper_2106_06150_amd import synth

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2106_06150_amd import binding as B
    from gpu_harness import GpuGns, full_parity, compare_cache, compare_blocks, AGG_RTOL

U, C, CF = 0, 1, 2          # UNIFORM, CACHE_ONLY, CACHE_FIRST


def _small(n=3000, avg=14, seed=3, hub=1):
    ip, ix = random_symmetric_csr(n, avg, np.random.default_rng(seed), hub_boost=hub)
    return torch.from_numpy(ip), torch.from_numpy(ix)


def _feat(n, F, seed=0):
    g = torch.Generator().manual_seed(seed)
    return torch.randn((n, F), dtype=torch.float32, generator=g)


@pytest.mark.parametrize("flag_mode", [0, 1])
@pytest.mark.parametrize("offsets", [torch.int32, torch.int64])
@pytest.mark.parametrize("fanouts,policies", [((10, 5), (U, C)), ((15, 10, 5), (U, U, C)), ((3, 2, 1), (C, C, C)),
                                              ((4, 4), (U, U)), ((20, 17), (U, C)), ((6, 12), (U, C)),
                                              ((15, 10, 5), (CF, CF, C)), ((6, 9), (CF, CF)), ((20, 40), (U, CF))])
def test_small_graph_parity(offsets, fanouts, policies, flag_mode):
    ip, ix = _small()
    n = ip.numel() - 1
    feat = _feat(n, 64)
    gns = GpuGns(ip.to(offsets), ix, feat, fanouts=fanouts, policies=policies, cache_size=300, max_seeds=200,
                 flag_mode=flag_mode)
    try:
        for trial in range(3):
            seeds = synth.uniform_seed_batch(n, 200 - 37 * trial, 100 + trial)
            full_parity(gns, cache_seed=9, epoch=trial, batch_seed=1000 + trial, seeds=seeds)
    finally:
        gns.close()


def _marked_by_slots(gns):
    """Whether the context marks its input layer's new nodes by slots of the cache: its table of 1/p^C has 8 bytes a node then, and
    the same context with an input layer that is not from the cache only 4."""
    other = B.make_config(gns.fanouts, gns.policies[:-1] + [CF], gns.cache_size, gns.config.max_seeds, gns.wmode, gns.config.flag_mode)
    return B.gns_workspace_bytes(gns.graph, gns.config) > B.gns_workspace_bytes(gns.graph, other)


@functools.lru_cache(maxsize=None)
def _graph_of_150k():
    return _small(n=150_000, avg=20, seed=150)


@pytest.mark.parametrize("n,avg,cache,fanouts,seeds,tile_words,by_slot", [
    (3000, 9, 64, (3, 9), 257, 0, True), (3000, 9, 65, (4, 4, 8), 256, 0, True), (4000, 9, 3000, (5, 17), 700, 0, True),
    (4000, 9, 3900, (2, 64), 1100, 0, True), (90_000, 9, 65_536, (12, 5), 1500, 0, True), (90_000, 9, 65_537, (12, 5), 1500, 0, True),
    (150_000, 20, 140_000, (16, 5), 400, 0, True), (150_000, 20, 140_000, (16, 20), 400, 512, True), (150_000, 9, 140_000, (16, 5), 400, 0, False)])
def test_input_layer_marked_by_slots(n, avg, cache, fanouts, seeds, tile_words, by_slot, monkeypatch):
    """Input layers from the cache only on the induced subgraph, whose new nodes are marked by their slots of the cache: caches up to
    what is finished in one launch and beyond (tiles of slots of the smallest and of the largest length), last words of marks that are
    full and not, rows around whole blocks, more slots a row than a thread has on its way; mini-batches one after the other, whose
    marks are cleared in between, and a second cache, whose structures lie elsewhere.  The last one has no place for the marks."""
    if tile_words:
        monkeypatch.setenv("GNS_MARK_TILE_WORDS", str(tile_words))
    ip, ix = _small(n=n, avg=avg, seed=n)
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=(U,) * (len(fanouts) - 1) + (C,), cache_size=cache, max_seeds=seeds, flag_mode=1)
    try:
        assert _marked_by_slots(gns) == by_slot
        for trial in range(3):
            batch = synth.uniform_seed_batch(n, seeds - 75 * trial, trial)
            full_parity(gns, cache_seed=9, epoch=trial // 2, batch_seed=50 + trial, seeds=batch)
    finally:
        gns.close()


@pytest.mark.parametrize("spins", ["256", "0"])
@pytest.mark.parametrize("tile_words", [64, 128, 256, 512])
def test_group_marked_by_slots_of_a_large_cache(tile_words, spins, monkeypatch):
    """Groups (the created context and forks of it) whose marks by slot are finished tile by tile, with tiles of 4096, 8192, 16,384 and 32,768
    slots, and with the counts of other tiles taken from the marks; a fork on its own; the fixed scratch; a second cache."""
    monkeypatch.setenv("GNS_MARK_TILE_WORDS", str(tile_words))
    monkeypatch.setenv("GNS_UNION_SPINS", spins)
    ip, ix = _graph_of_150k()
    n, cache, fanouts, policies, count = ip.numel() - 1, 140_000, (12, 16, 5), (U, CF, C), 3
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=cache, max_seeds=150, flag_mode=1)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        assert _marked_by_slots(gns)
        for epoch in range(2):
            B.gns_sample_cache(gns.ctx, 48, epoch)
            bitmap = oracle.sample_cache(ip.numpy(), 48, epoch, cache)[1]
            batches = [synth.uniform_seed_batch(n, 150 - 40 * b, 10 * epoch + b) for b in range(count)]
            refs = [oracle.sample_blocks(ip.numpy(), ix.numpy(), bitmap, cache, 70 + b, batches[b].numpy(), list(fanouts), list(policies))
                    for b in range(count)]
            on_gpu = [b.cuda() for b in batches]
            for _ in range(2):
                call.sample([70 + b for b in range(count)], on_gpu)
                call.wait()
                for b in range(count):
                    compare_blocks([bufs[b].views(j) for j in range(3)], refs[b])
            B.gns_sample_blocks(ctxs[2], 71, on_gpu[1], bufs[2].array)
            compare_blocks([bufs[2].views(j) for j in range(3)], refs[1])
            B.gns_sample_blocks_static(ctxs[1], 72, on_gpu[2], bufs[1].array)
            compare_blocks([bufs[1].views(j) for j in range(3)], refs[2])
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("flag", [2, -1, 64, -2 ** 31])
def test_any_flag_but_zero_means_64_bit_offsets(flag, monkeypatch):
    """gns_graph.indptr_is_i64 comes from a C caller as it pleases; the union step's reads of new nodes' extents go by it without a branch."""
    make_graph = B.make_graph

    def flagged(*args):
        g = make_graph(*args)
        g.indptr_is_i64 = flag
        return g

    monkeypatch.setattr(B, "make_graph", flagged)
    ip, ix = _small()
    for flag_mode in (0, 1):
        gns = GpuGns(ip.to(torch.int64), ix, None, fanouts=(9, 4, 3), policies=(U, U, C), cache_size=300, max_seeds=400, flag_mode=flag_mode)
        try:
            full_parity(gns, cache_seed=9, epoch=0, batch_seed=5, seeds=synth.uniform_seed_batch(ip.numel() - 1, 400, 6))
        finally:
            gns.close()


@pytest.mark.parametrize("cache", [60_000, 140_000])
@pytest.mark.parametrize("fanouts", [(16, 8), (17, 5), (5, 5, 5)])
@pytest.mark.parametrize("count", [1, 3])
def test_few_seeds_and_a_large_cache(cache, fanouts, count):
    """Mini-batches whose seeds take fewer blocks of the first launch (either kind of it) than clearing the marks by slot does, one after
    the other: what the one before marked is gone."""
    ip, ix = _graph_of_150k()
    n = ip.numel() - 1
    L = len(fanouts)
    policies = (U,) * (L - 1) + (C,)
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=cache, max_seeds=64, flag_mode=1)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        assert _marked_by_slots(gns)
        B.gns_sample_cache(gns.ctx, 47, 0)
        bitmap = oracle.sample_cache(ip.numpy(), 47, 0, cache)[1]
        for rnd in range(3):
            seeds = [synth.uniform_seed_batch(n, 64 - b, 10 * rnd + b).cuda() for b in range(count)]
            call.sample([90 * rnd + b for b in range(count)], seeds)
            call.wait()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), bitmap, cache, 90 * rnd + b, seeds[b].cpu().numpy(), list(fanouts), list(policies))
                compare_blocks([bufs[b].views(j) for j in range(L)], ref)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("F", [1, 3, 4, 32, 64, 96, 100, 128, 256, 260, 1024])
def test_feature_widths_and_host_store(F):
    ip, ix = _small(n=1500)
    n = ip.numel() - 1
    feat = _feat(n, F, seed=F)
    for on_host in (False, True):
        gns = GpuGns(ip, ix, feat, fanouts=(6, 4), policies=(U, C), cache_size=150, max_seeds=64, feat_on_host=on_host)
        try:
            seeds = synth.uniform_seed_batch(n, 64, 5)
            full_parity(gns, cache_seed=1, epoch=0, batch_seed=77, seeds=seeds)
        finally:
            gns.close()


@pytest.mark.parametrize("F,count,on_host", [(1, 700, False), (3, 700, False), (4, 600_000, False), (5, 700, False), (17, 90_000, False),
                                             (66, 700, True), (100, 700, False), (130, 700, False), (255, 5_000, True), (257, 700, False), (300, 700, False)])
def test_gather_of_any_list(F, count, on_host):
    """gns_gather_features alone on a list that no sampler made: cached and other nodes, repeated ones, ids outside the graph
    (rows of zeros); widths around multiples of four and of the lanes per row, an output that is aligned to four bytes only,
    more rows than a wave looks up at once, and nothing written past the last row."""
    ip, ix = _small()
    n = ip.numel() - 1
    feat = _feat(n, F, seed=F)
    gns = GpuGns(ip, ix, feat, fanouts=(4, 3), policies=(U, C), cache_size=n // 4, max_seeds=8, feat_on_host=on_host)
    try:
        B.gns_sample_cache(gns.ctx, 5, 0)
        rng = np.random.default_rng(F)
        nodes = rng.integers(-3, n + 3, size=count).astype(np.int32)
        nodes[:4] = (-1, n, np.iinfo(np.int32).max, np.iinfo(np.int32).min)
        buf = torch.full((count * F + 2,), 7.0, dtype=torch.float32, device="cuda:0")
        out = buf[1:1 + count * F].view(count, F)
        B.gns_gather_features(gns.ctx, torch.from_numpy(nodes).to("cuda:0"), count, out)
        torch.cuda.synchronize()
        ok = (nodes >= 0) & (nodes < n)
        want = np.where(ok[:, None], feat.numpy()[np.where(ok, nodes, 0)], np.float32(0))
        assert (out.cpu().numpy() == want).all()
        assert float(buf[0]) == 7.0 and float(buf[-1]) == 7.0
    finally:
        gns.close()


@pytest.mark.parametrize("F", [5, 17, 33, 100, 130])
@pytest.mark.parametrize("more", [0, 1])
def test_gather_from_tables_that_the_caches_keep_and_do_not(F, more):
    """gns_gather_features from a table in HBM of no more than 200 MB, which is read through the caches, and of more; a cached node's
    row, another's, and rows of zeros."""
    dev = torch.device("cuda:0")
    n = 200 * 2 ** 20 // (4 * F) + more
    ip = torch.arange(n + 1, dtype=torch.int32, device=dev) * 2
    i = torch.arange(n, device=dev)
    ix = torch.sort(torch.stack([(i - 1) % n, (i + 1) % n], 1), 1)[0].reshape(-1).to(torch.int32)
    feat = torch.randn((n, F), device=dev, generator=torch.Generator(device=dev).manual_seed(F))
    gns = GpuGns(ip, ix, feat, fanouts=(4, 3), policies=(U, C), cache_size=n // 3, max_seeds=8)
    try:
        B.gns_sample_cache(gns.ctx, 5, 0)
        nodes = torch.randint(-3, n + 3, (150_000,), device=dev, generator=torch.Generator(device=dev).manual_seed(F + 1)).to(torch.int32)
        nodes[:3] = torch.tensor([n - 1, n, -1])
        out = torch.full((nodes.numel() + 1, F), 7.0, device=dev)
        B.gns_gather_features(gns.ctx, nodes, nodes.numel(), out)
        ok = (nodes >= 0) & (nodes < n)
        assert torch.equal(out[:-1], torch.where(ok[:, None], feat[torch.where(ok, nodes, 0).long()], 0.0)) and (out[-1] == 7.0).all()
    finally:
        gns.close()


@pytest.mark.parametrize("F,rows,max_deg", [(128, 70_000, 5), (128, 3_000, 20), (64, 40_000, 9), (256, 20_000, 12),
                                            (100, 40_000, 9), (8, 5_000, 20), (1024, 600, 9)])
def test_aggregate_on_hand_made_blocks(F, rows, max_deg):
    """gns_aggregate alone on a block that no sampler made: rows with 0..max_deg edges (several rounds of the
    kernel's inner loop), more rows than one pass of the grid covers (the kernel's pipeline over rows), empty rows
    next to full ones, non-finite values in source row 0 (empty rows must still give 0), repeated sources."""
    rng = np.random.default_rng(F * 1000 + max_deg)
    num_src = rows + 500
    deg = rng.integers(0, max_deg + 1, size=rows)
    deg[rng.integers(0, rows, size=rows // 10)] = 0
    indptr = np.zeros(rows + 1, dtype=np.int32)
    indptr[1:] = np.cumsum(deg)
    E = int(indptr[-1])
    indices = rng.integers(1, num_src, size=E).astype(np.int32)          # source row 0 is only reached by padding
    weights = rng.uniform(0.5, 40.0, size=E).astype(np.float32)
    x = rng.standard_normal((num_src, F)).astype(np.float32)
    x[0, :] = np.inf
    x[0, ::2] = np.nan
    ref = oracle.aggregate(indptr, indices, weights, x)
    scale = np.zeros((rows, F))
    np.add.at(scale, np.repeat(np.arange(rows), deg), np.abs(weights[:, None].astype(np.float64) * x[indices]))
    scale /= np.maximum(deg, 1)[:, None]
    dev = torch.device("cuda:0")
    ip, ix = _small(n=300)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=10, max_seeds=8)      # a context to call through
    try:
        t = {k: torch.from_numpy(v).to(dev) for k, v in dict(indptr=indptr, indices=indices, weights=weights, x=x).items()}
        blk = B.gns_block()
        blk.num_dst, blk.num_src, blk.num_edges = rows, num_src, E
        blk.indptr, blk.indices, blk.weights = t["indptr"].data_ptr(), t["indices"].data_ptr(), t["weights"].data_ptr()
        out = torch.full((rows, F), 7.0, dtype=torch.float32, device=dev)
        B.gns_aggregate(gns.ctx, blk, t["x"], F, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert np.isfinite(got).all()
        assert (got[deg == 0] == 0).all()
        assert (np.abs(got.astype(np.float64) - ref) <= AGG_RTOL * scale + 1e-30).all()
    finally:
        gns.close()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("F", [1, 3, 4, 5, 16, 17, 31, 32, 33, 64, 66, 80, 81, 96, 99, 127, 128, 129, 161, 192, 193, 255, 256, 257, 300, 512, 516, 1023, 1028, 2100])
def test_aggregate_widths(F, shift):
    """gns_aggregate at the widths where its lanes per row change, and at buffers aligned to four bytes only: rows with 0..9 edges, one
    edge out of range (it is skipped), nothing written around the output."""
    rng = np.random.default_rng(F)
    rows = 3000 if F < 300 else 500
    num_src = rows + 200
    deg = rng.integers(0, 10, size=rows)
    deg[0] = 3
    indptr = np.zeros(rows + 1, dtype=np.int32)
    indptr[1:] = np.cumsum(deg)
    E = int(indptr[-1])
    indices = rng.integers(0, num_src, size=E).astype(np.int32)
    weights = rng.uniform(0.5, 40.0, size=E).astype(np.float32)
    x = rng.standard_normal((num_src, F)).astype(np.float32)
    x_ref, w_ref = x.astype(np.float64), weights.astype(np.float64)
    w_ref[1] = 0.0                                                       # of the edge that is skipped
    ref, scale = np.zeros((rows, F)), np.zeros((rows, F))
    owner = np.repeat(np.arange(rows), deg)
    np.add.at(ref, owner, w_ref[:, None] * x_ref[indices])
    np.add.at(scale, owner, np.abs(w_ref[:, None] * x_ref[indices]))
    ref /= np.maximum(deg, 1)[:, None]
    scale /= np.maximum(deg, 1)[:, None]
    indices[1] = num_src
    dev = torch.device("cuda:0")
    ip, ix = _small(n=300)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=10, max_seeds=8)
    try:
        t = {k: torch.from_numpy(v).to(dev) for k, v in dict(indptr=indptr, indices=indices, weights=weights).items()}
        xs = torch.zeros(num_src * F + 4, dtype=torch.float32, device=dev)[shift:shift + num_src * F].view(num_src, F)
        xs.copy_(torch.from_numpy(x))
        blk = B.gns_block()
        blk.num_dst, blk.num_src, blk.num_edges = rows, num_src, E
        blk.indptr, blk.indices, blk.weights = t["indptr"].data_ptr(), t["indices"].data_ptr(), t["weights"].data_ptr()
        buf = torch.full((rows * F + 8,), 7.0, dtype=torch.float32, device=dev)
        out = buf[4 + shift:4 + shift + rows * F].view(rows, F)
        B.gns_aggregate(gns.ctx, blk, xs, F, out)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        assert (got[deg == 0] == 0).all()
        assert (np.abs(got.astype(np.float64) - ref) <= AGG_RTOL * scale).all()
        assert (buf[:4 + shift] == 7.0).all() and (buf[4 + shift + rows * F:] == 7.0).all()
    finally:
        gns.close()


# Rows that make every lane group of the grid visit three of them, the last ones not all (four lanes a row: eight blocks of 64 groups on
# each of 256 CUs; eight lanes and one column each: six of 32; else four of 32, 16, 8 and 4).
@pytest.mark.parametrize("F,rows", [(2, 600_001), (4, 290_001), (13, 290_001), (16, 290_001), (17, 110_001), (20, 110_001), (32, 110_001)] +
                                   [(F, 72_001) for F in (36, 50, 64, 66, 80, 81, 96, 127, 128)] + [(F, 36_001) for F in (99, 100, 129, 160, 161, 192)] +
                                   [(F, 18_001) for F in (193, 255, 256, 260, 384, 388, 448, 512)] + [(F, 9_001) for F in (516, 768, 772, 896, 1024, 1028, 2100)])
@pytest.mark.parametrize("shift", [0, 1])
def test_aggregate_rows_ahead(F, rows, shift):
    """gns_aggregate with several rows per lane group, whose extents and edges are read ahead: rows of 0..9 edges and one of 40, two edges out of
    range.  Weights and sources are whole numbers, so sums are exact and the mean is either the sum divided by the number of edges, rounded once
    (widths and bases that are no multiple of four floats, and wide rows), or its product with the rounded reciprocal: to the last bit."""
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev).manual_seed(F)
    num_src = rows + 100
    deg = torch.randint(0, 10, (rows,), device=dev, generator=gen)
    deg[0], deg[rows // 2] = 3, 40
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device=dev)
    indptr[1:] = deg.cumsum(0)
    E = int(indptr[-1])
    indices = torch.randint(0, num_src, (E,), device=dev, generator=gen)
    weights = torch.randint(1, 65, (E,), device=dev, generator=gen).double()
    x = torch.randint(-1000, 1001, (num_src, F), device=dev, generator=gen).double()
    owner = torch.repeat_interleave(torch.arange(rows, device=dev), deg)
    w_ref = weights.clone()
    w_ref[1] = w_ref[E - 1] = 0.0                                        # of the edges that are skipped
    ref = torch.zeros((rows, F), dtype=torch.float64, device=dev)
    step = max(1, 2 ** 26 // F)
    for e in range(0, E, step):
        ref.index_add_(0, owner[e:e + step], w_ref[e:e + step, None] * x[indices[e:e + step]])
    n = deg.clamp(min=1).double()[:, None]
    divided = F % 4 or shift or F > 1024 or (F > 256 and F % 32)
    # (a quotient or a product of two floats, rounded to 53 bits and then to 24, is what it is rounded to 24 at once)
    want = (ref / n if divided else ref * (1.0 / n).float().double()).float()
    indices[1], indices[E - 1] = num_src, 2 ** 31 - 1
    ip, ix = _small(n=300)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=10, max_seeds=8)
    try:
        t = [v.contiguous() for v in (indptr.int(), indices.int(), weights.float())]
        xs = torch.zeros(num_src * F + 4, dtype=torch.float32, device=dev)[shift:shift + num_src * F].view(num_src, F)
        xs.copy_(x)
        blk = B.gns_block()
        blk.num_dst, blk.num_src, blk.num_edges = rows, num_src, E
        blk.indptr, blk.indices, blk.weights = (v.data_ptr() for v in t)
        buf = torch.full((rows * F + 8,), 7.0, dtype=torch.float32, device=dev)
        out = buf[4 + shift:4 + shift + rows * F].view(rows, F)
        B.gns_aggregate(gns.ctx, blk, xs, F, out)
        assert torch.equal(out, want)
        assert (buf[:4 + shift] == 7.0).all() and (buf[4 + shift + rows * F:] == 7.0).all()
    finally:
        gns.close()


@pytest.mark.parametrize("F,shift", [(1, 0), (3, 0), (4, 0), (4, 1), (5, 0), (20, 1), (64, 0), (66, 0), (128, 1), (130, 0), (260, 0), (1028, 0)])
def test_aggregate_of_infinities_nan_and_extremes(F, shift):
    """Means of rows with infinities, NaN, the largest and the smallest floats, in the widths that divide and those that multiply: float by
    float as numpy's fp32 sum and division, or product with 1 / n; results below the normal numbers within one unit of the smallest."""
    big, tiny = np.finfo(np.float32).max, np.finfo(np.float32).tiny
    vals = np.array([np.inf, -np.inf, np.nan, big, -big, tiny, 3 * tiny, 2.0 ** -149, 1.0, -7.0], np.float32)
    rows = [[v] for v in range(10)] + [[0, 8, 8], [0, 1], [1, 9], [3, 3], [3, 4], [3, 8, 8], [4, 9, 9], [5, 5, 5, 7, 7], [6] * 7, [7] * 3, [7] * 6 + [5],
            [3] + [7] * 9, [2, 8], [8] * 10 + [0], [9, 9, 8], []]
    deg = np.array([len(r) for r in rows])
    indptr = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    indices = np.array([v for r in rows for v in r], np.int32)
    # column c of a source row is its value times 2^-(c % 3): all columns differ from their neighbors
    x = (vals[:, None] * np.float32(0.5) ** (np.arange(F) % 3).astype(np.float32)).astype(np.float32)
    x = np.concatenate([x, np.zeros((30, F), np.float32)])
    divided = F % 4 or shift or F > 1024 or (F > 256 and F % 32)
    want = np.zeros((len(rows), F), np.float32)
    with np.errstate(all="ignore"):
        for r, edges in enumerate(rows):
            for v in edges:
                want[r] = want[r] + x[v]                                 # weight 1: one rounding, as the fma
            if edges:
                want[r] = want[r] / np.float32(len(edges)) if divided else want[r] * (np.float32(1) / np.float32(len(edges)))
    dev = torch.device("cuda:0")
    ip, ix = _small(n=300)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=10, max_seeds=8)
    try:
        t = [torch.from_numpy(v).to(dev) for v in (indptr, indices, np.ones(len(indices), np.float32))]
        xs = torch.zeros(x.size + 4, dtype=torch.float32, device=dev)[shift:shift + x.size].view(x.shape)
        xs.copy_(torch.from_numpy(x))
        out = torch.zeros(len(rows) * F + 4, dtype=torch.float32, device=dev)[shift:shift + len(rows) * F].view(len(rows), F)
        blk = B.gns_block()
        blk.num_dst, blk.num_src, blk.num_edges = len(rows), x.shape[0], len(indices)
        blk.indptr, blk.indices, blk.weights = (v.data_ptr() for v in t)
        B.gns_aggregate(gns.ctx, blk, xs, F, out)
        got = out.cpu().numpy()
    finally:
        gns.close()
    small = np.abs(want) < tiny
    assert np.array_equal(got[~small], want[~small], equal_nan=True)
    assert (np.abs(got[small].astype(np.float64) - want[small]) <= 2.0 ** -149).all()


@pytest.mark.parametrize("F", [1025, 65535 * 1024 + 1, 65536 * 1024 + 1030, 2 ** 30 + 5])
def test_aggregate_of_rows_beyond_a_grid_and_beyond_4_gb(F):
    """Rows of more columns than one grid has windows for, and of 2^32 bytes and more: the second of two source rows, copied by a
    single edge of weight 1, and a row without edges; the last window has one column, six and five."""
    dev = torch.device("cuda:0")
    ip, ix = _small(n=300)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=10, max_seeds=8)
    try:
        x = torch.empty((2, F), dtype=torch.float32, device=dev).uniform_(generator=torch.Generator(device=dev).manual_seed(F))
        out = torch.full((2, F), 7.0, dtype=torch.float32, device=dev)
        t = [torch.tensor(v, device=dev) for v in (np.array([0, 1, 1], np.int32), np.array([1], np.int32), np.array([1], np.float32))]
        blk = B.gns_block()
        blk.num_dst, blk.num_src, blk.num_edges = 2, 2, 1
        blk.indptr, blk.indices, blk.weights = (v.data_ptr() for v in t)
        B.gns_aggregate(gns.ctx, blk, x, F, out)
        assert torch.equal(out[0], x[1]) and not out[1].any()
    finally:
        gns.close()


@pytest.mark.parametrize("policies", [(U, C), (CF, CF)])
def test_unbiased_weight_mode(policies):
    ip, ix = _small()
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, _feat(n, 32), fanouts=(8, 3), policies=policies, cache_size=400, max_seeds=128,
                 wmode=B.GNS_W_UNBIASED)
    try:
        full_parity(gns, cache_seed=4, epoch=2, batch_seed=5, seeds=synth.uniform_seed_batch(n, 128, 9))
    finally:
        gns.close()


def _star_graph(n, hub_degree, extra_avg, seed):
    """A hub joined to `hub_degree` nodes plus a sparse random background, so one
    row spans several LDS segments of the per-row sampler."""
    rng = np.random.default_rng(seed)
    leaves = rng.choice(np.arange(1, n), size=hub_degree, replace=False)
    a = np.concatenate([np.zeros(hub_degree, dtype=np.int64), rng.integers(1, n, size=n * extra_avg // 2)])
    b = np.concatenate([leaves, rng.integers(1, n, size=n * extra_avg // 2)])
    keep = a != b
    a, b = a[keep], b[keep]
    key = np.unique(np.minimum(a, b) * n + np.maximum(a, b))
    a, b = key // n, key % n
    row = np.concatenate([a, b])
    col = np.concatenate([b, a])
    order = np.lexsort((col, row))
    row, col = row[order], col[order]
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(row, minlength=n), out=indptr[1:])
    return torch.from_numpy(indptr), torch.from_numpy(col.astype(np.int32))


@pytest.mark.parametrize("flag_mode", [0, 1])
@pytest.mark.parametrize("policy", [C, CF])
@pytest.mark.parametrize("hub_degree", [1000, 16385, 40000])
def test_hub_row_spanning_many_flag_words(hub_degree, policy, flag_mode):
    n = 60000
    ip, ix = _star_graph(n, hub_degree, 6, hub_degree)
    assert int(ip[1] - ip[0]) == hub_degree
    gns = GpuGns(ip, ix, None, fanouts=(5, 7), policies=(policy, policy), cache_size=3000, max_seeds=16,
                 flag_mode=flag_mode)
    try:
        seeds = torch.tensor([0, 5, 17, 9, 33], dtype=torch.int32)       # the hub is a seed
        full_parity(gns, cache_seed=2, epoch=0, batch_seed=3, seeds=seeds)
        views, ref = full_parity(gns, cache_seed=2, epoch=1, batch_seed=4, seeds=seeds)
        assert ref[0].row_eligible[0] > 7                                 # the hub really drew a subset
    finally:
        gns.close()


@pytest.mark.parametrize("degrees", [(20000,) * 8, (63, 64, 65, 0, 1), (130_000, 0, 2000), (2048 * 64 - 63, 1)])
def test_scan_plan_of_long_and_empty_rows(degrees):
    """A tile's list of chunks longer and shorter than the 2048 entries that the block looks up at a time, and of that length; rows
    that begin and end inside a chunk, rows without an entry first, in between and last."""
    n = 140_000
    rng = np.random.default_rng(sum(degrees))
    deg = np.zeros(n, dtype=np.int64)
    deg[1:1 + len(degrees)] = degrees
    deg[1000:3000] = rng.integers(0, 5, size=2000)
    ip = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=ip[1:])
    ix = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg if d]).astype(np.int32)
    gns = GpuGns(torch.from_numpy(ip), torch.from_numpy(ix), None, fanouts=(5,), policies=(C,), cache_size=900, max_seeds=600, flag_mode=0)
    try:
        first = np.arange(0, 2 + len(degrees))
        for batch, seeds in enumerate((first, np.concatenate([first[::-1], np.arange(1000, 1500)]))):
            full_parity(gns, cache_seed=2, epoch=batch, batch_seed=3 + batch, seeds=torch.from_numpy(seeds.astype(np.int32)))
    finally:
        gns.close()


def test_rows_with_no_neighbors_and_no_cached_neighbors():
    # nodes 0..9 isolated, the rest a ring; tiny cache -> most rows have N_C = 0
    n = 200
    ring = np.arange(10, n)
    a = ring
    b = np.concatenate([ring[1:], ring[:1]])
    row = np.concatenate([a, b])
    col = np.concatenate([b, a])
    order = np.lexsort((col, row))
    row, col = row[order], col[order]
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(row, minlength=n), out=indptr[1:])
    ip, ix = torch.from_numpy(indptr), torch.from_numpy(col.astype(np.int32))
    gns = GpuGns(ip, ix, _feat(n, 8), fanouts=(2, 2), policies=(U, C), cache_size=3, max_seeds=50)
    try:
        seeds = torch.arange(0, 50, dtype=torch.int32)                   # includes the isolated nodes
        views, ref = full_parity(gns, cache_seed=6, epoch=0, batch_seed=8, seeds=seeds)
        assert (np.diff(ref[1].indptr) == 0).any()
    finally:
        gns.close()


def test_maximum_fanout_and_maximum_depth():
    """The limits of the config: fan-out 64 at every policy, and 8 layers."""
    ip, ix = _small(n=2000, avg=40, seed=13, hub=4)
    n = ip.numel() - 1
    for policies in [(U, C), (CF, CF)]:
        gns = GpuGns(ip, ix, None, fanouts=(64, 64), policies=policies, cache_size=600, max_seeds=24)
        try:
            full_parity(gns, cache_seed=3, epoch=0, batch_seed=14, seeds=synth.uniform_seed_batch(n, 24, 2))
        finally:
            gns.close()
    gns = GpuGns(ip, ix, _feat(n, 8), fanouts=(2, 1, 2, 1, 2, 1, 2, 3), policies=(U, CF, U, CF, U, C, U, C), cache_size=300,
                 max_seeds=16)
    try:
        views, ref = full_parity(gns, cache_seed=5, epoch=1, batch_seed=15, seeds=synth.uniform_seed_batch(n, 16, 3))
        assert len(ref) == 8
    finally:
        gns.close()


def test_single_seed_and_repeatability():
    ip, ix = _small()
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, _feat(n, 16), fanouts=(5, 5), policies=(U, C), cache_size=100, max_seeds=8)
    try:
        seeds = torch.tensor([42], dtype=torch.int32)
        v1, _ = full_parity(gns, cache_seed=1, epoch=0, batch_seed=2, seeds=seeds)
        snap = [{k: (t.clone() if torch.is_tensor(t) else t) for k, t in v.items()} for v in v1]
        v2, _ = full_parity(gns, cache_seed=1, epoch=0, batch_seed=2, seeds=seeds)
        for a, b in zip(snap, v2):
            for k in ("indptr", "indices", "src_nodes", "weights"):
                assert torch.equal(a[k], b[k])
    finally:
        gns.close()


def test_graph_replays_and_eager_launches_agree_with_the_oracle():
    """The batch's launch sequence (twelve launches) is captured once per set of buffers and replayed; with stage timing on
    it is issued kernel by kernel instead.  Replays, eager runs and replays again, with different seeds and
    batch sizes on the same buffers, all against the oracle."""
    ip, ix = _small(n=4000, avg=18, seed=17)
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, _feat(n, 32), fanouts=(7, 5, 4), policies=(CF, U, C), cache_size=350, max_seeds=120)
    try:
        step = 0
        for mode in ("graph", "eager", "graph"):
            if mode == "eager":
                B.gns_profile_begin(gns.ctx, (1 << B.GNS_STAGE_SAMPLE) | (1 << B.GNS_STAGE_GATHER), 64)
            else:
                B.gns_profile_begin(gns.ctx, 0, 0)
            for _ in range(5):
                seeds = synth.uniform_seed_batch(n, 120 - 11 * (step % 4), 50 + step)
                full_parity(gns, cache_seed=8, epoch=step // 4, batch_seed=900 + step, seeds=seeds)
                step += 1
            if mode == "eager":
                ms, launches = B.gns_profile_collect(gns.ctx, B.GNS_STAGE_SAMPLE)
                assert launches == 5 and ms > 0
    finally:
        gns.close()


@pytest.mark.parametrize("fanouts,policies,flag_mode", [((6, 4, 3), (U, U, C), 0), ((5, 4), (C, U), 0), ((4, 3, 3, 2), (U, U, U, C), 1)])
def test_replays_on_alternating_streams_between_direct_launches(fanouts, policies, flag_mode):
    """Sequences of nine, eight and nine launches are replayed where the family's sequences alternate between streams and
    launched directly where they do not: two contexts on two streams, then both on one, then on two again, nothing waited for
    within a round, every mini-batch against the oracle."""
    ip, ix = _small(n=4000, avg=16, seed=43)
    n = ip.numel() - 1
    csize, bs = 300, 70
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=flag_mode)
    ctxs, keep, bufs, _ = _group_setup(gns, 2)
    calls = [B.GroupCall([c], [b.array]) for c, b in zip(ctxs, bufs)]
    try:
        streams = [torch.cuda.Stream() for _ in range(2)]
        cache = None
        for rnd, spread in enumerate((True, True, False, False, True, True)):
            if rnd % 2 == 0:
                B.gns_sample_cache(gns.ctx, 6, rnd)
                cache = oracle.sample_cache(ip.numpy(), 6, rnd, csize)
            seeds = [synth.uniform_seed_batch(n, bs - 9 * ((rnd + i) % 4), 10 * rnd + i).cuda() for i in range(2)]
            for i, call in enumerate(calls):
                call.sample([100 * rnd + i], [seeds[i]], streams[i if spread else 0])
            for i, call in enumerate(calls):
                call.wait(streams[i if spread else 0])
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 100 * rnd + i, seeds[i].cpu().numpy(),
                                           list(fanouts), list(policies))
                compare_blocks([bufs[i].views(j) for j in range(len(fanouts))], ref)
    finally:
        B.gns_destroy(ctxs[1])
        gns.close()


def test_error_paths():
    ip, ix = _small(n=500)
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, None, fanouts=(3, 2), policies=(U, C), cache_size=50, max_seeds=32)
    try:
        seeds = synth.uniform_seed_batch(n, 32, 1).cuda()
        with pytest.raises(B.GnsError) as e:                               # no cache drawn yet
            B.gns_sample_blocks(gns.ctx, 1, seeds, gns.blocks.array)
        assert e.value.status == B.GNS_ESTATE
        B.gns_sample_cache(gns.ctx, 1, 0)
        dup = seeds.clone()
        dup[5] = dup[4]
        with pytest.raises(B.GnsError) as e:
            B.gns_sample_blocks(gns.ctx, 1, dup, gns.blocks.array)
        assert e.value.status == B.GNS_EINVAL
        bad = seeds.clone()
        bad[0] = n
        with pytest.raises(B.GnsError) as e:
            B.gns_sample_blocks(gns.ctx, 1, bad, gns.blocks.array)
        assert e.value.status == B.GNS_EINVAL
        B.gns_sample_blocks(gns.ctx, 1, seeds, gns.blocks.array)          # still healthy afterwards
        ref_cache = oracle.sample_cache(ip.numpy(), 1, 0, 50)
        ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), ref_cache[1], 50, 1, seeds.cpu().numpy(), [3, 2], [U, C])
        compare_blocks([gns.blocks.views(i) for i in range(2)], ref)
        small = gns.blocks.array[1].cap_edges
        gns.blocks.array[1].cap_edges = small - 1
        with pytest.raises(B.GnsError) as e:
            B.gns_sample_blocks(gns.ctx, 1, seeds, gns.blocks.array)
        assert e.value.status == B.GNS_ECAPACITY
        gns.blocks.array[1].cap_edges = small
        with pytest.raises(B.GnsError) as e:                               # too many seeds
            B.gns_sample_blocks(gns.ctx, 1, torch.arange(33, dtype=torch.int32).cuda(), gns.blocks.array)
        assert e.value.status == B.GNS_EINVAL
        with pytest.raises(B.GnsError) as e:                               # no features configured
            B.gns_gather_features(gns.ctx, seeds, 4, torch.empty(4, device="cuda"))
        assert e.value.status == B.GNS_ESTATE
        with pytest.raises(B.GnsError) as e:                               # the config draws the cache by degree
            B.gns_cache_walk_probability(gns.ctx, seeds, 10)
        assert e.value.status == B.GNS_ESTATE
        with pytest.raises(B.GnsError) as e:
            B.gns_cache_probability_view(gns.ctx)
        assert e.value.status == B.GNS_ESTATE
    finally:
        gns.close()


def test_create_rejects_bad_graphs_and_configs():
    ip, ix = _small(n=300)
    n = ip.numel() - 1
    dev = torch.device("cuda:0")

    def create(indptr, indices, fanouts=(2,), policies=(C,), cache_size=10, ws_shrink=0):
        g = B.make_graph(indptr.to(dev), indices.to(dev))
        c = B.make_config(fanouts, policies, cache_size, 8)
        ws = B.alloc_workspace(g, c, dev)
        if ws_shrink:
            ws = ws[:ws.numel() - ws_shrink]
        ctx = B.gns_create(g, c, ws)
        B.gns_destroy(ctx)

    create(ip, ix)
    unsorted = ix.clone()
    b, e = int(ip[7]), int(ip[8])
    assert e - b >= 2
    unsorted[b], unsorted[b + 1] = ix[b + 1], ix[b]
    with pytest.raises(B.GnsError) as err:
        create(ip, unsorted)
    assert err.value.status == B.GNS_EINVAL
    out_of_range = ix.clone()
    out_of_range[3] = n
    with pytest.raises(B.GnsError):
        create(ip, out_of_range)
    bad_ip = ip.clone()
    bad_ip[5] = bad_ip[6] + 1
    with pytest.raises(B.GnsError):
        create(bad_ip, ix)
    with pytest.raises(B.GnsError) as err:                                  # more cache than nodes with neighbors
        create(ip, ix, cache_size=n + 1)
    assert err.value.status == B.GNS_EINVAL
    with pytest.raises(B.GnsError) as err:
        create(ip, ix, policies=(7,))
    assert err.value.status == B.GNS_EINVAL
    with pytest.raises(B.GnsError) as err:
        create(ip, ix, ws_shrink=256)
    assert err.value.status == B.GNS_ECAPACITY


@pytest.mark.parametrize("offsets", [torch.int32, torch.int64])
def test_walk_probability_cache_and_weights(offsets):
    """Section 3.2's random-walk cache probability: the integer weight vector, its prefix, the cache
    drawn from it and the Section 3.4 weights that use it, all against the oracle."""
    ip, ix = _small(n=5000, avg=12, seed=21)
    n = ip.numel() - 1
    train = torch.from_numpy(np.random.default_rng(4).permutation(n)[:150].astype(np.int32))
    fanouts, policies = (6, 4, 3), (CF, CF, C)
    gns = GpuGns(ip.to(offsets), ix, _feat(n, 16), fanouts=fanouts, policies=policies, cache_size=120, max_seeds=64,
                 cache_probability=B.GNS_PROB_WALK)
    try:
        with pytest.raises(B.GnsError) as err:                     # the probability has to be computed first
            B.gns_sample_cache(gns.ctx, 1, 0)
        assert err.value.status == B.GNS_ESTATE
        for scale in (12, 30):
            w, pre, total, support = gns.walk_probability(train, scale)
            w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), list(fanouts), scale_log2=scale)
            assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref)
            assert total == int(pre_ref[-1]) and support == int(np.count_nonzero(w_ref))
            gns.prob_prefix = pre_ref
            for trial in range(2):
                seeds = train[trial * 64:(trial + 1) * 64]
                full_parity(gns, cache_seed=31, epoch=trial, batch_seed=700 + trial, seeds=seeds)
        with pytest.raises(B.GnsError) as err:                     # 40 bits per node times fan-outs up to 6: too much
            big = GpuGns(ip, ix, None, fanouts=(60, 60, 60, 60, 60, 60, 60, 60), policies=(U,) * 7 + (C,), cache_size=50,
                         max_seeds=8, cache_probability=B.GNS_PROB_WALK)
            try:
                B.gns_cache_walk_probability(big.ctx, torch.arange(0, 200, dtype=torch.int32).cuda(), 40)
            finally:
                big.close()
        assert err.value.status == B.GNS_ECAPACITY
    finally:
        gns.close()


@pytest.mark.parametrize("n,scale", [(1, 3), (65, 24), (1_310_000, 24), (1_310_000, 31)])
def test_walk_probability_vector_widths(n, scale):
    """Bit, 32-bit and 64-bit vectors of the walk steps, a training bitmap beyond LDS, runs of 64 rows, a hub row
    over many chunks and empty rows."""
    rng = np.random.default_rng(n)
    hub = rng.choice(n, size=min(n, 3001), replace=False)
    key = np.unique(np.concatenate([rng.integers(0, n * n, size=3 * n), np.int64(n // 2) * n + np.sort(hub)]))
    ip = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=ip[1:])
    ip, ix = torch.from_numpy(ip.astype(np.int32)), torch.from_numpy((key % n).astype(np.int32))
    train = torch.from_numpy(rng.choice(n, size=max(1, n // 10), replace=False).astype(np.int32))
    gns = GpuGns(ip, ix, None, fanouts=(3, 2, 2), policies=(U, U, C), cache_size=1, max_seeds=1,
                 cache_probability=B.GNS_PROB_WALK)
    try:
        w, pre, _, _ = gns.walk_probability(train, scale)
        w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), [3, 2, 2], scale_log2=scale)
        assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref)
    finally:
        gns.close()


@pytest.mark.parametrize("n,degrees", [(3000, (0,)), (3000, (0, 0, 0, 7)), (3000, (1023, 1, 0)), (70000, (0, 1024, 0, 2049, 5, 0))])
def test_walk_windows_and_runs_of_empty_rows(n, degrees):
    """The first step's windows of 1024 entries: rows that end, begin and span where a window does, windows that begin
    inside the row before, runs of nothing but empty rows, in the middle and behind the last entry."""
    rng = np.random.default_rng(n + len(degrees))
    deg = np.zeros(n, dtype=np.int64)
    deg[500:700] = [degrees[i % len(degrees)] for i in range(200)]
    deg[[3, 64, 1200]] = (17, 1024, 33)
    ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    ix = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in deg if d]).astype(np.int32)
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    gns = GpuGns(ip, ix, None, fanouts=(3, 2), policies=(U, C), cache_size=2, max_seeds=8, cache_probability=B.GNS_PROB_WALK)
    try:
        train = torch.arange(1, n, 3, dtype=torch.int32)
        w, pre, _, _ = gns.walk_probability(train, 20)
        w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), [3, 2], scale_log2=20)
        assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref)
    finally:
        gns.close()


def test_cache_nearly_all_nodes():
    # the cache takes every node that has a neighbor: the stream must run until the rarest node shows up
    ip, ix = _small(n=300, avg=6)
    deg = (ip[1:] - ip[:-1])
    support = int((deg > 0).sum())
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(C,), cache_size=support, max_seeds=8)
    try:
        compare_cache(gns.sample_cache(3, 0), oracle.sample_cache(ip.numpy(), 3, 0, support))
    finally:
        gns.close()


@pytest.mark.parametrize("flag_mode", [0, 1])
def test_draw_of_many_chunks_fills_everything_once_it_is_complete(flag_mode):
    """A cache of nearly all nodes takes several rounds of two chunks: bitmap, list, induced subgraph, weights and feature
    table are those of the complete one."""
    ip, ix = _small(n=40_000, avg=6, seed=3)
    csize = min(39_000, int((ip[1:] > ip[:-1]).sum()))
    gns = GpuGns(ip, ix, _feat(40_000, 8), fanouts=(5, 4), policies=(CF, C), cache_size=csize, max_seeds=100, flag_mode=flag_mode)
    try:
        for epoch in range(3):
            assert oracle.sample_cache(ip.numpy(), 3, epoch, csize)[2] > 4 * 1.6 * csize
            full_parity(gns, cache_seed=3, epoch=epoch, batch_seed=50 + epoch, seeds=synth.uniform_seed_batch(40_000, 100, 20 + epoch))
    finally:
        gns.close()


def test_a_refused_draw_leaves_no_draw_to_activate():
    """One node of 6001 owns one of 12 M entries: drawing all of them is refused, and the copy of the cache structures that an
    enqueued draw had filled is gone with it."""
    wide, n = 2000, 6001
    ip = torch.cat([torch.arange(n, dtype=torch.int64) * wide, torch.tensor([(n - 1) * wide + 1])])
    ix = torch.cat([torch.arange(wide, dtype=torch.int32).repeat(n - 1), torch.zeros(1, dtype=torch.int32)])
    gns = GpuGns(ip, ix, None, fanouts=(3,), policies=(C,), cache_size=n, max_seeds=50)
    try:
        for epoch in range(20):
            B.gns_sample_cache_async(gns.ctx, 7, epoch)
            try:
                B.gns_sample_cache(gns.ctx, 7, epoch)
            except B.GnsError as e:
                assert e.status == B.GNS_ECAPACITY
                with pytest.raises(B.GnsError) as err:
                    B.gns_activate_cache(gns.ctx)
                assert err.value.status == B.GNS_ESTATE
                break
        else:
            pytest.fail("no draw was refused")
    finally:
        gns.close()


def _release_cached_memory():
    """Hand torch's cached device and pinned-host blocks back: the giant workloads need tens of
    GB of each, and blocks cached for an earlier test's shapes would be counted twice."""
    import gc
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch._C._host_emptyCache()


def _config_parity(cfg_id, batches, device_gen="cpu", flag_mode=0, check_features=True, upper=U):
    """Whole path on one of the five workloads against the oracle.  The big graphs are generated
    on the GPU (same recipe) and copied to the host for the oracle."""
    import time
    t0 = time.time()
    _release_cached_memory()
    c = synth.CONFIGS[cfg_id]
    sd = synth.config_seeds(cfg_id)
    g = synth.make_config_graph(cfg_id, device=device_gen)
    indptr, indices = g.indptr.cpu(), g.indices.cpu()
    print("cfg%d: n=%d nnz=%d max_degree=%d (generated in %.1fs)" % (cfg_id, c["n"], g.nnz, g.max_degree, time.time() - t0),
          flush=True)
    del g
    feat = None
    if check_features:
        feat = synth.node_features(c["n"], c["feat"], sd["feat"], device=device_gen, pin=c["feat_on_host"])
        if not c["feat_on_host"]:
            feat = feat.cpu()
    print("cfg%d: features ready after %.1fs" % (cfg_id, time.time() - t0), flush=True)
    cache_size = int(c["n"] * c["cache_frac"])
    L = len(c["fanouts"])
    policies = [upper] * (L - 1) + [C]
    gns = GpuGns(indptr, indices, feat, fanouts=c["fanouts"], policies=policies, cache_size=cache_size,
                 max_seeds=c["batch"], feat_on_host=c["feat_on_host"], flag_mode=flag_mode)
    try:
        epoch = None
        if "split" in c:                      # batches of one shuffled epoch over the training split
            split = synth.training_split(c["n"], c["split"], sd["split"])
            epoch = synth.epoch_batches(split, c["batch"], sd["split"] + 1)
        for b in range(batches):
            if epoch is not None:
                seeds = epoch[-1] if b == batches - 1 else epoch[b]      # the last one is the ragged tail
            else:
                seeds = synth.uniform_seed_batch(c["n"], c["batch"], sd["batch"] + b)
            views, ref = full_parity(gns, cache_seed=sd["cache"], epoch=b, batch_seed=sd["batch"] + b, seeds=seeds)
            print("cfg%d batch %d after %.1fs: rows/src/edges per layer %s" % (
                cfg_id, b, time.time() - t0, [(r.num_dst, r.num_src, r.num_edges) for r in ref]), flush=True)
    finally:
        gns.close()
        del gns, feat, indptr, indices
        _release_cached_memory()


def test_config1_tiny_graph():
    _config_parity(1, batches=3)


@pytest.mark.parametrize("flag_mode", [0, 1])
def test_config2_medium_graph(flag_mode):
    _config_parity(2, batches=2, flag_mode=flag_mode)


@pytest.mark.parametrize("flag_mode", [0, 1])
def test_config2_cache_first_on_the_upper_layers(flag_mode):
    """The paper's experimental setting (Section 4.1): GNS sampling on layers 3 and 2 with fan-outs
    15 and 10, the input layer only from the cache."""
    _config_parity(2, batches=1, flag_mode=flag_mode, upper=CF)


def test_async_pipeline_on_forked_contexts():
    """Three mini-batches in flight on three streams (the created context and two
    forks sharing its cache), no host synchronisation between sampling, gather and
    aggregation (counts stay on the device); every batch must still match the oracle."""
    ip, ix = _small(n=4000, avg=16, seed=11)
    n = ip.numel() - 1
    F = 32
    feat = _feat(n, F, seed=5)
    fanouts, policies, csize, bs = (6, 4, 3), (U, U, C), 250, 96
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs)
    forks, fork_ws = [], []
    try:
        ref_cache = oracle.sample_cache(ip.numpy(), 21, 3, csize)
        compare_cache(gns.sample_cache(21, 3), ref_cache)
        ctxs = [gns.ctx]
        for _ in range(2):
            ws = torch.empty(B.gns_fork_workspace_bytes(gns.ctx), dtype=torch.uint8, device=gns.device)
            fork_ws.append(ws)
            child = B.gns_fork(gns.ctx, ws)
            forks.append(child)
            ctxs.append(child)
        streams = [torch.cuda.Stream() for _ in ctxs]
        bufs = [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in ctxs]
        last = len(fanouts) - 1
        xin = [torch.zeros((b.array[last].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        out = [torch.zeros((b.array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for b in bufs]
        H = 24                                                # the update step rides along, counts on the device too
        gw = torch.Generator().manual_seed(77)
        w_dense = torch.randn((2 * F, H), generator=gw) / np.sqrt(2 * F)
        b_dense = torch.randn(H, generator=gw)
        w_dev, b_dev = w_dense.cuda(), b_dense.cuda()
        z = [torch.zeros((b.array[last].cap_dst, H), dtype=torch.float32, device=gns.device) for b in bufs]
        for rnd in range(2):
            seeds = [synth.uniform_seed_batch(n, bs - 7 * i, 300 + 10 * rnd + i).cuda() for i in range(len(ctxs))]
            torch.cuda.synchronize()
            for i, ctx in enumerate(ctxs):
                with torch.cuda.stream(streams[i]):
                    B.gns_sample_blocks_async(ctx, 900 + 10 * rnd + i, seeds[i], bufs[i].array, streams[i])
                    assert bufs[i].array[last].num_dst == -1 - last
                    B.gns_gather_features(ctx, bufs[i].tensors[last]["src_nodes"], -1, xin[i], streams[i])
                    B.gns_aggregate(ctx, bufs[i].array[last], xin[i], F, out[i], streams[i])
                    B.gns_sage_dense(ctx, xin[i], out[i], w_dev, b_dev, True, z[i], -1 - last, streams[i])
            for i, ctx in enumerate(ctxs):
                B.gns_sample_blocks_wait(ctx, bufs[i].array, streams[i])
            torch.cuda.synchronize()
            for i in range(len(ctxs)):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), ref_cache[1], csize, 900 + 10 * rnd + i,
                                           seeds[i].cpu().numpy(), list(fanouts), list(policies))
                compare_blocks([bufs[i].views(j) for j in range(len(fanouts))], ref)
                x_ref = oracle.gather(feat.numpy(), ref[last].src_nodes)
                assert xin[i][:ref[last].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
                o_ref = oracle.aggregate(ref[last].indptr, ref[last].indices, ref[last].weights, x_ref)
                from gpu_harness import compare_aggregate, aggregate_scale
                compare_aggregate(out[i][:ref[last].num_dst].cpu().numpy(), o_ref, aggregate_scale(ref[last], x_ref))
                # the update step saw the GPU's own aggregate; feed the oracle the same fp32 rows
                nd = ref[last].num_dst
                hs, hn = xin[i][:nd].cpu().numpy(), out[i][:nd].cpu().numpy()
                z_ref = oracle.sage_dense(hs, hn, w_dense.numpy(), b_dense.numpy(), True)
                scale = np.abs(np.concatenate([hs, hn], axis=1).astype(np.float64)) @ np.abs(w_dense.numpy().astype(np.float64)) \
                    + np.abs(b_dense.numpy().astype(np.float64))
                err = np.abs(z[i][:nd].cpu().numpy().astype(np.float64) - z_ref.astype(np.float64))
                assert np.all(err <= (2 * F + 3) * 2.0 ** -24 * scale)
        with pytest.raises(B.GnsError):                       # the cache belongs to the created context
            B.gns_sample_cache(forks[0], 1, 0)
    finally:
        for f in forks:
            B.gns_destroy(f)
        gns.close()


def test_bad_seed_in_an_earlier_batch_is_still_reported():
    """Three mini-batches enqueued before one wait, the first of them with a repeated seed: the wait reports
    it although the last batch was fine; the next wait is clean again."""
    ip, ix = _small(n=2000)
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, None, fanouts=(4, 3), policies=(U, C), cache_size=150, max_seeds=48)
    try:
        B.gns_sample_cache(gns.ctx, 3, 0)
        good = [synth.uniform_seed_batch(n, 48, 70 + i).cuda() for i in range(3)]
        bad = good[0].clone()
        bad[7] = bad[3]
        for sd_, t in ((1, bad), (2, good[1]), (3, good[2])):
            B.gns_sample_blocks_async(gns.ctx, sd_, t, gns.blocks.array)
        with pytest.raises(B.GnsError) as e:
            B.gns_sample_blocks_wait(gns.ctx, gns.blocks.array)
        assert e.value.status == B.GNS_EINVAL
        B.gns_sample_blocks_async(gns.ctx, 4, good[0], gns.blocks.array)
        B.gns_sample_blocks_wait(gns.ctx, gns.blocks.array)
        cache = oracle.sample_cache(ip.numpy(), 3, 0, 150)
        ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], 150, 4, good[0].cpu().numpy(), [4, 3], [U, C])
        compare_blocks([gns.blocks.views(i) for i in range(2)], ref)
    finally:
        gns.close()


def test_a_stream_that_is_being_captured_is_refused():
    """Stamps and batch ids are arguments of the launches, so a mini-batch cannot be replayed: the call says so, enqueues
    nothing, and the context goes on as before."""
    ip, ix = _small(n=2000)
    gns = GpuGns(ip, ix, None, fanouts=(4, 3), policies=(U, U), cache_size=0, max_seeds=48)
    try:
        seeds = synth.uniform_seed_batch(ip.numel() - 1, 48, 70).cuda()
        x = torch.zeros(64, device="cuda")
        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            graph.capture_begin()
            x.add_(1.0)
            with pytest.raises(B.GnsError) as e:
                B.gns_sample_blocks_async(gns.ctx, 4, seeds, gns.blocks.array, stream)
            graph.capture_end()
        assert e.value.status == B.GNS_EHIP
        B.gns_sample_blocks(gns.ctx, 4, seeds, gns.blocks.array)
        ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), None, 0, 4, seeds.cpu().numpy(), [4, 3], [U, U])
        compare_blocks([gns.blocks.views(i) for i in range(2)], ref)
    finally:
        gns.close()


def test_walk_probability_recomputed_while_batches_are_in_flight():
    """gns_cache_walk_probability invalidates the cache; mini-batches enqueued before it (on another stream,
    not yet waited for) keep the cache they were enqueued with, and the draw that follows fills the other
    copy of the cache structures instead of the one they read."""
    ip, ix = _small(n=6000, avg=18, seed=31)
    n = ip.numel() - 1
    F = 16
    feat = _feat(n, F, seed=2)
    fanouts, policies, csize, bs = (5, 4), (CF, C), 300, 80
    train = torch.from_numpy(np.random.default_rng(9).permutation(n)[:400].astype(np.int32))
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=1,
                 cache_probability=B.GNS_PROB_WALK)
    try:
        work = torch.cuda.Stream()
        nb = 6
        bufs = [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in range(nb)]
        xin = [torch.zeros((b.array[1].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        seeds = [train[40 * b:40 * b + bs].contiguous().cuda() for b in range(nb)]
        prefixes = []
        for rnd, scale in enumerate((10, 20)):
            w, pre, total, support = gns.walk_probability(train, scale)     # while the previous pass's batches may still run
            w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), list(fanouts), scale_log2=scale)
            assert np.array_equal(pre, pre_ref)
            prefixes.append(pre_ref)
            B.gns_sample_cache(gns.ctx, 12, rnd)
            for b in range(3 * rnd, 3 * rnd + 3):
                B.gns_sample_blocks_async(gns.ctx, 300 + b, seeds[b], bufs[b].array, work)
                B.gns_gather_features(gns.ctx, bufs[b].tensors[1]["src_nodes"], -1, xin[b], work)
        torch.cuda.synchronize()
        for b in range(nb):
            pre_ref = prefixes[b // 3]
            cache = oracle.sample_cache(pre_ref, 12, b // 3, csize)
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 300 + b, seeds[b].cpu().numpy(),
                                       list(fanouts), list(policies), prob_prefix=pre_ref)
            for j, r in enumerate(ref):
                t = bufs[b].tensors[j]
                assert np.array_equal(t["indptr"][:r.num_dst + 1].cpu().numpy(), r.indptr)
                assert np.array_equal(t["indices"][:r.num_edges].cpu().numpy(), r.indices)
                assert np.array_equal(t["src_nodes"][:r.num_src].cpu().numpy(), r.src_nodes)
                gw = t["weights"][:r.num_edges].cpu().numpy().astype(np.float64)
                assert np.all(np.abs(gw - r.weights) <= 1e-5 * np.abs(r.weights))
            x_ref = oracle.gather(feat.numpy(), ref[1].src_nodes)
            assert xin[b][:ref[1].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
    finally:
        gns.close()


def test_walk_probability_waits_for_a_draw_in_flight():
    """An asynchronous draw on a stream that is busy with other work, then the probability of other training nodes on another
    stream: the draw, its cache and its weights are those of the probability it was enqueued with."""
    ip, ix = _small(n=6000, avg=18, seed=31)
    n = ip.numel() - 1
    fanouts, policies, csize, bs = (5, 4), (CF, C), 300, 80
    nodes = torch.from_numpy(np.random.default_rng(9).permutation(n).astype(np.int32))
    first, second = nodes[:400].contiguous(), nodes[3000:3100].contiguous()
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=1,
                 cache_probability=B.GNS_PROB_WALK)
    try:
        gns.walk_probability(first, 20)
        busy = torch.cuda.Stream()
        a = torch.randn((4096, 4096), device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(busy):
            for _ in range(20):
                a = (a @ a).clamp_(-1.0, 1.0)
        B.gns_sample_cache_async(gns.ctx, 12, 0, busy)
        _, pre, _, _ = gns.walk_probability(second, 20)
        assert np.array_equal(pre, oracle.walk_weights(ip.numpy(), ix.numpy(), second.numpy(), list(fanouts), scale_log2=20)[1])
        B.gns_activate_cache(gns.ctx)
        nodes_ptr, size, _, draws = B.gns_cache_view(gns.ctx)
        _, pre_first = oracle.walk_weights(ip.numpy(), ix.numpy(), first.numpy(), list(fanouts), scale_log2=20)
        ref = oracle.sample_cache(pre_first, 12, 0, csize)
        assert draws == ref[2]
        assert np.array_equal(B.device_view_i32(nodes_ptr, size, gns.device).cpu().numpy(), ref[0])
        seeds = first[:bs].contiguous()
        blocks = oracle.sample_blocks(ip.numpy(), ix.numpy(), ref[1], csize, 7, seeds.numpy(), list(fanouts), list(policies),
                                      prob_prefix=pre_first)
        compare_blocks(gns.sample_blocks(7, seeds), blocks)
    finally:
        gns.close()


def test_cache_refresh_while_batches_are_in_flight():
    """A cache draw fills the copy of the cache structures that is not in use: batches enqueued before it
    (here on two forks, not yet waited for) must come out with the old cache, batches enqueued after it
    with the new one."""
    ip, ix = _small(n=6000, avg=20, seed=19)
    n = ip.numel() - 1
    F = 16
    feat = _feat(n, F, seed=6)
    fanouts, policies, csize, bs = (5, 4), (CF, C), 400, 64
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=1)
    forks, keep = [], []
    try:
        caches = [oracle.sample_cache(ip.numpy(), 77, e, csize) for e in range(3)]
        compare_cache(gns.sample_cache(77, 0), caches[0])
        for _ in range(2):
            ws = torch.empty(B.gns_fork_workspace_bytes(gns.ctx), dtype=torch.uint8, device=gns.device)
            keep.append(ws)
            forks.append(B.gns_fork(gns.ctx, ws))
        streams = [torch.cuda.Stream() for _ in forks]
        draw_stream = torch.cuda.Stream()
        bufs = [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in forks]
        xin = [torch.zeros((b.array[1].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        for epoch in (1, 2):
            seeds = [synth.uniform_seed_batch(n, bs, 40 + 2 * epoch + i).cuda() for i in range(2)]
            torch.cuda.synchronize()
            for i, f in enumerate(forks):                       # enqueued with the cache of epoch - 1
                B.gns_sample_blocks_async(f, 500 + i, seeds[i], bufs[i].array, streams[i])
                B.gns_gather_features(f, bufs[i].tensors[1]["src_nodes"], -1, xin[i], streams[i])
            B.gns_sample_cache(gns.ctx, 77, epoch, draw_stream)   # overlaps them
            for i, f in enumerate(forks):
                B.gns_sample_blocks_wait(f, bufs[i].array, streams[i])
            torch.cuda.synchronize()
            for i in range(2):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), caches[epoch - 1][1], csize, 500 + i,
                                           seeds[i].cpu().numpy(), list(fanouts), list(policies))
                compare_blocks([bufs[i].views(j) for j in range(2)], ref)
                x_ref = oracle.gather(feat.numpy(), ref[1].src_nodes)
                assert xin[i][:ref[1].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
            nodes_ptr, size, bitmap_ptr, _ = B.gns_cache_view(gns.ctx)
            assert np.array_equal(B.device_view_i32(nodes_ptr, size, gns.device).cpu().numpy(), caches[epoch][0])
            # and a batch enqueued now sees the new cache
            B.gns_sample_blocks(forks[0], 900, seeds[0], bufs[0].array, streams[0])
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), caches[epoch][1], csize, 900, seeds[0].cpu().numpy(),
                                       list(fanouts), list(policies))
            compare_blocks([bufs[0].views(j) for j in range(2)], ref)
    finally:
        for f in forks:
            B.gns_destroy(f)
        gns.close()


def test_cache_prepared_ahead_and_activated_later():
    """gns_sample_cache_async fills the copy of the cache structures that is not in use while batches of the
    current cache run; gns_activate_cache switches over.  Nothing here synchronises between the draws, the
    activations and the batches; every batch must match the oracle for the cache of its own period."""
    ip, ix = _small(n=7000, avg=22, seed=29)
    n = ip.numel() - 1
    F = 16
    feat = _feat(n, F, seed=4)
    fanouts, policies, csize, bs = (5, 4), (CF, C), 450, 96
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=1)
    try:
        work, draws = torch.cuda.Stream(), torch.cuda.Stream()
        periods, per = 4, 3
        nb = periods * per
        bufs = [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in range(nb)]
        xin = [torch.zeros((b.array[1].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        seeds = [synth.uniform_seed_batch(n, bs, 800 + b).cuda() for b in range(nb)]
        with pytest.raises(B.GnsError) as err:                     # nothing drawn yet
            B.gns_activate_cache(gns.ctx)
        assert err.value.status == B.GNS_ESTATE
        torch.cuda.synchronize()
        B.gns_sample_cache_async(gns.ctx, 66, 0, draws)
        for b in range(nb):
            if b % per == 0:
                B.gns_activate_cache(gns.ctx)                      # the cache of period b // per, drawn one period ago
                if b // per + 1 < periods:
                    B.gns_sample_cache_async(gns.ctx, 66, b // per + 1, draws)
            B.gns_sample_blocks_async(gns.ctx, 2000 + b, seeds[b], bufs[b].array, work)
            B.gns_gather_features(gns.ctx, bufs[b].tensors[1]["src_nodes"], -1, xin[b], work)
        torch.cuda.synchronize()
        for b in range(nb):
            cache = oracle.sample_cache(ip.numpy(), 66, b // per, csize)
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 2000 + b, seeds[b].cpu().numpy(),
                                       list(fanouts), list(policies))
            for j, r in enumerate(ref):
                t = bufs[b].tensors[j]
                assert np.array_equal(t["indptr"][:r.num_dst + 1].cpu().numpy(), r.indptr)
                assert np.array_equal(t["indices"][:r.num_edges].cpu().numpy(), r.indices)
                assert np.array_equal(t["src_nodes"][:r.num_src].cpu().numpy(), r.src_nodes)
                gw = t["weights"][:r.num_edges].cpu().numpy().astype(np.float64)
                assert np.all(np.abs(gw - r.weights) <= 1e-5 * np.abs(r.weights))
            x_ref = oracle.gather(feat.numpy(), ref[1].src_nodes)
            assert xin[b][:ref[1].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
        last = oracle.sample_cache(ip.numpy(), 66, periods - 1, csize)
        nodes_ptr, size, _, num_draws = B.gns_cache_view(gns.ctx)   # reads the asynchronous draw's outcome back
        assert np.array_equal(B.device_view_i32(nodes_ptr, size, gns.device).cpu().numpy(), last[0]) and num_draws == last[2]
    finally:
        gns.close()


def test_host_far_ahead_of_the_device_across_cache_refreshes():
    """Many mini-batches and several cache draws enqueued without waiting for any of them, the draws on a
    stream of their own: a draw must not overwrite the copy of the cache structures that batches the device
    has not reached yet still read (the library makes it wait for them on the device)."""
    ip, ix = _small(n=8000, avg=24, seed=23)
    n = ip.numel() - 1
    F = 32
    feat = _feat(n, F, seed=9)
    fanouts, policies, csize, bs = (6, 5), (U, C), 500, 128
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=1)
    try:
        work, draws = torch.cuda.Stream(), torch.cuda.Stream()
        nb, period = 24, 3
        bufs = [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in range(nb)]
        xin = [torch.zeros((b.array[1].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        seeds = [synth.uniform_seed_batch(n, bs, 600 + b).cuda() for b in range(nb)]
        torch.cuda.synchronize()
        for b in range(nb):
            if b % period == 0:
                B.gns_sample_cache(gns.ctx, 55, b // period, draws)
            B.gns_sample_blocks_async(gns.ctx, 1000 + b, seeds[b], bufs[b].array, work)
            B.gns_gather_features(gns.ctx, bufs[b].tensors[1]["src_nodes"], -1, xin[b], work)
        torch.cuda.synchronize()
        for b in range(nb):
            bufs[b].array[0].num_dst = 0                      # counts were never waited for: take them from the oracle
            cache = oracle.sample_cache(ip.numpy(), 55, b // period, csize)
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 1000 + b, seeds[b].cpu().numpy(),
                                       list(fanouts), list(policies))
            for j, r in enumerate(ref):
                t = bufs[b].tensors[j]
                assert np.array_equal(t["indptr"][:r.num_dst + 1].cpu().numpy(), r.indptr)
                assert np.array_equal(t["indices"][:r.num_edges].cpu().numpy(), r.indices)
                assert np.array_equal(t["src_nodes"][:r.num_src].cpu().numpy(), r.src_nodes)
            x_ref = oracle.gather(feat.numpy(), ref[1].src_nodes)
            assert xin[b][:ref[1].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
    finally:
        gns.close()


def test_config3_products_shaped_graph():
    _config_parity(3, batches=2, device_gen="cuda")


def test_config3_cache_first_per_cache_flags():
    _config_parity(3, batches=1, device_gen="cuda", flag_mode=1, upper=CF, check_features=False)


def test_config3_per_cache_flags_with_features():
    """The benchmark's default mode (one flag per CSR entry, built when the cache is drawn) on the
    products-shaped graph, gather and aggregation included."""
    _config_parity(3, batches=2, device_gen="cuda", flag_mode=1)


def test_config3_input_nodes_of_node_wise_sampling_against_gns():
    """Shape check after the paper's Table 3: on the products-shaped graph plain node-wise sampling (every layer
    UNIFORM) reaches several times more input nodes per mini-batch than GNS in the paper's setting (upper layers
    cache first, input layer from the cache only), a good share of the GNS input nodes are cached, and at the
    input layer the cached share of a row's neighbors, N_C(v)/deg(v), is about the share of all edge endpoints
    that cached nodes own.  The GPU counts are also the oracle's (first batch of every setting)."""
    _release_cached_memory()
    c = synth.CONFIGS[3]
    sd = synth.config_seeds(3)
    g = synth.make_config_graph(3, device="cuda")
    indptr, indices = g.indptr.cpu(), g.indices.cpu()
    del g
    ip, ix = indptr.numpy(), indices.numpy()
    cache_size = int(c["n"] * c["cache_frac"])
    cache_nodes, bitmap, _ = oracle.sample_cache(ip, sd["cache"], 0, cache_size)
    deg = np.diff(ip)
    endpoint_share = deg[cache_nodes].sum() / ip[-1]
    is_cached = np.zeros(c["n"], dtype=bool)
    is_cached[cache_nodes] = True
    batches = 3
    stats = {}
    for name, pol in (("ns", (U, U, U)), ("gns", (CF, CF, C))):
        gns = GpuGns(indptr, indices, None, fanouts=c["fanouts"], policies=pol, cache_size=cache_size,
                     max_seeds=c["batch"], flag_mode=1)
        try:
            if name == "gns":                       # a config with no cache layer has no cache to draw
                gns.sample_cache(sd["cache"], 0)
            inputs = cached = 0
            elig = degs = 0
            for b in range(batches):
                seeds = synth.uniform_seed_batch(c["n"], c["batch"], sd["batch"] + b)
                views = gns.sample_blocks(sd["batch"] + b, seeds)
                v = views[-1]
                src = v["src_nodes"].cpu().numpy()
                inputs += src.size
                cached += int(is_cached[src].sum())
                if name == "gns":
                    rows = v["row_eligible"].numel()
                    elig += int(v["row_eligible"].sum())
                    degs += int(deg[src[:rows]].sum())
                if b == 0:
                    ref = oracle.sample_blocks(ip, ix, bitmap, cache_size, sd["batch"], seeds.numpy(), list(c["fanouts"]),
                                               list(pol))
                    assert [r.num_src for r in ref] == [int(w["src_nodes"].numel()) for w in views]
            stats[name] = (inputs / batches, cached / batches, elig, degs)
        finally:
            gns.close()
            del gns
            _release_cached_memory()
    ns_in, gns_in, gns_cached = stats["ns"][0], stats["gns"][0], stats["gns"][1]
    row_share = stats["gns"][2] / stats["gns"][3]
    print("cfg3 input nodes per mini-batch: NS %.0f, GNS %.0f (%.0f cached); N_C/deg over the input layer's rows %.4f, "
          "cached share of edge endpoints %.4f" % (ns_in, gns_in, gns_cached, row_share, endpoint_share), flush=True)
    # Table 3 reports a factor 4.9 on OGBN-products (3.3 to 7.9 over its datasets): the same order here
    assert 2.0 < ns_in / gns_in < 20.0
    assert gns_cached > 0.1 * gns_in
    assert 0.5 * endpoint_share < row_share < 2.0 * endpoint_share


def test_config2_walk_probability_at_scale():
    """The random-walk cache probability on the medium graph from a 10 % training split: weights and prefix
    bit for bit, then one mini-batch drawn with that cache."""
    c = synth.CONFIGS[2]
    sd = synth.config_seeds(2)
    g = synth.make_config_graph(2)
    ip, ix = g.indptr, g.indices
    train = synth.training_split(c["n"], 100_000, sd["split"])
    gns = GpuGns(ip, ix, None, fanouts=c["fanouts"], policies=(CF, CF, C), cache_size=int(c["n"] * c["cache_frac"]),
                 max_seeds=c["batch"], flag_mode=1, cache_probability=B.GNS_PROB_WALK)
    try:
        w, pre, total, support = gns.walk_probability(train, 24)
        w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), list(c["fanouts"]), scale_log2=24)
        assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref) and total == int(pre_ref[-1])
        gns.prob_prefix = pre_ref
        full_parity(gns, cache_seed=sd["cache"], epoch=0, batch_seed=sd["batch"], seeds=train[:c["batch"]])
    finally:
        gns.close()


def test_config4_int64_offsets_and_host_features():
    _config_parity(4, batches=1, device_gen="cuda", flag_mode=1)


def test_config5_giant_graph():
    _config_parity(5, batches=2, device_gen="cuda", flag_mode=0)


def test_config5_giant_graph_per_cache_flags():
    """The flag pass over all 1.6 G CSR entries with the cache bitmap in global memory, then mini-batches that
    only read their rows' flag words: the mode the benchmark runs on this workload."""
    _config_parity(5, batches=2, device_gen="cuda", flag_mode=1)


@pytest.mark.parametrize("rows,f1,f2,hdim,relu,use_bias", [(1000, 128, 128, 256, True, True), (1, 4, 8, 12, False, False),
                                                            (129, 100, 128, 132, True, False), (517, 64, 32, 40, False, True)])
def test_sage_dense_update_step(rows, f1, f2, hdim, relu, use_bias):
    """h_u = g(W . (h_u, h_N(u))) on the matrix cores against the fp64 oracle.  fp32 products are
    exact in the fp32 accumulator up to one rounding per addition: K + 1 additions of terms bounded
    by S = sum |a||w| + |b| give an error of at most (K + 2) * 2^-24 * S; the oracle's own final
    rounding adds 2^-24 of the result."""
    ip, ix = _small(n=600)
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=0, max_seeds=8)
    try:
        g = torch.Generator().manual_seed(rows + hdim)
        hs = torch.randn((rows, f1), generator=g)
        hn = torch.randn((rows, f2), generator=g)
        w = torch.randn((f1 + f2, hdim), generator=g) / np.sqrt(f1 + f2)
        b = torch.randn(hdim, generator=g) if use_bias else None
        out = torch.full((rows, hdim), float("nan"), device=gns.device)
        B.gns_sage_dense(gns.ctx, hs.cuda(), hn.cuda(), w.cuda(), None if b is None else b.cuda(), relu, out, rows)
        torch.cuda.synchronize()
        ref = oracle.sage_dense(hs.numpy(), hn.numpy(), w.numpy(), None if b is None else b.numpy(), relu)
        a = np.concatenate([hs.numpy(), hn.numpy()], axis=1).astype(np.float64)
        scale = np.abs(a) @ np.abs(w.numpy().astype(np.float64)) + (0.0 if b is None else np.abs(b.numpy().astype(np.float64)))
        bound = (f1 + f2 + 3) * 2.0 ** -24 * scale
        err = np.abs(out.cpu().numpy().astype(np.float64) - ref.astype(np.float64))
        assert np.all(err <= bound), float(np.max(err / bound))
        with pytest.raises(B.GnsError):                           # widths must be multiples of 4
            B.gns_sage_dense(gns.ctx, hs.cuda()[:, :f1 - 1].contiguous(), hn.cuda(),
                             w.cuda()[1:].contiguous(), None, relu, out, rows)
    finally:
        gns.close()


@pytest.mark.parametrize("rows,f1,f2,hdim", [(12_289, 64, 68, 128), (6_150, 36, 220, 200), (12_300, 8, 12, 64), (12_290, 4, 4, 20),
                                             (6_145, 256, 256, 128), (3_073, 300, 400, 256), (40, 700, 600, 36), (33, 4, 28, 4)])
def test_sage_dense_slabs_and_split(rows, f1, f2, hdim):
    """Weight slabs of every width (edges of tiles, k remainders, columns past the last) and the split of k."""
    test_sage_dense_update_step(rows, f1, f2, hdim, rows % 2 == 0, True)


@pytest.mark.parametrize("rows,f1,f2,hdim", [(24_577, 32, 32, 128), (24_600, 64, 80, 100), (24_608, 160, 192, 128), (24_577, 176, 192, 128),
                                             (12_290, 336, 336, 256), (12_290, 336, 352, 256), (65_601, 20, 44, 128), (65_537, 100, 100, 128),
                                             (87_400, 36, 220, 96), (65_537, 24, 36, 128)])
def test_sage_dense_in_bf16_terms(rows, f1, f2, hdim):
    """Slabs of 64 and 32 columns in terms and the first K beyond them; widths that are multiples of 16 and that are not; odd
    numbers of steps; rows, k and columns past the last.  The bound is that of the fp32 products: a product of terms is exact
    in the accumulator's 24 bits, the two that are left out are below 2^-24 of |a||w|, and there are fewer additions."""
    test_sage_dense_update_step(rows, f1, f2, hdim, rows % 2 == 0, True)


def _one_pattern(bits):
    value = torch.tensor([bits], dtype=torch.int32).view(torch.float32).item()
    return lambda shape, g: (torch.randint(0, 2, shape, generator=g, device="cuda") * 2 - 1).float() * value


def _normal(shape, g):
    return torch.randn(shape, generator=g, device="cuda")


@pytest.mark.parametrize("f", [32, 128, 256])
@pytest.mark.parametrize("rows_of,weights_of", [
    (_normal, _normal), (_one_pattern(0x3F80FFFF),) * 2, (_one_pattern(0x3F808040),) * 2, (_one_pattern(0x3F807EC0),) * 2,
    (lambda s, g: _normal(s, g) * 1e-36, _normal), (_normal, lambda s, g: _normal(s, g) * 1e-37),
    (lambda s, g: _normal(s, g) * 1e-18, lambda s, g: _normal(s, g) * 1e-18), (lambda s, g: _normal(s, g) * 1e20, _normal),
    (lambda s, g: _normal(s, g) * torch.exp2(torch.randint(-60, 60, s, generator=g, device="cuda").float()), _normal),
])
def test_sage_dense_in_bf16_terms_is_no_further_from_64_bits_than_fp32_products(rows_of, weights_of, f):
    """A large product against 64 bits, and the same rows in two calls, each too small for the terms and therefore in fp32
    products: factors whose bits are cut badly, all of one sign of error; very small and very large ones; rows whose values
    span 36 decades."""
    rows, hdim = 24_576, 128
    g = torch.Generator(device="cuda").manual_seed(f)
    hs, hn, w = rows_of((rows, f), g), rows_of((rows, f), g), weights_of((2 * f, hdim), g)
    gns = GpuGns(*_small(n=600), None, fanouts=(2,), policies=(U,), cache_size=0, max_seeds=8)
    try:
        whole, parts = (torch.full((rows, hdim), 7.0, device="cuda") for _ in range(2))
        B.gns_sage_dense(gns.ctx, hs, hn, w, None, False, whole, rows)
        for lo in (0, rows // 2):
            part = slice(lo, lo + rows // 2)
            B.gns_sage_dense(gns.ctx, hs[part], hn[part], w, None, False, parts[part], rows // 2)
        a = torch.cat([hs, hn], dim=1).double()
        ref = a @ w.double()
        err_terms, err_fp32 = (((o.double() - ref).norm() / ref.norm()).item() for o in (whole, parts))
        assert 0 < err_terms <= err_fp32 < 1e-6, (err_terms, err_fp32)
        assert bool(((whole.double() - ref).abs() <= (2 * f + 3) * 2.0 ** -24 * (a.abs() @ w.double().abs())).all())
    finally:
        gns.close()


@pytest.mark.parametrize("count", [1, 31, 32, 33, 100])
def test_sage_dense_in_bf16_terms_with_few_rows_counted_on_the_device(count):
    """The kernel is chosen by the largest number of rows there may be; the number there is may be less than a tile."""
    ip, ix = _small(n=30_000, avg=4)
    F, H = 32, 100
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(U,), cache_size=0, max_seeds=25_000)
    try:
        B.gns_sample_blocks(gns.ctx, 5, synth.uniform_seed_batch(30_000, count, 3).cuda(), gns.blocks.array)
        g = torch.Generator(device="cuda").manual_seed(count)
        hs, hn = _normal((25_000, F), g), _normal((25_000, F), g)
        w, bias = _normal((2 * F, H), g), _normal((H,), g)
        out = torch.full((25_000, H), 7.0, device="cuda")
        B.gns_sage_dense(gns.ctx, hs, hn, w, bias, True, out, -1)
        a = torch.cat([hs, hn], dim=1)[:count].double()
        ref = (a @ w.double() + bias.double()).clamp_min(0)
        scale = a.abs() @ w.double().abs() + bias.double().abs()
        assert bool(((out[:count].double() - ref).abs() <= (2 * F + 3) * 2.0 ** -24 * scale).all())
        assert bool((out[count:] == 7.0).all())
    finally:
        gns.close()


def test_sage_dense_infinities_nan_and_the_largest_values():
    """Values whose bf16 terms do not add up to them, and the largest finite ones: as plain products have it."""
    rows, f, hdim = 24_600, 64, 128
    gns = GpuGns(*_small(n=600), None, fanouts=(2,), policies=(U,), cache_size=0, max_seeds=8)
    try:
        g = torch.Generator().manual_seed(4)
        a = torch.randn((rows, 2 * f), generator=g)
        w = torch.randn((2 * f, hdim), generator=g) / 16
        w[3, 5], w[70, 90] = 0.0, float("inf")
        a[17, 2], a[40, 100], a[41, 3], a[90, 70] = float("inf"), -float("inf"), float("inf"), 0.0
        a[300, 7], a[24_599, 127] = float("nan"), 3.0e38
        out = torch.full((rows, hdim), 7.0, device=gns.device)
        B.gns_sage_dense(gns.ctx, a[:, :f].contiguous().cuda(), a[:, f:].contiguous().cuda(), w.cuda(), None, False, out, rows)
        ref = (a.double() @ w.double()).float()
        out = out.cpu()
        assert torch.equal(torch.isnan(out), torch.isnan(ref))
        inf = torch.isinf(ref)
        assert torch.equal(out[inf], ref[inf]) and not torch.isinf(out[~inf]).any()
        ok = torch.isfinite(ref)
        scale = torch.where(torch.isfinite(a), a, 0.0).double().abs() @ torch.where(torch.isfinite(w), w, 0.0).double().abs()
        err = (out.double() - ref.double()).abs()
        assert bool((err[ok] <= (2 * f + 3) * 2.0 ** -24 * scale[ok]).all())
    finally:
        gns.close()


def _group_setup(gns, count):
    """count contexts (the created one and forks) with their own block buffers, feature buffers and a GroupCall."""
    ctxs, keep = [gns.ctx], []
    for _ in range(count - 1):
        ws = torch.empty(B.gns_fork_workspace_bytes(gns.ctx), dtype=torch.uint8, device=gns.device)
        keep.append(ws)
        ctxs.append(B.gns_fork(gns.ctx, ws))
    bufs = [gns.blocks] + [B.BlockBuffers(gns.graph, gns.config, gns.device) for _ in range(count - 1)]
    call = B.GroupCall(ctxs, [b.array for b in bufs])
    return ctxs, keep, bufs, call


def _check_group_batch(gns, buf, ref, feat, xin, hout, F):
    from gpu_harness import compare_aggregate, aggregate_scale
    L = len(ref)
    compare_blocks([buf.views(j) for j in range(L)], ref)
    if feat is None:
        return
    last = L - 1
    x_ref = oracle.gather(feat.numpy(), ref[last].src_nodes)
    assert xin[:ref[last].num_src].cpu().numpy().tobytes() == x_ref.tobytes()
    o_ref = oracle.aggregate(ref[last].indptr, ref[last].indices, ref[last].weights, x_ref)
    compare_aggregate(hout[:ref[last].num_dst].cpu().numpy(), o_ref, aggregate_scale(ref[last], x_ref))


@pytest.mark.parametrize("flag_mode", [0, 1])
@pytest.mark.parametrize("count,fanouts,policies", [(8, (6, 4, 3), (U, U, C)), (3, (5, 7), (CF, CF)), (1, (4, 4), (U, C)),
                                                    (5, (20, 3), (U, C))])
def test_group_of_mini_batches_in_one_launch_sequence(count, fanouts, policies, flag_mode):
    """gns_*_group: `count` mini-batches of different sizes per launch sequence, several rounds (direct launches, and graph
    replays where two layers scan their rows), a cache refresh in the middle; every batch against the oracle."""
    ip, ix = _small(n=5000, avg=16, seed=37)
    n = ip.numel() - 1
    F = 24
    feat = _feat(n, F, seed=8)
    csize, bs = 300, 90
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=flag_mode)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        L = len(fanouts)
        last = L - 1
        st = torch.cuda.Stream()
        xin = [torch.zeros((b.array[last].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        hout = [torch.zeros((b.array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for b in bufs]
        for rnd in range(5):
            epoch = rnd // 2
            if rnd % 2 == 0:
                B.gns_sample_cache(gns.ctx, 44, epoch, st)
            cache = oracle.sample_cache(ip.numpy(), 44, epoch, csize)
            seeds = [synth.uniform_seed_batch(n, bs - 11 * ((b + rnd) % 7), 100 * rnd + b).cuda() for b in range(count)]
            bseeds = [7000 + 10 * rnd + b for b in range(count)]
            call.sample(bseeds, seeds, st)
            call.gather([b.tensors[last]["src_nodes"] for b in bufs], [-1] * count, xin, st)
            call.aggregate(last, xin, F, hout, st)
            call.wait(st)
            torch.cuda.synchronize()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, bseeds[b], seeds[b].cpu().numpy(),
                                           list(fanouts), list(policies))
                _check_group_batch(gns, bufs[b], ref, feat, xin[b], hout[b], F)
        # a context of the group used on its own in between, then the group again (their stamps now differ)
        solo = synth.uniform_seed_batch(n, 33, 999).cuda()
        B.gns_sample_blocks(ctxs[-1], 31337, solo, bufs[-1].array, st)
        ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 31337, solo.cpu().numpy(), list(fanouts),
                                   list(policies))
        compare_blocks([bufs[-1].views(j) for j in range(L)], ref)
        seeds = [synth.uniform_seed_batch(n, bs, 5000 + b).cuda() for b in range(count)]
        call.sample(list(range(count)), seeds, st)
        call.wait(st)
        for b in range(count):
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, b, seeds[b].cpu().numpy(), list(fanouts),
                                       list(policies))
            compare_blocks([bufs[b].views(j) for j in range(L)], ref)
        # a bad seed in one batch of a group is reported by the group's wait
        bad = seeds[count // 2].clone()
        bad[1] = bad[0]
        seeds2 = list(seeds)
        seeds2[count // 2] = bad
        call.sample(list(range(count)), seeds2, st)
        with pytest.raises(B.GnsError) as e:
            call.wait(st)
        assert e.value.status == B.GNS_EINVAL
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


def test_group_argument_checks():
    ip, ix = _small(n=800)
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, None, fanouts=(3, 2), policies=(U, U), cache_size=0, max_seeds=16)
    other = GpuGns(ip, ix, None, fanouts=(3, 2), policies=(U, U), cache_size=0, max_seeds=16)
    try:
        seeds = synth.uniform_seed_batch(n, 16, 1).cuda()
        twice = B.GroupCall([gns.ctx, gns.ctx], [gns.blocks.array, other.blocks.array])
        with pytest.raises(B.GnsError) as e:
            twice.sample([1, 2], [seeds, seeds])
        assert e.value.status == B.GNS_EINVAL
        strangers = B.GroupCall([gns.ctx, other.ctx], [gns.blocks.array, other.blocks.array])
        with pytest.raises(B.GnsError) as e:
            strangers.sample([1, 2], [seeds, seeds])
        assert e.value.status == B.GNS_EINVAL
    finally:
        other.close()
        gns.close()


def test_config2_pipeline_as_the_benchmark_drives_it():
    """The medium workload driven the way bench.py times it: groups of mini-batches on two streams, device-side
    counts, graph replays, no host synchronisation between batches, a cache refresh in the middle; every
    batch compared with the oracle afterwards (blocks, gathered rows, aggregate)."""
    _release_cached_memory()
    cfg_id = 2
    c = synth.CONFIGS[cfg_id]
    sd = synth.config_seeds(cfg_id)
    g = synth.make_config_graph(cfg_id)
    n, F = c["n"], c["feat"]
    feat = synth.node_features(n, F, sd["feat"])
    fanouts, policies = list(c["fanouts"]), [U, U, C]
    csize = int(n * c["cache_frac"])
    gns = GpuGns(g.indptr, g.indices, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=c["batch"],
                 flag_mode=1)
    G, S = 4, 2                                       # batches per group, groups in flight
    ctxs, keep, bufs, _ = _group_setup(gns, G * S)
    try:
        calls = [B.GroupCall(ctxs[s * G:(s + 1) * G], [b.array for b in bufs[s * G:(s + 1) * G]]) for s in range(S)]
        streams = [torch.cuda.Stream() for _ in range(S)]
        last = len(fanouts) - 1
        rounds, refresh_at = 3, 2 * G                # 3 rounds of S groups of G batches; a refresh after 8 batches
        nb = rounds * S * G
        seeds = [synth.uniform_seed_batch(n, c["batch"], sd["batch"] + b).cuda() for b in range(nb)]
        # results are copied out of the reused buffers on the batch's own stream right behind the batch
        snap = {}
        xin = [torch.zeros((bufs[i].array[last].cap_src, F), dtype=torch.float32, device=gns.device) for i in range(G * S)]
        hout = [torch.zeros((bufs[i].array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for i in range(G * S)]
        torch.cuda.synchronize()
        b0 = 0
        for rnd in range(rounds):
            for s in range(S):
                ids = list(range(b0, b0 + G))
                if b0 % refresh_at == 0:
                    B.gns_sample_cache(gns.ctx, sd["cache"], b0 // refresh_at, streams[0])
                sl = slice(s * G, (s + 1) * G)
                with torch.cuda.stream(streams[s]):
                    calls[s].sample([sd["batch"] + b for b in ids], [seeds[b] for b in ids], streams[s])
                    calls[s].gather([bf.tensors[last]["src_nodes"] for bf in bufs[sl]], [-1] * G, xin[sl], streams[s])
                    calls[s].aggregate(last, xin[sl], F, hout[sl], streams[s])
                    for k, b in enumerate(ids):
                        i = s * G + k
                        snap[b] = ([{name: t.clone() for name, t in bufs[i].tensors[j].items()} for j in range(last + 1)],
                                   xin[i].clone(), hout[i].clone())
                b0 += G
        torch.cuda.synchronize()
        ip, ix = g.indptr.numpy(), g.indices.numpy()
        from gpu_harness import compare_aggregate, aggregate_scale
        caches = {}
        for b in (0, 1, G, 2 * G, 2 * G + 1, nb - 1):          # first group, across the refresh, the last batch
            epoch = b // refresh_at
            if epoch not in caches:
                caches[epoch] = oracle.sample_cache(ip, sd["cache"], epoch, csize)
            ref = oracle.sample_blocks(ip, ix, caches[epoch][1], csize, sd["batch"] + b, seeds[b].cpu().numpy(), fanouts, policies)
            tens, x, h = snap[b]
            for j, r in enumerate(ref):
                t = tens[j]
                assert np.array_equal(t["indptr"][:r.num_dst + 1].cpu().numpy(), r.indptr), (b, j)
                assert np.array_equal(t["indices"][:r.num_edges].cpu().numpy(), r.indices), (b, j)
                assert np.array_equal(t["src_nodes"][:r.num_src].cpu().numpy(), r.src_nodes), (b, j)
                assert np.array_equal(t["row_eligible"][:r.num_dst].cpu().numpy(), r.row_eligible), (b, j)
                gw = t["weights"][:r.num_edges].cpu().numpy().astype(np.float64)
                assert np.all(np.abs(gw - r.weights) <= 1e-5 * np.abs(r.weights)), (b, j)
            x_ref = oracle.gather(feat.numpy(), ref[last].src_nodes)
            assert x[:ref[last].num_src].cpu().numpy().tobytes() == x_ref.tobytes(), b
            o_ref = oracle.aggregate(ref[last].indptr, ref[last].indices, ref[last].weights, x_ref)
            compare_aggregate(h[:ref[last].num_dst].cpu().numpy(), o_ref, aggregate_scale(ref[last], x_ref))
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()
        _release_cached_memory()


@pytest.mark.parametrize("fanouts,policies,flag_mode", [((6, 4, 3), (U, U, C), 1), ((5, 7), (CF, CF), 0), ((20, 5), (U, C), 0)])
def test_mark_bitmap_summary_on_a_small_graph(fanouts, policies, flag_mode, monkeypatch):
    """Graphs with millions of nodes keep a summary of the frontier mark bitmap (one bit per word) so that the
    union step only reads words that carry marks.  Forced here on a small graph whose bitmap spans several
    summary words and tiles; group launches and repeated batches check that both levels are left clean."""
    monkeypatch.setenv("GNS_MARK_SUMMARY_MIN_WORDS", "1")
    ip, ix = _small(n=20000, avg=10, seed=43)
    n = ip.numel() - 1
    F = 8
    feat = _feat(n, F, seed=3)
    csize, bs, count = 500, 70, 3
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=flag_mode)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        L = len(fanouts)
        last = L - 1
        cache = oracle.sample_cache(ip.numpy(), 4, 0, csize)
        B.gns_sample_cache(gns.ctx, 4, 0)
        xin = [torch.zeros((b.array[last].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        hout = [torch.zeros((b.array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for b in bufs]
        for rnd in range(3):
            seeds = [synth.uniform_seed_batch(n, bs - 9 * b, 40 * rnd + b).cuda() for b in range(count)]
            bseeds = [600 + 10 * rnd + b for b in range(count)]
            call.sample(bseeds, seeds)
            call.gather([b.tensors[last]["src_nodes"] for b in bufs], [-1] * count, xin)
            call.aggregate(last, xin, F, hout)
            call.wait()
            torch.cuda.synchronize()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, bseeds[b], seeds[b].cpu().numpy(),
                                           list(fanouts), list(policies))
                _check_group_batch(gns, bufs[b], ref, feat, xin[b], hout[b], F)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("env", [{}, {"GNS_NO_GRAPH": "1"}, {"GNS_MARK_SUMMARY_MIN_WORDS": "1", "GNS_UNION_SPINS": "0"}])
@pytest.mark.parametrize("fanouts,policies,flag_mode", [((15, 10, 5), (U, U, U), 0), ((16, 8), (U, C), 1), ((4, 17, 3), (U, U, C), 1),
                                                        ((6, 5), (CF, C), 0), ((15, 10, 5), (CF, CF, C), 0)])
def test_sampler_kernel_choices_give_the_same_blocks(env, fanouts, policies, flag_mode, monkeypatch):
    """Layers by two-stage sampler, by a wave per row (fan-out 17) and by scans of the rows, whose sequences of ten and fourteen
    launches are replayed from a captured graph or, without it, enqueued one by one; the union step by the bitmap and by its
    summary, without a poll for another block's count.  In groups of three mini-batches, against the oracle."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    ip, ix = _small(n=20000, avg=12, seed=61)
    n = ip.numel() - 1
    F = 8
    feat = _feat(n, F, seed=6)
    csize, bs, count = 2000, 80, 3
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=flag_mode)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        last = len(fanouts) - 1
        uses_cache = any(p != U for p in policies)
        cache = oracle.sample_cache(ip.numpy(), 4, 0, csize)
        if uses_cache:
            B.gns_sample_cache(gns.ctx, 4, 0)
        xin = [torch.zeros((b.array[last].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
        hout = [torch.zeros((b.array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for b in bufs]
        for rnd in range(2):
            seeds = [synth.uniform_seed_batch(n, bs - 13 * b, 60 * rnd + b).cuda() for b in range(count)]
            bseeds = [900 + 10 * rnd + b for b in range(count)]
            call.sample(bseeds, seeds)
            call.gather([b.tensors[last]["src_nodes"] for b in bufs], [-1] * count, xin)
            call.aggregate(last, xin, F, hout)
            call.wait()
            torch.cuda.synchronize()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, bseeds[b], seeds[b].cpu().numpy(),
                                           list(fanouts), list(policies))
                _check_group_batch(gns, bufs[b], ref, feat, xin[b], hout[b], F)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("summary", [False, True])
def test_union_step_with_large_tiles_and_several_lds_passes(summary, monkeypatch):
    """The union step walks the frontier mark bitmap in tiles of up to 8192 words and passes a tile's marked
    words through LDS 1024 at a time.  Forced here: one tile of 4096 words over a 300 K-node graph, and a batch
    whose new nodes mark nearly every word of it (several passes), with and without the bitmap's summary."""
    monkeypatch.setenv("GNS_MARK_TILE_WORDS", "4096")
    monkeypatch.setenv("GNS_MARK_SUMMARY_MIN_WORDS", "1" if summary else "1000000000")
    ip, ix = random_symmetric_csr(300000, 8, np.random.default_rng(47))
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    n = ip.numel() - 1
    gns = GpuGns(ip, ix, None, fanouts=(12, 6), policies=(U, CF), cache_size=3000, max_seeds=3000, flag_mode=1)
    try:
        for trial in range(2):
            seeds = synth.uniform_seed_batch(n, 3000 - 500 * trial, 70 + trial)
            views, ref = full_parity(gns, cache_seed=5, epoch=trial, batch_seed=80 + trial, seeds=seeds)
            assert ref[1].num_src - ref[1].num_dst > 40000          # new nodes of the input layer: most words marked
    finally:
        gns.close()


def test_directed_adjacency():
    """Nothing in the path assumes a symmetric adjacency (deg(i) is the row length, the cache draw takes the
    owner row of a uniform entry): the symmetric graph and a directed thinning of it, both against the oracle."""
    ip, ix = _small(n=4000, avg=16, seed=53)
    n = ip.numel() - 1
    rng = np.random.default_rng(3)
    keep = rng.random(ix.numel()) < 0.7                                   # drop 30 % of the entries, one direction at a time
    row = np.repeat(np.arange(n), np.diff(ip.numpy()))
    ip_d = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(row[keep], minlength=n), out=ip_d[1:])
    ix_d = ix.numpy()[keep]
    for indptr, indices in ((ip, ix), (torch.from_numpy(ip_d), torch.from_numpy(ix_d))):
        gns = GpuGns(indptr, indices, _feat(n, 16), fanouts=(6, 5), policies=(CF, C), cache_size=300, max_seeds=100,
                     flag_mode=1)
        try:
            for trial in range(2):
                seeds = synth.uniform_seed_batch(n, 100 - 30 * trial, 11 + trial)
                full_parity(gns, cache_seed=14, epoch=trial, batch_seed=15 + trial, seeds=seeds)
        finally:
            gns.close()


@pytest.mark.parametrize("spins", ["0", "256"])
@pytest.mark.parametrize("fanouts,policies,flag_mode", [((16, 11, 1), (U, CF, C), 1), ((6, 10, 5), (CF, U, C), 1), ((17, 16), (U, C), 1),
                                                        ((8, 9, 12), (CF, U, C), 1), ((13, 8), (CF, C), 1),
                                                        ((20, 40), (CF, C), 1), ((5, 15), (CF, CF), 0)])
def test_sampler_unrolls_and_counts_taken_from_the_bitmap(spins, fanouts, policies, flag_mode, monkeypatch):
    """Fan-outs at the edges of the two-stage sampler's unroll lengths and above them; union blocks that do not wait
    for one another's counts (no polls at all) and that do."""
    monkeypatch.setenv("GNS_UNION_SPINS", spins)
    ip, ix = _small(n=30000, avg=14, seed=29, hub=40)
    gns = GpuGns(ip, ix, _feat(ip.numel() - 1, 4), fanouts=fanouts, policies=policies, cache_size=900, max_seeds=300, flag_mode=flag_mode)
    try:
        for trial, count in enumerate((300, 1, 67)):
            full_parity(gns, cache_seed=8, epoch=trial, batch_seed=50 + trial, seeds=synth.uniform_seed_batch(30000, count, 20 + trial))
    finally:
        gns.close()


def test_node_table_is_cleared_when_its_stamps_run_out():
    """Mini-batches are told apart in the node table by a stamp of few bits: more mini-batches than stamps."""
    ip, ix = random_symmetric_csr(300000, 6, np.random.default_rng(3))
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    gns = GpuGns(ip, ix, None, fanouts=(20, 16), policies=(U, U), cache_size=0, max_seeds=2000)
    try:
        seeds = synth.uniform_seed_batch(300000, 40, 5).cuda()
        for b in range(8300):                              # 19 bits of local id leave 13 for the stamp
            B.gns_sample_blocks_async(gns.ctx, b, seeds, gns.blocks.array)
        B.gns_sample_blocks_wait(gns.ctx, gns.blocks.array)
        full_parity(gns, cache_seed=0, epoch=0, batch_seed=9, seeds=seeds.cpu())
    finally:
        gns.close()


@pytest.mark.parametrize("spins", ["256", "0"])
@pytest.mark.parametrize("n,avg,csize", [(70, 3, 1), (64, 4, 40), (5000, 2, 1365), (40000, 6, 1366), (40000, 6, 39000), (300000, 4, 30000)])
def test_cache_draw_chunks_and_counts_taken_from_the_data(spins, n, avg, csize, monkeypatch):
    """Caches that the first chunk of the stream completes and that need several (most of the nodes cached), chunks at
    the edges of a tile of draws, rows found between two entries of the table; blocks that do not wait for one another's
    counts and that do.  Waited for and enqueued."""
    monkeypatch.setenv("GNS_UNION_SPINS", spins)
    ip, ix = _small(n=n, avg=avg, seed=n + csize)
    csize = min(csize, int((ip[1:] > ip[:-1]).sum()))
    gns = GpuGns(ip, ix, None, fanouts=(2,), policies=(C,), cache_size=csize, max_seeds=8)
    try:
        for epoch in range(3):
            compare_cache(gns.sample_cache(12, epoch), oracle.sample_cache(ip.numpy(), 12, epoch, csize))
        ref = oracle.sample_cache(ip.numpy(), 12, 3, csize)
        if ref[2] <= 8 * 65536:                            # what an enqueued draw takes from the stream
            B.gns_sample_cache_async(gns.ctx, 12, 3)
            B.gns_activate_cache(gns.ctx)
            _, _, _, draws = B.gns_cache_view(gns.ctx)
            assert draws == ref[2]
    finally:
        gns.close()


@pytest.mark.parametrize("count", [2, 7, 16])
@pytest.mark.parametrize("fanouts,policies,flag_mode", [((9, 4), (U, C), 1), ((18, 3), (C, U), 0)])
def test_group_sizes_that_share_the_xcds_unevenly(count, fanouts, policies, flag_mode):
    """A group's blocks are dealt to the eight XCDs in turns of eight per batch: sizes that divide the eight, that do not, and
    the largest, in launches whose number of blocks is no multiple of eight; every batch against the oracle."""
    ip, ix = _small(n=4000, avg=14, seed=61)
    csize, bs = 250, 70
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=flag_mode)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        B.gns_sample_cache(gns.ctx, 46, 0)
        cache = oracle.sample_cache(ip.numpy(), 46, 0, csize)
        seeds = [synth.uniform_seed_batch(4000, bs - b, 300 + b).cuda() for b in range(count)]
        for rnd in range(2):
            call.sample([90 * rnd + b for b in range(count)], seeds)
            call.wait()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 90 * rnd + b, seeds[b].cpu().numpy(),
                                           list(fanouts), list(policies))
                compare_blocks([bufs[b].views(j) for j in range(len(fanouts))], ref)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("fanout,policy", [(1, C), (5, CF), (8, C), (9, U), (12, CF), (13, C), (16, U), (16, CF)])
def test_ranks_sorted_by_waves_of_thirty_two_rows(fanout, policy):
    """Layers of more than 131,072 rows at most, whose waves take the most rows; fan-outs at the edges of the sorted lengths,
    rows with fewer entries than slots, with as many and with more, and last waves that are not full."""
    n, bs, csize, count = 40000, 2100, 0 if policy == U else 3000, 4
    ip, ix = _small(n=n, avg=12, seed=77, hub=60)
    gns = GpuGns(ip, ix, None, fanouts=(15, fanout), policies=(U, policy), cache_size=csize, max_seeds=bs, flag_mode=1)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    try:
        if csize:
            B.gns_sample_cache(gns.ctx, 47, 0)
        cache = oracle.sample_cache(ip.numpy(), 47, 0, max(csize, 1))
        seeds = [synth.uniform_seed_batch(n, bs - 700 * b, 400 + b).cuda() for b in range(count - 1)]
        seeds.append(seeds[0][:1].contiguous())
        call.sample([9 + b for b in range(count)], seeds)
        call.wait()
        for b in range(count):
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 9 + b, seeds[b].cpu().numpy(),
                                       [15, fanout], [U, policy])
            compare_blocks([bufs[b].views(j) for j in range(2)], ref)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("offsets", [torch.int32, torch.int64])
@pytest.mark.parametrize("n", [26_623, 26_625, 53_249, 130_000])
def test_walk_hot_nodes_in_lds(n, offsets):
    """Steps on 32-bit values keep the nodes with the longest rows of 26,624 slots in LDS: fewer nodes than slots, one and
    two more than a multiple of them, several per slot; a graph whose rows say nothing about how often a node is drawn from
    (directed, hubs among the columns only), rows of thousands of entries that no wave's share can be cut in."""
    rng = np.random.default_rng(n)
    cols = np.concatenate([rng.integers(0, n, size=4 * n), rng.integers(0, 50, size=n) * (n // 50)])
    rows = np.concatenate([rng.integers(0, n, size=4 * n), rng.integers(0, n, size=n)])
    rows[:9000] = n - 1
    rows[9000:15000] = 7
    key = np.unique(rows.astype(np.int64) * n + cols)
    ip = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=ip[1:])
    ip, ix = torch.from_numpy(ip), torch.from_numpy((key % n).astype(np.int32))
    train = torch.from_numpy(rng.choice(n, size=n // 7, replace=False).astype(np.int32))
    gns = GpuGns(ip.to(offsets), ix, None, fanouts=(7, 3, 2, 2), policies=(U, U, U, C), cache_size=1, max_seeds=1,
                 cache_probability=B.GNS_PROB_WALK)
    try:
        for scale in (10, 22, 33, 40):                 # 32-bit sums, products beyond 32 bits, 64-bit vectors from the second step on
            w, pre, _, _ = gns.walk_probability(train, scale)
            w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), [7, 3, 2, 2], scale_log2=scale)
            assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref)
    finally:
        gns.close()


@pytest.mark.parametrize("flag_mode", [0, 1])
@pytest.mark.parametrize("n", [1_310_021, 16_777_217, 17_000_003, 83_361_792, 83_361_793])
def test_cache_filter_of_graphs_whose_bitmap_does_not_fit_lds(n, flag_mode):
    """Cache bitmaps beyond LDS are tested through groups of ids, tags of hot nodes and, on the larger of these graphs, pairs
    of cached nodes per group: a run of neighboring ids that are nearly all cached (groups with many), the last ids of the
    graph, and nodes far apart (groups with one), sharing slots of the tags.  The last two sizes are the largest with that
    filter, whose groups have up to 81 ids, and the smallest with the coarse bitmap."""
    rng = np.random.default_rng(n)
    dense = np.arange(n - 30_000, n)                            # up to the last node
    spread = rng.choice(n - 30_000, size=30_000, replace=False)
    spread[:200] = 5 + 16384 * np.arange(200) % (n - 30_000)    # one slot
    spread = np.unique(spread)
    nodes = np.concatenate([dense, spread])
    a, b = nodes[rng.integers(0, len(nodes), size=400_000)], nodes[rng.integers(0, len(nodes), size=400_000)]
    a[:3000], b[:3000] = n - 1, nodes[rng.integers(0, len(nodes), size=3000)]       # a hub
    keep = a != b
    key = np.unique(np.concatenate([a[keep] * n + b[keep], b[keep] * n + a[keep]]))
    ip = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=ip[1:])
    ip, ix = torch.from_numpy(ip), torch.from_numpy((key % n).astype(np.int32))
    gns = GpuGns(ip.to(torch.int32), ix, None, fanouts=(6, 5), policies=(CF, C), cache_size=35_000, max_seeds=600, flag_mode=flag_mode)
    gns.indptr_cpu = ip
    try:
        seeds = torch.from_numpy(np.random.default_rng(3).choice(nodes, size=600, replace=False).astype(np.int32))
        for epoch in range(3):                                  # both copies of the filter, one of them twice
            full_parity(gns, cache_seed=48, epoch=epoch, batch_seed=900 + epoch, seeds=seeds)
    finally:
        gns.close()


@pytest.mark.parametrize("n,avg", [(60_000, 40), (1_400_000, 6)])
def test_short_and_long_lists_of_chunks_to_flag(n, avg):
    """Lists of up to eight chunks for each of 4096 waves are tested against the bitmap in global memory, longer ones against
    what is staged in LDS (the bitmap, or a filter where it does not fit): a row, lists on both sides of the line, and a
    group whose lists are short each and long together."""
    ip, ix = random_symmetric_csr(n, avg, np.random.default_rng(n))
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    fanouts, policies, csize, bs = (10, 5), (U, C), n // 50, 3600
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=bs, flag_mode=0)
    ctxs, keep, bufs, call = _group_setup(gns, 3)
    try:
        for trial, count in enumerate((1, 700, bs)):
            full_parity(gns, cache_seed=49, epoch=0, batch_seed=60 + trial, seeds=synth.uniform_seed_batch(n, count, 500 + trial))
        cache = oracle.sample_cache(ip.numpy(), 49, 0, csize)
        seeds = [synth.uniform_seed_batch(n, 1300 - b, 510 + b).cuda() for b in range(3)]
        call.sample([70 + b for b in range(3)], seeds)
        call.wait()
        for b in range(3):
            ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 70 + b, seeds[b].cpu().numpy(), list(fanouts), list(policies))
            compare_blocks([bufs[b].views(j) for j in range(2)], ref)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("count,seeds", [(1, 1), (2, 9), (2, 10), (1, 38), (1, 39), (16, 3), (5, 17)])
@pytest.mark.parametrize("fanouts,policies,wmode", [((10, 5), (U, C), 0), ((16, 1), (CF, CF), 1), ((3, 3, 3), (C, U, C), 0), ((5, 7), (U, U), 0),
                                                    ((2, 2, 2, 2), (CF, U, CF, C), 1)])
def test_small_batches_in_one_launch(count, seeds, fanouts, policies, wmode):
    """Mini-batches of a few seeds are sampled by a block each; the same contexts then take a batch too large for that, and a
    small one again.  Hub rows, rows without neighbors, clustered ids, bad seeds; every batch against the oracle."""
    ip, ix = _small(n=3000, avg=10, seed=67)
    n, F, bs = 3000, 12, 400
    feat = _feat(n, F, seed=9)
    uses_cache = any(p != U for p in policies)
    gns = GpuGns(ip, ix, feat, fanouts=fanouts, policies=policies, cache_size=200 if uses_cache else 0, max_seeds=bs, wmode=wmode, flag_mode=1)
    ctxs, keep, bufs, call = _group_setup(gns, count)
    last = len(fanouts) - 1
    try:
        bitmap = None
        if uses_cache:
            B.gns_sample_cache(gns.ctx, 47, 0)
        for rnd, size in enumerate((seeds, bs, 1, seeds)):
            if uses_cache and rnd == 3:
                B.gns_sample_cache(gns.ctx, 47, 1)
            if uses_cache:
                bitmap = oracle.sample_cache(ip.numpy(), 47, int(rnd == 3), 200)[1]
            ids = [synth.uniform_seed_batch(n, max(1, size - b % 2), 60 * rnd + b).cuda() for b in range(count)]
            call.sample([500 * rnd + b for b in range(count)], ids)
            xin = [torch.zeros((b.array[last].cap_src, F), dtype=torch.float32, device=gns.device) for b in bufs]
            hout = [torch.zeros((b.array[last].cap_dst, F), dtype=torch.float32, device=gns.device) for b in bufs]
            call.gather([b.tensors[last]["src_nodes"] for b in bufs], [-1] * count, xin)
            call.aggregate(last, xin, F, hout)
            call.wait()
            for b in range(count):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), bitmap, 200 if uses_cache else 0, 500 * rnd + b, ids[b].cpu().numpy(),
                                           list(fanouts), list(policies), wmode)
                _check_group_batch(gns, bufs[b], ref, feat, xin[b], hout[b], F)
        for bad in ([5, 5, 7], [5, -1, 7], [5, n, 7]):
            ids = [torch.tensor(bad if b == count - 1 else [b, b + 20], dtype=torch.int32).cuda() for b in range(count)]
            call.sample(list(range(count)), ids)
            with pytest.raises(B.GnsError) as e:
                call.wait()
            assert e.value.status == B.GNS_EINVAL
        call.sample(list(range(count)), [torch.tensor([b, b + 20], dtype=torch.int32).cuda() for b in range(count)])
        call.wait()                                             # reported once
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


def _guarded_blocks(gns):
    """Block buffers with sentinel words behind every array, and a check that they are untouched."""
    bufs, guards = B.BlockBuffers(gns.graph, gns.config, gns.device), []
    for b, t in zip(bufs.array, bufs.tensors):
        for name in ("indptr", "indices", "src_nodes", "row_eligible", "weights"):
            big = torch.full((t[name].numel() + 4096,), 77, dtype=t[name].dtype, device=gns.device)
            guards.append(big[t[name].numel():])
            t[name] = big[:t[name].numel()]
            setattr(b, name, big.data_ptr())
    return bufs, lambda: all(bool((g == 77).all()) for g in guards)


def _many_bad_seeds(n, count):
    """Seed lists whose rows do not fit beside the nodes they lead to: repeats, ids out of range, or both."""
    ids = torch.arange(count, dtype=torch.int32)
    return {"twice": ids // 2 % n, "one": torch.zeros_like(ids), "outside": ids + n, "negative": -1 - ids, "mixed": torch.where(ids % 3 == 0, ids + n, ids % n)}


@pytest.mark.parametrize("n,count,fanouts,policies", [(100, 1000, (4, 16), (U, U)), (1000, 1000, (4, 4), (U, C)), (1000, 1000, (4, 4), (CF, CF)),
                                                      (100, 500, (8, 2, 1), (U, CF, C)), (64, 200, (1, 16), (C, U))])
def test_small_batches_of_many_bad_seeds(n, count, fanouts, policies):
    """Repeated and invalid seeds in a mini-batch that a block of its own samples, more of them than the graph leaves room for:
    reported, nothing written past a buffer, no rows left for the calls behind, and the next mini-batch is right."""
    ip, ix = _small(n=n, avg=12, seed=71)
    csize = n // 4 if any(p != U for p in policies) else 0
    gns = GpuGns(ip, ix, _feat(n, 8), fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=count, flag_mode=1)
    last = len(fanouts) - 1
    try:
        gns.blocks, untouched = _guarded_blocks(gns)
        for seeds in _many_bad_seeds(n, count).values():
            if csize:
                B.gns_sample_cache(gns.ctx, 47, 0)
            B.gns_sample_blocks_async(gns.ctx, 5, seeds.cuda(), gns.blocks.array)
            x = torch.full((gns.blocks.array[last].cap_src, 8), 3.0, device=gns.device)
            h = torch.full((gns.blocks.array[last].cap_dst, 8), 3.0, device=gns.device)
            B.gns_gather_features(gns.ctx, gns.blocks.tensors[last]["src_nodes"], -1, x)
            B.gns_aggregate(gns.ctx, gns.blocks.array[last], x, 8, h)
            with pytest.raises(B.GnsError) as e:
                B.gns_sample_blocks_wait(gns.ctx, gns.blocks.array)
            assert e.value.status == B.GNS_EINVAL
            assert untouched()
            assert all(b.num_dst == b.num_src == b.num_edges == 0 for b in gns.blocks.array)
            assert bool((x == 3.0).all()) and bool((h == 3.0).all())
            full_parity(gns, cache_seed=47, epoch=0, batch_seed=6, seeds=torch.arange(0, n, 3, dtype=torch.int32))
            assert untouched()
    finally:
        gns.close()


@pytest.mark.parametrize("graph", ["small", "star"])
@pytest.mark.parametrize("fanouts,policies,flag_mode", [((15, 10), (U, C), 1), ((18, 3), (CF, C), 1), ((6, 4), (U, C), 0), ((9, 3), (C, CF), 0),
                                                        ((4, 4, 4), (U, U, U), 0)])
def test_many_bad_seeds(graph, fanouts, policies, flag_mode, monkeypatch):
    """As above for the sequences of launches, replayed ones and gns_sample_blocks_static among them: more seeds than nodes, nodes
    behind repeated seeds beyond the end of the list, and a hub's chunks a few thousand times over."""
    n, count = 900, 2600
    ip, ix = _small(n=n, avg=10, seed=73) if graph == "small" else _star_graph(n, 800, 4, 5)
    csize = 60 if any(p != U for p in policies) else 0
    monkeypatch.setenv("GNS_MARK_SUMMARY_MIN_WORDS", "1" if graph == "star" else "65536")
    gns = GpuGns(ip, ix, _feat(n, 8), fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=count, flag_mode=flag_mode)
    last = len(fanouts) - 1
    try:
        gns.blocks, untouched = _guarded_blocks(gns)
        if csize:
            B.gns_sample_cache(gns.ctx, 48, 0)
        hub = int((ip[1:] - ip[:-1]).argmax())
        for ids in list(_many_bad_seeds(n, count).values()) + [torch.full((count,), hub, dtype=torch.int32), torch.arange(1700, dtype=torch.int32) % 850]:
            seeds = ids.cuda()
            B.gns_sample_blocks_async(gns.ctx, 5, seeds, gns.blocks.array)
            x = torch.empty((gns.blocks.array[last].cap_src, 8), device=gns.device)
            h = torch.empty((gns.blocks.array[last].cap_dst, 8), device=gns.device)
            B.gns_gather_features(gns.ctx, gns.blocks.tensors[last]["src_nodes"], -1, x)
            B.gns_aggregate(gns.ctx, gns.blocks.array[last], x, 8, h)
            for wait in (lambda: B.gns_sample_blocks_wait(gns.ctx, gns.blocks.array),
                         lambda: B.gns_sample_blocks_static(gns.ctx, 5, seeds, gns.blocks.array)):
                with pytest.raises(B.GnsError) as e:
                    wait()
                assert e.value.status == B.GNS_EINVAL
                assert untouched()
                assert all(b.num_dst <= b.cap_dst and b.num_src <= b.cap_src and b.num_edges <= b.cap_edges for b in gns.blocks.array)
            full_parity(gns, cache_seed=48, epoch=0, batch_seed=6, seeds=torch.arange(1, n, dtype=torch.int32))
            assert untouched()
    finally:
        gns.close()


@pytest.mark.parametrize("n,avg", [(60_000, 40), (1_400_000, 6)])
@pytest.mark.parametrize("sizes", [(1,) * 16, (1, 90, 2, 300), (400, 1, 1, 1, 400), (3000, 1, 2900, 7, 3000, 1)])
def test_lists_of_chunks_of_a_group_shared_out_as_one(sizes, n, avg):
    """The waves' parts go on from one mini-batch's list to the next, in short lists and in long ones: lists of one row between
    others, lists that all fall to a few waves, and one that begins and ends in the middle of parts."""
    ip, ix = random_symmetric_csr(n, avg, np.random.default_rng(n + 1))
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    fanouts, policies, csize = (10, 5), (U, C), n // 50
    gns = GpuGns(ip, ix, None, fanouts=fanouts, policies=policies, cache_size=csize, max_seeds=max(sizes), flag_mode=0)
    ctxs, keep, bufs, call = _group_setup(gns, len(sizes))
    try:
        B.gns_sample_cache(gns.ctx, 49, 0)
        cache = oracle.sample_cache(ip.numpy(), 49, 0, csize)
        for rnd in range(2):
            seeds = [synth.uniform_seed_batch(n, size, 520 + 20 * rnd + b).cuda() for b, size in enumerate(sizes)]
            call.sample([80 + b for b in range(len(sizes))], seeds)
            call.wait()
            for b in range(len(sizes)):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 80 + b, seeds[b].cpu().numpy(), list(fanouts), list(policies))
                compare_blocks([bufs[b].views(j) for j in range(2)], ref)
    finally:
        for f in ctxs[1:]:
            B.gns_destroy(f)
        gns.close()


@pytest.mark.parametrize("n,degrees,hot", [(1_310_000, (0,), True), (1_310_000, (1023, 1, 0), True), (1_310_001, (0, 1024, 0, 2049, 5, 0), False),
                                           (3000, (0, 0, 0, 7), False), (26_625, (1023, 1, 0), False)])
def test_walk_windows_beyond_lds_and_without_the_hot_nodes(n, degrees, hot, monkeypatch):
    """The windows above where the training nodes' bits do not fit LDS, so that entries outside a list ask for none; and the
    steps on 32-bit values without the hot nodes' table, which graphs of more than 1.7 G nodes take."""
    if not hot:
        monkeypatch.setenv("GNS_WALK_NO_HOT", "1")
    rng = np.random.default_rng(n + len(degrees))
    deg = np.zeros(n, dtype=np.int64)
    deg[500:700] = [degrees[i % len(degrees)] for i in range(200)]
    deg[[3, 64, 1200]] = (17, 1024, 33)
    if n > 3000:
        deg[-70_000 if n > 100_000 else -20_000:-1] += rng.integers(0, 12, size=69_999 if n > 100_000 else 19_999)
    ip = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    ix = np.concatenate([np.unique(rng.integers(0, n, size=4 * d + 64))[:d] if d < n // 8 else np.sort(rng.choice(n, d, replace=False)) for d in deg if d]).astype(np.int32)
    assert len(ix) == ip[-1]
    ip, ix = torch.from_numpy(ip), torch.from_numpy(ix)
    gns = GpuGns(ip, ix, None, fanouts=(3, 2, 4), policies=(U, U, C), cache_size=2, max_seeds=8, cache_probability=B.GNS_PROB_WALK)
    try:
        train = torch.arange(1, n, 3, dtype=torch.int32)
        for scale in (20, 33):
            w, pre, _, _ = gns.walk_probability(train, scale)
            w_ref, pre_ref = oracle.walk_weights(ip.numpy(), ix.numpy(), train.numpy(), [3, 2, 4], scale_log2=scale)
            assert np.array_equal(w, w_ref) and np.array_equal(pre, pre_ref)
    finally:
        gns.close()


@pytest.mark.parametrize("offset", [0, 256, 4096 - 256, 3 * 4096, 7 * 4096 + 256])
def test_workspaces_at_any_place(offset):
    """A context's scratch begins at a place of its own in its workspace: workspaces of just the bytes asked for, which lie
    differently to the pages, hold it with all that is behind it; one byte less is refused."""
    ip, ix = _small(n=2500, avg=11, seed=79)
    n, csize, bs, place, guard = 2500, 200, 70, 1 << 15, 4096
    dev = torch.device("cuda:0")
    feat = _feat(n, 8).to(dev)
    ipd, ixd = ip.to(dev), ix.to(dev)
    graph, config = B.make_graph(ipd, ixd, feat), B.make_config([12, 5], [U, C], csize, bs, flag_mode=1)
    room = []

    def workspace(size):
        room.append((torch.full((size + 2 * place + guard,), 77, dtype=torch.uint8, device=dev), size))
        begin = -room[-1][0].data_ptr() % place + offset
        room[-1] += (begin,)
        return room[-1][0][begin:begin + size]

    size = B.gns_workspace_bytes(graph, config)
    with pytest.raises(B.GnsError) as e:
        B.gns_create(graph, config, workspace(size)[:-1])
    assert e.value.status == B.GNS_ECAPACITY
    ctxs = [B.gns_create(graph, config, workspace(size))]
    try:
        need = B.gns_fork_workspace_bytes(ctxs[0])
        with pytest.raises(B.GnsError) as e:
            B.gns_fork(ctxs[0], workspace(need)[:-1])
        assert e.value.status == B.GNS_ECAPACITY
        ctxs += [B.gns_fork(ctxs[0], workspace(need)) for _ in range(9)]
        bufs = [B.BlockBuffers(graph, config, dev) for _ in ctxs]
        cache = oracle.sample_cache(ip.numpy(), 50, 0, csize)
        B.gns_sample_cache(ctxs[0], 50, 0)
        call = B.GroupCall(ctxs, [b.array for b in bufs])
        seeds = [synth.uniform_seed_batch(n, bs, 700 + b).cuda() for b in range(len(ctxs))]
        for rnd in range(2):
            call.sample([90 + b for b in range(len(ctxs))], seeds)
            call.wait()
            for b in range(len(ctxs)):
                ref = oracle.sample_blocks(ip.numpy(), ix.numpy(), cache[1], csize, 90 + b, seeds[b].cpu().numpy(), [12, 5], [U, C])
                compare_blocks([bufs[b].views(j) for j in range(2)], ref)
        for t, size, begin in room:
            assert bool((t[:begin] == 77).all()) and bool((t[begin + size:] == 77).all())
    finally:
        for c in reversed(ctxs):
            B.gns_destroy(c)

"""Calls whose time follows from what they are given, whatever a graph's mean degree or a tuned size would suggest: kernel
durations (least of several) of two calls beside each other, with results against the CPU oracle."""
import numpy as np
import pytest

import chain
import oracle
from paper_2101_07706_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2101_07706_amd import csgs
    csgs.lib()
    return torch.device("cuda:0")


def _least_us(call, kernels, reps=10):
    """Sum over `kernels` of the least duration of a launch, in us."""
    from paper_2101_07706_amd import csgs
    call()
    torch.cuda.synchronize()
    csgs.csgs_profile_enable(True)
    for _ in range(reps):
        call()
    torch.cuda.synchronize()
    samples = csgs.csgs_profile_samples()
    csgs.csgs_profile_collect()
    csgs.csgs_profile_enable(False)
    return sum(min(samples[k]) for k in kernels if k in samples) * 1e3


def _hub_graph(rng, n, mean, hubs, hub_degree):
    """A graph whose rows have `mean` edges, but for `hubs` of them."""
    deg = np.full(n, mean)
    hub_rows = np.sort(rng.choice(n, hubs, replace=False)).astype(np.int32)
    deg[hub_rows] = hub_degree
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    step = np.repeat(n // deg, deg)
    col = (np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], deg)) * step + (rng.random(int(rowptr[-1])) * step).astype(np.int64)
    val = (1.0 / np.repeat(deg, deg)).astype(np.float32)
    return synth.Graph(n, rowptr, col.astype(np.int32), val, synth.partition_bounds(n, 8), 0, 1.0), hub_rows


# A million edges in a few rows of a sparse graph against the same number in ordinary rows.
def test_weight_scan_of_hub_rows(dev):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(11)
    n, mean, hubs, hub_degree = 200_000, 8, 256, 4000
    g, hub_rows = _hub_graph(rng, n, mean, hubs, hub_degree)
    ordinary = np.sort(rng.choice(np.setdiff1d(np.arange(n), hub_rows), hubs * hub_degree // mean, replace=False)).astype(np.int32)
    dg = pipeline.DeviceGraph(g, dev)
    us = []
    for S in (ordinary, hub_rows):
        print(f"[scan] {len(S)} rows", flush=True)
        ws = pipeline.Workspace(n, len(S), 1, g.nnz, dev)
        lb = pipeline.LayerBuffers(len(S), 1, n, 1, 8, dev)
        Sd = torch.from_numpy(S).to(dev)
        us.append(_least_us(lambda: csgs.csgs_build_probs(dg.c, Sd, 4.0, lb.cand_id, lb.cand_w, lb.cdf, None, lb.stats, ws.desc, lb.status),
                            ("scan_edges", "cand_partials")))
        want = oracle.build_probs(g, S, 4.0)
        n_c = len(want.cand_id)
        assert int(lb.status.item()) == 0 and int(lb.stats_host().n_cand) == n_c
        np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
        np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
    print(f"[scan] ordinary {us[0]:.1f} us, hubs {us[1]:.1f} us")
    assert us[1] < 2.0 * us[0]


# The sampled adjacency of the same two sets of rows.
def test_sampled_adjacency_of_hub_rows(dev):
    from types import SimpleNamespace
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(12)
    n, mean, hubs, hub_degree, B = 200_000, 8, 256, 4000, 1000
    g, hub_rows = _hub_graph(rng, n, mean, hubs, hub_degree)
    ordinary = np.sort(rng.choice(np.setdiff1d(np.arange(n), hub_rows), hubs * hub_degree // mean, replace=False)).astype(np.int32)
    dg = pipeline.DeviceGraph(g, dev)
    ids = np.arange(n, dtype=np.int32)
    cdf = np.cumsum(rng.integers(1, 1 << 20, n), dtype=np.uint64)
    draw = oracle.draw_nodes(SimpleNamespace(cand_id=ids, cdf=cdf), B, 5, 1, 0)
    ws = pipeline.Workspace(n, len(ordinary), B, g.nnz, dev)
    i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)
    S_next, mult, n_next, status, p = i32(B), i32(B), i32(1), i32(1), torch.zeros(B, dtype=torch.float32, device=dev)
    st = torch.frombuffer(bytearray(bytes(csgs.ProbStats(n_cand=n, total=int(cdf[-1])))), dtype=torch.int64).to(dev)
    csgs.csgs_draw_nodes(n, torch.from_numpy(ids).to(dev), torch.from_numpy(cdf.view(np.int64)).to(dev), st, B, 5, 1, 0, S_next, mult, p, n_next,
                         ws.desc, status)
    us = []
    for S in (ordinary, hub_rows):
        print(f"[adjacency] {len(S)} rows", flush=True)
        want = oracle.sampled_adjacency(g, S, draw)
        cap = want.adj_nnz + 5
        rp, ac, av, nnz = i32(len(S) + 1), i32(cap), torch.zeros(cap, dtype=torch.float32, device=dev), torch.zeros(1, dtype=torch.int64, device=dev)
        Sd = torch.from_numpy(S).to(dev)
        us.append(_least_us(lambda: csgs.csgs_sampled_adjacency(dg.c, Sd, rp, ac, av, nnz, ws.desc, status), ("adj_once", "adj_mark", "adj_place")))
        assert int(status.item()) == 0 and int(nnz.item()) == want.adj_nnz
        np.testing.assert_array_equal(rp.cpu().numpy(), want.adj_rowptr)
        np.testing.assert_array_equal(ac[:want.adj_nnz].cpu().numpy(), want.adj_col)
        chain.assert_close(av[:want.adj_nnz].cpu().numpy(), want.adj_val, chain.P_RTOL, 0.0, "adj_val")
    print(f"[adjacency] ordinary {us[0]:.1f} us, hubs {us[1]:.1f} us")
    assert us[1] < 2.0 * us[0]


# The compaction of the drawn positions reads a bitmap of one bit per candidate: sixteen times the candidates, sixteen times
# the bits at most.
def test_draw_from_many_candidates(dev):
    from paper_2101_07706_amd import csgs, pipeline
    B, us = 8192, []
    for n_c in (16_000_000, 256_000_000):
        print(f"[draw] {n_c} candidates", flush=True)
        ws = pipeline.Workspace(n_c, 1, B, 1, dev)
        ids = torch.arange(n_c, dtype=torch.int32, device=dev)
        cdf = torch.arange(1, n_c + 1, dtype=torch.int64, device=dev) * 1000003
        st = torch.frombuffer(bytearray(bytes(csgs.ProbStats(n_cand=n_c, total=n_c * 1000003))), dtype=torch.int64).to(dev)
        i32 = lambda k: torch.zeros(k, dtype=torch.int32, device=dev)
        S_next, mult, n_next, status, p = i32(B), i32(B), i32(1), i32(1), torch.zeros(B, dtype=torch.float32, device=dev)
        us.append(_least_us(lambda: csgs.csgs_draw_nodes(n_c, ids, cdf, st, B, 5, 1, 0, S_next, mult, p, n_next, ws.desc, status), ("hits",)))
        m = int(n_next.item())
        assert int(status.item()) == 0 and int(mult[:m].sum().item()) == B and bool((S_next[1:m] > S_next[:m - 1]).all())
        del ws, ids, cdf
    print(f"[draw] {us[0]:.1f} us, {us[1]:.1f} us")
    assert us[1] < 8.0 * us[0]


# The transpose of the aggregation gradient reads its columns' counts a bounded number of times.
def test_gradient_with_many_columns(dev):
    from paper_2101_07706_amd import csgs
    nS, F, us = 4096, 8, []
    gen = torch.Generator(device=dev).manual_seed(7)
    for n_cols in (4_000_000, 64_000_000):
        print(f"[aggregate grad] {n_cols} columns", flush=True)
        rp = (torch.arange(nS + 1, device=dev) * 4).to(torch.int32)
        col = torch.randperm(n_cols, generator=gen, device=dev)[:nS * 4].view(nS, 4).sort(1)[0].reshape(-1)   # a column of its own for every entry
        val = torch.rand(nS * 4, generator=gen, device=dev)
        dZ, dH = torch.randn((nS, F), generator=gen, device=dev), torch.full((n_cols, F), float("nan"), device=dev)
        scratch = torch.empty(csgs.csgs_aggregate_grad_scratch_bytes(n_cols, nS * 4) // 8 + 32, dtype=torch.int64, device=dev)
        c32 = col.to(torch.int32)
        us.append(_least_us(lambda: csgs.csgs_aggregate_grad(rp, c32, val, None, dZ, None, dH, scratch), ("adjT_prefix",), 3))
        want = (val[:, None].double() * dZ.double().repeat_interleave(4, 0)).float()
        assert bool((dH[col] == want).all()) and int(torch.count_nonzero(dH).item()) == int(torch.count_nonzero(want).item())
        del dH, scratch
    print(f"[aggregate grad] {us[0]:.1f} us, {us[1]:.1f} us")
    assert us[1] < 60.0 * us[0]


# The transpose in one launch beside the several launches of larger arrays (the same entries with more room behind them): never much
# dearer, with few entries, a column that thousands of rows share, several of those in one block, full arrays of many columns.
@pytest.mark.parametrize("nS,n_cols,entries,longest", [(8192, 8192, 20_000, 0), (16_384, 8192, 20_000, 1000), (16_384, 8192, 20_000, 8000), (65_536, 8192, 20_000, 60_000),
                                                       (65_536, 300, 60_000, 0), (16_384, 4, 50_000, 0), (65_536, 65_536, 390_000, 0), (65_536, 8192, 520_000, 0)])
def test_gradient_in_one_launch(dev, nS, n_cols, entries, longest):
    from paper_2101_07706_amd import csgs
    print(f"[aggregate grad] {entries} entries of {n_cols} columns, one of {longest}", flush=True)
    F, more, us, got = 8, (1 << 19) + 1, [], []
    gen = torch.Generator(device=dev).manual_seed(nS + longest)
    key = torch.randint(0, nS * n_cols, (entries,), generator=gen, device=dev)
    key = torch.unique(torch.cat([key, torch.randperm(nS, generator=gen, device=dev)[:longest] * n_cols + 5 % n_cols]))
    nnz, row = key.numel(), key // n_cols
    rp = torch.zeros(nS + 1, dtype=torch.int64, device=dev)
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=nS), 0)
    rp, col, val = rp.to(torch.int32), torch.zeros(more, dtype=torch.int32, device=dev), torch.rand(more, generator=gen, device=dev)
    col[:nnz] = (key % n_cols).to(torch.int32)
    dZ, dH = torch.randn((nS, F), generator=gen, device=dev), torch.empty((n_cols, F), device=dev)
    for cap in (nnz, more):
        scratch = torch.empty(csgs.csgs_aggregate_grad_scratch_bytes(n_cols, cap) // 8 + 32, dtype=torch.int64, device=dev)
        us.append(_least_us(lambda: csgs.csgs_aggregate_grad(rp, col[:cap], val[:cap], None, dZ, None, dH, scratch),
                            ("fill_zero", "adjT_count", "adjT_prefix", "adjT_fill", "adjT_order"), 4))
        got.append(dH.cpu().numpy())
    np.testing.assert_array_equal(got[0], got[1])   # the same transpose, summed by the same kernel
    chain.assert_close(got[0], oracle.aggregate_grad(rp.cpu().numpy(), col[:nnz].cpu().numpy(), val[:nnz].cpu().numpy(), n_cols, dZ.cpu().numpy(), None),
                       chain.RTOL, chain.ATOL, "dH")
    print(f"[aggregate grad] one launch {us[0]:.1f} us, several {us[1]:.1f} us")
    assert us[0] < 1.2 * us[1]


# Rows a little longer than those that a wavefront walks through: a tenth more edges, not half as much time again.  (2000 rows with
# F = 481: four rows a tile.)  A block of few rows: twice the edges in no more time, since all its wavefronts take part.
@pytest.mark.parametrize("fused,F,bf16,n_rows,short,longer", [(True, 128, False, 2048, 60, 66), (True, 128, False, 16_384, 60, 66), (False, 100, True, 65_536, 120, 132),
                                                              (False, 504, True, 65_536, 60, 66), (False, 481, False, 2000, 60, 66), (True, 128, False, 15, 60, 120)])
def test_rows_of_equal_length(dev, fused, F, bf16, n_rows, short, longer):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(F)
    n_cols, us = 100_000, []
    X = rng.standard_normal((n_cols, F)).astype(np.float32)
    Xh = synth.to_bf16_bits(X) if bf16 else X
    Xd = torch.from_numpy(Xh.view(np.int16) if bf16 else Xh).to(dev)
    W = rng.standard_normal((F, 64)).astype(np.float32)
    Wd, t = torch.from_numpy(W).to(dev), lambda a: torch.from_numpy(a).to(dev)
    for length in (short, longer):
        print(f"[rows] {n_rows} of {length} edges, F={F} bf16={bf16} fused={fused}", flush=True)
        rowptr = (np.arange(n_rows + 1) * length).astype(np.int32)
        col, val = rng.integers(0, n_cols, n_rows * length).astype(np.int32), rng.standard_normal(n_rows * length).astype(np.float32)
        rp, cd, vd = t(rowptr), t(col), t(val)
        Z, H = torch.zeros((n_rows, F), device=dev), torch.zeros((n_rows, 64), device=dev)
        if fused:
            us.append(_least_us(lambda: csgs.csgs_layer_forward(rp, cd, vd, None, Xd, None, None, True, Wd, H, Z), ("layer_forward",)))
        else:
            us.append(_least_us(lambda: csgs.csgs_aggregate(rp, cd, vd, None, Xd, None, None, True, Z), ("aggregate",)))
        few = 500
        want = oracle.aggregate(rowptr[:few + 1], col[:few * length], val[:few * length], Xh, relu_on_input=True)
        chain.assert_close(Z[:few].cpu().numpy(), want, chain.RTOL, chain.ATOL, f"{length} edges")
    print(f"[rows] {us[0]:.1f} us, {us[1]:.1f} us")
    assert us[1] < 1.3 * us[0]


# The split of the node set just sampled, with as many partitions as nodes sampled and more: level with a few partitions.
def test_remote_split_over_many_partitions(dev):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(13)
    n, B, us = 100_000, 200, []
    g, _ = _hub_graph(rng, n, 10, 1, 10)
    S = np.sort(rng.choice(n, B, replace=False)).astype(np.int32)
    for P in (8, 1024, 1500):
        print(f"[remote split] {P} partitions", flush=True)
        g.part_bounds = synth.partition_bounds(n, P)
        dg = pipeline.DeviceGraph(g, dev)
        ws, lb = pipeline.Workspace(n, B, B, g.nnz, dev), pipeline.LayerBuffers(B, B, n, 64 * B, P, dev)
        Sd = torch.from_numpy(S).to(dev)
        us.append(_least_us(lambda: pipeline.sample_step(dg, ws, Sd, 4.0, B, 5, 3, 0, lb), ("adj_once",)))
        m = int(lb.n_next.item())
        want = oracle.remote_count(lb.S_next[:m].cpu().numpy(), g.local_lo, g.local_hi, g.part_bounds)
        assert int(lb.status.item()) == 0 and int(lb.remote_total.item()) == want.remote_total
        np.testing.assert_array_equal(lb.per_part[:P].cpu().numpy(), want.per_part)
        np.testing.assert_array_equal(lb.src_row[:m].cpu().numpy(), want.src_row)
    print("[remote split] " + ", ".join(f"{u:.1f} us" for u in us))
    assert max(us[1:]) < 3.0 * us[0]


def _rows_by_target(rng, n, P, n_rows, degree, local_share):
    """`n_rows` rows of `degree` edges, row i with local_share[i] of them in the local range [0, n / P); the other rows are empty."""
    deg = np.zeros(n, np.int64)
    S = np.sort(rng.choice(n, n_rows, replace=False)).astype(np.int32)
    deg[S] = degree
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    local = rng.random((n_rows, degree)) < np.asarray(local_share)[:, None]
    col = np.where(local, rng.integers(0, n // P, (n_rows, degree)), rng.integers(n // P, n, (n_rows, degree)))
    col.sort(axis=1)
    return synth.Graph(n, rowptr, col.reshape(-1).astype(np.int32), np.full(n_rows * degree, 1.0 / degree, np.float32), synth.partition_bounds(n, P), 0, 1.0), S


# Few local targets: what the library chooses is level with atomics for all.  Chunks with local targets only beside chunks
# with hardly any: a call in which some chunks hand theirs over.
@pytest.mark.parametrize("P,n_rows,shares,timed", [(64, 16_000, (1 / 64, 1 / 64), True), (8, 4000, (1 / 8, 1 / 8), False), (2, 4000, (1.0, 0.02), False),
                                                   (2, 4000, (0.45, 0.41), False)])
def test_weight_scan_by_local_share(dev, P, n_rows, shares, timed):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(P + n_rows)
    n = 400_000
    g, S = _rows_by_target(rng, n, P, n_rows, 50, np.repeat(shares, n_rows // 2))
    dg, Sd = pipeline.DeviceGraph(g, dev), torch.from_numpy(S).to(dev)
    want = oracle.build_probs(g, S, 4.0)
    n_c, us = len(want.cand_id), {}
    for mode in (0, 1, 2):
        print(f"[scan] {n_rows} rows, local shares {shares}, mode {mode}", flush=True)
        ws, lb = pipeline.Workspace(n, n_rows, 1, g.nnz, dev, scan_mode=mode), pipeline.LayerBuffers(n_rows, 1, n, 1, 8, dev)
        us[mode] = _least_us(lambda: csgs.csgs_build_probs(dg.c, Sd, 4.0, lb.cand_id, lb.cand_w, lb.cdf, None, lb.stats, ws.desc, lb.status),
                             ("scan_edges", "cand_partials"))
        assert int(lb.status.item()) == 0 and int(lb.stats_host().n_cand) == n_c
        np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
        np.testing.assert_array_equal(lb.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
        np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
        assert int(torch.count_nonzero(ws.buf[:chain.csgs_clean_words(n)]).item()) == 0, "workspace not restored"
    print("[scan] " + ", ".join(f"mode {m} {u:.1f} us" for m, u in us.items()))
    if timed:
        assert us[0] < 1.2 * us[1]


def _scan_modes(dev, share, bins, n_rows, counts, kernels, limit):
    """csgs_build_probs for the first counts[i] of n_rows rows (8 edges each; 1.4 M nodes, one in eight local, four edges in five to those,
    `share` of all to the ids of `bins` blocks of the sums elsewhere): as the library chooses, against the form that sends remote edges through atomics."""
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(bins + int(100 * share))
    n, P, degree, at = 1_400_000, 8, 8, 146 * 4096
    kind, ids = rng.random((n, degree)), lambda lo, hi: rng.integers(lo, hi, (n, degree))
    col = np.where(kind < 0.8, ids(0, n // P), np.where(kind > 1 - share, ids(at, at + 4096 * bins), ids(n // P, n)))
    col.sort(axis=1)
    g = synth.Graph(n, np.arange(n + 1, dtype=np.int64) * degree, col.reshape(-1).astype(np.int32), np.full(n * degree, 1.0 / degree, np.float32), synth.partition_bounds(n, P), 0, 1.0)
    S = rng.permutation(n)[:n_rows].astype(np.int32)
    dg, Sd = pipeline.DeviceGraph(g, dev), torch.from_numpy(S).to(dev)
    for count in counts:
        want = oracle.build_probs(g, S[:count], 4.0)
        n_c, us, rows = len(want.cand_id), {}, torch.tensor([count], dtype=torch.int32, device=dev)
        for mode in (0, 2):
            print(f"[scan] {share:.0%} of the edges in {bins} blocks' ids, {count} rows, mode {mode}", flush=True)
            ws, lb = pipeline.Workspace(n, n_rows, 1, g.nnz, dev, scan_mode=mode), pipeline.LayerBuffers(n_rows, 1, n, 1, 8, dev)
            us[mode] = _least_us(lambda: csgs.csgs_build_probs(dg.c, Sd, 4.0, lb.cand_id, lb.cand_w, lb.cdf, None, lb.stats, ws.desc, lb.status, nS_dev=rows), kernels)
            assert int(lb.status.item()) == 0 and int(lb.stats_host().n_cand) == n_c
            np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
            np.testing.assert_array_equal(lb.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
            np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
            assert int(torch.count_nonzero(ws.buf[:chain.csgs_clean_words(n)]).item()) == 0, "workspace not restored"
        print(f"[scan] {share:.0%} in {bins}, {count} rows: mode 0 {us[0]:.1f} us, mode 2 {us[2]:.1f} us")
        assert us[0] < limit * us[2]


# Many edges, sorted by the block that sums their targets: some of them crowded into few blocks' ids outside the local range.
@pytest.mark.parametrize("share,bins", [(0.0, 1), (0.02, 1), (0.05, 1), (0.12, 1), (0.1, 8), (0.18, 64)])
def test_weight_scan_of_crowded_targets(dev, share, bins):
    _scan_modes(dev, share, bins, 400_000, [400_000], ("scan_edges", "cand_partials"), 1.25)


# Room for many rows, of which the device has few: runs of one, two and four steps, a last run that is short.
def test_weight_scan_of_few_of_many_rows(dev):
    _scan_modes(dev, 0.0, 1, 400_000, [40, 3000, 50_000, 131_072, 131_200, 200_000, 262_300], ("scan_edges", "cand_partials", "cand_emit"), 1.2)


# Thousands of rows without edges before, between and behind the ones that have some, by both forms of the weight scan: little dearer than the rows with
# edges alone, and the same candidates and entries.
@pytest.mark.parametrize("n,k,degree,first,limit", [(200_000, 10_000, 20, 190_000, 4.0), (200_000, 10_000, 20, 0, 4.0), (1_000_000, 50_000, 1, None, 5.0),
                                                    (1_400_000, 100_000, 32, 1_300_000, 2.0)])
def test_scan_of_rows_without_edges(dev, n, k, degree, first, limit):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(n + k)
    B, us = 500, []
    with_edges = np.arange(first, first + k) if first is not None else np.sort(rng.permutation(n)[:k])
    deg = np.zeros(n, np.int64)
    deg[with_edges] = degree
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = np.sort(rng.integers(0, n, (k, degree)), axis=1).reshape(-1).astype(np.int32)
    g = synth.Graph(n, rowptr, col, np.full(k * degree, 1.0 / degree, np.float32), synth.partition_bounds(n, 8), 0, 1.0)
    dg = pipeline.DeviceGraph(g, dev)
    ws, lb = pipeline.Workspace(n, n, B, g.nnz, dev), pipeline.LayerBuffers(n, B, n, g.nnz, 8, dev)
    for S in (with_edges.astype(np.int32), np.arange(n, dtype=np.int32)):
        print(f"[scan] {len(S)} rows, {k} with {degree} edges", flush=True)
        Sd = torch.from_numpy(S).to(dev)
        us.append(_least_us(lambda: pipeline.sample_step(dg, ws, Sd, 4.0, B, 5, 3, 0, lb), ("scan_edges",)))
        want = oracle.build_probs(g, S, 4.0)
        step, n_c = oracle.sample_layer(g, S, want, B, 5, 3, 0), len(want.cand_id)
        assert int(lb.status.item()) == 0 and int(lb.n_next.item()) == step.n_next and int(lb.adj_nnz.item()) == step.adj_nnz
        np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
        np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
        np.testing.assert_array_equal(lb.adj_rowptr[:len(S) + 1].cpu().numpy(), step.adj_rowptr)
        np.testing.assert_array_equal(lb.adj_col[:step.adj_nnz].cpu().numpy(), step.adj_col)
    print(f"[scan] alone {us[0]:.1f} us, among the others {us[1]:.1f} us")
    assert us[1] < limit * us[0]


# More edges than are handed over (8 Mi), just and by a quarter: whole runs go through the atomics, into the sums of the others.
def test_weight_scan_beyond_the_hand_over(dev):
    _scan_modes(dev, 0.05, 1, 1_310_000, [1_050_000, 1_310_000], ("scan_edges", "cand_partials", "cand_emit"), 1.3)


# Several instances of which one has most of the rows, beside as many rows shared out evenly: the device works on the large one as a whole.
def test_uneven_instances(dev):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(3)
    n, P, degree, B, K, nS = 400_000, 8, 40, 4096, 8, 32_768
    col = np.where(rng.random((n, degree)) < 0.8, rng.integers(0, n // P, (n, degree)), rng.integers(n // P, n, (n, degree)))
    col.sort(axis=1)
    g = synth.Graph(n, np.arange(n + 1, dtype=np.int64) * degree, col.reshape(-1).astype(np.int32), np.full(n * degree, 1.0 / degree, np.float32), synth.partition_bounds(n, P), 0, 1.0)
    dg, us = pipeline.DeviceGraph(g, dev), []
    lb = pipeline.LayerBuffers(nS, B, n, 64 * B, P, dev, n_inst=K)
    ws = pipeline.Workspace(n, nS, B, 2 * degree * nS, dev, n_inst=K, inst_stride=lb.stride)
    S = [rng.permutation(n)[:nS].astype(np.int32) for _ in range(K)]
    for counts in ([(nS + 7 * 2048) // K] * K, [2048] * 3 + [nS] + [2048] * 4):
        print(f"[instances] {counts} rows", flush=True)
        for k in range(K):
            lb.inst(k).S0.copy_(torch.from_numpy(S[k]).to(dev))
            lb.inst(k).q.view(torch.int32)[0] = counts[k]   # (a word of the instance's that the step leaves alone)
        us.append(_least_us(lambda: pipeline.sample_step(dg, ws, lb.S0, 4.0, B, 5, 3, 0, lb, want_q=False, nS_dev=lb.q.view(torch.int32)[:1]),
                            ("scan_edges", "cand_partials", "cand_emit", "draw", "hits", "adj_mark", "adj_place")))
        for k in (0, 3):
            want, one = oracle.build_probs(g, S[k][:counts[k]], 4.0), lb.inst(k)
            step = oracle.sample_layer(g, S[k][:counts[k]], want, B, 5, 3 + k, 0)
            m, nnz = step.n_next, step.adj_nnz
            assert int(one.status.item()) == 0 and int(one.n_next.item()) == m and int(one.adj_nnz.item()) == nnz
            np.testing.assert_array_equal(one.S_next[:m].cpu().numpy(), step.S_next)
            np.testing.assert_array_equal(one.adj_rowptr[:counts[k] + 1].cpu().numpy(), step.adj_rowptr)
            np.testing.assert_array_equal(one.adj_col[:nnz].cpu().numpy(), step.adj_col)
    print(f"[instances] even {us[0]:.1f} us, uneven {us[1]:.1f} us")
    assert us[1] < 1.5 * us[0]

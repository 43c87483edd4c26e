"""The sizes at which a call changes the shape of its launch, against the CPU oracle: edges of tiles, remainders, the
smallest and largest size of each variant.  Tolerances as in test_gpu_parity.py."""
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


def _csr(rng, lens, n_cols):
    rowptr = np.zeros(len(lens) + 1, np.int32)
    np.cumsum(lens, out=rowptr[1:])
    return rowptr, rng.integers(0, n_cols, int(rowptr[-1])).astype(np.int32), rng.standard_normal(int(rowptr[-1])).astype(np.float32)


# F, its type and its slices pick the lanes per row (4, 8, 16, 32, 64).  A wavefront takes 8 rows per lane group (at most 64),
# half as many until the launch has 512 blocks of four wavefronts: the row counts on both sides of every halving.
def _rows_around_halvings(lanes, slices):
    most, least = min(64 // lanes * 8, 64), max(64 // lanes // 2, 2)
    edges, tr = [], most
    while tr > least:
        last = 4 * tr * ((512 + slices - 1) // slices - 1)     # rows with which `tr` rows a wavefront are too few blocks still
        edges += [last, last + 1]
        tr //= 2
    return edges


@pytest.mark.parametrize("F,bf16,lanes,slices,rows", [(32, False, 4, 1, (1, 65, 700)), (64, False, 8, 1, (1, 33)), (256, False, 8, 4, (1, 9)),
                                                      (128, False, 16, 1, (7,)), (100, True, 32, 1, (3,)), (75, False, 64, 2, (1,)),
                                                      (264, True, 64, 1, (1, 5)), (504, True, 64, 1, (700,))])
def test_aggregate_rows_per_wavefront(dev, F, bf16, lanes, slices, rows):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(31 * F)
    n_cols = 3000
    X = rng.standard_normal((n_cols, F)).astype(np.float32)
    Xh = synth.to_bf16_bits(X) if bf16 else X
    Xd = torch.from_numpy(Xh.view(np.int16) if bf16 else Xh).to(dev)
    for n in rows + tuple(_rows_around_halvings(lanes, slices)):
        print(f"[aggregate] {n} rows, F={F} bf16={bf16}", flush=True)
        lens = rng.poisson(2, n)
        lens[rng.integers(0, n, 4)] = (0, 300, 257, 90)       # the block-wide path, and rows longer than a share
        rowptr, col, val = _csr(rng, lens, n_cols)
        want = oracle.aggregate(rowptr, col, val, Xh, relu_on_input=True)
        Z = torch.full((n + 3, F), float("nan"), dtype=torch.float32, device=dev)
        t = lambda a: torch.from_numpy(a).to(dev)
        csgs.csgs_aggregate(t(rowptr), t(col), t(val), None, Xd, None, None, True, Z[:n])
        torch.cuda.synchronize()
        chain.assert_close(Z[:n].cpu().numpy(), want, chain.RTOL, chain.ATOL, f"aggregate {n} rows F={F}")
        assert bool(torch.isnan(Z[n:]).all()), f"{n} rows: wrote past the last row"


# Rows around the lengths from which a block takes them together (256, and from 64 or 128 on by the lanes per row where the
# tile's other rows are shorter) and around its rounds of 256 edges, in 1, 3, 4 and 5 feature slices; columns outside the table; output rows closer and further apart than 2^24
@pytest.mark.parametrize("F,bf16,ld", [(256, False, 0), (300, False, 0), (602, False, 0), (100, True, 0), (640, True, 0), (264, True, 0), (504, True, 0),
                                       (64, False, (1 << 24) + 8),
                                       (64, False, (1 << 24) - 8)])
def test_aggregate_long_rows(dev, F, bf16, ld):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(F + ld)
    n_cols = 900
    X = rng.standard_normal((n_cols, F)).astype(np.float32)
    Xh = synth.to_bf16_bits(X) if bf16 else X
    Xd = torch.from_numpy(Xh.view(np.int16) if bf16 else Xh).to(dev)
    lens = np.array([64, 65, 0, 128, 129, 255, 256, 257, 1, 63, 511, 513, 5000])
    print(f"[aggregate] long rows, F={F} bf16={bf16} ld={ld}", flush=True)
    rowptr, col, val = _csr(rng, lens, n_cols)
    out = rng.random(len(col)) < 0.1                             # edges that must not count
    want = oracle.aggregate(rowptr, col, np.where(out, 0, val).astype(np.float32), Xh, relu_on_input=True)
    col[out] = rng.choice([-1, n_cols, 2**31 - 1], int(out.sum()))
    ld = ld or F
    Z = torch.as_strided(torch.full((len(lens) * ld,), float("nan"), dtype=torch.float32, device=dev), (len(lens), F), (ld, 1))
    t = lambda a: torch.from_numpy(a).to(dev)
    csgs.csgs_aggregate(t(rowptr), t(col), t(val), None, Xd, None, None, True, Z)
    torch.cuda.synchronize()
    chain.assert_close(Z.cpu().numpy(), want, chain.RTOL, chain.ATOL, f"long rows F={F}")


# Candidate counts at the ends of bitmap words, of a block's 16 words, and where the blocks (512, 16 words each) begin to take
# more words and then more than 64 at a time; budgets from a few hits to every position drawn, several draws in a row on one
# workspace (the position bitmap of one draw is cleared by the next)
@pytest.mark.parametrize("n_nodes,cases", [(1, ((1, 5),)), (1100, ((64, 3), (1023, 900), (65, 4000), (1, 7), (1025, 256))),
                                           (600_000, ((524_288, 3000), (524_289, 5000), (1025, 20_000), (600_000, 70_000))),
                                           (2_200_000, ((2_097_153, 9000), (2_200_000, 1), (100, 100))),
                                           # ... and where the prefix comes from the scan across blocks (beyond 49152 words)
                                           (3_300_000, ((3_145_728, 9000), (3_145_729, 9000), (1000, 500), (3_300_000, 100_000), (3_200_001, 1))),
                                           # ... and around the 256 samples of the CDF and the 128 draws of a block
                                           (1100, ((255, 127), (256, 128), (257, 129), (511, 300), (512, 300), (513, 300))),
                                           (70_000, ((2047, 4000), (2049, 4000), (16_641, 4000), (65_537, 4000)))])
def test_draws_by_candidate_count(dev, n_nodes, cases):
    from types import SimpleNamespace
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(n_nodes)
    B_max = max(B for _, B in cases)
    ws = pipeline.Workspace(n_nodes, 1, B_max, 1, dev)
    clean = chain.csgs_clean_words(n_nodes)
    for it, (n_c, B) in enumerate(cases):
        print(f"[draw] {n_c} candidates of {n_nodes} nodes, {B} draws", flush=True)
        ids = np.sort(rng.choice(n_nodes, n_c, replace=False)).astype(np.int32)
        cdf = np.cumsum(rng.integers(1, 1 << 30, n_c), dtype=np.uint64)
        want = oracle.draw_nodes(SimpleNamespace(cand_id=ids, cdf=cdf), B, 99, it, 2)
        stats = csgs.ProbStats(n_cand=n_c, total=int(cdf[-1]))
        st = torch.frombuffer(bytearray(bytes(stats)), dtype=torch.int64).to(dev)
        i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)
        S_next, mult, n_next, status, p = i32(B), i32(B), i32(1), i32(1), torch.zeros(B, dtype=torch.float32, device=dev)
        csgs.csgs_draw_nodes(n_nodes, torch.from_numpy(ids).to(dev), torch.from_numpy(cdf.view(np.int64)).to(dev), st, B, 99, it, 2, S_next, mult,
                             p, n_next, ws.desc, status)
        torch.cuda.synchronize()
        m = want.n_next
        assert int(n_next.item()) == m and int(status.item()) == 0
        np.testing.assert_array_equal(S_next[:m].cpu().numpy(), want.S_next)
        np.testing.assert_array_equal(mult[:m].cpu().numpy(), want.mult)
        chain.assert_close(p[:m].cpu().numpy(), want.p_incl, chain.P_RTOL, 0.0, "p_incl")
        assert int(torch.count_nonzero(S_next[m:]).item()) == 0, "wrote past the last hit"
        assert int(torch.count_nonzero(ws.buf[:clean]).item()) == 0, "workspace not restored"


# Calls whose edges exceed what the marking pass can leave for the placing pass (8 Mi edges), and the sizes around the
# choice between one pass and two (256 expected chunks of 1024 edges), with rows that have no edges at both ends
@pytest.mark.parametrize("n_nodes,degree,rows", [(70_000, 130, (70_000, 69_000, 1)), (20_000, 40, (0.29, 4000, 5300, 6500, 20_000))])
def test_sampled_adjacency_sizes(dev, n_nodes, degree, rows):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(n_nodes)
    deg = rng.poisson(degree, n_nodes)
    deg[[0, 1, 777, n_nodes - 2, n_nodes - 1]] = (0, 3000, 0, 1, 0)
    rowptr = np.zeros(n_nodes + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = rng.integers(0, n_nodes, int(rowptr[-1])).astype(np.int32)
    order = np.argsort(np.repeat(np.arange(n_nodes, dtype=np.int64), deg) * n_nodes + col, kind="stable")
    g = synth.Graph(n_nodes, rowptr, col[order], rng.uniform(0.01, 0.2, len(col)).astype(np.float32), synth.partition_bounds(n_nodes, 4), 0, 100.0)
    B = 900
    n_c = n_nodes // 2
    ids = np.sort(rng.choice(n_nodes, n_c, replace=False)).astype(np.int32)
    cdf = np.cumsum(rng.integers(1, 1 << 20, n_c), dtype=np.uint64)
    from types import SimpleNamespace
    draw = oracle.draw_nodes(SimpleNamespace(cand_id=ids, cdf=cdf), B, 5, 1, 0)
    dg = pipeline.DeviceGraph(g, dev)
    ws = pipeline.Workspace(n_nodes, n_nodes, B, g.nnz, dev)
    i32 = lambda n: torch.zeros(n, dtype=torch.int32, device=dev)
    S_next, mult, n_next, status, p = i32(B), i32(B), i32(1), i32(1), torch.zeros(B, dtype=torch.float32, device=dev)
    st = torch.frombuffer(bytearray(bytes(csgs.ProbStats(n_cand=n_c, total=int(cdf[-1])))), dtype=torch.int64).to(dev)
    csgs.csgs_draw_nodes(n_nodes, torch.from_numpy(ids).to(dev), torch.from_numpy(cdf.view(np.int64)).to(dev), st, B, 5, 1, 0, S_next, mult, p, n_next,
                         ws.desc, status)
    for n_rows in rows:
        # 0.29: rows without any edge
        sel = np.array([0, 777, n_nodes - 1], np.int32) if n_rows == 0.29 else rng.permutation(n_nodes)[:n_rows].astype(np.int32)
        print(f"[adjacency] {len(sel)} rows, {int(deg[sel].sum())} edges", flush=True)
        want = oracle.sampled_adjacency(g, sel, draw)
        cap = max(want.adj_nnz, 1) + 5
        rp, ac, av, nnz = i32(len(sel) + 1), i32(cap), torch.zeros(cap, dtype=torch.float32, device=dev), torch.zeros(1, dtype=torch.int64, device=dev)
        csgs.csgs_sampled_adjacency(dg.c, torch.from_numpy(sel).to(dev), rp, ac, av, nnz, ws.desc, status)
        torch.cuda.synchronize()
        assert int(status.item()) == 0 and int(nnz.item()) == want.adj_nnz
        np.testing.assert_array_equal(rp.cpu().numpy(), want.adj_rowptr)
        np.testing.assert_array_equal(ac[:want.adj_nnz].cpu().numpy(), want.adj_col)
        chain.assert_close(av[:want.adj_nnz].cpu().numpy(), want.adj_val, chain.P_RTOL, 0.0, "adj_val")
        assert int(torch.count_nonzero(ac[want.adj_nnz:]).item()) == 0, "wrote past the last kept edge"


# The weight scan's hand-over: local ranges that begin and end inside tiles of 1024 ids (one tile, many, the most it
# takes and one more), a tile's sums split over several blocks, weights too large for a handed-over entry (2^54; four rows
# whose norm is one edge's), more edges than it takes (8 Mi), and hardly any edge; by every form of the scan
@pytest.mark.parametrize("n_nodes,degree,n_rows,lo,hi,skew", [
    (6000, 60, 5000, 1000, 2050, 2.0),         # three tiles, blocks of several shares each
    (6000, 60, 5000, 1023, 1025, 8.0), (6000, 1.5, 4, 0, 6000, 1.0), (700, 0.01, 700, 5, 690, 1.0),
    (400_000, 3, 60_000, 1, 327_681, 2.0), (400_000, 3, 60_000, 1023, 327_681, 2.0),   # 321 and 320 tiles
    (70_000, 130, 70_000, 511, 30_001, 2.0),
    (1_048_576, 3, 40_000, 6500, 300_001, 2.0), (1_048_577, 3, 70_000, 6500, 300_001, 2.0), (1_048_577, 3, 70_000, 4096, 8192, 4.0),   # one and four tiles per block
])
def test_weight_scan_hand_over(dev, n_nodes, degree, n_rows, lo, hi, skew):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(n_nodes + hi)
    deg = rng.poisson(degree, n_nodes)
    rowptr = np.zeros(n_nodes + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = np.where(rng.random(int(rowptr[-1])) < 0.5, rng.integers(0, n_nodes, int(rowptr[-1])), rng.integers(lo, hi, int(rowptr[-1])))
    order = np.argsort(np.repeat(np.arange(n_nodes, dtype=np.int64), deg) * n_nodes + col, kind="stable")
    val = rng.uniform(0.01, 1.0, len(col)).astype(np.float32)
    if n_rows == 4:
        val[::2] = 33.0
    bounds = np.array(sorted({0, lo, hi, n_nodes}), np.int32)
    g = synth.Graph(n_nodes, rowptr, col[order].astype(np.int32), val, bounds, int(np.flatnonzero(bounds == lo)[0]))
    S = rng.permutation(n_nodes)[:n_rows].astype(np.int32)
    if n_rows == 4:
        S = np.flatnonzero(deg == 1)[:4].astype(np.int32)
    g.rownorm2_max = max(float(np.square(val[rowptr[i]:rowptr[i + 1]], dtype=np.float64).sum()) for i in S) * 1.001
    assert (g.local_lo, g.local_hi) == (lo, hi)
    dg = pipeline.DeviceGraph(g, dev)
    print(f"[hand-over] {n_rows} rows, {int(deg[S].sum())} edges, local [{lo}, {hi})", flush=True)
    S = S[np.argsort(deg[S] == 0, kind="stable")]   # rows with edges first
    few = max(1, min(n_rows // 2, 3))   # so few rows on the device that most shares of a tile hold no chunk
    wants = [(n_rows, oracle.build_probs(g, S, skew)), (few, oracle.build_probs(g, S[:few], skew))]
    if n_rows == 4:
        assert int(wants[0][1].cand_w.max()) >= 1 << 54, "no weight beyond an entry of the hand-over"
    for mode in (0, 1, 2):
        ws = pipeline.Workspace(n_nodes, n_rows, 1, max(g.nnz, 1), dev, scan_mode=mode)
        for rows, want in wants + wants[:1]:
            lb = pipeline.LayerBuffers(n_rows, 1, n_nodes, 1, 1, dev)
            csgs.csgs_build_probs(dg.c, torch.from_numpy(S).to(dev), skew, lb.cand_id, lb.cand_w, lb.cdf, None, lb.stats, ws.desc, lb.status,
                                  nS_dev=torch.tensor([rows], dtype=torch.int32, device=dev))
            torch.cuda.synchronize()
            n_c = len(want.cand_id)
            assert int(lb.stats_host().n_cand) == n_c and int(lb.status.item()) == (0 if n_c else csgs.ST_EMPTY_CANDIDATES)
            np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
            np.testing.assert_array_equal(lb.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
            np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
            assert int(torch.count_nonzero(ws.buf[:chain.csgs_clean_words(n_nodes)]).item()) == 0, "workspace not restored"


# Column counts around what one block of the transpose orders (16), what one takes of its prefix (2048) and several of those;
# fewer columns on the device than the bound; columns around the 64 entries that one wavefront orders.  (With that many entries to spare several
# launches transpose, else one.)
@pytest.mark.parametrize("spare", [3, 1 << 19])
@pytest.mark.parametrize("bound,n_cols", [(15, 15), (17, 16), (17, 17), (2047, 2047), (2049, 2048), (2049, 2049), (10_300, 10_241), (9000, 100), (50, 0)])
def test_aggregate_gradient_columns(dev, bound, n_cols, spare):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(bound + n_cols)
    nS, F = 700, 20
    print(f"[aggregate grad] {n_cols} of {bound} columns", flush=True)
    dense = rng.random((nS, n_cols)) < 2.0 / max(n_cols, 4)
    for c, k in zip(rng.permutation(n_cols)[:5], (63, 64, 65, 257, 700)):
        dense[:, c] = False
        dense[rng.choice(nS, k, replace=False), c] = True
    rows, col = np.nonzero(dense)
    rp = np.zeros(nS + 1, np.int32)
    np.cumsum(np.bincount(rows, minlength=nS), out=rp[1:])
    val = rng.standard_normal(len(col)).astype(np.float32)
    dZ, Hp = rng.standard_normal((nS, F)).astype(np.float32), rng.standard_normal((bound, F)).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    cap = len(col) + spare
    cold, vald = torch.zeros(cap, dtype=torch.int32, device=dev), torch.zeros(cap, dtype=torch.float32, device=dev)
    cold[:len(col)], vald[:len(col)] = t(col.astype(np.int32)), t(val)
    dH = torch.full((bound, F), float("nan"), dtype=torch.float32, device=dev)
    nbytes = csgs.csgs_aggregate_grad_scratch_bytes(bound, cap)
    scratch = torch.full((nbytes // 8 + 32,), -1, dtype=torch.int64, device=dev)
    csgs.csgs_aggregate_grad(t(rp), cold, vald, torch.tensor([n_cols], dtype=torch.int32, device=dev), t(dZ), t(Hp), dH, scratch)
    torch.cuda.synchronize()
    want = oracle.aggregate_grad(rp, col.astype(np.int32), val, n_cols, dZ, Hp[:n_cols])
    chain.assert_close(dH[:n_cols].cpu().numpy(), want, chain.RTOL, chain.ATOL, "dH_prev")
    assert bool(torch.isnan(dH[n_cols:]).all()), "wrote past the last column"


# The weight gradient with widths that are whole pieces of four columns and odd ones, odd strides and addresses; rows and columns around
# multiples of 128 and 32, fewer rows on the device than the bound
@pytest.mark.parametrize("M,m,K,N,pad", [(1, 1, 4, 1, 0), (31, 31, 124, 5, 0), (33, 20, 128, 32, 0), (1000, 970, 132, 33, 0), (4096, 4096, 300, 100, 0),
                                         (64, 64, 260, 64, 4), (500, 499, 128, 40, 1), (500, 500, 130, 31, 2), (40, 0, 8, 8, 0)])
def test_weight_gradient_loads(dev, M, m, K, N, pad):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(M + K + N)
    print(f"[dW] {m} of {M} rows, {K} x {N}, pad {pad}", flush=True)
    Z, G = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    Zd = torch.full((M, K + pad), float("nan"), dtype=torch.float32, device=dev)[:, :K]
    Zd.copy_(torch.from_numpy(Z))
    Gd = torch.from_numpy(G).to(dev)
    Zd[m:], Gd[m:] = float("nan"), float("inf")                  # rows beyond the count are never summed
    dW = torch.zeros((K, N), dtype=torch.float32, device=dev)
    scratch = torch.zeros(csgs.csgs_layer_gemm_grad_w_scratch_bytes(M, K, N) // 8 + 32, dtype=torch.int64, device=dev)
    csgs.csgs_layer_gemm_grad_w(Zd, Gd, dW, scratch, M_dev=torch.tensor([m], dtype=torch.int32, device=dev))
    torch.cuda.synchronize()
    want = oracle.layer_gemm_grad_w(Z[:m], G[:m]) if m else np.zeros((K, N), np.float32)
    chain.assert_close(dW.cpu().numpy(), want, chain.RTOL, chain.ATOL, "dW")


# The products around a wavefront's tiles of 16 rows and columns: K in chunks of 32 and what is left of them (in steps of four, room for 8 or 32), rows
# whose floats start anywhere.  (Most of these sizes are taken in tiles of 16 x 16: each larger one in test_product_shapes.  The last size takes the
# kernel for rows 2^24 floats apart and more; offsets that need its 64 bits in test_products_of_distant_rows.)
@pytest.mark.parametrize("M,K,N,pad", [(1, 1, 1, 0), (15, 31, 2, 1), (17, 32, 3, 0), (16, 33, 16, 3), (33, 36, 17, 0), (1023, 40, 7, 2), (1024, 64, 256, 0),
                                       (2048, 41, 250, 1), (4095, 63, 100, 0), (4096, 96, 512, 0), (4097, 34, 511, 1), (20001, 9, 201, 0), (65530, 8, 47, 1),
                                       (65537, 4, 130, 2), (3, 37, 5, 1 << 24)])
def test_product_tiles(dev, M, K, N, pad):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(7 * M + K + N)
    print(f"[products] {M} x {K} x {N}, pad {pad}", flush=True)

    def padded(a):
        t = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), dtype=torch.float32, device=dev)[:, :a.shape[1]]
        t.copy_(torch.from_numpy(a))
        return t
    Z, W, G = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (K, N), (M, N)))
    Zd, Wd, Gd = padded(Z), padded(W), padded(G)
    out = lambda r, c: torch.full((r + 1, c + 3), float("nan"), dtype=torch.float32, device=dev)
    H, dZ, dW = out(M, N), out(M, K), out(K, N)
    csgs.csgs_layer_gemm(Zd, Wd, H[:M, :N])
    csgs.csgs_layer_gemm_grad_z(Gd, Wd, dZ[:M, :K])
    scratch = torch.full((csgs.csgs_layer_gemm_grad_w_scratch_bytes(M, K, N) // 8,), -1, dtype=torch.int64, device=dev)
    csgs.csgs_layer_gemm_grad_w(Zd, Gd, dW[:K, :N], scratch)
    torch.cuda.synchronize()
    for got, want, what in ((H, oracle.layer_gemm(Z, W), "H"), (dZ, oracle.layer_gemm_grad_z(G, W), "dZ"), (dW, oracle.layer_gemm_grad_w(Z, G), "dW")):
        r, c = want.shape
        chain.assert_close(got[:r, :c].cpu().numpy(), want, chain.RTOL, chain.ATOL, what)
        assert bool(torch.isnan(got[r:]).all()) and bool(torch.isnan(got[:, c:]).all()), f"{what}: wrote outside"


# Every tile of the two products that go over the rows with every length of their last chunk (test_product_rules.py asks the rule whether these
# sizes take them): outputs that are no whole tiles in either direction, columns that are no multiple of a lane's
PRODUCT_SHAPES = [  # product, 16-row tiles, columns a lane, room for the last K % 32 k; M, K, N
    ("H", 2, 4, 0, 14088, 96, 97), ("H", 2, 4, 8, 14094, 66, 97), ("H", 2, 4, 32, 14089, 41, 103),
    ("H", 2, 3, 0, 13124, 96, 65), ("H", 2, 3, 8, 13191, 66, 65), ("H", 2, 3, 32, 13333, 42, 65),
    ("H", 2, 2, 0, 12290, 96, 49), ("H", 2, 2, 8, 12452, 65, 49), ("H", 2, 2, 32, 12692, 41, 49),
    ("H", 1, 4, 0, 5448, 96, 173), ("H", 1, 4, 8, 5446, 65, 163), ("H", 1, 4, 32, 5442, 42, 167),
    ("H", 1, 3, 0, 10939, 96, 35), ("H", 1, 3, 8, 10985, 65, 35), ("H", 1, 3, 32, 11022, 41, 35),
    ("H", 1, 2, 0, 8197, 96, 17), ("H", 1, 2, 8, 8223, 65, 17), ("H", 1, 2, 32, 8327, 41, 17),
    ("H", 2, 1, 0, 16397, 96, 5), ("H", 2, 1, 8, 16392, 65, 5), ("H", 2, 1, 32, 16625, 41, 5),
    ("H", 1, 1, 0, 17, 96, 5), ("H", 1, 1, 8, 17, 65, 5), ("H", 1, 1, 32, 17, 41, 5),
    ("dZ", 2, 4, 0, 14088, 97, 96), ("dZ", 2, 4, 8, 14094, 97, 66), ("dZ", 2, 4, 32, 14089, 103, 41),
    ("dZ", 2, 3, 0, 13124, 65, 96), ("dZ", 2, 3, 8, 13191, 65, 66), ("dZ", 2, 3, 32, 13333, 65, 42),
    ("dZ", 2, 2, 0, 12290, 49, 96), ("dZ", 2, 2, 8, 12452, 49, 65), ("dZ", 2, 2, 32, 12692, 49, 41),
    ("dZ", 1, 4, 0, 5448, 173, 96), ("dZ", 1, 4, 8, 5446, 163, 65), ("dZ", 1, 4, 32, 5442, 167, 42),
    ("dZ", 1, 3, 0, 10939, 35, 96), ("dZ", 1, 3, 8, 10985, 35, 65), ("dZ", 1, 3, 32, 11022, 35, 41),
    ("dZ", 1, 2, 0, 5453, 83, 96), ("dZ", 1, 2, 8, 841, 595, 65), ("dZ", 1, 2, 32, 1163, 439, 41),
    ("dZ", 2, 1, 0, 16397, 5, 96), ("dZ", 2, 1, 8, 16392, 5, 65), ("dZ", 2, 1, 32, 16625, 5, 41),
    ("dZ", 1, 1, 0, 17, 5, 96), ("dZ", 1, 1, 8, 17, 5, 65), ("dZ", 1, 1, 32, 17, 5, 41)]


@pytest.mark.parametrize("what,rt,nt,tail,M,K,N", PRODUCT_SHAPES)
def test_product_shapes(dev, what, rt, nt, tail, M, K, N):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(M + K + N)
    print(f"[products] {what} {M} x {K} x {N}: {16 * rt} x {16 * nt}, room for {tail}", flush=True)
    a, b, width = (M, K), (K, N), N
    if what == "dZ":
        a, width = (M, N), K
    A, W = rng.standard_normal(a).astype(np.float32), rng.standard_normal(b).astype(np.float32)
    out = torch.full((M + 1, width + 3), float("nan"), dtype=torch.float32, device=dev)
    call = csgs.csgs_layer_gemm if what == "H" else csgs.csgs_layer_gemm_grad_z
    call(torch.from_numpy(A).to(dev), torch.from_numpy(W).to(dev), out[:M, :width])
    torch.cuda.synchronize()
    want = oracle.layer_gemm(A, W) if what == "H" else oracle.layer_gemm_grad_z(A, W)
    chain.assert_close(out[:M, :width].cpu().numpy(), want, chain.RTOL, chain.ATOL, what)
    assert bool(torch.isnan(out[M:]).all()) and bool(torch.isnan(out[:, width:]).all()), "wrote outside"


# Rows so far apart that a lane's offset from its tile needs more than 32 bits, in each operand of the three products
def test_products_of_distant_rows(dev):
    from paper_2101_07706_amd import csgs
    M, K, N, ld = 40, 34, 17, 5 << 24
    assert 15 * ld * 4 > 1 << 32    # the last of a tile's rows from its first
    rng = np.random.default_rng(11)
    Z, W, G = (rng.standard_normal(s).astype(np.float32) for s in ((M, K), (K, N), (M, N)))
    print(f"[products] rows {ld} floats apart", flush=True)
    buf = torch.full((M, ld), float("nan"), dtype=torch.float32, device=dev)
    Zd, Wd, Gd = buf[:, :K], buf[:K, 64:64 + N], buf[:, 128:128 + N]
    for d, a in ((Zd, Z), (Wd, W), (Gd, G)):
        d.copy_(torch.from_numpy(a))
    H, dZ, dW = (torch.empty(s, dtype=torch.float32, device=dev) for s in ((M, N), (M, K), (K, N)))
    csgs.csgs_layer_gemm(Zd, Wd, H)
    csgs.csgs_layer_gemm_grad_z(Gd, Wd, dZ)
    scratch = torch.full((csgs.csgs_layer_gemm_grad_w_scratch_bytes(M, K, N) // 8,), -1, dtype=torch.int64, device=dev)
    csgs.csgs_layer_gemm_grad_w(Zd, Gd, dW, scratch)
    torch.cuda.synchronize()
    for got, want, what in ((H, oracle.layer_gemm(Z, W), "H"), (dZ, oracle.layer_gemm_grad_z(G, W), "dZ"), (dW, oracle.layer_gemm_grad_w(Z, G), "dW")):
        chain.assert_close(got.cpu().numpy(), want, chain.RTOL, chain.ATOL, what)
    del buf, Zd, Wd, Gd
    torch.cuda.empty_cache()


# The weight gradient's tiles and parts: each shape of its rule (2x2, 2x4, 2x3, 1x4, 1x2, 2x1, 1x1), one part and several, columns beside their
# edges, rows that are no multiple of a part's chunks
GRAD_W_SIZES = [(65, 64, 2), (7135, 47, 1), (63, 193, 322), (2400, 17, 66), (2433, 130, 306), (10847, 175, 1), (18817, 175, 17), (12287, 161, 33),
                (12033, 66, 318)]


@pytest.mark.parametrize("M,K,N", GRAD_W_SIZES)
def test_weight_gradient_tiles(dev, M, K, N):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(3 * M + K + N)
    print(f"[dW tiles] {M} rows, {K} x {N}", flush=True)
    Z, G = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((M, N)).astype(np.float32)
    dW = torch.full((K + 1, N + 3), float("nan"), dtype=torch.float32, device=dev)
    scratch = torch.full((csgs.csgs_layer_gemm_grad_w_scratch_bytes(M, K, N) // 8,), -1, dtype=torch.int64, device=dev)
    csgs.csgs_layer_gemm_grad_w(torch.from_numpy(Z).to(dev), torch.from_numpy(G).to(dev), dW[:K, :N], scratch)
    torch.cuda.synchronize()
    # one rounding to float of a sum held in double: half a unit in the last place, and what 2^-53 leaves of the summands
    want = Z.T.astype(np.float64) @ G.astype(np.float64)
    bound = 2.0 ** -24 * np.abs(want) + M * 2.0 ** -52 * (np.abs(Z).T.astype(np.float64) @ np.abs(G).astype(np.float64))
    assert (np.abs(dW[:K, :N].cpu().numpy() - want) <= bound).all()
    assert torch.isnan(dW[K]).all() and torch.isnan(dW[:, N:]).all()


# Rows that start anywhere: widths around the vectors' (2, 4, 8), the slices' (64 and 256 features) and the narrow rows' limits, tables and
# outputs that begin an element late with odd distances between rows, both types; nothing beside a row is written
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 8, 16, 17, 33, 65, 127, 128, 129, 200, 257, 264, 515])
def test_rows_that_start_anywhere(dev, F, bf16):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(F)
    n, n_local, n_remote = 5000 if 64 < F <= 128 else 300, 500, 90   # (narrow rows are cut by how many there are)
    print(f"[odd rows] F={F} bf16={bf16}", flush=True)

    def late(a, fill):   # the same values, one element late in rows that are longer by an odd number
        t = torch.full((a.shape[0], a.shape[1] + 3 - a.shape[1] % 2), fill, dtype=torch.int16 if a.dtype == np.int16 else torch.float32, device=dev)
        t[:, 1:1 + a.shape[1]] = torch.from_numpy(a).to(dev)
        return t[:, 1:1 + a.shape[1]]
    X = rng.standard_normal((n_local + n_remote, F)).astype(np.float32)
    Xh = synth.to_bf16_bits(X) if bf16 else X
    bits = Xh.view(np.int16) if bf16 else Xh
    Xl, Xr = late(bits[:n_local], -1 if bf16 else float("nan")), late(bits[n_local:], -1 if bf16 else float("nan"))
    n_cols = n_local + n_remote
    lens = rng.poisson(3, n)
    lens[rng.integers(0, n, 6)] = (0, 1, 300, 257, 90, 140)
    rowptr, col, val = _csr(rng, lens, n_cols)
    src = rng.permutation(n_cols).astype(np.int32)                 # column -> row of X
    src_row = np.where(src < n_local, src, n_local - 1 - src).astype(np.int32)
    want = oracle.aggregate(rowptr, src[col].astype(np.int32), val, Xh, relu_on_input=True)
    Zbuf = torch.full((n, F + 2 + F % 2), float("nan"), dtype=torch.float32, device=dev)
    t = lambda a: torch.from_numpy(a).to(dev)
    csgs.csgs_aggregate(t(rowptr), t(col), t(val), torch.tensor([n_cols], dtype=torch.int32, device=dev), Xl, Xr, t(src_row), True, Zbuf[:, 1:1 + F])
    few = torch.full((61, F), float("nan"), dtype=torch.float32, device=dev)   # a handful of rows
    csgs.csgs_aggregate(t(rowptr[:61]), t(col), t(val), torch.tensor([n_cols], dtype=torch.int32, device=dev), Xl, Xr, t(src_row), True, few[:60])
    ids = rng.integers(0, n_local, 70).astype(np.int32)
    out = torch.full((71, F + 2 + F % 2), 7, dtype=Xl.dtype, device=dev)
    csgs.csgs_gather_rows(Xl, t(ids), None, out[:70, 1:1 + F])
    torch.cuda.synchronize()
    chain.assert_close(Zbuf[:, 1:1 + F].cpu().numpy(), want, chain.RTOL, chain.ATOL, "Z")
    chain.assert_close(few[:60].cpu().numpy(), want[:60], chain.RTOL, chain.ATOL, "Z of few rows")
    assert bool(torch.isnan(few[60]).all()), "wrote past the last row"
    assert bool(torch.isnan(Zbuf[:, 0]).all()) and bool(torch.isnan(Zbuf[:, 1 + F:]).all()), "wrote beside a row"
    assert np.array_equal(out[:70, 1:1 + F].cpu().numpy(), bits[ids])
    assert bool((out[:, 0] == 7).all()) and bool((out[:, 1 + F:] == 7).all()) and bool((out[70] == 7).all()), "gathered beside a row"
    if not bf16:   # the gradient through the same kernel: output mask and table in odd places
        H = rng.standard_normal((n_cols, F)).astype(np.float32)
        dense = np.unique(np.stack([rng.integers(0, n, 900), rng.integers(0, n_cols, 900)], 1), axis=0)
        rp = np.zeros(n + 1, np.int32)
        np.cumsum(np.bincount(dense[:, 0], minlength=n), out=rp[1:])
        gcol, gval = dense[:, 1].astype(np.int32), rng.standard_normal(len(dense)).astype(np.float32)
        dZ = rng.standard_normal((n, F)).astype(np.float32)
        dH = torch.full((n_cols, F + 2 + F % 2), float("nan"), dtype=torch.float32, device=dev)
        scratch = torch.full((csgs.csgs_aggregate_grad_scratch_bytes(n_cols, len(gcol)) // 8 + 32,), -1, dtype=torch.int64, device=dev)
        csgs.csgs_aggregate_grad(t(rp), t(gcol), t(gval), torch.tensor([n_cols], dtype=torch.int32, device=dev), late(dZ, float("nan")),
                                 late(H, float("nan")), dH[:, 1:1 + F], scratch)
        torch.cuda.synchronize()
        chain.assert_close(dH[:, 1:1 + F].cpu().numpy(), oracle.aggregate_grad(rp, gcol, gval, n_cols, dZ, H), chain.RTOL, chain.ATOL, "dH")
        assert bool(torch.isnan(dH[:, 0]).all()) and bool(torch.isnan(dH[:, 1 + F:]).all()), "wrote beside a row"


# From 8192 tiles of 1024 ids on, over all instances, the candidate sums pack their tiles: tiles with all ids, with one, without any, the last,
# shorter one, tiles of the local range with and without a hand-over, one instance and several; the workspace is left clean
@pytest.mark.parametrize("n,n_inst", [(8192 * 1024 + 37, 1), (1366 * 1024 - 5, 6)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_packed_candidate_tiles(dev, n, n_inst, mode):
    from paper_2101_07706_amd import csgs, pipeline
    from test_gpu_scaling import _rows_by_target
    rng = np.random.default_rng(n_inst)
    P, n_rows, degree = 16, 4000, 50
    g, S = _rows_by_target(rng, n, P, n_rows, degree, np.full(n_rows, 0.7))
    cols = g.colidx.reshape(n_rows, degree)
    for first, row in ((9 * 1024, 0), ((n // P // 1024 + 40) * 1024, 21)):      # a local tile and a remote one, every id of them
        ids = np.arange(first, first + 21 * degree) % n
        cols[row:row + 21] = ids.reshape(21, degree)
    cols[42] = np.arange(n - degree, n)
    edge = (n // P) - degree // 2
    cols[43] = np.arange(edge, edge + degree)                                    # across the end of the local range
    print(f"[packed tiles] n={n} n_inst={n_inst} mode={mode}", flush=True)
    K, skew = n_inst, 4.0
    lb = pipeline.LayerBuffers(n_rows, 1, n, 1, P, dev, n_inst=K)
    ws = pipeline.Workspace(n, n_rows, 1, g.nnz, dev, n_inst=K, inst_stride=lb.stride, scan_mode=mode)
    dg = pipeline.DeviceGraph(g, dev)
    rows = [np.sort(rng.permutation(S)[:n_rows - 700 * k]).astype(np.int32) for k in range(K)]
    for k in range(K):
        lb.inst(k).S0[:n_rows].zero_()
        lb.inst(k).S0[:len(rows[k])].copy_(torch.from_numpy(rows[k]))
        lb.inst(k).n_next.fill_(len(rows[k]))
    for _ in range(2):                                                           # the second call finds what the first left
        csgs.csgs_build_probs(dg.c, lb.S0[:n_rows], skew, lb.cand_id, lb.cand_w, lb.cdf, lb.q, lb.stats, ws.desc, lb.status, nS_dev=lb.n_next)
    torch.cuda.synchronize()
    for k in range(K):
        one, want = lb.inst(k), oracle.build_probs(g, rows[k], skew)
        n_c = len(want.cand_id)
        assert int(one.status.item()) == 0 and int(one.stats_host().n_cand) == n_c
        np.testing.assert_array_equal(one.cand_id[:n_c].cpu().numpy(), want.cand_id)
        np.testing.assert_array_equal(one.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
        np.testing.assert_array_equal(one.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
        np.testing.assert_array_equal(one.q[:n_c].cpu().numpy(), want.q)
        at = k * ws.bytes_per_inst // 8
        assert int(torch.count_nonzero(ws.buf[at:at + chain.csgs_clean_words(n)]).item()) == 0, "workspace not restored"


# Staged rows in whole pieces of 2, 4 and 16 bytes while 64 lanes cover them at once, beyond in 16 bytes from any address: widths around the
# pieces and the limits (128 and 256 bytes), tables and outputs that begin on a piece and one element late; ids outside the table
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 7, 8, 9, 10, 12, 62, 63, 64, 65, 66, 127, 128, 129, 130, 132, 200, 333])
def test_gathered_row_pieces(dev, F, bf16):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(F)
    rows, cap, n = 300, 77, 70
    dtype = np.int16 if bf16 else np.float32
    X = rng.integers(-30000, 30000, (rows, F)).astype(dtype)
    ids = rng.integers(0, rows, cap).astype(np.int32)
    ids[3], ids[4] = -1, rows
    want = np.where(((ids >= 0) & (ids < rows))[:, None], X[np.clip(ids, 0, rows - 1)], 0)[:n].astype(dtype)
    for late in (0, 1):
        print(f"[gathered rows] F={F} bf16={bf16} late={late}", flush=True)
        place = lambda r, fill: torch.full((r, (F + 15) // 8 * 8 + late), fill, dtype=torch.from_numpy(X).dtype, device=dev)
        table, out = place(rows, 5), place(cap, 7)
        table[:, late:late + F] = torch.from_numpy(X).to(dev)
        csgs.csgs_gather_rows(table[:, late:late + F], torch.from_numpy(ids).to(dev), torch.tensor([n], dtype=torch.int64, device=dev),
                              out[:, late:late + F])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out[:n, late:late + F].cpu().numpy(), want)
        out[:n, late:late + F] = 7
        assert bool((out == 7).all()), "wrote beside the rows"


# Odd widths on either side of the row counts at which the lanes per row change (64, 1024, 4096, 8192 and 65536 rows), tables that begin on a
# pair (float rows of 258 to 320 features are then read in pairs) and one element late; rows without edges and long ones among them
@pytest.mark.parametrize("n,F", [(64, 15), (65, 15), (8192, 15), (8193, 9), (8193, 15), (65536, 11), (65537, 11), (8192, 17), (8193, 17), (8193, 31),
                                 (1024, 65), (1025, 65), (1025, 127), (4096, 127), (4097, 127), (4096, 258), (4097, 257), (4097, 258), (4097, 320), (4097, 322)])
def test_odd_widths_by_rows(dev, n, F):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(n + F)
    n_cols = 700
    lens = rng.poisson(1.5, n)
    lens[rng.integers(0, n, 4)] = (0, 70, 140, 300)
    rowptr, col, val = _csr(rng, lens, n_cols)
    X = rng.standard_normal((n_cols, F)).astype(np.float32)
    t = lambda a: torch.from_numpy(a).to(dev)
    adj, cols = [t(a) for a in (rowptr, col, val)], torch.tensor([n_cols], dtype=torch.int32, device=dev)
    for bf16 in (False, True):
        Xh = synth.to_bf16_bits(X) if bf16 else X
        want = oracle.aggregate(rowptr, col, val, Xh, relu_on_input=False)
        for late in (0, 1):
            print(f"[odd widths] {n} rows F={F} bf16={bf16} late={late}", flush=True)
            bits = Xh.view(np.int16) if bf16 else Xh
            table = torch.full((n_cols, F + F % 2 + late), -1 if bf16 else float("nan"), dtype=torch.int16 if bf16 else torch.float32, device=dev)
            table[:, late:late + F] = t(bits)
            Z = torch.full((n, F + F % 2 + late), float("nan"), dtype=torch.float32, device=dev)
            csgs.csgs_aggregate(*adj, cols, table[:, late:late + F], None, None, False, Z[:, late:late + F])
            torch.cuda.synchronize()
            chain.assert_close(Z[:, late:late + F].cpu().numpy(), want, chain.RTOL, chain.ATOL, "Z")
            assert bool(torch.isnan(Z[:, :late]).all()) and bool(torch.isnan(Z[:, late + F:]).all()), "wrote beside a row"


# The weight scan of many edges: every edge sorted by the block that sums its target.  Local ranges at the start, in the middle (bins of fewer than four
# tiles before and behind it), in the last partial tile, and too wide to have blocks of their own; a remote piece of 4096 ids that takes all remote edges (its
# runs go through the atomics); rows whose count only the device knows, few enough that an edge's weight does not fit an entry.
@pytest.mark.parametrize("n,lo,hi,n_rows,degree,remote_ids,count", [(300_001, 0, 37_500, 9000, 41, None, None), (300_001, 150_700, 190_001, 9000, 41, None, None),
                                                                     (299_900, 270_000, 299_900, 9000, 41, None, None), (400_000, 10, 390_000, 9000, 41, None, None),
                                                                     (300_001, 0, 37_500, 9000, 41, (204_800, 208_896), None), (300_001, 0, 37_500, 9000, 41, None, 5)])
def test_weight_scan_of_many_edges(dev, n, lo, hi, n_rows, degree, remote_ids, count):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(n + lo)
    K = 8
    remote = np.setdiff1d(np.arange(n), np.arange(lo, hi)) if remote_ids is None else np.arange(*remote_ids)
    col = np.where(rng.random((n, degree)) < 0.7, rng.integers(lo, hi, (n, degree)), remote[rng.integers(0, len(remote), (n, degree))]).astype(np.int32)
    col.sort(axis=1)
    val = rng.random((n, degree)).astype(np.float32) / degree
    if count is not None:
        val[:] = np.eye(1, degree, dtype=np.float32)   # 1, 0, 0, ...
    g = synth.Graph(n, np.arange(n + 1, dtype=np.int64) * degree, col.reshape(-1), val.reshape(-1), np.array([0, lo, hi, n], np.int32) if lo else np.array([0, hi, n], np.int32),
                    1 if lo else 0, 1.0)
    assert (g.local_lo, g.local_hi) == (lo, hi)
    dg = pipeline.DeviceGraph(g, dev)
    lb = pipeline.LayerBuffers(n_rows, 1, n, 1, dg.n_parts, dev, n_inst=K)
    ws = pipeline.Workspace(n, n_rows, 1, g.nnz, dev, n_inst=K, inst_stride=lb.stride)
    S = [np.sort(rng.choice(n, n_rows, replace=False)).astype(np.int32) for _ in range(K)]
    for k in range(K):
        lb.inst(k).S0.copy_(torch.from_numpy(S[k]).to(dev))
        lb.inst(k).n_next.fill_(n_rows if count is None else count)
    for again in range(2):   # the second call finds the workspace as the first has left it
        csgs.csgs_build_probs(dg.c, lb.S0[:n_rows], 4.0, lb.cand_id, lb.cand_w, lb.cdf, lb.q, lb.stats, ws.desc, lb.status, nS_dev=None if count is None else lb.n_next)
        torch.cuda.synchronize()
        for k in (0, 3, K - 1):
            want, b = oracle.build_probs(g, S[k] if count is None else S[k][:count], 4.0), lb.inst(k)
            n_c = len(want.cand_id)
            assert int(b.status.item()) == 0 and b.stats_host().n_cand == n_c and b.stats_host().n_local == int(((want.cand_id >= lo) & (want.cand_id < hi)).sum())
            np.testing.assert_array_equal(b.cand_id[:n_c].cpu().numpy(), want.cand_id)
            np.testing.assert_array_equal(b.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
            np.testing.assert_array_equal(b.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
    assert int(torch.count_nonzero(ws.buf.view(K, -1)[:, :csgs.csgs_workspace_clean_bytes(n) // 8]).item()) == 0


# The same with few edges to a bin, whose sums are one wavefront's: bins with none, with more than it has room for (the block's), with more than the scan
# hands over (through the table), bins cut by the local range; as many entries outside the local range as decide whether wavefronts or blocks take them
@pytest.mark.parametrize("lo,hi,local,hot", [(0, 106_000, 0.8, 0.0), (700_300, 806_001, 0.7, 0.02), (1_790_001, 1_900_001, 0.7, 0.25), (700_300, 806_001, 0.1, 0.0),
                                             (700_300, 806_001, 0.39, 0.0), (0, 106_000, 0.33, 0.0), (1_790_001, 1_900_001, 0.39, 0.3)])
def test_weight_scan_of_few_edges_a_bin(dev, lo, hi, local, hot):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(lo + 1)
    n, n_rows, degree, K, base = 1_900_001, 9000, 38, 8, 50_000
    print(f"[few edges a bin] local {lo}..{hi}, {hot} of the others in 4096 ids", flush=True)
    shape = (base, degree)
    remote = (hi + rng.integers(0, n - hi + lo, shape)) % n
    remote = np.where(rng.random(shape) < hot, 409_600 + rng.integers(0, 4096, shape), remote)
    col = np.where(rng.random(shape) < local, rng.integers(lo, hi, shape), remote).astype(np.int32)
    col[:, 0] = np.where(rng.random(base) < 0.1, 1_200_000 + rng.integers(0, 3, base), col[:, 0])   # (few ids with many edges)
    col.sort(axis=1)
    rows = -(-n // base)
    col = np.tile(col, (rows, 1))[:n]
    val = np.tile(rng.random(shape).astype(np.float32) / degree, (rows, 1))[:n]
    g = synth.Graph(n, np.arange(n + 1, dtype=np.int64) * degree, col.reshape(-1), val.reshape(-1), np.array([0, lo, hi, n], np.int32) if lo else np.array([0, hi, n], np.int32),
                    1 if lo else 0, 1.0)
    dg = pipeline.DeviceGraph(g, dev)
    lb = pipeline.LayerBuffers(n_rows, 1, n, 1, dg.n_parts, dev, n_inst=K)
    ws = pipeline.Workspace(n, n_rows, 1, g.nnz, dev, n_inst=K, inst_stride=lb.stride)
    S = [np.sort(rng.choice(n, n_rows, replace=False)).astype(np.int32) for _ in range(K)]
    counts = [n_rows] * (K - 1) + [n_rows // 30]
    for k in range(K):
        lb.inst(k).S0.copy_(torch.from_numpy(S[k]).to(dev))
        lb.inst(k).n_next.fill_(counts[k])
    for again in range(2):
        csgs.csgs_build_probs(dg.c, lb.S0[:n_rows], 4.0, lb.cand_id, lb.cand_w, lb.cdf, lb.q, lb.stats, ws.desc, lb.status, nS_dev=lb.n_next)
        torch.cuda.synchronize()
    for k in (0, 5, K - 1):
        want, b = oracle.build_probs(g, S[k][:counts[k]], 4.0), lb.inst(k)
        n_c = len(want.cand_id)
        assert int(b.status.item()) == 0 and b.stats_host().n_cand == n_c and b.stats_host().n_local == int(((want.cand_id >= lo) & (want.cand_id < hi)).sum())
        np.testing.assert_array_equal(b.cand_id[:n_c].cpu().numpy(), want.cand_id)
        np.testing.assert_array_equal(b.cand_w[:n_c].cpu().numpy().view(np.uint64), want.cand_w)
        np.testing.assert_array_equal(b.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
    assert int(torch.count_nonzero(ws.buf.view(K, -1)[:, :csgs.csgs_workspace_clean_bytes(n) // 8]).item()) == 0


# The transpose in one launch: a column that holds more entries than a block's lists, row pointers that start inside the arrays, empty rows, the most
# columns it takes and one more (several launches), two calls bit for bit.
@pytest.mark.parametrize("nS,n_cols,most,hub", [(20_000, 700, 6, True), (20_000, 65_536, 6, False), (20_000, 65_537, 6, False), (3, 1, 1, True), (700, 256, 300, True), (1, 257, 200, False)])
def test_aggregate_gradient_one_launch(dev, nS, n_cols, most, hub):
    from paper_2101_07706_amd import csgs
    rng = np.random.default_rng(nS + n_cols)
    F, skip = 12, 37
    cols = [np.unique(np.concatenate([rng.integers(0, n_cols, rng.integers(0, most + 1)), [min(5, n_cols - 1)] if hub else []])).astype(np.int32) for _ in range(nS)]
    rp = np.zeros(nS + 1, np.int32)
    np.cumsum([len(c) for c in cols], out=rp[1:])
    nnz = int(rp[-1])
    col, val = np.concatenate(cols + [np.zeros(1, np.int32)])[:max(nnz, 1)], rng.standard_normal(max(nnz, 1)).astype(np.float32)
    dZ, H = rng.standard_normal((nS, F)).astype(np.float32), rng.standard_normal((n_cols, F)).astype(np.float32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    pad = np.full(skip, 3 % n_cols, np.int32)   # entries before the first row's
    cold, vald = t(np.concatenate([pad, col])), t(np.concatenate([pad.astype(np.float32), val]))
    scratch = torch.full((csgs.csgs_aggregate_grad_scratch_bytes(n_cols, cold.numel()) // 8 + 32,), -1, dtype=torch.int64, device=dev)
    got = []
    for _ in range(2):
        dH = torch.full((n_cols, F), float("nan"), dtype=torch.float32, device=dev)
        csgs.csgs_aggregate_grad(t(rp + skip), cold, vald, None, t(dZ), t(H), dH, scratch)
        got.append(dH.cpu().numpy())
    chain.assert_close(got[0], oracle.aggregate_grad(rp, col, val, n_cols, dZ, H), chain.RTOL, chain.ATOL, "dH")
    np.testing.assert_array_equal(got[0], got[1])


# Where the last chunk of edges ends: rows without edges behind the last one that has some, in its tile of rows and in tiles of their own, before the first
# one, none at all; edges that end on a chunk's boundary, one short of it and one beyond; the adjacency in one pass and in two.
@pytest.mark.parametrize("before,with_edges,degree,behind", [(0, 500, 3, 20), (0, 1024, 1, 3000), (3, 341, 3, 3000), (1030, 41, 25, 2000), (0, 1, 2047, 1500), (2100, 5, 1, 0),
                                                             (0, 9000, 80, 2500), (40, 8192, 80, 0)])
def test_rows_without_edges_around_the_last_chunk(dev, before, with_edges, degree, behind):
    from paper_2101_07706_amd import csgs, pipeline
    rng = np.random.default_rng(before + with_edges)
    n, B = before + with_edges + behind + 900, 400
    deg = np.zeros(n, np.int64)
    deg[before:before + with_edges] = degree
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    col = np.concatenate([np.sort(rng.choice(n, d, replace=False)) for d in deg[deg > 0]]).astype(np.int32)
    g = synth.Graph(n, rowptr, col, (rng.random(len(col)) / degree).astype(np.float32), synth.partition_bounds(n, 3), 0, 1.0)
    S = np.arange(before + with_edges + behind, dtype=np.int32)
    dg, Sd = pipeline.DeviceGraph(g, dev), torch.from_numpy(S).to(dev)
    ws, lb = pipeline.Workspace(n, len(S), B, g.nnz, dev), pipeline.LayerBuffers(len(S), B, n, g.nnz, 3, dev)
    lb.adj_rowptr.fill_(-7)
    pipeline.sample_step(dg, ws, Sd, 4.0, B, 5, 3, 0, lb)
    want = oracle.build_probs(g, S, 4.0)
    got = oracle.sample_layer(g, S, want, B, 5, 3, 0)
    n_c, m, nnz = len(want.cand_id), got.n_next, got.adj_nnz
    assert int(lb.status.item()) == 0 and int(lb.n_next.item()) == m and int(lb.adj_nnz.item()) == nnz
    np.testing.assert_array_equal(lb.cand_id[:n_c].cpu().numpy(), want.cand_id)
    np.testing.assert_array_equal(lb.cdf[:n_c].cpu().numpy().view(np.uint64), want.cdf)
    np.testing.assert_array_equal(lb.adj_rowptr[:len(S) + 1].cpu().numpy(), got.adj_rowptr)
    np.testing.assert_array_equal(lb.adj_col[:nnz].cpu().numpy(), got.adj_col)

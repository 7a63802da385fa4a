"""GPU parity of the individual kernels (through the C ABI) against fp64 numpy / scipy on the oracle's graph."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle.graph import OracleGraph
from paper_2112_09335_amd import synth
from parity import say

pytestmark = pytest.mark.gpu

HYPER = dict(nu=1e-3, rho=1e-3, tau0=1e-3, theta0=1e-3, eta=2.0, max_backtrack=60, fista_iters=10)


@pytest.fixture(scope="module")
def ctx():
    import torch
    from paper_2112_09335_amd import binding
    w = synth.config(3, 0.03)        # N = 6000, 32 communities, degree 15: several tiles, ragged tails
    s = binding.Solver(0)
    s.build_graph(w.N, w.src, w.dst, w.M, w.comm)
    s.set_model([1030, 512, 512, 16], **HYPER)       # reserves scratch for the widest shapes below
    s.set_workspace()
    g = OracleGraph(w.N, w.src, w.dst, w.M, w.comm)
    yield s, g, torch
    s.close()


@pytest.fixture(scope="module")
def hub_ctx():
    """A graph with hub rows far beyond the split threshold (a few nodes adjacent to thousands of others),
    so that the split-row path of the aggregation (parts + ordered combine) is exercised, ragged sizes."""
    import torch
    from paper_2112_09335_amd import binding
    rng = np.random.default_rng(77)
    N, M = 5003, 5
    comm = rng.integers(0, M, size=N).astype(np.int32)
    src = [rng.integers(0, N, size=12000)]
    dst = [rng.integers(0, N, size=12000)]
    for hub, deg in ((0, 4000), (17, 1500), (N - 1, 385), (99, 384), (100, 383)):
        nb = rng.choice(N, size=deg, replace=False)
        src.append(np.full(deg, hub))
        dst.append(nb)
    src = np.concatenate(src).astype(np.int32)
    dst = np.concatenate(dst).astype(np.int32)
    s = binding.Solver(0)
    s.build_graph(N, src, dst, M, comm)
    s.set_model([300, 64, 16], **HYPER)
    s.set_workspace()
    g = OracleGraph(N, src, dst, M, comm)
    assert np.diff(g.row_ptr).max() > 3000
    yield s, g, torch
    s.close()


@pytest.mark.parametrize("width,tile", [(3, 0), (16, 0), (64, 0), (256, 0), (300, 0), (256, 32), (256, 64), (300, 128), (7, 4)])
def test_aggregate_with_hub_rows_and_column_tiles(hub_ctx, width, tile):
    s, g, torch = hub_ctx
    say("hub aggregate width", width, "tile", tile)
    rng = np.random.default_rng(width + tile)
    X = rng.standard_normal((g.N, width)).astype(np.float32)
    s.tune("spmm_tile_cols", tile)
    try:
        Y = s.op_aggregate(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
        P = s.op_aggregate_segments(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    finally:
        s.tune("spmm_tile_cols", 0)
    assert rel_err(Y, g.A @ X.astype(np.float64)) < 3e-6
    S = sp.csr_matrix((g.val, g.col, g.seg_ptr), shape=(g.n_segments, g.N))
    assert rel_err(P, (S @ X.astype(np.float64))[s.get_segment_order()]) < 3e-6


def test_kernel_calls_on_a_stream_that_takes_the_place_of_a_destroyed_one(hub_ctx):
    """The runtime may give a new stream the handle of a destroyed one whose work still runs; the calls share the buffer of
    split rows, so the second must wait for the first."""
    import ctypes
    s, g, torch = hub_ctx
    X = [torch.randn(g.N, 300, device="cuda") for _ in range(4)]
    want = [s.op_aggregate(x) for x in X]
    Y = [torch.empty_like(x) for x in X]
    torch.cuda.synchronize()
    for x, y in zip(X, Y):
        stream = ctypes.c_void_p()
        assert s.lib.hipStreamCreate(ctypes.byref(stream)) == 0
        assert s.lib.cadmm_op_stream(s.h, stream) == 0
        for _ in range(20):
            assert s.lib.cadmm_op_aggregate(s.h, x.data_ptr(), 300, y.data_ptr()) == 0
        assert s.lib.hipStreamDestroy(stream) == 0
    torch.cuda.synchronize()
    for y, w in zip(Y, want):
        assert torch.equal(y, w)


def rel_err(got, ref):
    return float(np.abs(got - ref).max() / max(np.abs(ref).max(), 1e-300))


@pytest.mark.parametrize("width", [1, 3, 7, 16, 64, 100, 128, 256, 500, 512, 1030])
def test_aggregate_matches_sparse_product(ctx, width):
    s, g, torch = ctx
    say("aggregate width", width)
    rng = np.random.default_rng(width)
    X = rng.standard_normal((g.N, width)).astype(np.float32)
    Y = s.op_aggregate(torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    ref = g.A @ X.astype(np.float64)
    assert rel_err(Y.cpu().numpy().astype(np.float64), ref) < 2e-6


@pytest.fixture(scope="module")
def one_community_ctx():
    """40000 rows in one community, whose rows fit an XCD's L2 in no more than 32 columns: the tile rules part here."""
    import torch
    from paper_2112_09335_amd import binding
    rng = np.random.default_rng(78)
    N = 40000
    src, dst = rng.integers(0, N, 150000).astype(np.int32), rng.integers(0, N, 150000).astype(np.int32)
    s = binding.Solver(0)
    s.build_graph(N, src, dst, 1, np.zeros(N, np.int32))
    s.set_model([516, 64, 16], **HYPER)
    s.set_workspace()
    yield s, OracleGraph(N, src, dst, 1, np.zeros(N, np.int32)), torch
    s.close()


@pytest.mark.parametrize("width", [33, 48, 64, 96, 100, 130, 256, 261, 300, 320, 516])
def test_aggregate_in_whole_rows_even_tiles_and_tiles_of_a_line(one_community_ctx, width):
    s, g, torch = one_community_ctx
    say("one community, width", width)
    X = np.random.default_rng(width).standard_normal((g.N, width)).astype(np.float32)
    Y = s.op_aggregate(torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    assert rel_err(Y, g.A @ X.astype(np.float64)) < 2e-6


@pytest.mark.parametrize("n,widths", [(1 << 24, (4, 5, 16, 32)), ((1 << 24) + 3, (4, 5, 16, 32)), (1 << 22, (256,)), ((1 << 22) + 3, (256,)),
                                      (1 << 18, (4096,)), ((1 << 18) + 1, (4096, 4095))])
def test_aggregate_on_both_sides_of_the_32_bit_offsets(n, widths):
    """Up to 2^24 rows and 4 GiB a gather's offset is formed in 32 bits, beyond in 64: one to many lanes per gathered row, few rows
    of many columns and the other way round.  A few edges between far ends of the numbering; a node without edges
    keeps its row.  Three terms at most per entry: within 1e-6 of their magnitudes."""
    import torch
    from paper_2112_09335_amd import binding
    say("row offsets", n, widths)
    rng = np.random.default_rng(9)
    nodes = np.unique(np.concatenate([[0, n - 1, n - 2], rng.integers(0, n, size=997)])).astype(np.int32)
    src, dst = nodes[:-1], nodes[1:]                       # a path through them
    src, dst = np.append(src, 0).astype(np.int32), np.append(dst, n - 1).astype(np.int32)
    s = binding.Solver(0)
    try:
        s.build_graph(n, src, dst, 1, None)
        s.set_model([max(widths), 5, 3], **HYPER)
        s.set_workspace()
        for width in widths:
            X = torch.randn(n, width, device="cuda")
            Y = s.op_aggregate(X)
            want = X.clone()
            x = X[torch.from_numpy(nodes).cuda().long()].double()          # every touched node has two neighbours: 1/3 each
            want[torch.from_numpy(nodes).cuda().long()] = ((x + x.roll(1, 0) + x.roll(-1, 0)) / 3.0).float()
            assert want.sub_(Y).abs_().max().item() <= 1e-6 * X.abs().max().item()
            del X, Y, want
    finally:
        s.close()


def test_aggregate_is_exact_on_integers_scaled_by_the_values(ctx):
    """With X = e_j (unit columns) the result reproduces the stored values of A~ bit for bit."""
    s, g, torch = ctx
    say("aggregate unit columns")
    cols = [0, 17, g.N - 1]
    X = np.zeros((g.N, 4), np.float32)
    for k, j in enumerate(cols):
        X[j, k] = 1.0
    Y = s.op_aggregate(torch.from_numpy(X).cuda()).cpu().numpy()
    A32 = g.A.astype(np.float32).toarray() if g.N <= 8000 else None
    for k, j in enumerate(cols):
        assert np.array_equal(Y[:, k], A32[:, j])


@pytest.mark.parametrize("width", [3, 10, 16, 256])
def test_aggregate_segments_matches_per_community_products(ctx, width):
    s, g, torch = ctx
    say("aggregate_segments width", width)
    rng = np.random.default_rng(100 + width)
    V = rng.standard_normal((g.N, width)).astype(np.float32)
    P = s.op_aggregate_segments(torch.from_numpy(V).cuda()).cpu().numpy().astype(np.float64)
    # the segments of a row partition its entries, so seg_ptr is the row pointer of an n_seg x N matrix
    S = sp.csr_matrix((g.val, g.col, g.seg_ptr), shape=(g.n_segments, g.N))
    ref = (S @ V.astype(np.float64))[s.get_segment_order()]
    assert P.shape == ref.shape
    assert rel_err(P, ref) < 2e-6
    # summing a row's segments gives the full aggregation
    full = np.zeros((g.N, width))
    np.add.at(full, g.seg_row[s.get_segment_order()], P)
    assert rel_err(full, g.A @ V.astype(np.float64)) < 2e-6


@pytest.mark.parametrize("n,K,C", [(1000, 256, 256), (777, 500, 128), (300, 128, 3), (1000, 7, 64), (129, 16, 256),
                                   (4100, 512, 512), (513, 10, 256), (2000, 256, 16), (64, 64, 64), (1, 5, 2)])
def test_transform_matches_fp64_product(ctx, n, K, C):
    s, g, torch = ctx
    say("transform", n, K, C)
    rng = np.random.default_rng(n + K + C)
    A = rng.standard_normal((n, K)).astype(np.float32)
    B = rng.standard_normal((K, C)).astype(np.float32)
    out = s.op_transform(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()).cpu().numpy().astype(np.float64)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert rel_err(out, ref) < 1e-5


@pytest.mark.parametrize("n,K,C", [(6000, 256, 256), (5000, 500, 128), (3000, 128, 3), (6000, 512, 512), (4097, 256, 16),
                                   (100, 7, 5), (17, 300, 40)])
def test_wgrad_matches_fp64_product(ctx, n, K, C):
    s, g, torch = ctx
    say("wgrad", n, K, C)
    rng = np.random.default_rng(n + K + C + 1)
    A = rng.standard_normal((n, K)).astype(np.float32)
    G = rng.standard_normal((n, C)).astype(np.float32)
    out = s.op_wgrad(torch.from_numpy(A).cuda(), torch.from_numpy(G).cuda()).cpu().numpy().astype(np.float64)
    ref = A.astype(np.float64).T @ G.astype(np.float64)
    assert rel_err(out, ref) < 1e-5


@pytest.mark.parametrize("n,K,C", [(3000, 512, 512), (1031, 500, 200), (2000, 128, 256), (640, 37, 129)])
def test_products_agree_on_the_fp32_and_the_bf16_split_matrix_core_paths(ctx, n, K, C):
    """Results wider than 32 columns run on the bf16 matrix cores with both operands split exactly into three bf16
    parts; the fp32 MFMA kernels stay selectable.  Both must sit at fp32 rounding of the fp64 product, also for
    operands whose rows span many orders of magnitude."""
    s, g, torch = ctx
    say("split products", n, K, C)
    rng = np.random.default_rng(n * 7 + K + C)
    A = (rng.standard_normal((n, K)) * np.exp(3.0 * rng.standard_normal((n, 1)))).astype(np.float32)
    B = (rng.standard_normal((K, C)) * np.exp(2.0 * rng.standard_normal((1, C)))).astype(np.float32)
    G = (rng.standard_normal((n, C)) * np.exp(3.0 * rng.standard_normal((n, 1)))).astype(np.float32)
    ref_nn = A.astype(np.float64) @ B.astype(np.float64)
    mag_nn = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    ref_tn = A.astype(np.float64).T @ G.astype(np.float64)
    mag_tn = np.abs(A).astype(np.float64).T @ np.abs(G).astype(np.float64)
    At, Bt, Gt = (torch.from_numpy(x).cuda() for x in (A, B, G))
    try:
        for split in (0, 1):
            s.tune("gemm_split", split)
            nn = s.op_transform(At, Bt).cpu().numpy().astype(np.float64)
            tn = s.op_wgrad(At, Gt).cpu().numpy().astype(np.float64)
            assert (np.abs(nn - ref_nn) / mag_nn).max() < 2e-6, split
            assert (np.abs(tn - ref_tn) / mag_tn).max() < 2e-6, split
    finally:
        s.tune("gemm_split", 1)


@pytest.mark.parametrize("n,K,C", [(63, 17, 33), (65, 129, 65), (2047, 300, 200), (32640, 37, 200), (32641, 37, 200),
                                   (65408, 37, 7), (65409, 37, 7), (32641, 300, 201), (3, 1, 1), (20011, 128, 32)])
def test_products_on_both_sides_of_the_tile_rules(ctx, n, K, C):
    """64-row tiles against 128-row ones (wide results), 32-row against 128-row workgroups (narrow ones), chunks from 64 rows:
    the sizes where a rule changes sides, remainders of tiles, chunks and quads.  fp32 sums of at most 2048 terms: the same
    2e-6 of |A||B| as above."""
    s, g, torch = ctx
    say("tile rules", n, K, C)
    rng = np.random.default_rng(n + 3 * K + C)
    A = rng.standard_normal((n, K)).astype(np.float32)
    B = rng.standard_normal((K, C)).astype(np.float32)
    G = rng.standard_normal((n, C)).astype(np.float32)
    At, Bt, Gt = (torch.from_numpy(x).cuda() for x in (A, B, G))
    for got, X, Y in ((s.op_transform(At, Bt), A, B), (s.op_wgrad(At, Gt), A.T, G)):
        ref = X.astype(np.float64) @ Y.astype(np.float64)
        mag = np.abs(X).astype(np.float64) @ np.abs(Y).astype(np.float64)
        assert (np.abs(got.cpu().numpy() - ref) / mag).max() < 2e-6


@pytest.mark.parametrize("n,K,C", [(100, 37, 7), (70001, 37, 7), (50, 130, 16), (77, 5, 3)])
def test_an_infinity_in_the_last_row_stays_an_infinity_in_narrow_products(ctx, n, K, C):
    """Steps past the end of the contraction repeat the last row of an operand: it must not meet the zeros of the other."""
    s, g, torch = ctx
    say("infinity", n, K, C)
    A, B = torch.ones(n, K, device="cuda"), torch.ones(K, C, device="cuda")
    B[K - 1, 1] = float("inf")
    want = torch.full((n, C), float(K), device="cuda")
    want[:, 1] = float("inf")
    assert torch.equal(s.op_transform(A, B), want)
    A[n - 1, 2] = float("-inf")
    G, want = torch.ones(n, C, device="cuda"), torch.full((K, C), float(n), device="cuda")
    want[2] = float("-inf")
    assert torch.equal(s.op_wgrad_noalloc(A, G), want)


# 128 x 128 tiles (two of A's columns, one and three of G's) and 64 x 64 ones (49161 rows); last chunks that end inside a step
@pytest.mark.parametrize("n,K,C", [(50003, 129, 33), (49161, 256, 128), (60001, 500, 129), (65537, 129, 300)])
@pytest.mark.parametrize("kind", ["even", "growing", "late", "columns", "masked", "opposed"])
def test_wgrad_of_rows_and_columns_of_unlike_size(ctx, n, K, C, kind):
    """Columns that grow by 2^80 from row to row, that start with thousands of zeros, or that are 1e-20 to 1e20 of each other must
    come out as from 32-bit products, also where the largest entries of a column meet zeros (a node whose features are 1e7 times the
    others', all of its units inactive) or every row of A is as much larger as that of G is smaller: an operand is held in all
    24 bits whatever the rest of its column is like."""
    import torch
    s, g, _ = ctx
    say("wgrad of unlike rows", n, K, C, kind)
    gen = torch.Generator(device="cuda").manual_seed(n + K)
    A = torch.randn((n, K), generator=gen, device="cuda")
    G = torch.randn((n, C), generator=gen, device="cuda") * 1e-3
    if kind == "growing":
        A *= torch.exp2(torch.arange(n, device="cuda") * (40.0 / n))[:, None]
        G *= torch.exp2(torch.arange(n, device="cuda") * (80.0 / n) - 60.0)[:, None]
    elif kind == "late":
        A[: n // 3, ::2] = 0
        G[: n // 2, 1::3] = 0
    elif kind == "columns":
        A *= 10.0 ** torch.randint(-20, 1, (1, K), generator=gen, device="cuda")
        G *= 10.0 ** torch.randint(0, 20, (1, C), generator=gen, device="cuda")
    elif kind == "masked":
        A[5::1000] *= 1e7
        G[5::1000] = 0
    elif kind == "opposed":
        size = torch.exp(4.0 * torch.randn((n, 1), generator=gen, device="cuda"))
        A *= size
        G /= size
    got = s.op_wgrad_noalloc(A, G).double()
    ref, mag = A.double().t() @ G.double(), A.double().abs().t() @ G.double().abs()
    # (fp32 sums over chunks of at most a few hundred rows; the tolerance of the other products)
    assert ((got - ref).abs() / mag).max().item() < 2e-6


def base_chunk_rows(n, K, C):
    """Rows per chunk of the W-gradient product at its base: about 1024 workgroups of 128-row tiles, at least 256 rows."""
    tiles = -(-K // 128) * -(-C // (128 if C > 32 else 32))
    chunks = max(1, min(-(-1024 // tiles), -(-n // 256)))
    return -(-(-(-n // chunks)) // 16) * 16


# 48 and 49 tiles, the limit on the partial matrices (512 x 512), 64-row tiles (476 x 347, 500 x 128), narrow results
FP32_SUM_SHAPES = [(13752, 767, 1000), (32114, 896, 896), (20000, 512, 512), (16956, 476, 347), (20000, 500, 128), (5000, 100, 20)]


@pytest.mark.parametrize("split", [1, 0])
@pytest.mark.parametrize("n,K,C", FP32_SUM_SHAPES)
def test_fp32_sums_of_the_wgrad_product_are_no_longer_than_a_base_chunk(n, K, C, split):
    """Chunks are added in fp64, so how many rows are summed in fp32 can be counted: 2^29 in the first row swallows the ones
    behind it (half a unit in its last place is 32, sixteen rows are added at a time) until the chunk ends.  -2^29 in the last row brings
    the sum back to a small whole number; the chunk it closes is rounded once, by at most 32."""
    import torch
    from paper_2112_09335_amd import binding
    say("fp32 sums", n, K, C, split)
    s = binding.Solver(0)
    s.tune("gemm_split", split)                      # process-wide
    try:
        A, G = torch.ones(n, K, device="cuda"), torch.ones(n, C, device="cuda")
        G[0] = 2.0 ** 29
        G[n - 1] = -2.0 ** 29
        lost = n - 2 - s.op_wgrad_noalloc(A, G)
        assert lost.abs().max().item() <= base_chunk_rows(n, K, C) + 32
        # the same through the hidden-layer prologue: a graph without edges (A~ = 1), T_1 = 1 everywhere and nu = 1 make
        # nu (T_1 - Z_1) those numbers, and the search reports the squared norm of their sums
        s.build_graph(n, np.zeros(0, np.int32), np.zeros(0, np.int32), 1, None)
        s.set_model([K, C, 3], **dict(HYPER, nu=1.0))
        s.set_workspace()
        s.set_data(np.ones((n, K), np.float32), np.zeros(n, np.int32))
        W1 = np.zeros((K, C), np.float32)
        W1[0] = 1.0
        s.init([W1, np.zeros((C, 3), np.float32)])
        Z1 = np.zeros((n, C), np.float32)
        Z1[0], Z1[n - 1] = -2.0 ** 29, 2.0 ** 29
        s.set_state(Z=[Z1, None])
        s.run(1)
        lost = n - 2 - (s.get_steps()[3][0] / (K * C)) ** 0.5
        assert abs(lost) <= base_chunk_rows(n, K, C) + 32
    finally:
        s.tune("gemm_split", 1)
        s.close()


def test_calibration_kernels_report_a_rate(ctx):
    s, g, torch = ctx
    assert s.op_calibrate("copy", 1 << 22, 3) > 10.0        # GB/s
    assert s.op_calibrate("update", 1 << 22, 3) > 10.0
    assert s.op_calibrate("mfma", 200, 3) > 1.0             # TFLOP/s
    assert s.op_calibrate("mfma_bf16", 200, 3) > 1.0
    assert s.op_calibrate("mfma_bf16_valu6", 200, 3) > 1.0


def test_profile_counts_kernel_calls_that_still_run_on_another_stream():
    """Eight products of more than a millisecond each on torch's stream: collecting the records waits for them."""
    import torch
    from paper_2112_09335_amd import binding
    n, K, C = 400000, 512, 512
    s = binding.Solver(0)
    try:
        A, B = torch.zeros(n, K, device="cuda"), torch.zeros(K, C, device="cuda")
        s.op_transform(A, B)
        torch.cuda.synchronize()
        for reset in (False, True):
            s.profile(True)
            for _ in range(8):
                s.op_transform(A, B)
            if reset:
                s.profile(True)                      # clears what was enqueued before
            rec = [r for r in s.get_profile().values() if r["records"]]
            torch.cuda.synchronize()
            assert sum(r["records"] for r in rec) == (0 if reset else 8)
            if not reset:
                assert rec[0]["ms"] > 0 and rec[0]["flops"] == 8 * 2.0 * n * K * C
        s.profile(False)
    finally:
        s.close()


def test_kernel_calls_are_ordered_with_the_sweep_and_can_be_captured():
    """A kernel-level call runs on torch's current stream, after the iterations enqueued before it and before those enqueued
    later (they share scratch memory), and inside a captured graph."""
    import torch
    from paper_2112_09335_amd import binding
    w = synth.config(2, 0.1)
    a, b = binding.Solver.from_workload(w, 0), binding.Solver.from_workload(w, 0)
    try:
        side = torch.cuda.Stream()
        X = torch.randn(w.N, 128, device="cuda")
        torch.cuda.synchronize()
        want = b.op_aggregate(X * 2)
        torch.cuda.synchronize()
        for _ in range(3):
            a.run(2)
            with torch.cuda.stream(side):
                got = a.op_aggregate(X * 2)
            here = a.op_aggregate(X + X)
            a.run(1)
            b.run(3)
            torch.cuda.synchronize()
            assert torch.equal(got, want) and torch.equal(here, want)
        for l in range(1, w.L + 1):
            assert np.array_equal(a.get_W(l), b.get_W(l)) and np.array_equal(a.get_Z(l), b.get_Z(l))
        G, out = torch.randn(w.N, 3, device="cuda"), torch.empty(128, 3, device="cuda")
        graph = torch.cuda.CUDAGraph()
        a.op_wgrad_noalloc(X, G, out)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            a.op_wgrad_noalloc(X, G, out)
        for k in range(3):
            X.mul_(1.5)
            eager = b.op_wgrad_noalloc(X, G)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager), k
            a.run(1)
    finally:
        a.close()
        b.close()


def test_a_capture_of_the_own_stream_leaves_the_order_of_the_calls_around_it():
    """A call on torch's stream still runs while the context's own stream is captured; what the own stream does after the
    capture waits for that call, and replays give the eager result."""
    import torch
    from paper_2112_09335_amd import binding
    w = synth.config(2, 0.1)
    a, b = binding.Solver.from_workload(w, 0), binding.Solver.from_workload(w, 0)
    try:
        X, G, out = torch.randn(w.N, 500, device="cuda"), torch.randn(w.N, 128, device="cuda"), torch.empty(500, 128, device="cuda")
        want = b.op_wgrad(X, G)
        torch.cuda.synchronize()
        a.run(1)
        for _ in range(50):
            got = a.op_wgrad(X, G)                       # (shares the scratch of the partial matrices with the sweep)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(a.stream):
            graph.capture_begin()
            a.op_wgrad_noalloc(X, G, out)
            graph.capture_end()
        a.run(2)
        b.run(3)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        for l in range(1, w.L + 1):
            assert np.array_equal(a.get_W(l), b.get_W(l)) and np.array_equal(a.get_Z(l), b.get_Z(l))
        for k in range(3):
            X.mul_(1.5)
            eager = b.op_wgrad_noalloc(X, G)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, eager), k
            a.run(1)
    finally:
        a.close()
        b.close()


@pytest.mark.parametrize("own", [False, True])
def test_calls_on_the_null_stream_and_on_another_one_in_turn(own):
    """The calls share their scratch: one on another stream (a side stream, the context's own) waits for those on the null
    stream before it, and they for it, although the calls before the first change of stream leave no event behind."""
    import torch
    from paper_2112_09335_amd import binding
    s = binding.Solver(0)
    try:
        side = s.stream if own else torch.cuda.Stream()
        gen = torch.Generator(device="cuda").manual_seed(3)
        A = [torch.randn(20000, 256, generator=gen, device="cuda") for _ in range(2)]
        G = [torch.randn(20000, 200, generator=gen, device="cuda") for _ in range(2)]
        want = []
        for a, g in zip(A, G):
            want.append(s.op_wgrad_noalloc(a, g))
            torch.cuda.synchronize()
        out = [torch.empty_like(want[0]) for _ in range(12)]
        torch.cuda.synchronize()
        for i, o in enumerate(out):
            if i % 3 == 2:
                with torch.cuda.stream(side):
                    s.op_wgrad_noalloc(A[i % 2], G[i % 2], o)
            else:
                s.op_wgrad_noalloc(A[i % 2], G[i % 2], o)
        torch.cuda.synchronize()
        for i, o in enumerate(out):
            assert torch.equal(o, want[i % 2]), i
    finally:
        s.close()


@pytest.mark.parametrize("mode", ["global", "relaxed"])
def test_the_first_change_of_stream_while_some_other_stream_is_captured(mode):
    """The event behind calls on the null stream is recorded when the first call goes to another stream: also where the thread
    is capturing a stream that has nothing to do with either.  The capture is whole and replays give the eager result."""
    import torch
    from paper_2112_09335_amd import binding
    s = binding.Solver(0)
    try:
        A, G = torch.randn(20000, 256, device="cuda"), torch.randn(20000, 200, device="cuda")
        x, y = torch.randn(1000, device="cuda"), torch.zeros(1000, device="cuda")
        side, captured = torch.cuda.Stream(), torch.cuda.Stream()
        out = [torch.empty(256, 200, device="cuda") for _ in range(2)]
        want = A.double().t() @ G.double()
        torch.cuda.synchronize()
        for _ in range(20):
            s.op_wgrad_noalloc(A, G, out[0])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=captured, capture_error_mode=mode):
            torch.add(x, 1.0, out=y)
            with torch.cuda.stream(side):
                s.op_wgrad_noalloc(A, G, out[1])
            y.mul_(2.0)
        torch.cuda.synchronize()
        for o in out:
            assert (o - want).norm() <= 1e-5 * want.norm()
        for k in range(3):
            x.add_(1.0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, (x + 1.0) * 2.0), k
    finally:
        s.close()


def test_a_refused_call_between_kernel_calls_on_two_streams_keeps_their_order():
    """set_data makes the own stream wait for the call before it, then refuses the labels and enqueues nothing: a call on a
    third stream still waits for the one on the first, with which it shares the scratch of the partial matrices."""
    import torch
    from paper_2112_09335_amd import binding
    w = synth.config(2, 0.1)
    s = binding.Solver.from_workload(w, 0)
    try:
        X = [torch.randn(w.N, 500, device="cuda") for _ in range(2)]
        G = [torch.randn(w.N, 128, device="cuda") for _ in range(2)]
        want = [s.op_wgrad(x, g) for x, g in zip(X, G)]
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        for _ in range(5):
            for _ in range(50):
                first = s.op_wgrad(X[0], G[0])
            with pytest.raises(binding.CadmmError):
                s.set_data(w.X, np.full(w.N, w.dims[-1], np.int32))
            with torch.cuda.stream(side):
                second = s.op_wgrad(X[1], G[1])
            torch.cuda.synchronize()
            assert torch.equal(first, want[0]) and torch.equal(second, want[1])
    finally:
        s.close()


def test_kernel_calls_and_readouts_while_another_device_is_current():
    """The events of a context belong to its own device, whichever the calling thread has current."""
    import torch
    from paper_2112_09335_amd import binding
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    w = synth.make_workload("two-devices", 5, 20000, 4, [256, 64, 4], 4, 2, graph="sbm", features="gaussian", avg_degree=6,
                            frac_intra=0.8)
    s = binding.Solver.from_workload(w, 0)
    try:
        X = torch.randn(w.N, 64, device="cuda:0")
        with torch.cuda.device(0):
            want = s.op_aggregate(X)
            s.run(2)
            Z = [s.get_Z(1) for _ in range(2)]
        with torch.cuda.device(1):
            t = binding.Solver.from_workload(w, 0)
            torch.cuda.set_device(1)
            got = t.op_aggregate(X)
            t.run(2)
            assert torch.equal(got, want)
            for _ in range(2):                           # (the second large readout goes through the pinned pieces)
                assert np.array_equal(t.get_Z(1), Z[0])
            t.close()
    finally:
        s.close()

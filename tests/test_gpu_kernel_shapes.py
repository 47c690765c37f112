"""Kernels and dispatch rules at the sizes where they can go wrong: tile edges, remainders, smallest and largest of a
range.  Every comparison is against the CPU oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from util import assert_close

pytestmark = pytest.mark.gpu


def G():
    import paper_2005_03300_amd as g
    return g


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def host(x):
    return x.detach().cpu().numpy()


@pytest.mark.parametrize("K,M,N", [
    (1, 70, 70), (15, 64, 33), (17, 33, 33), (63, 65, 40), (130, 48, 34),          # fewer rows than a workgroup's trip
    (5000, 64, 41), (3001, 41, 64), (4096, 64, 64), (3000, 65, 17),                # one and two column groups, four and two row sets
    (2001, 192, 48), (2500, 256, 64), (3007, 602, 64), (1500, 256, 100),           # three, four and ten groups; 16 to 64 columns of B
    (1100, 520, 130), (700, 1100, 65), (900, 2100, 20),                            # more columns than one workgroup takes
    (300_000, 64, 64), (200_000, 64, 16)])                                         # two-stage reduction of the partial results
def test_gemm_tn_any_shape(K, M, N):
    g = G()
    H = synth.normal_features(K, M, 41)
    S = synth.normal_features(K, N, 42)
    Yd = torch.full((M, N), float("nan"), device="cuda")
    g.gcn_gemm(1, 0, dev(H), dev(S), Yd)
    first = host(Yd)
    want = H.astype(np.float64).T @ S.astype(np.float64)
    assert_close(first, want, f"TN {K}: {M}x{N}")
    g.gcn_gemm(1, 0, dev(H), dev(S), Yd)
    np.testing.assert_array_equal(first.view(np.uint32), host(Yd).view(np.uint32))


def test_gemm_tn_epilogues_and_pitch():
    g = G()
    K, M, N = 3000, 70, 50
    H = synth.normal_features(K, M, 43)
    S = synth.normal_features(K, N, 44)
    bias = synth.normal_features(1, N, 45)[0]
    Zp = synth.normal_features(M, N, 46)
    Hd = dev(np.concatenate([H, np.full((K, 7), np.nan, np.float32)], 1))[:, :M]
    Cd = torch.full((M, N + 3), float("nan"), device="cuda")
    want = H.astype(np.float64).T @ S.astype(np.float64)
    g.gcn_gemm(1, 0, Hd, dev(S), Cd[:, :N], bias=dev(bias), epilogue=g.EPI_RELU)
    assert np.all(np.isnan(host(Cd)[:, N:]))
    assert_close(host(Cd)[:, :N], np.maximum(want + bias, 0), "TN + bias + relu")
    g.gcn_gemm(1, 0, Hd, dev(S), Cd[:, :N], epilogue=g.EPI_MASK, Zprev=dev(Zp))
    assert_close(host(Cd)[:, :N], np.where(Zp > 0, want, 0), "TN + mask")


@pytest.mark.parametrize("M,N,lda", [(33, 16, 64), (70, 16, 96), (129, 41, 160), (301, 16, 320), (302, 64, 352)])
def test_gemm_tn_of_padded_rows(M, N, lda):
    """Rows of A that are whole 128-byte lines but whose last four columns start at any multiple of 4 bytes (the loads of these
    rows carry the non-temporal hint)."""
    g = G()
    K = 2500
    H, S = synth.normal_features(K, M, 47), synth.normal_features(K, N, 48)
    Hd = torch.full((K, lda), float("nan"), device="cuda")[:, :M].copy_(dev(H))
    assert Hd.data_ptr() % 128 == 0
    Cd = torch.full((M, N), float("nan"), device="cuda")
    g.gcn_gemm(1, 0, Hd, dev(S), Cd)
    assert_close(host(Cd), H.astype(np.float64).T @ S.astype(np.float64), f"TN {M}x{N}, pitch {lda}")


@pytest.mark.parametrize("M,K,N", [(4100, 256, 64), (2049, 602, 64), (1000, 602, 256), (130, 1000, 48), (70, 1900, 20),
                                   (65, 2300, 17), (300, 240, 41), (1025, 512, 32)])
def test_gemm_nn_wide_second_operand(M, K, N):
    """op(B) between 40 KB and a compute unit's LDS, in one or several column passes, and beyond it."""
    g = G()
    A = synth.normal_features(M, K, 47)
    B = synth.normal_features(K, N, 48)
    Cd = torch.full((M, N), float("nan"), device="cuda")
    g.gcn_gemm(0, 0, dev(A), dev(B), Cd)
    want = A.astype(np.float64) @ B.astype(np.float64)
    assert_close(host(Cd), want, f"NN {M}x{K}x{N}")
    Zp = synth.normal_features(M, N, 49)
    g.gcn_gemm(0, 1, dev(A), dev(np.ascontiguousarray(B.T)), Cd, epilogue=g.EPI_MASK, Zprev=dev(Zp))
    assert_close(host(Cd), np.where(Zp > 0, want, 0), f"NT + mask {M}x{K}x{N}")


@pytest.mark.parametrize("n,f", [(1, 1), (127, 3), (129, 41), (5000, 64), (4097, 65), (2500, 130), (200_001, 5)])
def test_bias_gradient(n, f):
    """dbias of the per-layer backward call: column sums of G."""
    g = G()
    src = np.arange(n, dtype=np.int32)
    a = g.gcn_csr_create(n, dev(src), dev(np.roll(src, 1)), g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    Gm = synth.normal_features(n, f, 50)
    Hin = synth.normal_features(n, f, 51)
    W = torch.eye(f, device="cuda")
    S, Y, db = torch.empty(n, f, device="cuda"), torch.empty(f, f, device="cuda"), torch.full((f,), float("nan"), device="cuda")
    g.gcn_layer_backward(a, dev(Hin), None, W, dev(Gm), S, S, Y, None, order=g.ORDER_GEMM_FIRST, dbias=db)
    want = Gm.astype(np.float64).sum(0)
    assert np.all(np.abs(host(db) - want) <= 1e-5 * np.sqrt(n) * np.maximum(1.0, np.abs(want)))
    a.close()


@pytest.mark.parametrize("n", [1, 63, 64, 65, 511, 513, 8191, 8192, 8193, 16_385, 70_001])
@pytest.mark.parametrize("width", [0, 1, 2, 3])
def test_radix_sort_tile_edges(n, width):
    """Keys that put whole wavefronts, whole tiles or single keys on one digit; payloads of every size."""
    g = G()
    rs = np.random.default_rng(61 + width)
    for keys in (rs.integers(0, 1 << 40, n, dtype=np.uint64), np.arange(n, dtype=np.uint64) // np.uint64(64),
                 np.full(n, 77, np.uint64), rs.integers(0, 2, n, dtype=np.uint64) * np.uint64(0xFF00FF)):
        pay = None
        if width:
            pay = rs.integers(-(1 << 31), 1 << 31, (n, width), dtype=np.int64).astype(np.int32)
            pay[:, 0] = np.arange(n, dtype=np.int32)
        order = np.argsort(keys, kind="stable")
        out, pout = g.gcn_radix_sort(dev(keys.view(np.int64)), None if pay is None else dev(pay))
        assert np.array_equal(host(out).view(np.uint64), keys[order])
        if width:
            assert np.array_equal(host(pout), pay[order])


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 4097])
@pytest.mark.parametrize("loops", [False, True])
def test_csr_create_at_powers_of_two_of_n(n, loops):
    """Packed keys at vertex counts where a column takes one bit more, with and without the diagonal: against the oracle,
    A and A^T, for symmetric (one set of arrays for both) and directed input."""
    g = G()
    rs = np.random.default_rng(62 + n)
    src, dst = [rs.integers(0, n, 6 * n, dtype=np.int64).astype(np.int32) for _ in range(2)]
    src[:3] = dst[:3] = n - 1                                       # loops in the input, at the largest id
    for sym in (False, True):
        A = oracle.build_csr(n, src, dst, symmetrise=sym, self_loops=loops, norm="sym" if sym else "none")
        flags = g.BUILD_TRANSPOSE | (g.ADD_SELF_LOOPS if loops else 0) | ((g.SYMMETRISE | g.NORM_SYM) if sym else 0)
        a = g.gcn_csr_create(n, dev(src), dev(dst), flags)
        for trans, want in ((False, A), (True, oracle.transpose(A))):
            rowptr, colidx, val, deg = [host(t) for t in a.arrays(trans)]
            assert np.array_equal(rowptr, want.rowptr) and np.array_equal(colidx, want.colidx)
            assert np.array_equal(val.view(np.uint32), want.val.view(np.uint32))
        a.close()


def test_matrices_of_changing_size_reuse_memory_safely():
    """Matrices of changing size come and go, on two streams in turn, and their products are checked: blocks given back by one
    are taken by the next (two threads at the same time: see below)."""
    g = G()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in range(6):
        n = [5000, 1200, 40_000][k % 3]
        rs = np.random.default_rng(70 + k)
        src, dst = [rs.integers(0, n, 8 * n, dtype=np.int64).astype(np.int32) for _ in range(2)]
        A = oracle.build_csr(n, src, dst)
        X = synth.normal_features(n, 16, 71 + k)
        with torch.cuda.stream(streams[k % 2]):
            a = g.gcn_csr_create(n, dev(src), dev(dst), g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE)
            Z = torch.empty(n, 16, device="cuda")
            g.gcn_spmm(a, 1, dev(X), Z)
            a.close()
            assert_close(host(Z), oracle.spmm(A, X), f"matrix {k}")
    g.gcn_scratch_release()


def _rows_matrix(lengths, ncols, seed):
    """A rectangular matrix with the given row lengths (0 allowed), random ascending columns and values."""
    rs = np.random.default_rng(seed)
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    col = [np.sort(rs.choice(ncols, k, replace=False)) for k in lengths if k]
    colidx = (np.concatenate(col) if col else np.zeros(0)).astype(np.int32)
    return rowptr, colidx, rs.standard_normal(colidx.size).astype(np.float32)


@pytest.mark.parametrize("f", [1, 3, 4, 5, 7, 16, 17, 31, 33, 41, 64, 65, 66, 67, 130])
@pytest.mark.parametrize("shape", ["ends_on_chunk", "crosses_one", "covers_chunks", "mixed", "one_row"])
def test_spmm_rows_across_chunks_any_width(f, shape):
    """Rows that end on, cross or cover the 512-entry chunks of the nonzero-split kernels (also in the last, short chunk),
    at widths that are no multiple of a lane's 16 bytes; operands with a pitch; every epilogue."""
    g = G()
    lengths = {"ends_on_chunk": [512, 256, 256, 100, 412, 512, 3], "crosses_one": [300] * 12 + [1, 0, 511, 2],
               "covers_chunks": [5, 1600, 3, 512, 1024, 509, 1000], "mixed": [0, 1, 700, 0, 31, 32, 33, 1500, 20, 0, 64, 0],
               "one_row": [1700]}[shape]
    n, nc = len(lengths), 2000
    rowptr, colidx, val = _rows_matrix(lengths, nc, 80)
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), g.BUILD_TRANSPOSE)
    A = np.zeros((n, nc))
    for i in range(n):
        A[i, colidx[rowptr[i]:rowptr[i + 1]]] = val[rowptr[i]:rowptr[i + 1]]
    X = synth.normal_features(nc, f, 81)
    Zp = synth.normal_features(n, f, 82)
    Xd = dev(np.concatenate([X, np.full((nc, 3), np.nan, np.float32)], 1))[:, :f]
    want = A @ X.astype(np.float64)
    for epi, ref in ((g.EPI_NONE, want), (g.EPI_RELU, np.maximum(want, 0)), (g.EPI_MASK, np.where(Zp > 0, want, 0))):
        Zd = torch.full((n, f + 5), float("nan"), device="cuda")
        g.gcn_spmm(a, 0, Xd, Zd[:, :f], epi, dev(Zp) if epi == g.EPI_MASK else None)
        assert_close(host(Zd)[:, :f], ref, f"{shape} f={f} epilogue {epi}")
        assert np.all(np.isnan(host(Zd)[:, f:]))
    Xt = synth.normal_features(n, f, 83)
    Zt = torch.full((nc, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 1, dev(Xt), Zt)                                   # mostly empty and one-entry rows
    assert_close(host(Zt), A.T @ Xt.astype(np.float64), f"{shape} transposed f={f}")
    a.close()


@pytest.mark.parametrize("f", [7, 16, 21, 33, 41, 64, 67])
def test_spmm_few_chunks_and_many_chunks_add_alike(f):
    """The kernel for matrices of few chunks, the one for more and the one for many keep every row's order of additions:
    the first rows of a matrix give the same bits whichever kernel runs."""
    g = G()
    rs = np.random.default_rng(84)
    lengths = np.concatenate([rs.integers(0, 90, 3000), [2000, 700], rs.integers(0, 30, 1000)])
    X = synth.normal_features(5000, f, 85)
    rowptr, colidx, val = _rows_matrix(lengths, 5000, 86)
    first = None
    for repeat in (1, 12, 60):                                      # the same rows again and again behind themselves
        rp = np.concatenate([[0]] + [rowptr[1:] + k * rowptr[-1] for k in range(repeat)])
        a = g.gcn_csr_create_from_csr_rect(rp.size - 1, 5000, dev(rp), dev(np.tile(colidx, repeat)), dev(np.tile(val, repeat)), 0)
        g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1)
        Z = torch.empty(rp.size - 1, f, device="cuda")
        g.gcn_spmm(a, 0, dev(X), Z)
        got = host(Z)[:4000].view(np.uint32)
        first = got if first is None else first
        assert np.array_equal(got, first), repeat
        a.close()


@pytest.mark.parametrize("f", [1, 7, 16, 21, 32, 41, 64, 130])
@pytest.mark.parametrize("longest", [1, 4, 900])
def test_spmm_mask_of_many_rows_per_chunk(f, longest):
    """Chunks that begin anything between no row and 512 rows, more than the kernels keep the derivative mask of: the masked
    product is the plain one with the masked places set to zero, bit by bit."""
    g = G()
    rs = np.random.default_rng(87)
    lengths = rs.integers(1, longest + 1, 1_200_000 // (longest + 1))
    n, nc = lengths.size, 3000
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    within = np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lengths)
    colidx = (np.repeat(rs.integers(0, nc - longest, n), lengths) + within).astype(np.int32)
    val = rs.standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1)
    X, Zp = dev(synth.normal_features(nc, f, 88)), dev(synth.normal_features(n, f, 89))
    plain, masked = torch.empty(n, f, device="cuda"), torch.full((n, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, X, plain)
    g.gcn_spmm(a, 0, X, masked, g.EPI_MASK, Zp)
    want = np.add.reduceat(dev(val)[:, None].mul(X[dev(colidx).long()]).cpu().numpy(), rowptr[:-1], axis=0, dtype=np.float64)
    assert_close(host(plain), want, f"rows of 1 to {longest}, f={f}")
    np.testing.assert_array_equal(host(masked), np.where(host(Zp) > 0, host(plain), 0))
    a.close()


@pytest.mark.parametrize("f", [1, 3, 5, 7, 9, 17, 31, 33, 41, 63, 65, 130])
@pytest.mark.parametrize("edges,blocks", [(3000, 1), (90_000, 1), (900_000, 1), (90_000, 3)])
def test_layer_products_of_ragged_width(f, edges, blocks):
    """Products that no ReLU decides on (the last layer's, the backward ones) at widths that are no whole 16-byte pieces,
    with short rows, with rows over several chunks, over column blocks; bias and activation in one pass."""
    g = G()
    n, f_in = 1501, 140
    rs = np.random.default_rng(90)
    src = rs.integers(0, n, edges).astype(np.int32)
    dst = (n * rs.random(edges) ** 3).astype(np.int32)
    flags = g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE
    a = g.gcn_csr_create(n, dev(src), dev(dst), flags)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, blocks)
    A = oracle.build_csr(n, src, dst, symmetrise=False, norm="row")
    At = oracle.transpose(A)
    H, W = synth.normal_features(n, f_in, 92), synth.glorot_weights((f_in, f), 93)[0]
    b, Gl, Zprev = synth.normal_features(1, f, 94)[0], synth.normal_features(n, f, 95), synth.normal_features(n, f_in, 96)
    buf = torch.empty(n * f + 1, device="cuda")
    for first in (0, 1):                                            # 16-byte aligned, and not
        Z, Ho, T = buf[first:first + n * f].view(n, f), torch.empty(n, f, device="cuda"), torch.empty(n, f, device="cuda")
        for act, name in ((g.ACT_NONE, "none"), (g.ACT_RELU, "relu")):
            for bias in (None, b):
                Z.fill_(float("nan")), Ho.fill_(float("nan"))
                g.gcn_layer_forward(a, dev(H), dev(W), Z, Ho, T, g.ORDER_GEMM_FIRST, act, bias=None if bias is None else dev(bias))
                Zref, Href = oracle.layer_forward(At, H, W, name, bias=bias)
                assert_close(host(Z), Zref, f"Z {name}")
                np.testing.assert_array_equal(host(Ho), host(Z) if name == "none" else np.maximum(host(Z), 0))
    S, Y, Gp = torch.empty(n, f, device="cuda"), torch.empty(f_in, f, device="cuda"), torch.empty(n, f_in, device="cuda")
    Sref, Yref, Gpref, _ = oracle.layer_backward(A, H, Zprev, W, Gl)
    g.gcn_layer_backward(a, dev(H), dev(Zprev), dev(W), dev(Gl), None, S, Y, Gp, g.ORDER_GEMM_FIRST)
    assert_close(host(S), Sref, "S = A G")
    assert_close(host(Y), Yref, "Y")
    assert_close(host(Gp), Gpref, "Gprev")
    # the other direction and order: the products have the width of the input, the mask in their epilogue
    Hw, Ww, Gw = synth.normal_features(n, f, 97), synth.glorot_weights((f, 20), 98)[0], synth.normal_features(n, 20, 99)
    Zp = synth.normal_features(n, f, 100)
    T, Z, S = torch.empty(n, f, device="cuda"), torch.empty(n, 20, device="cuda"), torch.empty(n, f, device="cuda")
    Y, Gp = torch.empty(f, 20, device="cuda"), torch.full((n, f), float("nan"), device="cuda")
    g.gcn_layer_forward(a, dev(Hw), dev(Ww), Z, None, T, g.ORDER_SPMM_FIRST, g.ACT_NONE)
    assert_close(host(Z), oracle.layer_forward(At, Hw, Ww, "none")[0], "Z, sparse product first")
    g.gcn_layer_backward(a, dev(Hw), dev(Zp), dev(Ww), dev(Gw), T, S, Y, Gp, g.ORDER_SPMM_FIRST)
    _, Yref, Gpref, _ = oracle.layer_backward(A, Hw, Zp, Ww, Gw)
    assert_close(host(Y), Yref, "Y, sparse product first")
    assert_close(host(Gp), Gpref, "Gprev, sparse product first")
    a.close()


def _far(rows, cols, pitch):
    """A rows x cols matrix in device memory whose rows are `pitch` floats apart (4 GB and more)."""
    return torch.empty((rows - 1) * pitch + cols, device="cuda").as_strided((rows, cols), (pitch, 1))


@pytest.mark.parametrize("which,trans", [("X", 1), ("Z", 0), ("Zprev", 0)])
@pytest.mark.parametrize("f", [5, 16, 41])
def test_spmm_rows_four_gigabytes_apart(which, trans, f):
    """Leading dimensions from 2^30 floats on, where a row's pitch in bytes no longer fits 32 bits, in each operand of each
    entry point of the product; the matrix has three rows of chunks enough for every nonzero-split kernel."""
    g = G()
    nc, pitch = 250_000, (1 << 30) + 4
    rs = np.random.default_rng(101)
    rowptr = np.array([0, 200_000, 370_000, 570_000])
    colidx = np.concatenate([np.sort(rs.choice(nc, k, replace=False)) for k in np.diff(rowptr)]).astype(np.int32)
    val = rs.standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(3, nc, dev(rowptr), dev(colidx), dev(val), g.BUILD_TRANSPOSE)
    xrows, zrows = (3, nc) if trans else (nc, 3)
    X, Zp = synth.normal_features(xrows, f, 102), synth.normal_features(zrows, f, 103)
    Xd, Zd, Pd = [_far(r, f, pitch) if which == k else torch.empty(r, f, device="cuda")
                  for k, r in (("X", xrows), ("Z", zrows), ("Zprev", zrows))]
    Xd.copy_(dev(X)), Pd.copy_(dev(Zp))
    row = np.repeat(np.arange(3), np.diff(rowptr))

    def product(v):
        out = np.zeros((zrows, f))
        for i in range(3):
            k = row == i
            if trans:
                out[colidx[k]] += v[k, None] * X[i].astype(np.float64)
            else:
                out[i] = v[k].astype(np.float64) @ X[colidx[k]].astype(np.float64)
        return np.where(Zp > 0, out, 0)
    for call in (g.gcn_spmm, g.gcn_spmm_static):
        Zd.fill_(float("nan"))
        call(a, trans, Xd, Zd, g.EPI_MASK, Pd)
        assert_close(host(Zd.contiguous()), product(val), call.__name__)
    Zd.fill_(float("nan"))
    g.gcn_spmm_pattern(a, trans, Xd, Zd, None, g.EPI_MASK, Pd)
    assert_close(host(Zd.contiguous()), product(np.ones_like(val)), "gcn_spmm_pattern")
    a.close()


@pytest.mark.parametrize("algo,blocks", [(0, 0), (2, 1), (2, 3), (3, 0), (4, 0)])
@pytest.mark.parametrize("f", [3, 16, 41, 51])
def test_spmm_mask_that_is_the_output(f, algo, blocks):
    """Zprev == Z, with rows inside a chunk, over several chunks, over column blocks, deferred by the hub schedule, and at widths
    whose last lane repeats columns: the result is that of the same call with the mask in a buffer of its own."""
    g = G()
    n = 3000
    rs = np.random.default_rng(104)
    src = rs.integers(0, n, 200_000).astype(np.int32)
    dst = (n * rs.random(200_000) ** 4).astype(np.int32)
    a = g.gcn_csr_create(n, dev(src), dev(dst), g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE)
    for key, value in ((g.CFG_SPMM_ALGO, algo), (g.CFG_SPMM_BLOCKS, blocks), (g.CFG_SWEEP_HEAVY, 64), (g.CFG_HUB_DMIN, 16),
                       (g.CFG_HUB_BLOCK_COLS, 64)):
        g.gcn_csr_config(a, key, value)
    X, M = dev(synth.normal_features(n, f, 105)), dev(synth.normal_features(n, f, 106))
    pitched = torch.full((n, f + 3), float("nan"), device="cuda")
    ones = torch.ones(n, device="cuda")
    calls = [lambda Z, P: g.gcn_spmm(a, 1, X, Z, g.EPI_MASK, P), lambda Z, P: g.gcn_spmm_static(a, 0, X, Z, g.EPI_MASK, P),
             lambda Z, P: g.gcn_spmm_pattern(a, 0, X, Z, ones, g.EPI_MASK, P)]
    for k, call in enumerate(calls):
        apart = torch.empty(n, f, device="cuda")
        call(apart, M)
        for Z in (M.clone(), pitched[:, :f].copy_(M)):
            call(Z, Z)
            assert_close(host(Z), host(apart), f"call {k}")
    assert torch.isnan(pitched[:, f:]).all()
    # the backward call of a layer in sparse-product-first order
    W, Gl, Y = dev(synth.glorot_weights((f, 20), 107)[0]), dev(synth.normal_features(n, 20, 108)), torch.empty(f, 20, device="cuda")
    apart, S, Gp = torch.empty(n, f, device="cuda"), torch.empty(n, f, device="cuda"), M.clone()
    g.gcn_layer_backward(a, X, M, W, Gl, X, S, Y, apart, g.ORDER_SPMM_FIRST)
    g.gcn_layer_backward(a, X, Gp, W, Gl, X, S, Y, Gp, g.ORDER_SPMM_FIRST)
    assert_close(host(Gp), host(apart), "Gprev")
    a.close()


def test_build_count_is_what_was_built():
    """Each stored order counts once, when it is there: a matrix that equals its transpose builds one for both directions, a
    directed one builds two; a matrix that the hub schedule rejects builds none."""
    g = G()
    n = 5000
    rs = np.random.default_rng(109)
    src = dev(rs.integers(0, n, 120_000).astype(np.int32))
    dst = dev((n * rs.random(120_000) ** 4).astype(np.int32))

    def built(a, trans):
        before = g.gcn_build_count()
        g.gcn_spmm_prepare(a, trans, 16)
        return g.gcn_build_count() - before
    sym = g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE
    for flags, again in ((sym, 0), (g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE, 1)):
        for settings, count in (((g.CFG_SPMM_ALGO, 2, g.CFG_SPMM_BLOCKS, 4), 1),                   # the column-blocked order
                                ((g.CFG_SPMM_ALGO, 3, g.CFG_SPMM_BLOCKS, 1, g.CFG_SWEEP_HEAVY, 1 << 20), 1),    # no long rows
                                ((g.CFG_SPMM_ALGO, 3, g.CFG_SPMM_BLOCKS, 1, g.CFG_SWEEP_HEAVY, 30), 2),
                                ((g.CFG_SPMM_ALGO, 3, g.CFG_SPMM_BLOCKS, 4, g.CFG_SWEEP_HEAVY, 30), 3)):
            a = g.gcn_csr_create(n, src, dst, flags)
            for key, value in zip(settings[::2], settings[1::2]):
                g.gcn_csr_config(a, key, value)
            assert [built(a, 0), built(a, 1), built(a, 0), built(a, 1)] == [count, again * count, 0, 0], (flags, settings)
            a.close()
    a = g.gcn_csr_create(n, src, dst, sym)
    for key, value in ((g.CFG_SPMM_ALGO, 4), (g.CFG_HUB_DMIN, 16), (g.CFG_HUB_BLOCK_COLS, 64)):
        g.gcn_csr_config(a, key, value)
    assert [built(a, 0), built(a, 1)] == [2, 0] and g.gcn_spmm_describe(a, 0, 16).startswith("hub(")
    g.gcn_csr_config(a, g.CFG_HUB_DMIN, 4900)                       # longer than any row: rejected
    assert built(a, 0) == 0 and g.gcn_spmm_describe(a, 0, 16).startswith("split(")
    a.close()


def test_split_lds_setting():
    """The LDS padding of the narrow nonzero-split kernels: 0 is the default, a value holds as it is, and no value changes a
    result; what is out of range is refused."""
    g = G()
    n = 40_000
    rs = np.random.default_rng(110)
    src, dst = [rs.integers(0, n, 600_000).astype(np.int32) for _ in range(2)]
    a = g.gcn_csr_create(n, dev(src), dev(dst), g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1)
    for f in (3, 16):
        X, Zp = dev(synth.normal_features(n, f, 111)), dev(synth.normal_features(n, f, 112))
        first = None
        for kb in (0, 18, 28, 38, 64):
            g.gcn_csr_config(a, g.CFG_SPLIT_LDS_KB, kb)
            for epi in (g.EPI_NONE, g.EPI_MASK):
                Z = torch.full((n, f), float("nan"), device="cuda")
                g.gcn_spmm(a, 0, X, Z, epi, Zp)
                first = Z if first is None else first
                assert torch.equal(Z, first if epi == g.EPI_NONE else torch.where(Zp > 0, first, 0.0)), (f, kb, epi)
    for kb in (-1, 17, 65):
        with pytest.raises(g.GcnError):
            g.gcn_csr_config(a, g.CFG_SPLIT_LDS_KB, kb)
    a.close()


@pytest.mark.parametrize("f", [17, 20, 32, 33, 64, 128])
@pytest.mark.parametrize("lengths", [[3, 4], [4], [1], [1, 1, 1, 0, 900] + [1] * 500, [2, 0, 3]])
def test_spmm_mask_on_both_sides_of_its_rule(f, lengths):
    """Matrices whose mean row is just up to, and just beyond, the length below which the mask is looked up when a row ends, with
    rows that cross chunks and empty rows among them; value-free with row factors too: the masked product is the plain
    one with the masked places set to zero, bit by bit."""
    g = G()
    nc = 2000
    lens = np.tile(lengths, 500_000 // sum(lengths))
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    within = np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lens)
    colidx = (np.repeat(np.random.default_rng(113).integers(0, nc - 900, lens.size), lens) + within).astype(np.int32)
    n = lens.size
    val = np.random.default_rng(114).standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1)
    X, M = dev(synth.normal_features(nc, f, 115)), dev(synth.normal_features(n, f, 116))
    scale = dev(synth.normal_features(n, 1, 117)[:, 0])
    for call in (lambda Z, *m: g.gcn_spmm(a, 0, X, Z, *m), lambda Z, *m: g.gcn_spmm_pattern(a, 0, X, Z, scale, *m)):
        plain, masked = torch.empty(n, f, device="cuda"), torch.full((n, f), float("nan"), device="cuda")
        call(plain)
        call(masked, g.EPI_MASK, M)
        assert torch.equal(masked, torch.where(M > 0, plain, 0.0))
    a.close()


@pytest.mark.parametrize("full,length,f,kernel", [
    (1000, 65, 13, "k_spmm_split<16,1>"), (1000, 65, 16, "k_spmm_few<4>"), (1000, 65, 64, "k_spmm_few<8>"), (1000, 65, 41, "k_spmm_ragged"),
    (9000, 65, 3, "k_spmm_split<4,1>"), (9000, 65, 16, "k_spmm_split<4,4>"), (9000, 65, 64, "k_spmm_split<8,4>"),
    (9000, 65, 41, "k_spmm_line<1>"), (9000, 65, 67, "k_spmm_line<2>"), (9000, 65, 130, "k_spmm_line<1>"), (9000, 65, 132, "k_spmm_split<8,4>")])
@pytest.mark.parametrize("share", [1, 20, 21, 63, 64, 65, 80, 81, 160, 161, 240, 241, 511, 512, 513])
def test_rows_without_entries_go_with_the_chunks(full, length, f, kernel, share):
    """As many empty rows per chunk as fit one step of the zeroing, one less and one more; as many as small products take with their chunks
    (20 stores of 1 to 16 rows, 240 rows) and one more, and as a chunk takes at the most and one more (a launch of their own); a last chunk with a smaller share or none: they are zero, the other rows have the bits of the
    matrix without empty rows, and nothing between the rows of a wider output is touched."""
    g = G()
    chunks = (full * length + 511) // 512
    empty = (share - 1) * chunks + max(1, chunks // 3)
    rs = np.random.default_rng(118)
    lens = np.zeros(full + empty, np.int64)
    has = np.sort(rs.choice(full + empty, full, replace=False))
    lens[has] = length
    colidx = (rs.integers(0, 2000 - length, full)[:, None] + np.arange(length)).astype(np.int32).reshape(-1)
    val = rs.standard_normal(colidx.size).astype(np.float32)
    rowptr = lambda l: dev(np.concatenate([[0], np.cumsum(l)]).astype(np.int64))
    a = g.gcn_csr_create_from_csr_rect(full + empty, 2000, rowptr(lens), dev(colidx), dev(val), 0)
    b = g.gcn_csr_create_from_csr_rect(full, 2000, rowptr(lens[has]), dev(colidx), dev(val), 0)
    X, M = dev(synth.normal_features(2000, f, 119)), dev(synth.normal_features(full + empty, f, 120))
    at = torch.from_numpy(has).cuda()
    for m in (a, b):
        g.gcn_csr_config(m, g.CFG_SPMM_BLOCKS, 1)
        assert kernel in g.gcn_spmm_describe(m, 0, f)
    for epi in (g.EPI_NONE, g.EPI_RELU, g.EPI_MASK):
        Z = torch.full((full + empty, f + 3), float("nan"), device="cuda")
        g.gcn_spmm(a, 0, X, Z[:, :f], epi, M if epi == g.EPI_MASK else None)
        want = torch.zeros(full + empty, f, device="cuda")
        want[at] = g.gcn_spmm(b, 0, X, torch.empty(full, f, device="cuda"), epi, M[at].contiguous() if epi == g.EPI_MASK else None)
        assert torch.equal(Z[:, :f], want) and bool(Z[:, f:].isnan().all()), epi
    a.close()
    b.close()


@pytest.mark.parametrize("rows,length,f,blocks,want", [
    (1000, 17, 16, 0, "split(chunks=34,kernel=k_spmm_short<4>)"), (1000, 17, 41, 0, "split(chunks=34,kernel=k_spmm_short<16>)"),
    (1000, 65, 16, 0, "split(chunks=127,kernel=k_spmm_few<4>)"), (1000, 65, 64, 0, "split(chunks=127,kernel=k_spmm_few<8>)"),
    (1000, 65, 3, 0, "split(chunks=127,kernel=k_spmm_split<4,1>)"), (1000, 65, 21, 0, "split(chunks=127,kernel=k_spmm_split<32,1>)"),
    (1000, 65, 41, 0, "split(chunks=127,kernel=k_spmm_ragged)"), (9000, 65, 41, 0, "split(chunks=1143,kernel=k_spmm_line<1>)"),
    (9000, 65, 67, 0, "split(chunks=1143,kernel=k_spmm_line<2>)"), (9000, 65, 16, 0, "split(chunks=1143,kernel=k_spmm_split<4,4>)"),
    (9000, 65, 32, 0, "split(chunks=1143,kernel=k_spmm_split<8,4>)"),
    (9000, 65, 64, 2, "blocked(blocks=2,cols_per_block=1024,partial_rows=18000,chunks=1143,kernel=k_spmm_split<16,4>)")])
def test_describe_names_the_kernel(rows, length, f, blocks, want):
    """Which kernel a product goes through is part of its description (a stored measurement is tied to it); the product runs
    and is right."""
    g = G()
    nc = 2000
    rowptr = np.arange(rows + 1, dtype=np.int64) * length
    step = nc // length                                             # entries on both sides of the middle column
    colidx = np.tile(np.arange(length) * step, rows).astype(np.int32)
    val = np.random.default_rng(118).standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(rows, nc, dev(rowptr), dev(colidx), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, blocks)
    assert g.gcn_spmm_describe(a, 0, f) == want
    X = synth.normal_features(nc, f, 119)
    Z = torch.full((rows, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, dev(X), Z)
    assert_close(host(Z), val.reshape(rows, length).astype(np.float64) @ X[:step * length:step].astype(np.float64), want)
    a.close()


def test_two_threads_build_use_and_destroy_matrices_at_the_same_time():
    """Two host threads, each with matrices and a stream of its own, whose constructions, products and destructions overlap (the
    library's calls run outside the interpreter's lock): memory that one gives back is taken by the other while its
    work is still running, and every array and result is the oracle's.  A third thread gives kept memory back to the
    device now and then."""
    import threading
    g = G()
    g.lib()
    cases = []
    for k, (n, edges) in enumerate([(3000, 30_000), (700, 60_000), (20_000, 90_000), (9000, 200_000)]):
        rs = np.random.default_rng(120 + k)
        src, dst = rs.integers(0, n, edges).astype(np.int32), (n * rs.random(edges) ** 2).astype(np.int32)
        A = oracle.build_csr(n, src, dst)
        X = synth.normal_features(n, 16, 130 + k)
        cases.append((n, dev(src), dev(dst), A, dev(X), oracle.spmm(A, X)))
    flags = g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE
    start, failed, done = threading.Barrier(2), [], threading.Event()
    torch.cuda.synchronize()

    def work(first):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(60)
                for turn in range(24):
                    n, src, dst, A, X, want = cases[(first + turn) % len(cases)]
                    a = g.gcn_csr_create(n, src, dst, flags)
                    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, [1, 3][turn % 2])       # with and without another stored order
                    Z = torch.full((n, 16), float("nan"), device="cuda")
                    g.gcn_spmm(a, turn % 2, X, Z)
                    rowptr, colidx, val, deg = a.arrays(bool(turn % 2))
                    a.close()
                    torch.cuda.current_stream().synchronize()
                    assert np.array_equal(host(rowptr), A.rowptr) and np.array_equal(host(colidx), A.colidx), turn
                    assert np.array_equal(host(val).view(np.uint32), A.val.view(np.uint32)), turn
                    assert_close(host(Z), want, f"turn {turn}")
        except BaseException as e:
            failed.append(e)
            start.abort()

    def release():
        while not done.wait(0.02):
            g.gcn_scratch_release()
    threads = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    third = threading.Thread(target=release)
    for t in threads + [third]:
        t.start()
    for t in threads:
        t.join(100)
    done.set()
    third.join(20)
    assert not failed, failed
    assert not any(t.is_alive() for t in threads + [third])


@pytest.mark.parametrize("f", [4, 7, 8, 13, 16, 21, 32, 33, 41, 64, 66, 130])
def test_spmm_short_rows_add_alike_in_every_kernel(f):
    """The kernel for few and short rows keeps the order of additions of the others: the same rows give the same bits on their
    own, with one longer row behind them, and in a matrix of many chunks."""
    g = G()
    lengths = np.random.default_rng(140).integers(0, 65, 1000)
    rowptr, colidx, val = _rows_matrix(lengths, 3000, 141)
    longer = _rows_matrix([65], 3000, 142)
    X = dev(synth.normal_features(3000, f, 143))
    results, kernels = [], []
    for kind in ("alone", "longer", "repeated"):
        if kind == "alone":
            m = (rowptr, colidx, val)
        elif kind == "longer":
            m = (np.append(rowptr, rowptr[-1] + 65), np.concatenate([colidx, longer[1]]), np.concatenate([val, longer[2]]))
        else:
            m = (np.concatenate([[0]] + [rowptr[1:] + k * rowptr[-1] for k in range(80)]), np.tile(colidx, 80), np.tile(val, 80))
        a = g.gcn_csr_create_from_csr_rect(m[0].size - 1, 3000, dev(m[0]), dev(m[1]), dev(m[2]), 0)
        g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1)
        kernels.append(g.gcn_spmm_describe(a, 0, f).split("kernel=")[1].split("<")[0].rstrip(")"))
        Z = torch.full((m[0].size - 1, f), float("nan"), device="cuda")
        g.gcn_spmm(a, 0, X, Z)
        results.append(Z[:1000].clone())
        a.close()
    assert kernels[0] == "k_spmm_short" and "k_spmm_short" not in kernels[1:]
    assert torch.equal(results[0], results[1]) and torch.equal(results[0], results[2]), kernels


@pytest.mark.parametrize("f", [4, 16, 20, 32, 36])
@pytest.mark.parametrize("shape", ["one_row", "task_of_rows", "two_tasks", "trips", "few_long", "gaps", "six_tasks"])
def test_sweep_tasks_trips_and_padding(f, shape):
    """The column sweep at the edges of its tasks (511 rows at up to 16 columns, 255 beyond), trips (128 and 64 entries) and pairs
    of steps: rows that fill a window of 64 entries by themselves, tasks without entries, every epilogue, with and
    without stored values.  What padding entries add must not reach a row of the result: row 0 of X holds an infinity."""
    g = G()
    rs = np.random.default_rng(120)
    lengths = {"one_row": [700], "task_of_rows": [1] * 511, "two_tasks": [2] * 255 + [0, 3],
               "trips": [1] * 64 + [63] + [1] * 2 + [0] * 444 + [128] + [0] * 511 + [129],
               "few_long": [600, 0, 590, 1, 580] + [1] * 300, "gaps": [0] * 1100 + [5, 0, 40] + [0] * 600,
               "six_tasks": list(rs.integers(0, 60, 511 * 5 + 9))}[shape]
    n, nc = len(lengths), 900
    rowptr, colidx, val = _rows_matrix(lengths, nc - 1, 121)
    colidx += 1                                                     # column 0 is nobody's
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_ALGO, 3)
    g.gcn_csr_config(a, g.CFG_SWEEP_HEAVY, 1 << 30)
    rows = np.repeat(np.arange(n), lengths)
    X, Zp = synth.normal_features(nc, f, 122), synth.normal_features(n, f, 123)
    want, plain = np.zeros((n, f)), np.zeros((n, f))
    np.add.at(want, rows, val[:, None].astype(np.float64) * X[colidx])
    np.add.at(plain, rows, X[colidx].astype(np.float64))
    X[0] = np.inf
    Xd, Zpd = dev(X), dev(Zp)
    assert g.gcn_spmm_describe(a, 0, f).startswith("sweep(")
    for epi, of in ((g.EPI_NONE, lambda z: z), (g.EPI_RELU, lambda z: np.maximum(z, 0)), (g.EPI_MASK, lambda z: np.where(Zp > 0, z, 0))):
        for waves in (9, 2):
            g.gcn_csr_config(a, g.CFG_SWEEP_WAVES, waves)
            Zd = torch.full((n, f), float("nan"), device="cuda")
            g.gcn_spmm(a, 0, Xd, Zd, epi, Zpd)
            assert_close(host(Zd), of(want), f"{shape} f={f} epilogue {epi}")
            g.gcn_spmm_pattern(a, 0, Xd, Zd, None, epi, Zpd)
            assert_close(host(Zd), of(plain), f"{shape} f={f} epilogue {epi}, value-free")
    a.close()


@pytest.mark.parametrize("graph,f,want", [("wide", 16, "sweep("), ("wide", 32, "sweep("), ("wide", 20, "sweep("), ("wide", 48, "sweep("),
                                          ("few_blocks", 32, "blocked(blocks=4,"), ("few_blocks", 64, "blocked(blocks=4,")])
def test_schedule_by_cost_against_the_one_by_sizes(graph, f, want):
    """Products whose schedule is chosen by estimated cost (A X, and A^T X with a mask), with operands of every pitch and alignment, in
    both forms, against the products that keep the schedule of the sizes (A^T X: the matrix is symmetric) and against the
    oracle: as far from it as those are, and no further."""
    g = G()
    rs = np.random.default_rng(124)
    n, pairs = (500_000, 10_000_000) if graph == "wide" else (150_000, 5_000_000)
    src, dst = [rs.integers(0, n, pairs).astype(np.int32) for _ in range(2)]
    a = g.gcn_csr_create(n, dev(src), dev(dst), g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE)
    assert g.gcn_spmm_describe(a, 0, f).startswith(want) and not g.gcn_spmm_describe(a, 1, f).startswith(want)
    ref = oracle.build_csr(n, src, dst)
    X, Zp = synth.uniform_features(n, f, 125), synth.normal_features(n, f, 126)
    exact = oracle.spmm(ref, X.astype(np.float64))
    Xd, Zpd = dev(X), dev(Zp)
    Zd = torch.empty(n, f, device="cuda")

    def error():
        return float((Zd.double() - dev(exact)).norm() / np.linalg.norm(exact))
    g.gcn_spmm(a, 1, Xd, Zd)
    usual = error()
    kept = host(Zd)
    g.gcn_spmm(a, 0, Xd, Zd)
    first = host(Zd)
    assert error() <= 1.02 * usual, (error(), usual)
    assert_close(first, exact, "A X")
    g.gcn_spmm(a, 0, Xd, Zd)
    assert np.array_equal(first.view(np.uint32), host(Zd).view(np.uint32))
    for trans, pad, off in ((0, 4, 0), (1, 1, 0), (0, 3, 1), (1, 0, 2)):
        Xp = torch.full((n * (f + pad) + off,), float("nan"), device="cuda")[off:].view(n, f + pad)
        Xp[:, :f] = Xd
        Zw = torch.full((n, f + pad), float("nan"), device="cuda")
        g.gcn_spmm(a, trans, Xp[:, :f], Zw[:, :f], g.EPI_RELU)
        assert torch.equal(Zw[:, :f], dev(np.maximum(kept if trans else first, 0))) and bool(torch.isnan(Zw[:, f:]).all()), (trans, pad, off)
        g.gcn_spmm(a, trans, Xp[:, :f], Zw[:, :f], g.EPI_MASK, Zpd)
        assert torch.equal(Zw[:, :f], dev(np.where(Zp > 0, first, 0))), (trans, pad, off)
    g.gcn_spmm_pattern(a, 0, Xd, Zd)
    assert_close(host(Zd), oracle.spmm_pattern(ref, X.astype(np.float64)), "value-free")
    a.close()


@pytest.mark.parametrize("n,m", [(1, 1), (2, 3), (300, 64), (300, 127), (5000, 4096), (5000, 4097), (70_000, 20_481)])
@pytest.mark.parametrize("symmetrise", [False, True])
@pytest.mark.parametrize("loops", [False, True])
def test_csr_create_from_pairs_at_tile_edges(n, m, symmetrise, loops):
    """Small matrices, all of which the sort by buckets of rows takes: pair counts at the edges of its tiles, repeated pairs and pairs of equal
    ends, rows that stay empty at either end, both normalisations; an id outside the range is refused wherever it stands."""
    g = G()
    rs = np.random.default_rng(127)
    src = rs.integers(0, max(1, n // 3), m).astype(np.int32) + n // 3          # (the outer thirds stay empty without loops)
    dst = rs.integers(0, max(1, n // 3), m).astype(np.int32) + n // 3
    src[::5], dst[::7] = src[0], dst[0]
    dst[::11] = src[::11]
    src, dst = np.minimum(src, n - 1), np.minimum(dst, n - 1)
    for norm, flag in (("none", 0), ("sym", g.NORM_SYM), ("row", g.NORM_ROW)):
        flags = flag | (g.SYMMETRISE if symmetrise else 0) | (g.ADD_SELF_LOOPS if loops else 0) | g.BUILD_TRANSPOSE
        a = g.gcn_csr_create(n, dev(src), dev(dst), flags)
        for trans in (False, True):
            ref = oracle.build_csr(n, src, dst, symmetrise=symmetrise, self_loops=loops, norm=norm)
            ref = oracle.transpose(ref) if trans else ref
            rowptr, colidx, val, _ = a.arrays(trans)
            assert np.array_equal(host(rowptr), ref.rowptr) and np.array_equal(host(colidx), ref.colidx), (norm, trans)
            assert np.array_equal(host(val).view(np.uint32), ref.val.view(np.uint32)), (norm, trans)
        a.close()
    for where, bad in ((0, -1), (m - 1, n), (m // 2, 2**31 - 1)):
        for arr in (src, dst):
            kept, arr[where] = arr[where], bad
            with pytest.raises(g.GcnError):
                g.gcn_csr_create(n, dev(src), dev(dst), g.SYMMETRISE if symmetrise else 0)
            arr[where] = kept


def uneven_pairs(kind):
    """Pairs whose rows do not fall into even buckets, or whose columns do not spread over them."""
    rs = np.random.default_rng(131)
    pairs = lambda n, m: (rs.integers(0, n, m), rs.integers(0, n, m))
    if kind == "even":                           # as many buckets as there may be, tiles that end anywhere
        n = 4_000_037
        src, dst = pairs(n, 1_200_007)
    elif kind == "wide":                         # a bucket is one row of a few, with thousands of keys
        n = 700
        src, dst = pairs(n, 1_500_000)
    elif kind == "hub":                          # two rows fill several pieces each, the columns of one lie close together
        n = 300_007
        src, dst = pairs(n, 1_000_000)
        src[:150_000] = 77
        src[150_000:260_000], dst[150_000:260_000] = 123_456, rs.integers(5000, 90_000, 110_000)
    elif kind == "star":                         # one row has nearly everything: by keys
        n = 500_000
        src, dst = pairs(n, 600_000)
        src[:] = 3
    elif kind == "band":                         # neighbouring columns in every row, thirty at the most: places beyond a window
        n = 60_001
        src = np.repeat(np.arange(n), 30)
        dst = np.minimum(src + np.tile(np.arange(30), n), n - 1)
    elif kind == "repeats":                      # pairs that come back a hundred times: places of few distinct keys
        n = 40_000
        src, dst = (np.tile(x, 100) for x in pairs(n, 9_000))
    elif kind == "same":                         # one pair fills more than a piece
        n = 300_000
        src, dst = pairs(n, 400_000)
        src[:100_000], dst[:100_000] = 1234, 4321
    else:                                        # "last": one row that fills its bucket nearly, or more than that
        n = 1 << 19
        src, dst = pairs(n, 300_000)
        rows = int(kind[4:])
        src[:rows], dst[:rows] = 2047 + 2048 * 7, rs.permutation(n)[:rows]
    return n, src.astype(np.int32), dst.astype(np.int32)


@pytest.mark.parametrize("kind", ["even", "wide", "hub", "star", "band", "repeats", "same", "last23000", "last24577"])
@pytest.mark.parametrize("symmetrise", [False, True])
def test_csr_create_from_uneven_pairs(kind, symmetrise):
    """Uneven rows and columns (buckets in the LDS, pieces of large buckets, crowded places, all of it by 64-bit keys), bit for bit against the
    oracle, and the transpose, whose sort starts from the sorted keys."""
    g = G()
    n, src, dst = uneven_pairs(kind)
    for loops, norm, flag in ((True, "sym", g.NORM_SYM), (False, "row", g.NORM_ROW)):
        flags = flag | (g.SYMMETRISE if symmetrise else 0) | (g.ADD_SELF_LOOPS if loops else 0) | g.BUILD_TRANSPOSE
        a = g.gcn_csr_create(n, dev(src), dev(dst), flags)
        for trans in (False, True):
            ref = oracle.build_csr(n, src, dst, symmetrise=symmetrise, self_loops=loops, norm=norm)
            ref = oracle.transpose(ref) if trans else ref
            rowptr, colidx, val, _ = a.arrays(trans)
            assert np.array_equal(host(rowptr), ref.rowptr) and np.array_equal(host(colidx), ref.colidx), (norm, trans)
            assert np.array_equal(host(val).view(np.uint32), ref.val.view(np.uint32)), (norm, trans)
        a.close()


@pytest.mark.parametrize("M,N", [(16, 16), (64, 16), (300, 16), (602, 16), (130, 32), (200, 48), (100, 64), (700, 64), (7, 3), (24, 7)])
@pytest.mark.parametrize("trips", [1, 2, 7, 8, 9, 16, 17])
def test_gemm_tn_trips_and_sums(M, N, trips):
    """Numbers of 16-row trips at which the pipeline of the A^T B kernel ends, its sums are put aside, or the last trip is short; wide and
    narrow, one and several column groups per wavefront.  The error against 64 bits is what single precision gives: chains of at most 8
    trips, 3.5e-7 of the norm was measured up to 14 M rows."""
    g = G()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for K in (trips * 16, trips * 16 * cus + 5, trips * 64 * cus - 1):
        if K * (M + N) > 4e7:
            continue
        H, S = synth.normal_features(K, M, 128), synth.normal_features(K, N, 129)
        Y = torch.full((M, N), float("nan"), device="cuda")
        g.gcn_gemm(1, 0, dev(H), dev(S), Y)
        want = H.astype(np.float64).T @ S.astype(np.float64)
        assert np.linalg.norm(host(Y) - want) <= 5e-7 * np.linalg.norm(want), (K, M, N)


@pytest.mark.parametrize("n,C", [(1, 1), (3, 2), (70, 3), (255, 1), (257, 2), (5000, 2), (513, 3), (300, 4), (129, 5), (1000, 7), (300, 9), (257, 41), (64, 63), (65, 65), (100, 67), (33, 130), (40, 255), (20, 257)])
@pytest.mark.parametrize("pad,off", [(0, 0), (1, 0), (3, 2), (4, 4)])
def test_softmax_of_ragged_rows(n, C, pad, off):
    """Rows that are no multiple of a lane's 16 bytes, at any pitch and alignment: loss, gradient, nothing written beside the rows."""
    g = G()
    rs = np.random.default_rng(130)
    Z = synth.normal_features(n, C, 131) * 4
    y = rs.integers(0, C, n).astype(np.int32)
    y[1::3] = -1
    buf = torch.full((n * (C + pad) + off,), float("nan"), device="cuda")[off:].view(n, C + pad)
    buf[:, :C] = dev(Z)
    Gd = torch.full((n * (C + pad) + off,), float("nan"), device="cuda")[off:].view(n, C + pad)
    loss = torch.zeros(1, device="cuda")
    m = int((y >= 0).sum())
    g.gcn_softmax_nll_masked(buf[:, :C], dev(y), m, loss, Gd[:, :C])
    Zd = Z.astype(np.float64)
    p = np.exp(Zd - Zd.max(1, keepdims=True))
    p /= p.sum(1, keepdims=True)
    on = y >= 0
    want = np.where(on[:, None], (p - (np.arange(C) == y[:, None])) / m, 0)
    assert_close(host(Gd)[:, :C], want, f"G {n}x{C}")
    assert np.all(np.isnan(host(Gd)[:, C:]))
    nll = -np.log(p[on, y[on]]).mean()
    assert abs(loss.item() - nll) <= 1e-5 * max(1.0, abs(nll))


@pytest.mark.parametrize("f,kernel,chunks", [(f, kernel, least + more) for f, kernel, least in (
    (16, "k_spmm_split<4,4>", 769), (31, "k_spmm_split<32,1>", 769), (64, "k_spmm_split<16,4>", 769),
    (41, "k_spmm_line<1>", 1025), (67, "k_spmm_line<2>", 1025)) for more in (0, 3, 30, 31, 32, 62, 64)])
def test_column_blocks_walked_by_one_xcd_each(f, kernel, chunks):
    """Over column blocks an XCD takes one stretch of the chunks: numbers of chunks that leave the last stretch short, or the last
    workgroup without one, in both kernels that take so many chunks (fewer go to others, which do not deal them out)."""
    g = G()
    lengths = np.full(chunks, 512)
    lengths[::9] -= 40
    lengths[4::9] += 40
    lengths[-1] = chunks * 512 - int(lengths[:-1].sum()) - 3
    rowptr, colidx, val = _rows_matrix(lengths, 2500, 132)
    X = synth.uniform_features(2500, f, 133)
    a = g.gcn_csr_create_from_csr_rect(len(lengths), 2500, dev(rowptr), dev(colidx), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 2)
    assert f"chunks={chunks},kernel={kernel}" in g.gcn_spmm_describe(a, 0, f)
    Zd = torch.full((len(lengths), f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, dev(X), Zd)
    A = torch.sparse_csr_tensor(torch.from_numpy(rowptr), torch.from_numpy(colidx).long(), torch.from_numpy(val).double(), (len(lengths), 2500))
    assert_close(host(Zd), (A @ torch.from_numpy(X).double()).numpy(), f"{chunks} chunks f={f}")
    a.close()


@pytest.mark.parametrize("f", [2, 4, 16, 20, 64])
@pytest.mark.parametrize("blocks", [2, 4, 5, 9])
def test_partial_rows_are_added_in_the_order_of_the_blocks(f, blocks):
    """Rows of 0 to `blocks` partial rows, each the rounded product of one entry: the sums are those of adding one by one, bit for bit."""
    g = G()
    n, width = 700, 1024                                        # (columns of a block)
    rows = [[b * width + (i * 7 + b) % width for b in range(blocks) if (i + b) % 3 or i % (blocks + 1) == blocks][:i % (blocks + 1)] for i in range(n)]
    rowptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    col = np.concatenate([np.asarray(r, np.int32) for r in rows if r])
    val = synth.normal_features(len(col), 1, 71)[:, 0].copy()
    X = synth.uniform_features(blocks * width, f, 72)
    a = g.gcn_csr_create_from_csr_rect(n, blocks * width, dev(rowptr), dev(col), dev(val), 0)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, blocks)
    Z = torch.full((n, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, dev(X), Z)
    want = np.zeros((n, f), np.float32)
    for i in range(n):
        for k in range(rowptr[i], rowptr[i + 1]):
            want[i] = want[i] + val[k] * X[col[k]]
    np.testing.assert_array_equal(host(Z), want)
    a.close()


@pytest.mark.parametrize("strips", [1, 3, 4, 5, 16, 17, 252, 256, 257, 1008, 1024, 2052, 8192, 8199, 32_768, 33_001])
@pytest.mark.parametrize("C", [3, 16, 41, 130])
def test_last_layer_sums_of_workgroups(strips, C):
    """The fused last layer's weight gradient and loss from 1 to 2048 workgroups' partial results: fewer than the 64 groups of threads that
    add them, a multiple of eight times as many, and others; the last strip is short."""
    g = G()
    n = strips * 16 - 5
    rs = np.random.default_rng(134)
    P0, W = synth.normal_features(n, 16, 135), synth.normal_features(16, C, 136) * np.float32(0.3)
    y = rs.integers(0, C, n).astype(np.int32)
    y[2::5] = -1
    a = g.gcn_csr_create(n, dev(np.zeros(1, np.int32)), dev(np.zeros(1, np.int32)), g.ADD_SELF_LOOPS | g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE)
    Y, loss = torch.full((16, C), float("nan"), device="cuda"), torch.zeros(1, device="cuda")
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, [16, C]), dtype=torch.uint8, device="cuda")
    m = int((y >= 0).sum())
    g.gcn_epoch_preaggregated(a, [16, C], dev(P0), dev(y), m, [dev(W)], [Y], 0.0, loss, ws)
    Z = P0.astype(np.float64) @ W
    lse = np.log(np.exp(Z - Z.max(1, keepdims=True)).sum(1)) + Z.max(1)
    Gd = np.where((y >= 0)[:, None], (np.exp(Z - lse[:, None]) - (np.arange(C) == y[:, None])) / m, 0)
    assert_close(host(Y), P0.T.astype(np.float64) @ Gd, f"Y {strips} {C}")
    nll = (lse - Z[np.arange(n), np.maximum(y, 0)])[y >= 0].mean()
    assert abs(loss.item() - nll) <= 1e-5 * max(1.0, abs(nll))
    a.close()


@pytest.mark.parametrize("C", [3, 16, 41, 64, 130])
@pytest.mark.parametrize("labelled", [True, False])
def test_last_layer_with_logits_at_the_ends_of_the_range(C, labelled):
    """A logit of minus infinity counts for nothing; a NaN in a labelled row reaches the loss and all of Y, as the separate kernels do it."""
    g = G()
    n = 100
    P0, W = synth.normal_features(n, 16, 151), synth.normal_features(16, C, 152) * np.float32(0.3)
    P0[:, 15], W[15] = 0, 0
    P0[7, :], P0[7, 15], W[15, 0] = 0, 1e30, -1e30                     # logits of row 7: -inf, 0, 0, ...
    y = np.full(n, 1, np.int32)
    y[50] = 1 if labelled else -1
    a = g.gcn_csr_create(n, dev(np.zeros(1, np.int32)), dev(np.zeros(1, np.int32)), g.ADD_SELF_LOOPS | g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE)
    m = int((y >= 0).sum())
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, [16, C]), dtype=torch.uint8, device="cuda")

    def run(P):
        Y, loss = torch.full((16, C), float("nan"), device="cuda"), torch.zeros(1, device="cuda")
        g.gcn_epoch_preaggregated(a, [16, C], dev(P), dev(y), m, [dev(W)], [Y], 0.0, loss, ws)
        return host(Y), loss.item()
    Y, loss = run(P0)
    Z = P0.astype(np.float64) @ W
    Z[7, 0] = -np.inf
    lse = np.log(np.exp(Z - Z.max(1, keepdims=True)).sum(1)) + Z.max(1)
    Gd = np.where((y >= 0)[:, None], (np.exp(Z - lse[:, None]) - (np.arange(C) == y[:, None])) / m, 0)
    assert_close(Y, P0.T.astype(np.float64) @ Gd, f"Y {C}")
    assert abs(loss - (lse - Z[:, 1])[y >= 0].mean()) <= 1e-5 * abs(loss)
    P0[50, 3] = np.nan
    Y, loss = run(P0)
    assert np.isnan(loss) == labelled and (np.isnan(Y).all() or not labelled)
    a.close()


@pytest.mark.parametrize("tied", [[], [(1, 2)], [(0, 1), (1, 2), (16, 17)], [(3, 18)]])
def test_update_of_many_and_of_tied_layers(tied):
    """All layers' W are updated side by side, more of them than a launch takes, and one after another where they share a matrix."""
    g = G()
    rs = np.random.default_rng(137)
    n, L = 200, 20
    dims = [6] * (L + 1)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, 800).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE)
    W = [dev(np.eye(6, dtype=np.float32) + synth.normal_features(6, 6, 138 + l) * np.float32(0.1)) for l in range(L)]
    for l, k in tied:
        W[k] = W[l]
    Y = [torch.empty(6, 6, device="cuda") for _ in range(L)]
    H0, y, loss = dev(np.abs(synth.normal_features(n, 6, 139))), dev(rs.integers(0, 6, n).astype(np.int32)), torch.zeros(1, device="cuda")
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, dims), dtype=torch.uint8, device="cuda")
    g.gcn_epoch(a, dims, H0, y, W, Y, 0.0, loss, ws)
    want, gradients = {w.data_ptr(): host(w).copy() for w in W}, [host(v).copy() for v in Y]
    for w, v in zip(W, gradients):
        want[w.data_ptr()] -= np.float32(0.5) * v
    g.gcn_epoch(a, dims, H0, y, W, Y, 0.5, loss, ws)
    for w, v, k in zip(W, gradients, range(L)):
        assert np.array_equal(host(Y[k]), v) and np.abs(v).max() > 0, k
        assert np.allclose(host(w), want[w.data_ptr()], rtol=3e-7, atol=1e-9), k       # a rounding of the product may be fused away
    a.close()


@pytest.mark.parametrize("longest", [1, 4, 5, 8, 9, 16, 33, 63, 64])
@pytest.mark.parametrize("f", [4, 7, 16, 20, 32, 41, 64])
def test_spmm_short_rows_at_equal_pitch(longest, f):
    """Rows of up to `longest` entries at a pitch of whole fours: rounds of eight that end inside and behind a row, rows without entries, a
    first row of the operand that no entry names and that is not finite (what lies behind a row's last entry points there), epilogues, the
    transpose, the value-free form; an odd number of rows."""
    g = G()
    rs = np.random.default_rng(151)
    n, nc = 1403, 977
    lengths = rs.integers(0, longest + 1, n)
    lengths[5] = longest
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rs.choice(nc - 1, k, replace=False)) + 1 for k in lengths]).astype(np.int32)
    val = rs.standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), g.BUILD_TRANSPOSE)
    assert "k_spmm_short" in g.gcn_spmm_describe(a, 0, f)
    X = synth.normal_features(nc, f, 152)
    A = np.zeros((n, nc))
    A[np.repeat(np.arange(n), lengths), colidx] = val
    want, Zp = A @ X.astype(np.float64), synth.normal_features(n, f, 153)
    X[0] = np.where(np.arange(f) % 2, np.inf, np.nan)
    Z = torch.full((n, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, dev(X), Z)
    plain = host(Z).copy()
    assert_close(plain, want, f"{longest} {f}")
    g.gcn_spmm(a, 0, dev(X), Z, g.EPI_MASK, dev(Zp))
    assert np.array_equal(host(Z), np.where(Zp > 0, plain, 0))
    scale = rs.random(n).astype(np.float32) + 0.5
    g.gcn_spmm_pattern(a, 0, dev(X), Z, dev(scale))
    assert_close(host(Z), scale[:, None] * ((A != 0) @ np.where(np.arange(nc)[:, None] == 0, 0, X).astype(np.float64)), f"value-free {longest} {f}")
    Xt = synth.normal_features(n, f, 154)
    Zt = torch.full((nc, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 1, dev(Xt), Zt)
    assert_close(host(Zt), A.T @ Xt.astype(np.float64), f"transposed {longest} {f}")
    a.close()


@pytest.mark.parametrize("rows,power,kernel", [(60_001, 4, "k_spmm_split<8,1>"), (44_001, 4, "k_spmm_short<2>"), (60_001, 80, "k_spmm_short<2>")])
@pytest.mark.parametrize("f", [5, 7])
def test_short_rows_on_both_sides_of_the_padded_copy(rows, power, kernel, f):
    """Rows of 0 to 64 entries, most of them short: many whose padded copy would be mostly padding, fewer, and many of which hardly any are long;
    epilogues and the transpose, whose rows are another distribution."""
    g = G()
    rs = np.random.default_rng(158)
    lengths = (rs.random(rows) ** power * 64.99).astype(np.int64)
    lengths[11] = 64
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    colidx = (np.repeat(rs.integers(0, rows - 65 * 7, rows), lengths) + 7 * (np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], lengths))).astype(np.int32)
    val = rs.standard_normal(colidx.size).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(rows, rows, dev(rowptr), dev(colidx), dev(val), g.BUILD_TRANSPOSE)
    assert kernel in g.gcn_spmm_describe(a, 0, f)
    X, M = synth.normal_features(rows, f, 159), synth.normal_features(rows, f, 160)
    A = torch.sparse_coo_tensor(torch.from_numpy(np.stack([np.repeat(np.arange(rows), lengths), colidx.astype(np.int64)])),
                                torch.from_numpy(val).double(), (rows, rows)).coalesce()
    Z = torch.full((rows, f), float("nan"), device="cuda")
    g.gcn_spmm(a, 0, dev(X), Z)
    plain = host(Z).copy()
    assert_close(plain, torch.sparse.mm(A, torch.from_numpy(X).double()).numpy(), f"{rows} {f}")
    for epi, want in ((g.EPI_RELU, np.maximum(plain, 0)), (g.EPI_MASK, np.where(M > 0, plain, 0))):
        g.gcn_spmm(a, 0, dev(X), Z, epi, dev(M))
        assert np.array_equal(host(Z), want), epi
    g.gcn_spmm(a, 1, dev(X), Z)
    assert_close(host(Z), torch.sparse.mm(A.t(), torch.from_numpy(X).double()).numpy(), f"transposed {rows} {f}")
    a.close()


@pytest.mark.parametrize("K,N,M", [(100, 16, 65_536), (300, 16, 195_740), (300, 16, 195_735), (64, 32, 917_504), (128, 32, 40_000), (64, 16, 32_768), (16, 8, 32_784),
                                   (64, 16, 14_336), (256, 64, 14_336), (500, 24, 8192), (602, 64, 5000)])
def test_gemm_nn_on_both_sides_of_its_rules(K, N, M):
    """Row counts at which the product goes to another kernel or to workgroups of another size: the first rows keep their bits, the last ones are
    what 64 bits give."""
    g = G()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(155)
    A, B = torch.randn(M + 17, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    few = torch.empty(4000, N, device="cuda")
    g.gcn_gemm(0, 0, A[:4000], B, few)
    assert_close(host(few), host(A[:4000].double() @ B.double()), f"{K} {N}")
    for rows in (M - 1, M, M + 17):
        C = torch.full((rows, N), float("nan"), device="cuda")
        g.gcn_gemm(0, 0, A[:rows], B, C)
        assert torch.equal(C[:4000], few), rows
        assert_close(host(C[-200:]), host(A[rows - 200:rows].double() @ B.double()), f"{rows} {K} {N}")


@pytest.mark.parametrize("n,dims", [(70_001, (7, 3, 3, 3)), (500, (64, 16, 16, 16)), (5000, (100, 16, 16, 41)), (500, (5, 130, 130, 300)),
                                    (300, (12,) * 7 + (9,)), (300, (12,) * 8 + (9,))])
def test_reductions_at_the_end_of_the_epoch(n, dims):
    """Gradients, loss and update that an epoch adds up in one kernel: the bits of the reductions one by one, which an epoch whose second and
    third layer share their weights runs; with partial results folded first, both products of width 16 in one pass, the fused last layer, many
    classes, as many layers as the kernel takes and one more."""
    g = G()
    rs = np.random.default_rng(141)
    L = len(dims) - 1
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, 4 * n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE)
    H0, y = dev(synth.normal_features(n, dims[0], 142)), dev(rs.integers(-1, dims[-1], n).astype(np.int32))
    W = [dev(w) for w in synth.glorot_weights(dims, 143)]
    tied = dims[1] == dims[2] == dims[3]
    if tied:
        W[2].copy_(W[1])
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, dims), dtype=torch.uint8, device="cuda")
    got = []
    for share in (False, True):
        Ws = list(W)
        if share and tied:
            Ws[2] = Ws[1]
        elif share:                                                # the last layer's gradient beside the first one's weights, one float shared
            both = torch.empty(W[0].numel() + W[-1].numel() - 1, device="cuda")
            both[:W[0].numel()] = W[0].reshape(-1)
            Ws[0] = both[:W[0].numel()].view_as(W[0])
        Y = [torch.full_like(w, float("nan")) for w in Ws]
        if share and not tied:
            Y[-1] = both[W[0].numel() - 1:].view_as(W[-1])
        loss = torch.full((1,), float("nan"), device="cuda")
        ws.fill_(255)
        g.gcn_epoch_masked(a, dims, H0, y, int((y >= 0).sum()), Ws, Y, 0.0, loss, ws)
        got.append([host(loss)] + [host(v).copy() for v in Y])
        if not share:
            before = [host(w).copy() for w in Ws]
            ws.fill_(255)
            g.gcn_epoch_masked(a, dims, H0, y, int((y >= 0).sum()), Ws, Y, 0.5, loss, ws)
            for w, b, v in zip(Ws, before, got[0][1:]):
                assert np.allclose(host(w), b - np.float32(0.5) * v, rtol=3e-7, atol=1e-9)
                w.copy_(dev(b))
    for l in range(L + 1):
        if tied or l not in (1, L):                                # (without tied layers the shared float changes W[0] under way)
            assert np.isfinite(got[0][l]).all() and np.array_equal(got[0][l], got[1][l]), l
    a.close()


@pytest.mark.parametrize("value_free", [0, 1])
@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("n,classes", [(70, 16), (3000, 16), (3000, 8), (3000, 40)])
def test_partial_results_in_idle_memory(n, classes, given, value_free):
    """The partial results that an epoch adds up at its end lie where the scaled operand would, or the first layer's T, by whether the products are
    value-free and whether A^T H0 is given: the bits of the epoch whose tied weights make it add them one by one."""
    g = G()
    rs = np.random.default_rng(161)
    dims = (40, 16, 16, classes)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, 4 * n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE)
    g.gcn_csr_config(a, g.CFG_PATTERN_SPMM, value_free)
    H0, y = dev(synth.normal_features(n, dims[0], 162)), dev(rs.integers(-1, classes, n).astype(np.int32))
    W = [dev(w) for w in synth.glorot_weights(dims, 163)]
    run = g.gcn_epoch_preaggregated if given else g.gcn_epoch_masked
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, dims), dtype=torch.uint8, device="cuda")
    got = []
    for shared in (False, True):
        both = torch.empty(W[0].numel() + W[1].numel() - 1, device="cuda")
        Y = [both[:W[0].numel()].view_as(W[0]) if shared else torch.empty_like(W[0]), torch.empty_like(W[1]), torch.empty_like(W[2])]
        if shared:                                                  # one float of the first two gradients; the first is written last
            Y[1] = both[W[0].numel() - 1:].view_as(W[1])
        loss = torch.full((1,), float("nan"), device="cuda")
        ws.fill_(255)
        run(a, dims, H0, y, int((y >= 0).sum()), W, Y, 0.0, loss, ws)
        got.append([host(loss), host(Y[0]), host(Y[1]).reshape(-1)[1:], host(Y[2])])
    for k, (p, q) in enumerate(zip(*got)):
        assert np.isfinite(p).all(), k
        # (losses are added up in double by other groups of rows where a product makes them: the last bit of the float may differ)
        assert np.array_equal(p, q) if k else abs(p - q) <= 2.0 ** -23 * abs(q), k
    a.close()


@pytest.mark.parametrize("n,dims,rows", [
    (63, (20, 16, 8), "short"), (64, (20, 16, 8), "short"), (65, (64, 16, 8), "short"), (4097, (64, 16, 16, 12), "short"), (1000, (8, 8, 4), "short"),
    (333, (33, 12, 12, 16), "short"), (1000, (16, 4, 12, 4), "short"), (1000, (64, 16, 7), "short"), (1000, (64, 32, 16, 8), "short"),
    (32_768, (16, 8, 4), "short"), (1000, (40, 16, 20), "short"), (1000, (64, 16, 8), "long"), (300, (20, 16, 8), "empty")])
def test_epoch_on_short_rows_is_the_calls_one_by_one(n, dims, rows):
    """The dense product in front of the next sparse one, its masked counterpart in the backward pass and the loss where the kernel of few and
    short rows makes the rows: the bits of the layer and loss calls, whose kernels run one by one.  One row more or less than
    the dense kernel takes, the last 16 rows not whole, widths of 4 to 16, as many rows as the kernel is taken for; widths and rows beside its range."""
    g = G()
    rs = np.random.default_rng(151)
    u, v = rs.integers(0, n, (2, 3 * n)).astype(np.int32)
    flags = g.NORM_SYM | g.SYMMETRISE | g.BUILD_TRANSPOSE
    if rows == "long":
        u[:200] = 0
    if rows == "empty":
        u, v = u // 2, v // 2                                      # the upper half of the rows has no entries
    else:
        flags |= g.ADD_SELF_LOOPS
    a = g.gcn_csr_create(n, dev(u), dev(v), flags)
    assert ("k_spmm_short" in g.gcn_spmm_describe(a, 0, dims[1])) == (rows != "long")
    H0, y = dev(synth.normal_features(n, dims[0], 152)), dev(rs.integers(-1, dims[-1] + 1, n).astype(np.int32))      # (a label too large counts as the last class)
    count, L = int((y >= 0).sum()), len(dims) - 1
    W = [dev(w) for w in synth.glorot_weights(dims, 153)]
    Y = [torch.full_like(w, float("nan")) for w in W]
    loss = torch.full((1,), float("nan"), device="cuda")
    ws = torch.empty(g.gcn_epoch_workspace_bytes(n, dims), dtype=torch.uint8, device="cuda")
    g.gcn_csr_config(a, g.CFG_FUSED_LAST_LAYER, 0)
    empty = lambda k: torch.full((n, k), float("nan"), device="cuda")
    Z, T, Gr = ([empty(d) for d in dims[1:]] for _ in range(3))
    T = [empty(min(p, q)) for p, q in zip(dims, dims[1:])]
    x = H0
    for l in range(L):
        g.gcn_layer_forward(a, x, W[l], Z[l], Z[l] if l < L - 1 else None, T[l], act=g.ACT_RELU if l < L - 1 else g.ACT_NONE)
        x = Z[l]
    want_loss = torch.zeros(1, device="cuda")
    g.gcn_softmax_nll_masked(Z[-1], y, count, want_loss, Gr[-1])
    want_Y = [torch.empty_like(w) for w in W]
    for l in range(L - 1, -1, -1):
        g.gcn_layer_backward(a, Z[l - 1] if l else H0, Z[l - 1] if l else None, W[l], Gr[l], T[l], empty(T[l].shape[1]), want_Y[l], Gr[l - 1] if l else None)
    for rep in range(2):
        ws.fill_(255)
        g.gcn_epoch_masked(a, dims, H0, y, count, W, Y, 0.0, loss, ws)
        for l in range(L):
            got_Z, got_G = g.gcn_epoch_view(n, dims, g.ORDER_AUTO, ws, l + 1)
            assert torch.equal(got_Z, Z[l]) and torch.equal(got_G, Gr[l]) and torch.equal(Y[l], want_Y[l]), (rep, l)
        # losses are added up in double, here by rows of 16, there by workgroups: the last bit of the float may differ
        assert abs(float(loss) - float(want_loss)) <= 2.0 ** -23 * abs(float(want_loss))
    a.close()


@pytest.mark.parametrize("n", [64, 65, 127, 129, 1023, 32_768])
@pytest.mark.parametrize("dims", [(1, 16, 4), (15, 4, 4), (16, 16, 16), (17, 12, 8), (63, 16, 16, 12), (64, 8, 8, 4), (65, 16, 4)])
def test_gradients_beside_short_rows(n, dims):
    """Weight gradients made by the kernel of short rows, on both sides of its range (64 columns of H, 16 of Z), the last 64 rows not whole: as
    close to 64 bits as single launches, and their bits; nothing is written behind the workspace."""
    g = G()
    rs = np.random.default_rng(171)
    u, v = rs.integers(0, n, (2, 2 * n)).astype(np.int32)
    a = g.gcn_csr_create(n, dev(u), dev(v), g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    assert "k_spmm_short" in g.gcn_spmm_describe(a, 0, dims[1])
    H0, y = dev(synth.normal_features(n, dims[0], 172)), dev(rs.integers(0, dims[-1], n).astype(np.int32))
    W, L = [dev(w) for w in synth.glorot_weights(dims, 173)], len(dims) - 1
    Y, loss = [torch.full_like(w, float("nan")) for w in W], torch.zeros(1, device="cuda")
    size = g.gcn_epoch_workspace_bytes(n, dims)
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device="cuda")
    g.gcn_epoch(a, dims, H0, y, W, Y, 0.0, loss, ws[:size])
    assert bool((ws[size:] == 255).all())
    rowptr, col, val, _ = a.arrays()
    A = torch.sparse_csr_tensor(rowptr, col.long(), val.double(), (n, n))
    for l in range(L - 1, -1, -1):
        Gl = g.gcn_epoch_view(n, dims, g.ORDER_AUTO, ws[:size], l + 1)[1]
        Hin = g.gcn_epoch_view(n, dims, g.ORDER_AUTO, ws[:size], l)[0] if l else H0
        if dims[l + 1] > dims[l]:
            continue                                                # (A^T H first: another kernel's gradient)
        assert_close(host(Y[l]), host(Hin.double().T @ (A @ Gl.double())), f"{n} {dims} layer {l + 1}")
        S, want = torch.empty(n, dims[l + 1], device="cuda"), torch.empty_like(W[l])
        g.gcn_layer_backward(a, Hin, None, W[l], Gl, None, S, want, None)
        assert torch.equal(Y[l], want), (n, dims, l)
    a.close()


# dense products among an epoch's launches, forward and backward, counted by hand; others: an (empty) span of each layer that goes forward, and the sums with the update
@pytest.mark.parametrize("dims,n,gemm,other", [((64, 16, 8), n, 1, 3) for n in (64, 65, 127, 128, 129, 1000, 1023, 4095, 4096, 4097, 10_001, 16_383, 16_384)] +
                         [((64, 16, 8), 16_385, 2, 3), ((65, 16, 8), 4096, 2, 3), ((64, 16, 8), 63, 6, 3), ((32, 16, 8), 32_768, 1, 3), ((33, 16, 16, 12), 5000, 1, 4),
                          ((16, 8), 200, 1, 2), ((63, 16), 4097, 1, 2), ((64, 16, 41), 4097, 2, 2), ((16, 64, 8), 4096, 4, 3), ((8, 64, 4), 1024, 4, 3)])
def test_launches_of_an_epoch_on_short_rows(dims, n, gemm, other):
    """Weight gradients of up to 64 columns beside the rows at any number of them, the loss beside the rows, and all sums and the update in one launch, also where a layer
    widens; the bits of the layer calls."""
    g = G()
    rs = np.random.default_rng(176)
    u, v = rs.integers(0, n, (2, 2 * n)).astype(np.int32)
    a = g.gcn_csr_create(n, dev(u), dev(v), g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    assert all("k_spmm_short" in g.gcn_spmm_describe(a, 0, min(p, q)) for p, q in zip(dims, dims[1:]))
    H0, y = dev(synth.normal_features(n, dims[0], 177)), dev(rs.integers(0, dims[-1], n).astype(np.int32))
    W, L = [dev(w) for w in synth.glorot_weights(dims, 178)], len(dims) - 1
    first = [w.clone() for w in W]
    Y, loss = [torch.full_like(w, float("nan")) for w in W], torch.zeros(1, device="cuda")
    size = g.gcn_epoch_workspace_bytes(n, dims)
    ws = torch.full((size + 4096,), 255, dtype=torch.uint8, device="cuda")
    g.gcn_epoch_prepare(a, dims)
    g.gcn_config(g.CFG_TIMING, 1)
    try:
        g.gcn_timing_read_phases()
        g.gcn_epoch(a, dims, H0, y, W, Y, 0.5, loss, ws[:size])
        spans = g.gcn_timing_read_phases()
    finally:
        g.gcn_config(g.CFG_TIMING, 0)
    assert (spans["gemm"][0], spans["other"][0]) == (gemm, other), spans
    assert bool((ws[size:] == 255).all())
    assert all(torch.equal(w, w0 - 0.5 * y1) for w, w0, y1 in zip(W, first, Y))
    for l in range(L - 1, -1, -1):
        if dims[l + 1] > dims[l]:
            continue                                                # (A^T H first: its T is the epoch's own)
        Gl = g.gcn_epoch_view(n, dims, g.ORDER_AUTO, ws[:size], l + 1)[1]
        Hin = g.gcn_epoch_view(n, dims, g.ORDER_AUTO, ws[:size], l)[0] if l else H0
        S, want = torch.empty(n, dims[l + 1], device="cuda"), torch.empty_like(W[l])
        g.gcn_layer_backward(a, Hin, None, first[l], Gl, None, S, want, None)
        assert torch.equal(Y[l], want), l
    a.close()


@pytest.mark.parametrize("f", [4, 7, 16, 20, 32, 41, 48, 64, 130])
@pytest.mark.parametrize("pairs,loops,blocks", [(500, True, 0), (400_000, True, 1), (400_000, True, 3), (400_000, False, 1), (400_000, False, 3)])
@pytest.mark.parametrize("values", [0, 1])
def test_layer_end_in_the_product(f, pairs, loops, blocks, values):
    """Bias and activation where the product stores its rows, or in a pass behind it (few chunks, ragged widths, rows without
    entries): the same bits as the product, plus the bias, clamped; H beside Z, in place, over T; nothing but H and Z is written."""
    g = G()
    rs = np.random.default_rng(140)
    n = 3001
    src, dst = [np.concatenate([rs.integers(0, n - 5, pairs), np.full(1500, 7)]).astype(np.int32) for _ in range(2)]
    dst[-1500:] = rs.integers(0, n - 5, 1500)                       # a row over several chunks
    a = g.gcn_csr_create(n, dev(src), dev(dst), (g.ADD_SELF_LOOPS if loops else 0) | g.SYMMETRISE | g.NORM_SYM | g.BUILD_TRANSPOSE)
    g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, blocks)
    g.gcn_csr_config(a, g.CFG_PATTERN_SPMM, values)
    X, W, b = dev(synth.normal_features(n, 24, 141)), dev(synth.normal_features(24, f, 142)), dev(synth.normal_features(1, f, 143)[0])
    T, Z, want = [torch.full((n, f), float("nan"), device="cuda") for _ in range(3)]
    room = torch.full((n + 2, f), float("nan"), device="cuda")
    for bias in (b, None):
        H = room[1:-1].fill_(float("nan"))
        g.gcn_layer_forward(a, X, W, Z, H, T, g.ORDER_GEMM_FIRST, g.ACT_RELU, bias=bias)
        g.gcn_gemm(0, 0, X, W, T)
        xs = T
        g.gcn_csr_config(a, g.CFG_PATTERN_SPMM, 0)                  # the layer calls have no room for a scaled operand
        g.gcn_spmm(a, 1, xs, want)
        g.gcn_csr_config(a, g.CFG_PATTERN_SPMM, values)
        if bias is not None:
            want += bias
        assert torch.equal(Z, want) and torch.equal(H, want.clamp(min=0)), bias is None
        assert bool(torch.isnan(room[0]).all() and torch.isnan(room[-1]).all())
        g.gcn_layer_forward(a, X, W, Z, T, T, g.ORDER_GEMM_FIRST, g.ACT_RELU, bias=bias)           # H over T
        assert torch.equal(Z, want) and torch.equal(T, want.clamp(min=0))
        g.gcn_layer_forward(a, X, W, Z, Z, T, g.ORDER_GEMM_FIRST, g.ACT_RELU, bias=bias)           # in place
        assert torch.equal(Z, want.clamp(min=0))
        for Ho in (None, H):                                                                       # without an activation
            g.gcn_layer_forward(a, X, W, Z, Ho, T, g.ORDER_GEMM_FIRST, g.ACT_NONE, bias=bias)
            assert_close(host(Z), host(want).astype(np.float64), "no activation")
            assert Ho is None or torch.equal(H, Z)
    a.close()


@pytest.mark.parametrize("n", [63, 64, 65, 79, 128, 129, 1000, 8192, 70_001])
@pytest.mark.parametrize("pad,own", [(0, True), (0, False), (4, False), (1, False)])
def test_backward_products_of_width_16(n, pad, own):
    """Y = H^T S and Gprev = (S W^T) masked, in one pass where rows are aligned (not: pitch 17, below 64 rows): last trips of every
    length, the mask from H itself and from a matrix of its own, Gprev over H and over S."""
    g = G()
    rs = np.random.default_rng(144)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, 3 * n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [synth.normal_features(k, 16, 145 + i) for i, k in enumerate((n, n, 16, n))]
    Hd = torch.full((n, 16 + pad), float("nan"), device="cuda")
    Hd[:, :16] = dev(H)
    Hd, Wd = Hd[:, :16], dev(W)
    Zd = Hd if own else dev(Zp)
    S, Y = torch.empty(n, 16, device="cuda"), torch.full((16, 16), float("nan"), device="cuda")
    Gp = torch.full((n + 2, 16), float("nan"), device="cuda")
    g.gcn_layer_backward(a, Hd, Zd, Wd, dev(Gm), None, S, Y, Gp[1:-1], g.ORDER_GEMM_FIRST)
    Sx = host(S).astype(np.float64)
    wantY, wantG = H.T.astype(np.float64) @ Sx, np.where((H if own else Zp) > 0, Sx @ W.T, 0)
    assert np.linalg.norm(host(Y) - wantY) <= 5e-7 * np.linalg.norm(wantY)
    assert_close(host(Gp)[1:-1], wantG, f"{n} {pad}")
    assert bool(torch.isnan(Gp[0]).all() and torch.isnan(Gp[-1]).all())
    plain = torch.empty(n, 16, device="cuda")
    g.gcn_gemm(0, 1, S, Wd, plain, epilogue=g.EPI_MASK, Zprev=Zd)
    assert torch.equal(Gp[1:-1], plain)
    first = Y.clone()
    for over in ([S] if pad else [S, Hd]):
        g.gcn_layer_backward(a, Hd, Zd, Wd, dev(Gm), None, S, Y, over, g.ORDER_GEMM_FIRST)
        assert torch.equal(over, plain) and torch.equal(Y, first)
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("M,K", [(195_768, 300), (200_003, 300), (277_000, 212), (262_161, 228), (400_001, 148), (459_000, 128)])
@pytest.mark.parametrize("N", [4, 12, 16])
def test_dense_products_beyond_the_caches(M, K, N):
    """Strips through LDS, whose results leave in bursts: the last burst of every wavefront not whole, the last strip not either, columns behind the
    last one; all epilogues, and the rows around C untouched."""
    g = G()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(321)
    A, B, bias, Zp = [torch.randn(r, c, generator=gen, device="cuda") for r, c in ((M, K), (K, N), (1, N), (M, N))]
    plain = A.double() @ B.double() + bias.double()
    bound = (K + 2) * 2.0 ** -24 * (A.abs().double() @ B.abs().double() + bias.abs().double())
    for epilogue, want in ((g.EPI_NONE, plain), (g.EPI_RELU, plain.clamp(min=0)), (g.EPI_MASK, torch.where(Zp > 0, plain, 0.0))):
        C = torch.full((M + 2, N), float("nan"), device="cuda")
        g.gcn_gemm(0, 0, A, B, C[1:-1], bias=bias.view(-1), epilogue=epilogue, Zprev=Zp if epilogue == g.EPI_MASK else None)
        assert bool(((C[1:-1].double() - want).abs() <= bound).all()), epilogue
        assert bool(torch.isnan(C[0]).all() and torch.isnan(C[-1]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 63, 1000, 33_000])
@pytest.mark.parametrize("f_in,f_out", [(1, 1), (16, 16), (64, 41), (300, 16), (20, 70), (16, 200)])
def test_bias_gradient_beside_the_weight_gradient(n, f_in, f_out):
    """With a bias gradient the sums of both are one launch: the same bits of Y and Gprev as without, with and without Gprev, twice in a row, and the
    column sums of G; a weight gradient in place of the weights comes before Gprev as it does without."""
    g = G()
    rs = np.random.default_rng(311)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [dev(synth.normal_features(r, c, 312 + i)) for i, (r, c) in enumerate(((n, f_in), (n, f_in), (f_in, f_out), (n, f_out)))]
    w = min(f_in, f_out)
    T, S, empty = dev(synth.normal_features(n, w, 316)), torch.empty(n, w, device="cuda"), lambda r, c: torch.full((r, c), float("nan"), device="cuda")
    for Gp in (empty(n, f_in), None):
        Y, want, db = empty(f_in, f_out), empty(f_in, f_out), empty(1, f_out).view(-1)
        g.gcn_layer_backward(a, H, Zp, W, Gm, T, S, want, Gp)
        want_G = None if Gp is None else Gp.clone()
        for _ in range(2):
            g.gcn_layer_backward(a, H, Zp, W, Gm, T, S, Y, Gp, dbias=db)
            assert torch.equal(Y, want) and (Gp is None or torch.equal(Gp, want_G))
            bound = 16 * 2.0 ** -24 * host(Gm.double().abs().sum(0))                # chains of a few hundred rows, and their sums
            assert np.all(np.abs(host(db) - host(Gm.double().sum(0))) <= bound)
    W1, W2, G1, G2 = W.clone(), W.clone(), empty(n, f_in), empty(n, f_in)
    g.gcn_layer_backward(a, H, Zp, W1, Gm, T, S, W1, G1)
    g.gcn_layer_backward(a, H, Zp, W2, Gm, T, S, W2, G2, dbias=db)
    assert torch.equal(W1, W2) and torch.equal(G1, G2)
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("C", [1, 2, 3, 4, 7, 16, 41, 130, 256, 300])
def test_loss_of_rows_with_infinities(C):
    """Logits of minus infinity are classes that have no share; a NaN or an infinity makes its own row NaN and no other; a row outside the split counts for
    nothing whatever it holds."""
    g = G()
    n = 777
    Z, labels = synth.normal_features(n, C, 391), np.zeros(n, np.int32)
    rs = np.random.default_rng(392)
    if C > 1:
        Z[:400][rs.random((400, C)) < 0.5] = -np.inf
        Z[np.arange(400), rs.integers(0, C, 400)] = 0.5
        labels[:400] = Z[:400].argmax(1)
        labels[400:] = rs.integers(0, C, n - 400)
    odd = {700: np.nan, 701: np.inf, 702: -np.inf, 703: np.nan}
    for row, value in odd.items():
        Z[row, (0 if row < 702 else slice(None))] = value
    for inside in (False, True):
        labels[700:704] = 0 if inside else -1
        keep = labels >= 0
        Gd, loss = torch.full((n, C), 7.0, device="cuda"), torch.zeros(1, device="cuda")
        g.gcn_softmax_nll_masked(dev(Z), dev(labels), int(keep.sum()), loss, Gd)
        got = host(Gd)
        with np.errstate(invalid="ignore"):
            z = Z.astype(np.float64)
            p = np.exp(z - z.max(1, keepdims=True))
            s = p.sum(1, keepdims=True)
            want = (p / s - np.eye(C)[np.maximum(labels, 0)]) / keep.sum()
            nll = np.log(s[:, 0]) - (z - z.max(1, keepdims=True))[np.arange(n), np.maximum(labels, 0)]
        want[~keep] = 0
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        finite = ~np.isnan(want)
        # a share has a relative error of a few roundings of the exponential, of the sum and of the division
        assert np.all(np.abs(got[finite] - want[finite]) <= (20 + C) * 2.0 ** -24 / keep.sum())
        if inside:
            assert np.isnan(float(loss))
        else:
            assert abs(float(loss) - nll[keep].mean()) <= 1e-6 * max(1.0, abs(nll[keep].mean()))


@pytest.mark.gpu
@pytest.mark.parametrize("dims", [((64, 41), (64, 41)), ((16, 16), (100, 70)), ((300, 16), (8, 200))])
def test_layer_calls_of_two_threads_on_one_stream(dims):
    """Two threads, a matrix each, one stream: no call's partial results lie where another call's do."""
    import threading
    g = G()
    stream = torch.cuda.Stream()
    work = []
    for i, (f_in, f_out) in enumerate(dims):
        n = 3000 + 7 * i
        rs = np.random.default_rng(361 + i)
        a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
        H, Zp, W, Gm = [dev(synth.normal_features(r, c, 362 + 10 * i + k)) for k, (r, c) in enumerate(((n, f_in), (n, f_in), (f_in, f_out), (n, f_out)))]
        w = min(f_in, f_out)
        T, S, Gp = dev(synth.normal_features(n, w, 366 + 10 * i)), torch.empty(n, w, device="cuda"), torch.empty(n, f_in, device="cuda")
        g.gcn_spmm_prepare(a, 0, w)
        call = lambda Y, db, a=a, H=H, Zp=Zp, W=W, Gm=Gm, T=T, S=S, Gp=Gp: g.gcn_layer_backward(a, H, Zp, W, Gm, T, S, Y, Gp, dbias=db)
        outs = [(torch.empty_like(W), torch.empty(f_out, device="cuda")) for _ in range(100)]
        want = torch.empty_like(W), torch.empty(f_out, device="cuda")
        call(*want)
        work.append((a, call, outs, want))
    torch.cuda.synchronize()
    errors = []

    def run(call, outs):
        try:
            with torch.cuda.stream(stream):
                for Y, db in outs:
                    call(Y, db)
        except Exception as e:                                          # (reported by the test's own thread)
            errors.append(e)
    threads = [threading.Thread(target=run, args=(call, outs)) for _, call, outs, _ in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for a, _, outs, want in work:
        assert all(torch.equal(Y, want[0]) and torch.equal(db, want[1]) for Y, db in outs)
        a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("f_in,f_out", [(64, 16), (64, 41), (300, 300)])
def test_layer_backward_with_a_bias_in_a_graph(f_in, f_out):
    """Captured after one call of its sizes, replayed between other work and eager calls: the eager results every time."""
    g = G()
    n = 5000
    rs = np.random.default_rng(371)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [dev(synth.normal_features(r, c, 372 + k)) for k, (r, c) in enumerate(((n, f_in), (n, f_in), (f_in, f_out), (n, f_out)))]
    w = min(f_in, f_out)
    T, empty = dev(synth.normal_features(n, w, 376)), lambda r, c: torch.zeros(r, c, device="cuda")
    S, Y, Gp, db = empty(n, w), empty(f_in, f_out), empty(n, f_in), empty(1, f_out).view(-1)
    call = lambda: g.gcn_layer_backward(a, H, Zp, W, Gm, T, S, Y, Gp, dbias=db)
    g.gcn_spmm_prepare(a, 0, w)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        call()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        call()
    for rep in range(4):
        Gm.copy_(dev(synth.normal_features(n, f_out, 380 + rep)))
        for x in (S, Y, Gp, db):
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in (S, Y, Gp, db)]
        call()
        assert all(torch.equal(p, q) for p, q in zip(got, (S, Y, Gp, db))), rep
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 64, 97, 416, 600, 1000])
@pytest.mark.parametrize("f_in,f_out", [(256, 256), (257, 256), (40, 1700), (1000, 70)])
def test_bias_gradient_beside_large_weight_gradients(n, f_in, f_out):
    """On both sides of 64 K numbers, with 1 to 32 partial results, of which the last are fewer than a step or a single one: the bits that a call without a bias
    gradient leaves, and the weight gradient as close to 64 bits as its chains of up to 64 rows and their sums allow."""
    g = G()
    a = g.gcn_csr_create(n, *[torch.arange(n, dtype=torch.int32, device="cuda")] * 2, g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [dev(synth.normal_features(r, c, 351 + i)) for i, (r, c) in enumerate(((n, f_in), (n, f_in), (f_in, f_out), (n, f_out)))]
    w = min(f_in, f_out)
    T, empty = dev(synth.normal_features(n, w, 356)), lambda r, c: torch.full((r, c), float("nan"), device="cuda")
    S, S1, Y, Y1, Gp, Gp1, db = empty(n, w), empty(n, w), empty(f_in, f_out), empty(f_in, f_out), empty(n, f_in), empty(n, f_in), empty(1, f_out).view(-1)
    g.gcn_layer_backward(a, H, Zp, W, Gm, T, S1, Y1, Gp1)
    g.gcn_layer_backward(a, H, Zp, W, Gm, T, S, Y, Gp, dbias=db)
    assert torch.equal(Y, Y1) and torch.equal(Gp, Gp1)
    left, right = (H, S) if f_out <= f_in else (T, Gm)
    want, scale = left.double().T @ right.double(), left.double().abs().T @ right.double().abs()
    assert bool(((Y.double() - want).abs() <= 100 * 2.0 ** -24 * scale).all())
    assert np.all(np.abs(host(db) - host(Gm.double().sum(0))) <= 16 * 2.0 ** -24 * host(Gm.double().abs().sum(0)))
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 2, 3, 5, 6, 7, 15, 17, 18, 19, 21, 22, 23, 31, 33, 35, 41, 47, 63, 65, 66, 67, 70, 80, 96, 130, 131])
@pytest.mark.parametrize("M,K,tb", [(64, 16, 0), (79, 3, 0), (1001, 64, 0), (1001, 64, 1), (333, 300, 0), (333, 602, 0), (5000, 41, 1)])
def test_dense_products_of_ragged_rows(M, K, tb, N):
    """Rows of C that are no whole 16 bytes: the last columns alone in their tile or behind others of it, in one or more shares of the columns, C at any
    address and pitch; bias and both epilogues; nothing between the rows is written.  The same bits as in rows at a pitch of 16 bytes."""
    g = G()
    A, B = synth.normal_features(M, K, 301), synth.normal_features(*((N, K) if tb else (K, N)), 302)
    bias, Zp = synth.normal_features(1, N, 303)[0], synth.normal_features(M, N, 304)
    plain = A.astype(np.float64) @ (B.T if tb else B).astype(np.float64)
    Ad, Bd, bd, Zd = dev(A), dev(B), dev(bias), dev(Zp)
    # a chain of K products, each step rounded once at the size of the sum of magnitudes, and the bias
    bound = (K + 2) * 2.0 ** -24 * (np.abs(A).astype(np.float64) @ np.abs(B.T if tb else B) + np.abs(bias)) + 1e-30
    for epilogue, want in ((g.EPI_NONE, plain + bias), (g.EPI_RELU, np.maximum(plain + bias, 0)), (g.EPI_MASK, np.where(Zp > 0, plain + bias, 0))):
        got = []
        for pitch, first in ((N, 0), (N + 1, 3), ((N + 3) // 4 * 4, 0)):
            memory = torch.full((M * pitch + 8,), 7.0, device="cuda")
            C = memory[first:first + M * pitch].view(M, pitch)[:, :N]
            Z = torch.full((M, (N + 3) // 4 * 4), float("nan"), device="cuda")[:, :N]
            Z.copy_(Zd)
            g.gcn_gemm(0, tb, Ad, Bd, C, bias=bd, epilogue=epilogue, Zprev=Z if epilogue == g.EPI_MASK else None)
            got.append(C.clone())
            assert np.all(np.abs(host(C) - want) <= bound), (pitch, epilogue)
            C.fill_(7.0)
            assert bool((memory == 7.0).all()), (pitch, epilogue)
        assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.gpu
@pytest.mark.parametrize("N", [65, 66, 67, 79, 82, 95, 111, 113, 127])
@pytest.mark.parametrize("K", [3, 44, 144, 145])
def test_dense_products_of_ragged_rows_beyond_the_caches(N, K):
    """Rows of 65 to 127 columns leave from one wavefront where operand and result are beyond the memory-side cache, up to 144 rows of op(B); pieces of the rows are
    other launches.  The same bits, with a bias and either epilogue."""
    g = G()
    M = (192 << 20) // (4 * (K + N)) + 21
    gen = torch.Generator(device="cuda")
    gen.manual_seed(331)
    A, B, bias, Zp = [torch.randn(r, c, generator=gen, device="cuda") for r, c in ((M, K), (K, N), (1, N), (M, N))]
    for epilogue in (g.EPI_NONE, g.EPI_RELU, g.EPI_MASK):
        C, pieces = torch.full((M + 2, N), float("nan"), device="cuda"), torch.empty(M, N, device="cuda")
        args = lambda r: dict(bias=bias.view(-1), epilogue=epilogue, Zprev=Zp[r] if epilogue == g.EPI_MASK else None)
        g.gcn_gemm(0, 0, A, B, C[1:-1], **args(slice(None)))
        for r in (slice(0, M // 3), slice(M // 3, 2 * (M // 3)), slice(2 * (M // 3), M)):
            g.gcn_gemm(0, 0, A[r], B, pieces[r], **args(r))
        assert torch.equal(C[1:-1], pieces), epilogue
        assert bool(torch.isnan(C[0]).all() and torch.isnan(C[-1]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n,C", [(3, 300), (1024, 300), (1025, 300), (2048, 300), (2049, 300), (8192, 300), (8197, 300), (131_072, 2), (131_073, 2)])
def test_loss_sums_on_both_sides_of_two_terms_a_thread(n, C):
    """Partial sums of the loss, 1 to 2048: up to 512 are added as they come, more of them eight at a time.  A row's loss is off by the roundings of its C exponentials' sum
    and of a few operations behind it, the sum over the rows in double by none of that size."""
    g = G()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(347)
    Z, y = torch.randn(n, C, generator=gen, device="cuda"), torch.randint(0, C, (n,), generator=gen, device="cuda", dtype=torch.int32)
    loss, again, grad = torch.full((1,), float("nan"), device="cuda"), torch.empty(1, device="cuda"), torch.empty(n, C, device="cuda")
    g.gcn_softmax_nll(Z, y, loss, grad)
    want = float(torch.nn.functional.cross_entropy(Z.double().cpu(), y.long().cpu()))
    assert abs(float(loss) - want) <= (C + 32) * 2.0 ** -24 * max(1.0, want)
    g.gcn_softmax_nll(Z, y, again)
    assert torch.equal(again, loss)


@pytest.mark.gpu
@pytest.mark.parametrize("M", [32768, 32769, 36001, 65535, 65537])
@pytest.mark.parametrize("K,N", [(300, 1), (302, 15), (409, 7), (602, 14)])
def test_dense_products_of_single_columns(M, K, N):
    """Up to 15 columns over 32 K to 64 K rows of 300 floats and more leave as single columns, pieces of the rows four columns at a time: the same bits, with and without a
    bias, with either epilogue and a mask that is the result, and nothing between the rows is written."""
    g = G()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(337)
    A, B, bias, Zp = [torch.randn(r, c, generator=gen, device="cuda") for r, c in ((M, K), (K, N), (1, N), (M, N))]
    parts = [slice(0, M // 3), slice(M // 3, 2 * (M // 3)), slice(2 * (M // 3), M)]
    for epilogue in (g.EPI_NONE, g.EPI_RELU, g.EPI_MASK):
        for b in (None, bias.view(-1)):
            C, pieces = torch.full((M + 2, N + 2), float("nan"), device="cuda"), torch.empty(M, N, device="cuda")
            args = lambda r: dict(bias=b, epilogue=epilogue, Zprev=Zp[r] if epilogue == g.EPI_MASK else None)
            g.gcn_gemm(0, 0, A, B, C[1:-1, :N], **args(slice(None)))
            for r in parts:
                g.gcn_gemm(0, 0, A[r], B, pieces[r], **args(r))
            assert torch.equal(C[1:-1, :N], pieces), epilogue
            assert bool(torch.isnan(C[0]).all() and torch.isnan(C[-1]).all() and torch.isnan(C[:, N:]).all())
            if epilogue == g.EPI_MASK:
                over = Zp.clone()
                g.gcn_gemm(0, 0, A, B, over, bias=b, epilogue=epilogue, Zprev=over)
                assert torch.equal(over, pieces)
    rows = torch.randint(0, M, (200,), generator=gen, device="cuda")
    g.gcn_gemm(0, 0, A, B, C[1:-1, :N])
    assert_close(host(C[1:-1, :N][rows]), host(A[rows].double() @ B.double()), f"{M} x {K} x {N}")


@pytest.mark.gpu
@pytest.mark.parametrize("N", [1, 2, 3, 6, 7, 18, 23, 41, 62, 63, 66, 70, 95, 127, 130, 243, 255])
@pytest.mark.parametrize("M,K,tb", [(64, 16, 0), (1001, 30, 1), (333, 602, 0)])
def test_result_over_its_own_mask(M, K, tb, N):
    """A mask that is the result itself: the last columns of a row are read and stored by two lanes."""
    g = G()
    A, B, Zp = dev(synth.normal_features(M, K, 341)), dev(synth.normal_features(*((N, K) if tb else (K, N)), 342)), dev(synth.normal_features(M, N, 343))
    want = torch.empty(M, N, device="cuda")
    g.gcn_gemm(0, tb, A, B, want, epilogue=g.EPI_MASK, Zprev=Zp)
    g.gcn_gemm(0, tb, A, B, Zp, epilogue=g.EPI_MASK, Zprev=Zp)
    assert torch.equal(Zp, want)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [63, 64, 65, 79, 127, 129, 1000, 33_000, 70_001])
@pytest.mark.parametrize("f_in,f_out", [(16, 1), (16, 5), (16, 15), (16, 16), (32, 3), (32, 16), (32, 17), (32, 32), (64, 2), (64, 16), (64, 17), (64, 33), (64, 41),
                                        (64, 48), (64, 49), (64, 64)])
@pytest.mark.parametrize("pad,own", [(0, True), (4, False), (1, False)])
def test_backward_products_of_one_pass(n, f_in, f_out, pad, own):
    """Y = H^T S and Gprev = (S W^T) masked where they are one kernel (not: pitches that are no whole 16 bytes, below 64 rows, Gprev over H):
    columns and rows of S at the edges of its tiles and trips, S at no 16-byte address.  Gprev has the bits of the product of its own."""
    g = G()
    rs = np.random.default_rng(244)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [synth.normal_features(r, c, 245 + i) for i, (r, c) in enumerate(((n, f_in), (n, f_in), (f_in, f_out), (n, f_out)))]
    Hd = torch.full((n, f_in + pad), float("nan"), device="cuda")
    Hd[:, :f_in] = dev(H)
    Hd, Wd, Gd = Hd[:, :f_in], dev(W), dev(Gm)
    Zd = Hd if own else dev(Zp)
    S = torch.full((n * f_out + 2,), float("nan"), device="cuda")[1:-1].view(n, f_out)
    Y = torch.full((f_in, f_out), float("nan"), device="cuda")
    Gp = torch.full((n + 2, f_in), float("nan"), device="cuda")
    g.gcn_layer_backward(a, Hd, Zd, Wd, Gd, None, S, Y, Gp[1:-1], g.ORDER_GEMM_FIRST)
    Sx = S.double()
    wantY, scale = Hd.double().T @ Sx, float((Hd.double().T.abs() @ Sx.abs()).norm())
    # sums of up to 70 K products, in chains of 128 and the sums of those: a few roundings of the sums' size, which is below that of the magnitudes
    assert float((Y.double() - wantY).norm()) <= 4 * 2.0 ** -24 * scale
    plain = torch.empty(n, f_in, device="cuda")
    g.gcn_gemm(0, 1, S, Wd, plain, epilogue=g.EPI_MASK, Zprev=Zd)
    assert torch.equal(Gp[1:-1], plain)
    assert_close(host(plain), host(torch.where(Zd > 0, Sx @ Wd.double().T, 0.0)), f"{n} {f_in} {f_out}")
    assert bool(torch.isnan(Gp[0]).all() and torch.isnan(Gp[-1]).all())
    if pad == 0:
        over, first = torch.clone(Hd), Y.clone()
        g.gcn_layer_backward(a, over, over, Wd, Gd, None, S, Y, over, g.ORDER_GEMM_FIRST)
        assert torch.equal(over, plain) and float((Y - first).norm()) <= 4 * 2.0 ** -24 * scale
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [64, 1000, 70_001])
@pytest.mark.parametrize("ldh,first,over", [(20, 0, 0), (20, 0, 4), (16, 16, 0), (16, 0, 16), (24, 8, 0)])
def test_backward_products_of_width_16_with_gprev_across_the_rows_of_h(n, ldh, first, over):
    """Gprev in H's memory at another pitch or offset: row i of Gprev lies over other rows of H, all of which Y needs first."""
    g = G()
    rs = np.random.default_rng(146)
    a = g.gcn_csr_create(n, *[dev(rs.integers(0, n, 3 * n).astype(np.int32)) for _ in range(2)], g.ADD_SELF_LOOPS | g.NORM_ROW | g.BUILD_TRANSPOSE)
    H, Zp, W, Gm = [synth.normal_features(k, 16, 147 + i) for i, k in enumerate((n, n, 16, n))]
    memory = torch.zeros(n * ldh + 64, device="cuda")
    Hd = memory[first:first + n * ldh].view(n, ldh)[:, :16]
    Hd.copy_(dev(H))
    Gp = memory[over:over + n * 16].view(n, 16)
    S, Y = torch.empty(n, 16, device="cuda"), torch.full((16, 16), float("nan"), device="cuda")
    g.gcn_layer_backward(a, Hd, dev(Zp), dev(W), dev(Gm), None, S, Y, Gp, g.ORDER_GEMM_FIRST)
    Sx = host(S).astype(np.float64)
    wantY = H.T.astype(np.float64) @ Sx
    assert np.linalg.norm(host(Y) - wantY) <= 5e-7 * np.linalg.norm(wantY)
    assert_close(host(Gp), np.where(Zp > 0, Sx @ W.T, 0), f"{n} {ldh} {first} {over}")
    a.close()


@pytest.mark.gpu
@pytest.mark.parametrize("f", [16, 32])
def test_a_relu_does_not_change_the_sums(f):
    """A X may take another order of additions than A^T X; with a ReLU each of them is the clamp of the plain product, bit by bit, and
    A^T X that of the layer call."""
    g = G()
    n, pairs = 500_000, 10_000_000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(161)
    src, dst = [torch.randint(n, (pairs,), generator=gen, device="cuda", dtype=torch.int32) for _ in range(2)]
    a = g.gcn_csr_create(n, src, dst, g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE)
    X = torch.rand(n, f, generator=gen, device="cuda") - 0.5
    assert g.gcn_spmm_describe(a, 0, f) != g.gcn_spmm_describe(a, 1, f)
    for trans in (0, 1):
        plain, relu = torch.empty(n, f, device="cuda"), torch.empty(n, f, device="cuda")
        g.gcn_spmm(a, trans, X, plain)
        g.gcn_spmm(a, trans, X, relu, g.EPI_RELU)
        assert torch.equal(relu, plain.clamp(min=0)), trans
    T, Z = torch.empty(n, f, device="cuda"), torch.empty(n, f, device="cuda")
    g.gcn_layer_forward(a, X, torch.eye(f, device="cuda"), Z, Z, T, g.ORDER_SPMM_FIRST)
    assert torch.equal(T, plain) and torch.equal(Z, relu)
    a.close()


def drawn_graph(kind, n, pairs, seed):
    """Endpoints on the GPU: uniform, by a power law with exponent 2.3 (heaviest first), within a band, or mostly inside communities that lie
    one after another; the last three numbered so that the order of the vertices says something."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    u = lambda: torch.rand(pairs, generator=gen, device="cuda", dtype=torch.float64)
    if kind == "power":
        b, i0 = 1 - 1 / 1.3, 20.0
        return [((u() * ((n + i0) ** b - i0 ** b) + i0 ** b) ** (1 / b) - i0).clamp(0, n - 1).int() for _ in range(2)], gen
    src = (u() * n).int()
    if kind == "band":
        return [src, ((src + torch.randn(pairs, generator=gen, device="cuda") * 5000) % n).int().clamp(0, n - 1)], gen
    dst = (u() * n).int()
    if kind == "communities":
        inside = u() < 0.8
        dst = torch.where(inside, (src // 5000 * 5000 + (u() * 5000).int()).clamp(max=n - 1), dst)
    return [src, dst], gen


@pytest.mark.parametrize("kind", ["band", "communities", "power"])
def test_ordered_matrices_keep_the_schedule_of_the_sizes(kind):
    """The estimates take the vertices' order for random.  Vertices numbered along a band, by communities or by degree: A X runs as A^T X does, by
    the sizes; the same graph renamed at random does not."""
    g = G()
    n, pairs = 500_000, 10_000_000
    (src, dst), gen = drawn_graph(kind, n, pairs, 171)
    rename = torch.randperm(n, generator=gen, device="cuda").int()
    for ordered in (True, False):
        s, d = (src, dst) if ordered else (rename[src], rename[dst])
        a = g.gcn_csr_create(n, s, d, g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM | g.BUILD_TRANSPOSE)
        same = [g.gcn_spmm_describe(a, 0, f) == g.gcn_spmm_describe(a, 1, f) for f in (16, 32, 64)]
        assert all(same) if ordered else not all(same), (kind, ordered, same)
        a.close()


@pytest.mark.parametrize("nnz", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 3, (1 << 20) + 2049])
def test_columns_are_sampled_inside_the_matrix(nnz):
    """The smallest matrices that are sampled, entries not a multiple of the loads' width, transposes not stored: products as without."""
    g = G()
    rs = np.random.default_rng(172)
    n, nc, f = 30_000, 200_000, 8
    lengths = rs.multinomial(nnz, np.full(n, 1 / n))
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rs.choice(nc, k, replace=False)) for k in lengths]).astype(np.int32)
    val = rs.standard_normal(nnz).astype(np.float32)
    a = g.gcn_csr_create_from_csr_rect(n, nc, dev(rowptr), dev(colidx), dev(val), 0)
    X = synth.normal_features(nc, f, 173)
    want = np.zeros((n, f))
    np.add.at(want, np.repeat(np.arange(n), lengths), val[:, None].astype(np.float64) * X[colidx])
    assert_close(host(g.gcn_spmm(a, 0, dev(X), torch.empty(n, f, device="cuda"))), want, str(nnz))
    a.close()


@pytest.mark.parametrize("kind,mean", [("uniform", 12), ("uniform", 17), ("uniform", 21), ("uniform", 41), ("power", 13), ("power", 20), ("power", 41)])
@pytest.mark.parametrize("norm", ["sym", "row"])
def test_schedules_by_cost_are_no_less_exact(kind, mean, norm):
    """The error of A X against sums in 64 bits is no larger than that of the nonzero split, whatever schedule is taken, at mean rows where one sum
    per row in the sweep would be a longer chain; values 1 / sqrt(d_i d_j), whose long rows are small, and 1 / d_i."""
    g = G()
    n = 800_000
    (src, dst), gen = drawn_graph(kind, n, n * (mean - 1) // (2 if norm == "sym" else 1), 174)
    rename = torch.randperm(n, generator=gen, device="cuda").int()
    flags = g.SYMMETRISE | g.NORM_SYM if norm == "sym" else g.NORM_ROW
    a = g.gcn_csr_create(n, rename[src], rename[dst], flags | g.ADD_SELF_LOOPS | g.BUILD_TRANSPOSE)
    rowptr, colidx, val, _ = a.arrays(False)
    rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr[1:] - rowptr[:-1])
    for f in (16, 32):
        X = torch.rand(n, f, generator=gen, device="cuda") * 2 - 1
        exact = torch.zeros(n, f, dtype=torch.float64, device="cuda")
        for k in range(0, a.nnz, 1 << 22):
            part = slice(k, k + (1 << 22))
            exact.index_add_(0, rows[part], val[part, None].double() * X[colidx[part].long()])
        error = []
        for algo in (0, 2):
            g.gcn_csr_config(a, g.CFG_SPMM_ALGO, algo)
            g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1 if algo else 0)
            error.append(float((g.gcn_spmm(a, 0, X, torch.empty(n, f, device="cuda")).double() - exact).norm() / exact.norm()))
        g.gcn_csr_config(a, g.CFG_SPMM_ALGO, 0)
        g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 0)
        print(kind, mean, norm, f, g.gcn_spmm_describe(a, 0, f)[:90], error)
        assert error[0] <= 1.005 * error[1], (kind, mean, norm, f, g.gcn_spmm_describe(a, 0, f), error)
    a.close()


@pytest.mark.parametrize("kind,mean", [("uniform", 17), ("power", 20), ("power", 41)])
@pytest.mark.parametrize("values", ["none", "row", "sym", "given"])
def test_schedules_by_cost_of_the_transpose_are_no_less_exact(kind, mean, values):
    """As above for A^T X (with a mask that lets all through, so that its schedule is free) on directed graphs, whose rows are as long as vertices have
    incoming edges while the values follow from the outgoing ones, and for A X with values 1 and with the caller's, on rows in
    proportion to 1 / d_i."""
    g = G()
    n = 800_000
    (src, dst), gen = drawn_graph(kind, n, n * (mean - 1), 175)
    rename = torch.randperm(n, generator=gen, device="cuda").int()
    norm = {"none": 0, "row": g.NORM_ROW, "sym": g.NORM_SYM, "given": g.NORM_ROW}[values]
    a = g.gcn_csr_create(n, rename[src], rename[dst], norm | g.ADD_SELF_LOOPS | g.BUILD_TRANSPOSE)
    if values == "given":
        rowptr, colidx, val, _ = a.arrays(False)
        b = g.gcn_csr_create_from_csr(n, rowptr.clone(), colidx.clone(), val.clone(), g.BUILD_TRANSPOSE)
        a.close()
        a = b
    g.gcn_csr_config(a, g.CFG_PATTERN_SPMM, 0)
    f = 16
    X, ones = torch.rand(n, f, generator=gen, device="cuda") * 2 - 1, torch.ones(n, f, device="cuda")
    for trans in ((0, 1) if values in ("none", "given") else (1,)):
        rowptr, colidx, val, _ = a.arrays(bool(trans))
        rows = torch.repeat_interleave(torch.arange(n, device="cuda"), rowptr[1:] - rowptr[:-1])
        exact = torch.zeros(n, f, dtype=torch.float64, device="cuda")
        for k in range(0, a.nnz, 1 << 22):
            part = slice(k, k + (1 << 22))
            exact.index_add_(0, rows[part], val[part, None].double() * X[colidx[part].long()])
        error = []
        for algo in (0, 2):
            g.gcn_csr_config(a, g.CFG_SPMM_ALGO, algo)
            g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 1 if algo else 0)
            error.append(float((g.gcn_spmm(a, trans, X, torch.empty(n, f, device="cuda"), g.EPI_MASK, ones).double() - exact).norm() / exact.norm()))
        sched = g.gcn_csr_last_spmm_schedule(a)
        g.gcn_csr_config(a, g.CFG_SPMM_ALGO, 0)
        g.gcn_csr_config(a, g.CFG_SPMM_BLOCKS, 0)
        print(kind, mean, values, trans, g.gcn_spmm_describe(a, 0, f)[:90] if not trans else sched, error)
        assert error[0] <= 1.005 * error[1], (kind, mean, values, trans, error)
    a.close()


@pytest.mark.parametrize("kind,n,mean", [("power", 250_000, 60), ("power", 800_000, 20), ("power", 810_000, 72), ("power", 980_000, 90), ("uniform", 500_000, 25)])
@pytest.mark.parametrize("norm", ["none", "row", "sym"])
def test_prepared_products_with_and_without_values_build_nothing(kind, n, mean, norm):
    """gcn_spmm_prepare builds what gcn_spmm and gcn_spmm_pattern need at that width, also where the one knows the values and the other does not
    and they take different schedules: no call after it builds an order."""
    g = G()
    (src, dst), gen = drawn_graph(kind, n, n * (mean - 1), 176)
    rename = torch.randperm(n, generator=gen, device="cuda").int()
    a = g.gcn_csr_create(n, rename[src], rename[dst], {"none": 0, "row": g.NORM_ROW, "sym": g.NORM_SYM}[norm] | g.ADD_SELF_LOOPS | g.BUILD_TRANSPOSE)
    for f in (8, 16, 32, 64):
        X, Z, ones = torch.rand(n, f, device="cuda"), torch.empty(n, f, device="cuda"), torch.ones(n, f, device="cuda")
        for trans in (0, 1):
            g.gcn_spmm_prepare(a, trans, f)
            built = g.gcn_build_count()
            for epi in (g.EPI_NONE, g.EPI_RELU, g.EPI_MASK):
                g.gcn_spmm(a, trans, X, Z, epi, ones)
                g.gcn_spmm_pattern(a, trans, X, Z, None, epi, ones)
            assert g.gcn_build_count() == built, (kind, n, mean, norm, f, trans)
    a.close()


@pytest.mark.parametrize("n,k,f,usual", [(500_000, 41, 16, "split("), (500_000, 41, 32, "split("), (600_000, 100, 32, "split(")])
def test_rows_that_fill_no_set_are_not_swept(n, k, f, usual):
    """Row i selects the columns k i to k i + k - 1 (mod n): as long as the rows and columns of a uniform matrix, and as many different columns, but
    a task's rows come one after the other and a sweep copy would be padding for the most part.  Neither the estimates nor (mean of 64
    and more) the sizes take it, it is asked for once, and the product is right; asked for by the caller it is built."""
    g = G()
    rowptr = torch.arange(0, (n + 1) * k, k, device="cuda")
    cols = (torch.arange(n, device="cuda")[:, None] * k + torch.arange(k, device="cuda")) % n
    a = g.gcn_csr_create_from_csr(n, rowptr, cols.sort(1).values.int().reshape(-1), None, 0)
    assert g.gcn_spmm_describe(a, 0, f).startswith(usual)
    built = g.gcn_build_count()
    X = torch.rand(n, f, device="cuda") * 2 - 1
    Z = g.gcn_spmm(a, 0, X, torch.empty(n, f, device="cuda"))
    g.gcn_spmm(a, 0, X, Z)
    assert g.gcn_build_count() == built
    want = torch.zeros(n, f, device="cuda", dtype=torch.float64)
    for c in cols.unbind(1):
        want += X[c]
    assert_close(host(Z), host(want), f"{n} {k} {f}")
    if n == 500_000 and f == 16:
        g.gcn_csr_config(a, g.CFG_SPMM_ALGO, 3)
        assert g.gcn_spmm_describe(a, 0, f).startswith("sweep(")
        assert_close(host(g.gcn_spmm(a, 0, X, Z)), host(want), "asked for")
        g.gcn_csr_config(a, g.CFG_SPMM_ALGO, 0)
        assert g.gcn_spmm_describe(a, 0, f).startswith(usual)
    a.close()


@pytest.mark.parametrize("offset", [0, 1])
def test_export_in_a_graph(offset):
    """Captured on a stream of its own and replayed, by the kernel and by the runtime's copies."""
    from paper_2005_03300_amd import binding
    g = G()
    rs = np.random.default_rng(171)
    a = g.gcn_csr_create(5000, *[dev(rs.integers(0, 5000, 40_000).astype(np.int32)) for _ in range(2)], g.SYMMETRISE | g.ADD_SELF_LOOPS | g.NORM_SYM)
    want = a.arrays()
    room = [torch.empty(w.numel() + 4, dtype=w.dtype, device="cuda") for w in want]
    dst = [r[offset:offset + w.numel()] for r, w in zip(room, want)]
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        binding._check(binding.lib().gcn_csr_export(a._h, 0, *map(binding._ptr, dst), binding._stream()))
    for k in range(3):
        for r in room:
            r.fill_(-7 - k)
        graph.replay()
        torch.cuda.synchronize()
        for d, r, w in zip(dst, room, want):
            assert torch.equal(d, w) and int((r == -7 - k).sum()) >= 4, k
    a.close()


@pytest.mark.parametrize("nnz", [1, 4, 7, 4095, 4096, 4098, 3 * 4096 + 1, 1_000_003])
@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_export_fills_the_callers_arrays_and_no_more(nnz, offset):
    """Tiles of 4096 words and their remainders; destinations in pieces of 16 bytes and, `offset` words into an allocation, not; some left out."""
    from paper_2005_03300_amd import binding
    g = G()
    n = nnz // 3 + 1
    gen = torch.Generator(device="cuda").manual_seed(nnz)
    cut = torch.sort(torch.randint(0, nnz + 1, (n - 1,), generator=gen, device="cuda")).values
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), cut, torch.full((1,), nnz, device="cuda")])
    cols = (torch.arange(nnz, device="cuda") % (nnz + 5)).int()
    val = torch.rand(nnz, generator=gen, device="cuda")
    a = g.gcn_csr_create_from_csr_rect(n, nnz + 5, rowptr, cols, val, 0)
    deg = (rowptr[1:] - rowptr[:-1]).int()
    want = [rowptr, cols, val, deg]
    for keep in (15, 10):
        room = [torch.full((w.numel() + 8,), -7, dtype=w.dtype, device="cuda") for w in want]
        dst = [r[offset:] if keep >> i & 1 else None for i, r in enumerate(room)]
        binding._check(binding.lib().gcn_csr_export(a._h, 0, *(binding._ptr(d) if d is not None else None for d in dst), binding._stream()))
        for i, (r, w) in enumerate(zip(room, want)):
            expect = torch.full_like(r, -7)
            if keep >> i & 1:
                expect[offset:offset + w.numel()] = w
            assert torch.equal(r, expect), (i, keep)
    a.close()

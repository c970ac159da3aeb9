"""Small products against the oracle, every bit of C: sizes at the edges of the 64 x 64, 128 x 128 and 256 x 256 tiles of
the products, inner dimensions at the edges of a k-tile and of the one-pass conversion's forms, both orientations of either
operand, operands split one and two levels deep, and infinities / NaNs in the last vector of the last workgroup."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2504_08009_amd as oz
from oracle import oracle as orc


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x.T)).cuda().t()


def _gemm(ta, tb, A, B, N, beta=0.0):
    opA, opB = (A.T if ta == "T" else A), (B.T if tb == "T" else B)
    m, k = opA.shape
    n = opB.shape[1]
    rng = np.random.default_rng(m + n)
    C0 = np.asfortranarray(rng.standard_normal((m, n)))
    dA, dB, dC = _dev(A), _dev(B), _dev(C0)
    ws = oz.Workspace(m, n, k, N)
    oz.oz2_dgemm_ex(ta, tb, m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), B.shape[0], beta, dC.data_ptr(), m, N)
    torch.cuda.synchronize()
    flag = int(ws.view(oz.workspace_layout(m, n, k, N)["flags"], 1, torch.int64).item())
    return dC.cpu().numpy(), orc.dgemm_ex(ta, tb, 1.0, A, B, beta, C0, N), flag


def _choice(m, n, k, N):
    return oz.host_kernel_choice(m, n, k, N, torch.cuda.get_device_properties(0).multi_processor_count)


def _route(m, n, k, N, ta="N", tb="N", call="dgemm"):
    return oz.host_route(m, n, k, N, torch.cuda.get_device_properties(0).multi_processor_count, call, ta, tb)


def _mat(rng, r, c):
    return np.asfortranarray((rng.random((r, c)) - 0.5) * np.exp(rng.standard_normal((r, c))))


@pytest.mark.parametrize("m,n", [(1, 1), (63, 64), (65, 127), (128, 129), (191, 257), (256, 7), (9, 520), (300, 385), (640, 600)])
@pytest.mark.parametrize("k", [1, 64, 65, 200, 1024, 1025])
def test_edges_of_the_tiles_and_of_the_one_pass_conversion(m, n, k):
    rng = np.random.default_rng(m * 1000 + n + k)
    ta, tb = [("N", "N"), ("T", "N"), ("N", "T"), ("T", "T")][(m + k) % 4]
    N = [14, 9, 16, 22][(n + k) % 4]  # 22: elements of more than 75 bits, split two levels deep
    print("small: m=%d n=%d k=%d N=%d op=%s%s" % (m, n, k, N, ta, tb), flush=True)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    got, ref, flag = _gemm(ta, tb, A, B, N, beta=float(k % 2))
    assert flag == 0 and np.array_equal(got, ref)


@pytest.mark.parametrize("k", [1, 63, 65, 129, 193, 256, 257, 320, 449, 512, 513, 577, 960, 1000])
@pytest.mark.parametrize("m,n,N", [(70, 45, 3), (300, 500, 15), (40, 4200, 5), (3900, 30, 22)])
def test_one_pass_conversion_by_four_and_by_eight_vectors(m, n, N, k):
    """Every number of k-tiles up to eight and beyond (waves that share a k-tile, with fewer moduli than waves among them), vectors
    enough for workgroups of eight at every length and few enough for four, loads in flight that end inside a batch."""
    rng = np.random.default_rng(m + 7 * n + k)
    ta, tb = [("N", "N"), ("T", "T")][k % 2]
    print("one pass: m=%d n=%d k=%d N=%d op=%s%s" % (m, n, k, N, ta, tb), flush=True)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    got, ref, flag = _gemm(ta, tb, A, B, N, beta=float(m % 4 == 0))
    assert flag == 0 and np.array_equal(got, ref)


@pytest.mark.parametrize("N", range(2, 27))
@pytest.mark.parametrize("m,n", [(45, 70), (601, 500)])
def test_every_number_of_moduli(m, n, N):
    """Stage 3 of small results takes the planes eight or four at a time, by the number of moduli, in pieces of two and of four rows."""
    k = 40
    rng = np.random.default_rng(m + N)
    print("moduli: m=%d n=%d k=%d N=%d" % (m, n, k, N), flush=True)
    got, ref, flag = _gemm("N", "N", _mat(rng, m, k), _mat(rng, k, n), N, beta=float(N % 2))
    assert flag == 0 and np.array_equal(got, ref)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("m,n,k,N,vectors", [
    (2000, 2300, 250, 6, 8), (4000, 300, 512, 7, 8), (4200, 100, 1024, 5, 8), (60, 40, 1025, 3, 2), (300, 200, 1999, 14, 2), (700, 500, 2432, 9, 4),
    (700, 500, 2433, 9, 2), (1200, 100, 2433, 5, 2), (40, 700, 3393, 15, 2), (300, 800, 3393, 15, 4), (2000, 100, 4928, 4, 4), (700, 500, 4929, 6, 2),
    (70, 300, 4929, 16, 2), (256, 130, 6209, 22, 2), (30, 20, 9920, 21, 2), (30, 20, 9921, 21, 0)])
def test_one_pass_conversion_of_long_vectors(m, n, k, N, vectors, mode):
    """Two, four and eight vectors per workgroup in every shift mode; four and two at the longest that fit into LDS (2432 is the last
    inner dimension of eight, at which four are taken, 4928 that of four and 9920 that of two) and at one more."""
    rng = np.random.default_rng(3 * m + n + k)
    ta, tb = [("N", "N"), ("T", "T"), ("N", "T")][(k + mode) % 3]
    print("long: m=%d n=%d k=%d N=%d mode=%d op=%s%s" % (m, n, k, N, mode, ta, tb), flush=True)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    A[(m // 2, slice(None)) if ta == "N" else (slice(None), m // 2)] = 0.0  # an all-zero vector
    opA, opB = np.asfortranarray(A.T if ta == "T" else A), np.asfortranarray(B.T if tb == "T" else B)
    dA, dB, dC = _dev(A), _dev(B), _dev(np.ones((m, n), order="F"))
    ws = oz.Workspace(m, n, k, N)
    flags = ws.view(oz.workspace_layout(m, n, k, N)["flags"], 1, torch.int64)
    oz.oz2_set_shift_mode(mode)
    try:
        assert _choice(m, n, k, N)[0] == vectors
        args = (ta, tb, m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), B.shape[0], 0.0, dC.data_ptr(), m, N)
        oz.oz2_dgemm_ex(*args)
        torch.cuda.synchronize()
        assert int(flags.item()) == 0
        assert np.array_equal(dC.cpu().numpy(), orc.dgemm(opA, opB, N, mode=mode).C)
        dA[-1, -1] = float("nan")
        oz.oz2_dgemm_ex(*args)
        torch.cuda.synchronize()
        assert int(flags.item()) == 1 and bool(torch.isnan(dC[m - 1]).all()) and bool(torch.isfinite(dC[: m - 1]).all())
    finally:
        oz.oz2_set_shift_mode(0)


@pytest.mark.parametrize("lda,shift", [(1280, 0), (1281, 0), (1288, 0), (1296, 0), (1296, 1)])
def test_many_strided_vectors_in_whole_lines_and_not(lda, shift):
    """Rows of A that are whole cache lines by sixteens take the separate launches, others the one-pass conversion: leading dimensions that
    are a multiple of 16 and not, and an array that starts inside a line."""
    m, n, k, N = 1280, 140, 7424, 9
    assert _choice(m, n, k, N) == (0, 0, 128)
    rng = np.random.default_rng(lda + shift)
    A, B = _mat(rng, m, k), _mat(rng, k, n)
    print("lines: lda=%d shift=%d" % (lda, shift), flush=True)
    buf = torch.full((k * lda + 16,), float("nan"), dtype=torch.float64, device="cuda")
    assert buf.data_ptr() % 128 == 0
    dA = buf[shift:shift + k * lda].view(k, lda)
    dA[:, :m] = torch.from_numpy(np.ascontiguousarray(A.T)).cuda()
    dB, dC = _dev(B), torch.zeros((n, m), dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    ws.buf.fill_(0x7f)
    oz.oz2_dgemm(m, n, k, dA.data_ptr(), lda, dB.data_ptr(), k, dC.data_ptr(), m, N)
    torch.cuda.synchronize()
    rows = np.concatenate([np.arange(40), np.arange(m - 40, m)])
    assert np.array_equal(dC.t()[rows].cpu().numpy(), orc.dgemm(A, B, N, rows=rows).C)
    del ws


@pytest.mark.parametrize("k,n", [(1100, 40), (2500, 30), (3500, 20)])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("side,uplo,ta", [("L", "L", "N"), ("L", "U", "T"), ("R", "U", "N"), ("R", "L", "T"), ("L", "U", "N")])
def test_one_pass_conversion_of_a_triangular_operand(side, uplo, ta, mode, k, n):
    """Triangular operands whose vectors fit into LDS: NaNs in the half that is not referenced, every element against the oracle
    on the matrix that the convention defines."""
    rng = np.random.default_rng(k + n + mode)
    m_, n_, N = (k, n, 12) if side == "L" else (n, k, 12)
    A = _mat(rng, k, k)
    T = np.tril(A) if uplo == "L" else np.triu(A)
    A[np.triu_indices(k, 1) if uplo == "L" else np.tril_indices(k, -1)] = np.nan
    X = _mat(rng, m_, n_)
    opT = np.asfortranarray(T.T if ta == "T" else T)
    ref = orc.dgemm(opT, X, N, mode=mode).C if side == "L" else orc.dgemm(X, opT, N, mode=mode).C
    dA, dX = _dev(A), _dev(X)
    ws = oz.Workspace(m_, n_, k, N)
    oz.oz2_set_shift_mode(mode)
    try:
        oz.oz2_dtrmm(side, uplo, ta, "N", m_, n_, 1.0, dA.data_ptr(), k, dX.data_ptr(), m_, N)
        torch.cuda.synchronize()
    finally:
        oz.oz2_set_shift_mode(0)
    assert np.array_equal(dX.cpu().numpy(), ref)
    del ws


def _norm_bounds(vectors):
    """S of each row: with e = floor(log2 max |x|) and q_l = ceil(|x_l| 2^(19 - e)), the sum of q_l^2 (0 for a row of zeros)."""
    x = np.abs(np.asarray(vectors))
    e = np.frexp(x.max(axis=1))[1] - 1
    q = np.ceil(np.ldexp(x, (19 - e)[:, None])).astype(np.int64)
    return (q * q).sum(axis=1)


@pytest.mark.parametrize("entry", ["dgemm", "dsyrk", "dtrmm"])
@pytest.mark.parametrize("k", [300, 1500, 5000, 10300])
def test_norm_bounds_that_whole_calls_leave_in_the_workspace(entry, k):
    """Cauchy-Schwarz mode, inner dimensions on either side of what the one-pass conversion takes: the documented entries of the
    workspace hold the norm bounds, zero in the padding; an infinity in one row changes no other row's."""
    if entry == "dtrmm" and k > 1500:
        k = 900
    rng = np.random.default_rng(k)
    m, n, N = {"dgemm": (70, 300, 9), "dsyrk": (130, 130, 9), "dtrmm": (k, 40, 9)}[entry]
    A, B = _mat(rng, m, k), _mat(rng, k, n)
    A[m // 2, : k - 1] = 0.0
    print("norms: %s m=%d n=%d k=%d" % (entry, m, n, k), flush=True)
    dC = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    lay = oz.workspace_layout(m, n, k, N)
    flags = ws.view(lay["flags"], 1, torch.int64)

    def norms(name, pad):
        return ws.view(lay[name], lay[pad], torch.int64).cpu().numpy()

    oz.oz2_set_shift_mode(oz.OZ2_SHIFT_CAUCHY_SCHWARZ)
    try:
        for bad in (False, True):
            if bad:
                A[3, 2] = np.inf
            ws.buf.fill_(0x7f)
            dA, dB = _dev(A), _dev(B)
            if entry == "dgemm":
                oz.oz2_dgemm(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, dC.data_ptr(), m, N)
            elif entry == "dsyrk":
                oz.oz2_dsyrk("L", "N", m, k, 1.0, dA.data_ptr(), m, 0.0, dC.data_ptr(), m, N)
            else:
                oz.oz2_dtrmm("L", "L", "N", "N", m, n, 1.0, dA.data_ptr(), m, dB.data_ptr(), m, N)
            torch.cuda.synchronize()
            assert int(flags.item()) == int(bad)
            rows = np.where(np.arange(m) == 3, 0.0 if bad else 1.0, 1.0).astype(bool)
            stored = np.tril(A) if entry == "dtrmm" else A
            got = norms("rownorm", "m_pad")
            assert np.array_equal(got[:m][rows], _norm_bounds(stored[rows])) and not got[m:].any()
            if entry != "dsyrk":
                got = norms("colnorm", "n_pad")
                assert np.array_equal(got[:n], _norm_bounds(B.T)) and not got[n:].any()
    finally:
        oz.oz2_set_shift_mode(oz.OZ2_SHIFT_MAX)
    del ws


@pytest.mark.parametrize("entry,m,n,k,mode", [
    ("dgemm", 60, 50, 1100, 0), ("dgemm", 300, 300, 1500, 0), ("dgemm", 300, 200, 5000, 0), ("dgemm", 1000, 900, 1400, 0),
    ("dgemm", 500, 500, 1500, 1), ("dgemm", 1000, 1000, 1088, 1), ("dgemm", 2040, 2048, 2048, 1), ("dgemm", 9000, 150, 1100, 1),
    ("dgemm", 9000, 150, 1100, 0),
    ("dgemm", 1000, 1000, 2000, 2), ("dgemm", 700, 700, 700, 2), ("dgemm", 1000, 1000, 7000, 0),
    ("dsyrk", 500, 500, 3000, 0), ("dsyrk", 1500, 1500, 1500, 0), ("dsyrk", 700, 700, 1200, 1), ("dtrmm", 1500, 300, 1500, 0),
    ("dtrmm", 1100, 1000, 1100, 1)])
def test_products_are_left_out_of_calls_on_infinities(entry, m, n, k, mode):
    """Vectors longer than 1024 (INT8-product mode: of any length): an infinity in the last row or column leaves the product planes as
    they were (those that the fallback of an in-place product and the bound product do not use), and the next finite call fills them.
    9000 x 150: more reports than a workgroup fetches."""
    rng = np.random.default_rng(m + n + k)
    N = 14
    print("left out: %s m=%d n=%d k=%d mode=%d" % (entry, m, n, k, mode), flush=True)
    dA = torch.from_numpy(rng.standard_normal((k, m))).cuda()
    B = torch.from_numpy(rng.standard_normal((n, k))).cuda()
    dC = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    lay = oz.workspace_layout(m, n, k, N)
    flags = ws.view(lay["flags"], 1, torch.int64)
    area = lay["m_pad"] * lay["n_pad"]
    planes = ws.view(lay["c_planes"] + 8 * area, (N - 8) * area, torch.uint8)
    oz.oz2_set_shift_mode(mode)
    try:
        for bad in (True, False):
            dB = B.clone()
            (dB if entry == "dgemm" else dA)[-1, -1] = float("inf") if bad else 1.0
            ws.buf.fill_(0xff)  # no residue: all moduli but 256 are below it
            if entry == "dgemm":
                oz.oz2_dgemm(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, dC.data_ptr(), m, N)
            elif entry == "dsyrk":
                oz.oz2_dsyrk("L", "N", m, k, 1.0, dA.data_ptr(), m, 0.0, dC.data_ptr(), m, N)
            else:
                oz.oz2_dtrmm("L", "L", "N", "N", m, n, 1.0, dA.data_ptr(), m, dB.data_ptr(), m, N)
            torch.cuda.synchronize()
            assert int(flags.item()) == int(bad)
            assert bool((planes == 0xff).all()) == bad
    finally:
        oz.oz2_set_shift_mode(0)
    del ws


@pytest.mark.parametrize("delta", [30, -30])
def test_one_operand_split_deeper_than_the_other(delta):
    """21 moduli and a bit split of 30: one operand needs the two-level split, the other does not."""
    rng = np.random.default_rng(5)
    m, n, k, N = 130, 70, 300, 21
    A, B = _mat(rng, m, k), _mat(rng, k, n)
    oz.oz2_set_bit_split(delta)
    try:
        dA, dB, dC = _dev(A), _dev(B), _dev(np.zeros((m, n), order="F"))
        ws = oz.Workspace(m, n, k, N)
        oz.oz2_dgemm(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, dC.data_ptr(), m, N)
        torch.cuda.synchronize()
    finally:
        oz.oz2_set_bit_split(0)
    assert np.array_equal(dC.cpu().numpy(), orc.dgemm(A, B, N, delta=delta).C)
    del ws


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("where", ["first of A", "last of A", "last of B"])
@pytest.mark.parametrize("m,n,k", [(300, 131, 200), (1400, 1300, 70), (2100, 2000, 64)])
def test_nonfinite_inputs_reach_the_fallback(m, n, k, where, bad):
    """The reports of the one-pass conversion become the flag in the launch of the products; the fallback's blocks ride with
    stage 3 (below 2^24 elements of C)."""
    rng = np.random.default_rng(7)
    A, B = _mat(rng, m, k), _mat(rng, k, n)
    if where == "first of A":
        A[0, 0] = bad
    elif where == "last of A":
        A[m - 1, k - 1] = bad
    else:
        B[k - 1, n - 1] = bad
    got, ref, flag = _gemm("N", "N", A, B, 14)
    assert flag == 1
    finite = np.isfinite(ref)
    assert np.array_equal(got[~finite], ref[~finite], equal_nan=True) and np.all(np.isfinite(got[finite]))
    # finite elements are FP64 sums of k products in both, the oracle's with one rounding per product and sum, the kernel's
    # with one per fused multiply-add: each within (k + 1) 2^-53 |A||B| of the exact sum
    A0, B0 = np.where(np.isfinite(A), A, 0.0), np.where(np.isfinite(B), B, 0.0)
    bound = 2 * (k + 1) * 2.0**-53 * (np.abs(A0) @ np.abs(B0))
    assert np.all(np.abs(got[finite] - ref[finite]) <= bound[finite])
    # the next call on the same shape starts from a clear flag
    A[0, 0] = A[m - 1, k - 1] = B[k - 1, n - 1] = 1.0
    got, ref, flag = _gemm("N", "N", A, B, 14)
    assert flag == 0 and np.array_equal(got, ref)


@pytest.mark.parametrize("call,m,n,k", [("dgemm", 3000, 3000, 1000), ("dgemm", 8192, 8192, 64), ("dgemm", 30000, 3000, 1000),
                                        ("dsyrk", 5000, 5000, 1000), ("dsyrk", 4096, 4096, 1000), ("dtrmm", 1000, 16384, 1000)])
def test_long_products_are_not_formed_for_nonfinite_inputs(call, m, n, k):
    """The one-pass conversion leaves the flag word to the launch after it.  Long products (walked by one workgroup per compute
    unit, small tiles, more reports than every workgroup reads, one triangle, a triangular operand) find out before they start:
    nothing is written over the product planes.  The next call, on finite values, forms them."""
    N = 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + k)
    A = torch.randn((k, m), dtype=torch.float64, device="cuda", generator=gen)  # m x k column-major
    B = torch.randn((n, k), dtype=torch.float64, device="cuda", generator=gen)
    print("%s: m=%d n=%d k=%d" % (call, m, n, k), flush=True)
    ws = oz.Workspace(m, n, k, N)
    lay = oz.workspace_layout(m, n, k, N)
    planes = ws.view(lay["c_planes"], N * lay["n_pad"] * lay["m_pad"], torch.uint8)
    flags = ws.view(lay["flags"], 1, torch.int64)

    def run():
        if call == "dtrmm":
            C = B.clone()
            oz.oz2_dtrmm("L", "L", "N", "N", m, n, 1.0, A.data_ptr(), m, C.data_ptr(), m, N)
            ref = torch.matmul(B, torch.tril(A.t()).t().contiguous())
        elif call == "dsyrk":
            C = torch.zeros((n, n), dtype=torch.float64, device="cuda")
            oz.oz2_dsyrk("L", "N", n, k, 1.0, A.data_ptr(), n, 0.0, C.data_ptr(), n, N)
            ref = torch.triu(torch.matmul(A.t().contiguous(), A))
        else:
            C = torch.zeros((n, m), dtype=torch.float64, device="cuda")
            oz.oz2_dgemm(m, n, k, A.data_ptr(), m, B.data_ptr(), k, C.data_ptr(), m, N)
            ref = torch.matmul(B, A)
        torch.cuda.synchronize()
        return C, ref

    kept = A[k - 1, m - 1].item()
    A[k - 1, m - 1] = float("inf")  # last row of op(A)
    planes.fill_(0x7f)
    C, ref = run()
    free = 8 * m * n if call == "dtrmm" else 0  # (the triangular product's fallback keeps its result at the region's front)
    flag, untouched, last = int(flags.item()), bool((planes[free:] == 0x7f).all()), float(C[0, m - 1])
    assert flag == 1 and untouched and not np.isfinite(last)
    # (FP64 sums of k terms of order one on both sides: k (k + 1) 2^-53 < 1e-9 at most)
    error = float((C[:, :m - 1] - ref[:, :m - 1]).abs().max())
    assert error < 1e-9
    A[k - 1, m - 1] = kept
    C, ref = run()
    flag, untouched, error = int(flags.item()), bool((planes[-planes.numel() // N:][:m] == 0x7f).all()), float((C - ref).abs().max())
    assert flag == 0 and not untouched and error < 1e-9
    del ws


@pytest.mark.parametrize("n,k", [(4200, 64), (4200, 520), (4400, 520)])
@pytest.mark.parametrize("uplo", ["L", "U"])
def test_symmetric_update_with_more_than_2_24_elements(uplo, n, k):
    """Stage 3, here without the matrix cores, skips what lies in the other triangle;
    with the longer inner dimension the products take 256 x 256 tiles, 17 or 18 rows of them, of one triangle only."""
    N = 6
    rng = np.random.default_rng(3)
    A = _mat(rng, n, k)
    dA = _dev(A)
    dC = torch.full((n, n), 7.0, dtype=torch.float64, device="cuda")
    ws = oz.Workspace(n, n, k, N)
    oz.oz2_dsyrk(uplo, "N", n, k, 1.0, dA.data_ptr(), n, 0.0, dC.data_ptr(), n, N)
    torch.cuda.synchronize()
    got = dC.t().cpu().numpy()
    inside = np.tril(np.ones((n, n), bool)) if uplo == "L" else np.triu(np.ones((n, n), bool))
    assert np.all(got[~inside] == 7.0)
    rows = np.concatenate([np.arange(0, 40), np.arange(240, 280), np.arange(2030, 2070), np.arange(n - 150, n)])
    ref = orc.dgemm(A, np.asfortranarray(A.T), N, rows=rows, cols=np.arange(n)).C
    mine = inside[rows]
    assert np.array_equal(got[rows][mine], ref[mine])
    del ws


@pytest.mark.parametrize("n,k", [(7110, 64), (7110, 520), (7300, 520)])
@pytest.mark.parametrize("uplo", ["L", "U"])
def test_symmetric_update_whose_crt_runs_on_the_matrix_cores(uplo, n, k):
    """Rows and columns around the 256 x 16 blocks of the matrix-core kernel; with the longer inner dimension 256 x 256 tiles, 28 or 29
    rows of them."""
    assert _route(n, n, k, 6, call="dsyrk")[3] == 2 and _route(4400, 4400, k, 6, call="dsyrk")[3] == 1
    test_symmetric_update_with_more_than_2_24_elements(uplo, n, k)


@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 200, 256, 257, 320, 385, 600, 700])
@pytest.mark.parametrize("uplo", ["L", "U"])
def test_symmetric_update_by_small_tiles_of_one_triangle(uplo, n):
    """Even and odd numbers of rows of 64 x 64 and 128 x 128 tiles, whose triangle is launched as a rectangle."""
    k, N = 1101, 14
    rng = np.random.default_rng(n)
    A = _mat(rng, n, k)
    C0 = np.asfortranarray(rng.standard_normal((n, n)))
    dA, dC = _dev(A), _dev(C0)
    ws = oz.Workspace(n, n, k, N)
    ws.buf.fill_(0x5a)
    print("dsyrk: n=%d k=%d uplo=%s" % (n, k, uplo), flush=True)
    oz.oz2_dsyrk(uplo, "N", n, k, -1.0, dA.data_ptr(), n, 1.0, dC.data_ptr(), n, N)
    torch.cuda.synchronize()
    got = dC.cpu().numpy()
    assert np.array_equal(got, orc.dsyrk(uplo, "N", -1.0, A, 1.0, C0, N))
    del ws


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("m,n,k", [(5, 300, 12288), (5, 300, 12289), (300, 200, 12353), (700, 300, 12300), (17, 700, 12345), (33, 40, 70001),
                                   (9, 200, 10240), (9, 200, 10241)])
def test_few_long_vectors_in_the_other_shift_modes(m, n, k, mode):
    """Inner dimensions around the line from which few vectors take separate launches for maxima, norms and shifts, an
    infinity in the last place included."""
    rng = np.random.default_rng(k + m)
    ta, tb = [("N", "N"), ("T", "N"), ("N", "T"), ("T", "T")][(m + k) % 4]
    print("few long vectors: mode %d m=%d n=%d k=%d op=%s%s" % (mode, m, n, k, ta, tb), flush=True)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    opA, opB = np.asfortranarray(A.T if ta == "T" else A), np.asfortranarray(B.T if tb == "T" else B)
    dA, dB, dC = _dev(A), _dev(B), _dev(np.zeros((m, n), order="F"))
    ws = oz.Workspace(m, n, k, 14)
    flags = ws.view(oz.workspace_layout(m, n, k, 14)["flags"], 1, torch.int64)
    oz.oz2_set_shift_mode(mode)
    try:
        args = (ta, tb, m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), B.shape[0], 0.0, dC.data_ptr(), m, 14)
        oz.oz2_dgemm_ex(*args)
        torch.cuda.synchronize()
        assert int(flags.item()) == 0
        assert np.array_equal(dC.cpu().numpy(), orc.dgemm(opA, opB, 14, mode=mode).C)
        dB[-1, -1] = float("inf")
        oz.oz2_dgemm_ex(*args)
        torch.cuda.synchronize()
        assert int(flags.item()) == 1 and not torch.isfinite(dC).all()
    finally:
        oz.oz2_set_shift_mode(0)
    del ws


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("n,k,trans", [(70, 8192, "N"), (70, 8193, "T"), (300, 8200, "N"), (300, 12001, "T")])
def test_symmetric_update_of_few_long_vectors_in_the_other_shift_modes(n, k, trans, mode):
    rng = np.random.default_rng(k + n)
    A = _mat(rng, *((n, k) if trans == "N" else (k, n)))
    C0 = np.asfortranarray(rng.standard_normal((n, n)))
    print("few long vectors: dsyrk mode %d n=%d k=%d %s" % (mode, n, k, trans), flush=True)
    dA, dC = _dev(A), _dev(C0)
    ws = oz.Workspace(n, n, k, 14)
    oz.oz2_set_shift_mode(mode)
    try:
        oz.oz2_dsyrk("L", trans, n, k, 1.0, dA.data_ptr(), A.shape[0], 1.0, dC.data_ptr(), n, 14)
        torch.cuda.synchronize()
    finally:
        oz.oz2_set_shift_mode(0)
    assert np.array_equal(dC.cpu().numpy(), orc.dsyrk("L", trans, 1.0, A, 1.0, C0, 14, mode=mode))
    del ws


@pytest.mark.parametrize("thin", [1, 32, 33, 97, 128])
@pytest.mark.parametrize("ta,tb,first", [("N", "N", True), ("T", "N", True), ("N", "N", False), ("N", "T", False)])
def test_thin_products_convert_the_large_operand_on_the_way(thin, ta, tb, first):
    """A large operand of ragged extents against few vectors of the other one (oz2_thin.hip), either side, either orientation,
    whole and partial groups of moduli, elements split one and two levels deep."""
    large, k = 12337, 1101
    N = {1: 16, 32: 15, 33: 24, 97: 8, 128: 23}[thin]
    m, n = (large, thin) if first else (thin, large)
    assert _choice(m, n, k, N)[1] == (1 if first else 2)
    rng = np.random.default_rng(thin)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    print("thin: m=%d n=%d k=%d N=%d op=%s%s" % (m, n, k, N, ta, tb), flush=True)
    dA, dB = _dev(A), _dev(B)
    dC = torch.full((n, m), 5.0, dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    oz.oz2_dgemm_ex(ta, tb, m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), B.shape[0], 0.0, dC.data_ptr(), m, N)
    torch.cuda.synchronize()
    got = dC.t().cpu().numpy()
    opA, opB = np.asfortranarray(A.T if ta == "T" else A), np.asfortranarray(B.T if tb == "T" else B)
    pick = np.unique(np.concatenate([np.arange(70), np.arange(large - 90, large), rng.integers(0, large, 60)]))
    rows, cols = (pick, np.arange(n)) if first else (np.arange(m), pick)
    ref = orc.dgemm(opA, opB, N, rows=rows, cols=cols).C
    assert np.array_equal(got[np.ix_(rows, cols)], ref)
    # and every element against the products formed through planes (the staged calls)
    dD = torch.empty((n, m), dtype=torch.float64, device="cuda")
    if ta == "N" and tb == "N":
        oz.oz2_stage1_convert(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, N)
        oz.oz2_stage2_gemm(m, n, k, N)
        oz.oz2_stage3_crt(m, n, k, dD.data_ptr(), m, N)
        torch.cuda.synchronize()
        assert torch.equal(dC, dD)
    # an infinity in the large operand's last vector reaches the fallback
    if first and ta == "N":
        A[m - 1, k - 1] = np.inf
        dA = _dev(A)
        oz.oz2_dgemm_ex(ta, tb, m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), B.shape[0], 0.0, dC.data_ptr(), m, N)
        torch.cuda.synchronize()
        got = dC.t().cpu().numpy()
        assert np.all(np.isinf(got[m - 1])) and np.all(np.isfinite(got[:m - 1]))
    del ws


@pytest.mark.parametrize("side,uplo,ta", [(s, u, t) for s in "LR" for u in "LU" for t in "NT"])
def test_triangular_operand_of_which_only_the_used_half_is_converted(side, uplo, ta):
    """Orders above the one-pass conversion's 1024: scan and conversion walk only the blocks that the products read.  The
    workspace is full of other bytes beforehand, and the array's other triangle of NaNs."""
    order, other, N = 1300, 70, 9
    m, n = (order, other) if side == "L" else (other, order)
    rng = np.random.default_rng(order + len(side + uplo + ta) + ord(side) + ord(uplo) + ord(ta))
    A, B = _mat(rng, order, order), _mat(rng, m, n)
    keep = np.tril(np.ones((order, order), bool)) if uplo == "L" else np.triu(np.ones((order, order), bool))
    A[~keep] = np.nan
    print("dtrmm: %s%s%s order %d" % (side, uplo, ta, order), flush=True)
    dA, dB = _dev(A), _dev(B)
    ws = oz.Workspace(m, n, order, N)
    ws.buf.fill_(0x7f)
    oz.oz2_dtrmm(side, uplo, ta, "N", m, n, 1.0, dA.data_ptr(), order, dB.data_ptr(), m, N)
    torch.cuda.synchronize()
    assert np.array_equal(dB.cpu().numpy(), orc.dtrmm(side, uplo, ta, "N", 1.0, A, B, N))
    del ws


@pytest.mark.parametrize("k", [1025, 1088, 1120, 1152, 1153, 1216, 1279])
@pytest.mark.parametrize("ta", ["N", "T"])
def test_thin_products_at_the_ends_of_the_inner_dimension(k, ta):
    """Even and odd numbers of k-tiles, the last one whole or not: the loop takes two at a time."""
    m, n, N = 12337, 40, 16
    assert _choice(m, n, k, N)[1] == 1
    rng = np.random.default_rng(k)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, k, n)
    print("thin: m=%d n=%d k=%d N=%d op=%s" % (m, n, k, N, ta), flush=True)
    dA, dB = _dev(A), _dev(B)
    dC = torch.full((n, m), 5.0, dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    oz.oz2_dgemm_ex(ta, "N", m, n, k, 1.0, dA.data_ptr(), A.shape[0], dB.data_ptr(), k, 0.0, dC.data_ptr(), m, N)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(70), np.arange(m - 70, m), rng.integers(0, m, 40)]))
    opA = np.asfortranarray(A.T if ta == "T" else A)
    assert np.array_equal(dC.t().cpu().numpy()[rows], orc.dgemm(opA, B, N, rows=rows, cols=np.arange(n)).C)
    del ws


@pytest.mark.parametrize("k", [1025, 1089, 1153, 1217, 1281, 1344])
@pytest.mark.parametrize("large,thin,N,first", [(5003, 20, 16, True), (5003, 32, 15, False), (5003, 96, 16, True), (7003, 70, 13, False),
                                                (5003, 31, 23, True), (5003, 90, 24, False)])
def test_thin_products_two_k_tiles_at_a_time(large, thin, N, first, k):
    """One and three 32-vector tiles of the thin operand with at most one workgroup per compute unit, elements split one and two levels
    deep, every remainder of the number of k-tiles that the loop's rounds and its last fetches can meet."""
    m, n = (large, thin) if first else (thin, large)
    assert _choice(m, n, k, N)[1] == (1 if first else 2)
    rng = np.random.default_rng(thin + k)
    A, B = _mat(rng, m, k), _mat(rng, k, n)
    print("thin pairs: m=%d n=%d k=%d N=%d" % (m, n, k, N), flush=True)
    dA, dB = _dev(A), _dev(B)
    dC = torch.full((n, m), 5.0, dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, N)
    oz.oz2_dgemm(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, dC.data_ptr(), m, N)
    torch.cuda.synchronize()
    pick = np.unique(np.concatenate([np.arange(66), np.arange(large - 70, large), rng.integers(0, large, 40)]))
    rows, cols = (pick, np.arange(n)) if first else (np.arange(m), pick)
    assert np.array_equal(dC.t().cpu().numpy()[np.ix_(rows, cols)], orc.dgemm(A, B, N, rows=rows, cols=cols).C)
    del ws


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("mode,delta,N,k,ta,tb", [(1, 0, 16, 1101, "N", "T"), (2, 0, 16, 1101, "T", "N"), (1, 0, 16, 3000, "T", "T"),
                                                  (2, 0, 15, 3000, "N", "N"), (0, 30, 21, 1101, "N", "N"), (0, -30, 21, 3000, "T", "N"),
                                                  (1, 25, 21, 3000, "N", "N"), (2, -25, 21, 1101, "N", "T"), (0, 0, 16, 3000, "N", "T")])
def test_thin_products_under_the_other_settings(mode, delta, N, k, ta, tb, first):
    """The shift modes of Section 4.1, bit splits of which one operand needs the two-level split and the other does not, an update
    of C with leading dimensions of its own, and operands beyond the 2^25 elements up to which one launch finds the shifts."""
    large, thin = 12337, 40
    m, n = (large, thin) if first else (thin, large)
    rng = np.random.default_rng(100 * N + mode + k)
    A = _mat(rng, *((m, k) if ta == "N" else (k, m)))
    B = _mat(rng, *((k, n) if tb == "N" else (n, k)))
    print("thin: mode %d split %d m=%d n=%d k=%d N=%d op=%s%s" % (mode, delta, m, n, k, N, ta, tb), flush=True)

    def padded(x, more):  # column-major with `more` unused rows of NaN below each column
        buf = torch.full((x.shape[1], x.shape[0] + more), float("nan"), dtype=torch.float64, device="cuda")
        buf[:, :x.shape[0]] = torch.from_numpy(np.ascontiguousarray(x.T)).cuda()
        return buf

    dA, dB = padded(A, 3), padded(B, 2)
    C0 = np.asfortranarray(rng.standard_normal((m, n)))
    dC = padded(C0, 1)
    ws = oz.Workspace(m, n, k, N)
    lay = oz.workspace_layout(m, n, k, N)
    ws.buf.fill_(0x7f)
    pad = lay["m_pad"] if first else lay["n_pad"]
    second_plane = ws.view(lay["a_planes" if first else "b_planes"] + pad * lay["k_pad"], pad * lay["k_pad"], torch.uint8)
    oz.oz2_set_shift_mode(mode)
    oz.oz2_set_bit_split(delta)
    try:
        oz.oz2_dgemm_ex(ta, tb, m, n, k, -0.5, dA.data_ptr(), dA.shape[1], dB.data_ptr(), dB.shape[1], 2.0, dC.data_ptr(), m + 1, N)
        torch.cuda.synchronize()
    finally:
        oz.oz2_set_bit_split(0)
        oz.oz2_set_shift_mode(0)
    untouched = bool((second_plane == 0x7f).all())
    assert untouched  # the large operand was converted on the way, its planes were not written
    got = dC[:, :m].t().cpu().numpy()
    assert bool(torch.isnan(dC[:, m]).all())
    opA, opB = np.asfortranarray(A.T if ta == "T" else A), np.asfortranarray(B.T if tb == "T" else B)
    pick = np.unique(np.concatenate([np.arange(66), np.arange(large - 70, large), rng.integers(0, large, 40)]))
    rows, cols = (pick, np.arange(n)) if first else (np.arange(m), pick)
    P = orc.dgemm(opA, opB, N, rows=rows, cols=cols, mode=mode, delta=delta).C
    sub = C0[np.ix_(rows, cols)]
    # alpha is a power of two and beta doubles: fma(alpha, P, beta C) rounds alpha P + beta C once, as this sum does
    assert np.array_equal(got[np.ix_(rows, cols)], -0.5 * P + 2.0 * sub)
    del ws


@pytest.mark.parametrize("mode,k", [(0, 2500), (0, 4928), (1, 4929), (0, 9920), (2, 9919)])
def test_many_long_contiguous_vectors_in_one_pass(mode, k):
    """More elements than the last-level cache keeps, in contiguous vectors: one pass.  The same operands stored the other way round take
    the separate launches; every bit of C is the same, with an infinity too."""
    m, N = 300, 4
    n = ((19 << 20) // k // 256 + 1) * 256 - 3
    gen = torch.Generator(device="cuda").manual_seed(k)
    At = torch.randn((m, k), dtype=torch.float64, device="cuda", generator=gen)  # columns of the stored k x m matrix: rows of op(A)
    B = torch.randn((n, k), dtype=torch.float64, device="cuda", generator=gen)
    A, Bt = At.t().contiguous(), B.t().contiguous()
    ctx = oz.Context()
    ctx.set(oz.OZ2_OPT_SHIFT_MODE, mode)
    ctx.allocate_workspace(m, n, k, N, device="cuda:0")
    for infinity in (False, True):
        print("one pass over long vectors: k=%d n=%d mode=%d infinity=%d" % (k, n, mode, infinity), flush=True)
        if infinity:
            B[7, k - 1] = Bt[k - 1, 7] = float("inf")
        C1, C2 = (torch.zeros((n, m), dtype=torch.float64, device="cuda") for _ in range(2))
        ctx.dgemm("T", "N", m, n, k, 1.0, At.data_ptr(), k, B.data_ptr(), k, 0.0, C1.data_ptr(), m, N)
        ctx.dgemm("N", "T", m, n, k, 1.0, A.data_ptr(), m, Bt.data_ptr(), n, 0.0, C2.data_ptr(), m, N)
        torch.cuda.synchronize()
        assert bool(torch.isinf(C1).any()) == infinity
        assert torch.equal(C1.view(torch.int64), C2.view(torch.int64))


@pytest.mark.parametrize("mode,k", [(0, 2500), (0, 4928), (1, 4929), (0, 9920), (2, 9919)])
def test_many_long_contiguous_vectors_take_the_one_pass(mode, k):
    """The routes of the test above: one pass with contiguous vectors, separate launches with the others."""
    n = ((19 << 20) // k // 256 + 1) * 256 - 3
    oz.oz2_set_shift_mode(mode)
    try:
        assert _route(300, n, k, 4, "T", "N")[0] == 3 and _route(300, n, k, 4, "N", "T")[0] == 0
    finally:
        oz.oz2_set_shift_mode(oz.OZ2_SHIFT_MAX)


@pytest.mark.parametrize("m,n,k", [(3200, 3000, 4928), (3000, 2900, 4929), (2600, 2500, 9920), (9000, 5000, 2500)])
def test_one_operand_in_one_pass_and_the_other_in_two(m, n, k):
    """Strided vectors of one operand, contiguous ones of the other, more elements than the last-level cache keeps: bit for bit what the
    operands give stored the other way round, with an infinity in either of them too."""
    N = 4
    gen = torch.Generator(device="cuda").manual_seed(k)
    A = torch.randn((k, m), dtype=torch.float64, device="cuda", generator=gen)
    B = torch.randn((n, k), dtype=torch.float64, device="cuda", generator=gen)
    assert (m + n) * k > 190 << 17 and m + n >= 20 * 250
    ctx = oz.Context()
    ctx.allocate_workspace(m, n, k, N, device="cuda:0")
    for infinite in ("none", "A", "B"):
        print("one operand in one pass: m=%d n=%d k=%d infinite=%s" % (m, n, k, infinite), flush=True)
        X, Y = A.clone(), B.clone()
        if infinite == "A":
            X[k - 1, m - 1] = float("inf")
        if infinite == "B":
            Y[n - 1, 0] = float("-inf")
        got = []
        for ta, tb in (("N", "N"), ("T", "T"), ("T", "N")):
            x, y = (X if ta == "N" else X.t().contiguous()), (Y if tb == "N" else Y.t().contiguous())
            C = torch.zeros((n, m), dtype=torch.float64, device="cuda")
            ctx.dgemm(ta, tb, m, n, k, 1.0, x.data_ptr(), x.shape[1], y.data_ptr(), y.shape[1], 0.0, C.data_ptr(), m, N)
            torch.cuda.synchronize()
            got.append(C)
        assert bool(torch.isinf(got[0]).any()) == (infinite != "none")
        assert all(torch.equal(got[0].view(torch.int64), c.view(torch.int64)) for c in got[1:])


@pytest.mark.parametrize("m,n,k,alone", [(3200, 3000, 4928, [2, 1]), (3000, 2900, 4929, [2, 1]), (2600, 2500, 9920, [2, 1]), (9000, 5000, 2500, [2, 1]),
                                         (3500, 2500, 9911, [0, 1])])
def test_the_operand_that_takes_the_one_pass(m, n, k, alone):
    """The routes of the test above; and, of the longest vectors, strided ones that are not whole cache lines by sixteens, which do not
    take that route."""
    assert [_route(m, n, k, 4, ta, tb)[0] for ta, tb in (("N", "N"), ("T", "T"), ("T", "N"))] == alone + [3]
    if 0 in alone:
        test_one_operand_in_one_pass_and_the_other_in_two(m, n, k)

"""Residues that the GEMM epilogues leave (Algorithm 1 lines 6-7), all moduli.

Rows of A' and columns of B' are constant, so element (i, j) of C' is k a_i b_j exactly.  The first test covers one to five k-tiles,
reductions between blocks of one k-tile, and an inner dimension of 65536, of which the epilogue sees what a reduction after
61440 terms leaves and 4096 terms more; the others the longest sums that an epilogue can see, 61440 terms of 128 * 128 and
-128 * 127, in each of the kernels.  Planes are written into the workspace directly; whole numbers, no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2504_08009_amd as oz
from oracle import oracle as orc

N = 26


def _fill(ws, lay, name, rows_pad, vals, k):
    """plane t, row r, inner positions below k: vals[t][r]; the rest zero"""
    kp = lay["k_pad"]
    v = ws.view(lay[name], N * rows_pad * kp, torch.int8).view(N, rows_pad // 256, kp // 64, 256, 64)
    v.zero_()
    d = torch.from_numpy(vals).to(v.device)  # N x rows_pad
    for b in range((k + 63) // 64):
        n = min(64, k - 64 * b)
        v[:, :, b, :, :n] = d.view(N, rows_pad // 256, 256, 1)


@pytest.mark.parametrize("kblock", [65536, 64])
@pytest.mark.parametrize("k", [1, 64, 65, 192, 260, 65536])
def test_residues_of_products_over_the_int32_range(k, kblock):
    if kblock < 65536 and k not in (65, 260):
        pytest.skip("reduction between k-blocks: two depths are enough")
    mods, _ = oz.get_moduli(N)
    m, n = 256, 512
    print("epilogue: k=%d kblock=%d" % (k, kblock), flush=True)
    ws = oz.Workspace(m, n, k, N, product_format=oz.OZ2_PRODUCT_RESIDUE_U8)
    lay = oz.workspace_layout(m, n, k, N)
    lo = np.array([-(p // 2) for p in mods])
    hi = np.array([(p - 1) // 2 for p in mods])
    rng = np.random.default_rng(k)
    a = np.clip(np.arange(m)[None, :] - 128, lo[:, None], hi[:, None]).astype(np.int8)
    b = np.clip(np.concatenate([np.arange(256) - 128, rng.integers(-128, 128, 256)])[None, :], lo[:, None],
                hi[:, None]).astype(np.int8)
    _fill(ws, lay, "a_planes", lay["m_pad"], a, k)
    _fill(ws, lay, "b_planes", lay["n_pad"], b, k)
    oz.oz2_set_kblock(kblock)
    try:
        oz.oz2_stage2_gemm(m, n, k, N)
    finally:
        oz.oz2_set_kblock(65536)
    torch.cuda.synchronize()
    got = ws.view(lay["c_planes"], N * lay["n_pad"] * lay["m_pad"], torch.uint8).view(N, lay["n_pad"], lay["m_pad"])
    got = got[:, :n, :m].cpu().numpy()
    for t, p in enumerate(mods):
        ref = (k * b[t].astype(np.int64)[:, None] * a[t].astype(np.int64)[None, :]) % p
        assert np.array_equal(got[t], ref), "modulus %d" % p


@pytest.mark.parametrize("k", [34960, 49416, 61440])
@pytest.mark.parametrize("m,n", [(128, 128), (256, 512), (768, 768)])
def test_residues_of_the_longest_sums_without_a_reduction(m, n, k):
    """Up to 61440 terms reach the epilogue as one sum (up to 2^30 - 2^26).  The three results take the 64 x 64, the 128 x 128
    and the 256 x 256 tiles of the products."""
    mods, _ = oz.get_moduli(N)
    print("longest sums: m=%d n=%d k=%d" % (m, n, k), flush=True)
    ws = oz.Workspace(m, n, k, N, product_format=oz.OZ2_PRODUCT_RESIDUE_U8)
    lay = oz.workspace_layout(m, n, k, N)
    lo = np.array([-(p // 2) for p in mods])
    hi = np.array([(p - 1) // 2 for p in mods])
    rng = np.random.default_rng(k + m)

    def vectors(count):
        # (120 x -122 over 49416 terms modulo 255: one of the smallest byte sums there is)
        v = np.concatenate([[120, -122, 127, -127, -128, 126, -126, 1], rng.permutation(256) - 128, rng.integers(-128, 128, count)])
        return np.clip(v[None, :count], lo[:, None], hi[:, None]).astype(np.int8)

    a, b = vectors(lay["m_pad"]), vectors(lay["n_pad"])
    _fill(ws, lay, "a_planes", lay["m_pad"], a, k)
    _fill(ws, lay, "b_planes", lay["n_pad"], b, k)
    oz.oz2_stage2_gemm(m, n, k, N)
    torch.cuda.synchronize()
    got = ws.view(lay["c_planes"], N * lay["n_pad"] * lay["m_pad"], torch.uint8).view(N, lay["n_pad"], lay["m_pad"])
    got = got[:, :n, :m].cpu().numpy()
    for t, p in enumerate(mods):
        ref = (k * b[t, :n].astype(np.int64)[:, None] * a[t, :m].astype(np.int64)[None, :]) % p
        assert np.array_equal(got[t], ref), "modulus %d" % p
    del ws


@pytest.mark.parametrize("first", [True, False])
def test_thin_products_of_the_longest_sums(first):
    """Constant vectors of whole numbers with the residues 120, -122 ... modulo 255, long enough for sums near the INT32 limit, a
    large operand against few vectors (oz2_thin.hip).  Every product is k a b, known as a Python integer."""
    large, thin, k, moduli = 8192, 20, 49416, 14
    _, kappa = oz.get_moduli(moduli, k)
    rng = np.random.default_rng(11)
    wanted = [120, -122, 127, -127, 126, -126, 1, 0]

    def numbers(count):  # kappa bits each: the shifts are zero and nothing is truncated
        v = 2 ** (kappa - 1) + 255 + rng.integers(0, 2 ** (kappa - 2), count)
        r = np.array([wanted[i % 8] for i in range(count)])
        return [int(x) for x in v - (v - r) % 255]

    va, vb = numbers(large), numbers(thin)
    assert all(2 ** (kappa - 1) <= x < 2**kappa for x in va + vb)
    print("thin longest sums: first=%s" % first, flush=True)
    dl = torch.tensor(va, dtype=torch.float64, device="cuda")
    dt = torch.tensor(vb, dtype=torch.float64, device="cuda")
    if first:  # A: large x k column-major, B: k x thin
        A, B = dl.expand(k, large).contiguous(), dt[:, None].expand(thin, k).contiguous()
        m, n = large, thin
    else:
        A, B = dt.expand(k, thin).contiguous(), dl[:, None].expand(large, k).contiguous()
        m, n = thin, large
    dC = torch.empty((n, m), dtype=torch.float64, device="cuda")
    ws = oz.Workspace(m, n, k, moduli)
    oz.oz2_dgemm(m, n, k, A.data_ptr(), m, B.data_ptr(), k, dC.data_ptr(), m, moduli)
    torch.cuda.synchronize()
    got = dC.cpu().numpy()
    ref = np.array([[float(k * x * y) for x in va] for y in vb])
    assert np.array_equal(got if first else got.T, ref)
    del ws


@pytest.mark.parametrize("m,n,N,k,int32", [(2299, 2227, 12, k, True) for k in [1, 64, 65, 130, 193, 257, 321, 400, 513]] +
                         [(2047, 2040, 4, k, False) for k in [1, 64]] + [(2047, 2040, 8, k, False) for k in [65, 128, 130, 192]] +
                         [(2299, 2227, 12, k, False) for k in [193, 257, 321, 400, 513]])
def test_large_tiles_with_few_k_tiles_several_per_workgroup(m, n, N, k, int32):
    """The main loop of the large tiles, whose ring has four stages, on inner dimensions of one k-tile to nine, more tiles than compute
    units, both result formats, ragged last tiles.  With UINT8 residues two or three k-tiles take the large tiles at two per workgroup, a
    single one only where each workgroup has one tile."""
    rng = np.random.default_rng(k)
    print("large tiles: m=%d n=%d k=%d N=%d int32=%s" % (m, n, k, N, int32), flush=True)
    A = np.asfortranarray(rng.standard_normal((m, k)))
    B = np.asfortranarray(rng.standard_normal((k, n)))
    dA = torch.from_numpy(np.ascontiguousarray(A.T)).cuda().t()
    dB = torch.from_numpy(np.ascontiguousarray(B.T)).cuda().t()
    dC = torch.zeros((n, m), dtype=torch.float64, device="cuda")
    oz.oz2_set_product_format(oz.OZ2_PRODUCT_INT32 if int32 else oz.OZ2_PRODUCT_RESIDUE_U8)
    try:
        assert oz.host_kernel_choice(m, n, k, N, torch.cuda.get_device_properties(0).multi_processor_count)[2] == 256
        ws = oz.Workspace(m, n, k, N)
        oz.oz2_dgemm(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k, dC.data_ptr(), m, N)
        torch.cuda.synchronize()
    finally:
        oz.oz2_set_product_format(oz.OZ2_PRODUCT_RESIDUE_U8)
    rows = [r for r in [0, 15, 16, 127, 128, 255, 256, 1111, 1792, 2046, 2047, 2048, m - 1] if r < m]
    got = dC.t()[rows].cpu().numpy()
    assert np.array_equal(got, orc.dgemm(A, B, N, rows=rows).C)
    del ws


@pytest.mark.parametrize("m,n", [(1024, 1000), (2048, 2040)])
@pytest.mark.parametrize("k", [64, 512, 1023, 1024, 1025])
def test_residues_of_short_sums_in_large_tiles(m, n, k):
    """Up to 1024 terms the large tiles take the residue from one product with 2^32 / p rounded, whose error grows with the sum: all
    products of all residues, -128 * -128 included, stored through the caches and past them; the first longer sum too."""
    mods, _ = oz.get_moduli(N)
    print("short sums: m=%d n=%d k=%d" % (m, n, k), flush=True)
    ws = oz.Workspace(m, n, k, N, product_format=oz.OZ2_PRODUCT_RESIDUE_U8)
    lay = oz.workspace_layout(m, n, k, N)
    if k >= 512:
        assert oz.host_kernel_choice(m, n, k, N, torch.cuda.get_device_properties(0).multi_processor_count)[2] == 256
    lo = np.array([-(p // 2) for p in mods])
    hi = np.array([(p - 1) // 2 for p in mods])
    a = np.clip((np.arange(lay["m_pad"]) % 256 - 128)[None, :], lo[:, None], hi[:, None]).astype(np.int8)
    b = np.clip((np.arange(lay["n_pad"]) * 85 // 256 % 256 - 128)[None, :], lo[:, None], hi[:, None]).astype(np.int8)
    b[:, :256] = np.clip((np.arange(256) - 128)[None, :], lo[:, None], hi[:, None])
    _fill(ws, lay, "a_planes", lay["m_pad"], a, k)
    _fill(ws, lay, "b_planes", lay["n_pad"], b, k)
    oz.oz2_stage2_gemm(m, n, k, N)
    torch.cuda.synchronize()
    got = ws.view(lay["c_planes"], N * lay["n_pad"] * lay["m_pad"], torch.uint8).view(N, lay["n_pad"], lay["m_pad"])
    for t, p in enumerate(mods):
        at, bt = (torch.from_numpy(v[t].astype(np.int64)).cuda() for v in (a, b))
        ref = torch.remainder(k * bt[:n, None] * at[None, :m], p).to(torch.uint8)
        assert torch.equal(got[t, :n, :m], ref), "modulus %d" % p

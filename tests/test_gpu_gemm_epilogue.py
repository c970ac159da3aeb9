"""Residues that the GEMM epilogue leaves (Algorithm 1 lines 6-7) for products over the whole INT32 range, all moduli.

Rows of A' and columns of B' are constant, so element (i, j) of C' is k a_i b_j exactly: from 0 to the extremes of
65536 terms of 128 * 128 and -128 * 127.  Planes are written into the workspace directly; whole numbers, no tolerance."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_2504_08009_amd as oz

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

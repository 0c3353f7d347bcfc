"""H.V on block rows at the edges of the adjacent-column and one-lane kernels:
ragged column counts (the last lanes of a group move back and share columns),
every lane count, leading dimensions above nvec, inputs one element off a wide
word, targets in the last representatives (rows beyond n_Gamma would lie past
the array) and representatives with fewer than d_Gamma rows.  Against the
oracle; the lane layouts bit for bit against each other."""
import numpy as np
import pytest

from gpu_helpers import lib_block, oracle_block, oracle_sector, rel_err_cols
from oracle import hv

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2607_17429_amd")

TOL = {"float64": 1e-12, "float32": 2e-7, "float16": 2.0 ** -11 + 2.0 ** -24}
CASES = [  # (cluster, 2s, 2M, irrep): d = 1, 2, 3, 4, 5, 6, 8; tiny, small and larger sectors
    ("icosahedron", 1, 0, 0), ("cuboctahedron", 2, 0, 4), ("icosahedron", 1, 2, 3), ("dodecahedron", 1, 4, 6),
    ("dodecahedron", 1, 0, 8), ("petersen", 3, 0, 6), ("square4x4", 1, 0, 19), ("square6x6", 1, 28, 12),
]


@pytest.mark.parametrize("dtype", ["float64", "float32", "float16"])
@pytest.mark.parametrize("name,two_s,two_M,gi", CASES)
def test_block_rows(name, two_s, two_M, gi, dtype):
    _, H = oracle_sector(name, two_s, two_M)
    B = oracle_block(name, two_s, two_M, gi)
    LB = lib_block(name, two_s, two_M, gi)
    rng = np.random.default_rng(11)
    for nvec, ld, skew in ((1, 1, 0), (1, 3, 0), (2, 2, 1), (3, 3, 0), (4, 4, 1), (4, 6, 0), (5, 5, 0), (7, 7, 1), (13, 13, 0),
                           (24, 24, 0), (24, 27, 1), (25, 25, 0), (70, 70, 0)):
        X = rng.standard_normal((B.D, nvec)).astype(dtype)
        buf = torch.full((B.D * ld + 8,), float("nan"), dtype=getattr(torch, dtype), device="cuda")
        Xt = buf[skew:skew + B.D * ld].view(B.D, ld)[:, :nvec]
        Xt.copy_(torch.from_numpy(X))
        out = torch.full((B.D, ld), 7.0, dtype=Xt.dtype, device="cuda")
        Y = LB.apply_H(Xt, out[:, :nvec])
        assert rel_err_cols(Y.cpu().numpy(), hv.apply(B, H, X.astype(np.float64))) <= TOL[dtype], (nvec, ld)
        assert torch.all(out[:, nvec:] == 7.0)
        for lanes in (1, 2, 4, 8, 16, 64):
            if lanes * 8 < nvec and nvec <= 64:
                continue
            Yl, _ = LB.apply_H_ex(Xt, torch.zeros_like(out)[:, :nvec], layout=P.LAYOUT_BLOCK, lanes=lanes)
            assert torch.equal(Yl, Y), (nvec, ld, lanes)
        # the epilogue's sums count every column once
        sb = torch.tensor([[1.0, 0.0]] * nvec, dtype=torch.float64, device="cuda")
        dots = torch.full((nvec,), float("nan"), dtype=torch.float64, device="cuda")
        Ye, _ = LB.apply_H_ex(Xt, torch.zeros_like(out)[:, :nvec], layout=P.LAYOUT_BLOCK, scale=sb, dots=dots)
        p = Xt.double() * Ye.double()
        assert torch.all((dots - p.sum(0)).abs() <= 1e-12 * p.abs().sum(0) + 1e-300)


@pytest.mark.parametrize("name,two_M,irrep", [("ring20_C", 0, 3), ("ring20_C", 2, 10), ("ring20_C", 4, 1), ("icosahedron", 12, 0),
                                              ("dodecahedron", 0, 9), ("ring20_C", 16, 2)])
def test_row_offsets(name, two_M, irrep):
    """Row offsets built by one workgroup (up to 8,192 representatives) and by
    the scan (above), sectors of 1 to 9,252: the exported offsets are the
    prefix sums of n_Gamma, and a product that finds its targets through them
    equals the padded-row product, whose targets need none, bit for bit."""
    from synth import clusters
    cl = clusters.get(name)
    B = P.Block(P.Sector(cl, P.Group(cl.N, cl.gens), two_M, two_s=1), irrep)
    ex = B.export()
    n = ex["n_gamma"].astype(np.int64)
    live = n > 0
    assert np.array_equal(ex["offsets"].astype(np.int64)[live], (np.cumsum(n) - n)[live]) and n.sum() == B.D
    rows = np.concatenate([i * B.d_gamma + np.arange(n[i]) for i in np.nonzero(live)[0]])
    X = torch.from_numpy(np.random.default_rng(2).standard_normal((B.D, 3))).cuda()
    Xp = torch.zeros((B.D_pad, 3), dtype=torch.float64, device="cuda")
    Xp[torch.from_numpy(rows).cuda()] = X
    Yp, _ = B.apply_H_ex(Xp, layout=P.LAYOUT_PADDED)
    assert torch.equal(B.apply_H(X), Yp[torch.from_numpy(rows).cuda()])

"""The autotuner against the default lane layout: the default is among the
layouts timed (small sectors take more lanes than columns), and it stays
unless another one is clearly faster."""
import numpy as np
import pytest

from synth import clusters

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2607_17429_amd")


def block(name, two_M, irrep):
    cl = clusters.get(name)
    return P.Block(P.Sector(cl, P.Group(cl.N, cl.gens), two_M, two_s=1), irrep)


def lanes_used(B, nvec, layout=None):
    """Lanes of the launch that Lanczos runs make (epilogue) on block B."""
    X = torch.ones((B.D, nvec), dtype=torch.float64, device="cuda")
    sb = torch.ones((nvec, 2), dtype=torch.float64, device="cuda")
    return B.apply_H_ex(X, layout=P.LAYOUT_BLOCK, scale=sb)[1]["lanes_used"]


@pytest.mark.parametrize("name,two_M,irrep,nvec", [("icosahedron", 0, 3, 1), ("dodecahedron", 0, 8, 1), ("dodecahedron", 0, 8, 24),
                                                   ("ring20_C", 0, 1, 2), ("ring20_C", 0, 0, 13), ("square6x6", 30, 12, 3)])
def test_default_is_timed_and_not_lost(name, two_M, irrep, nvec):
    B = block(name, two_M, irrep)
    P.autotune_clear()
    default = lanes_used(B, nvec)
    best, ms, tried = B.autotune(nvec, P.F64)
    P.autotune_clear()
    assert default in tried and tried[best] == ms
    assert ms <= tried[default]


def test_tuned_lanes_stay_in_their_size_class(tmp_path):
    """Lanes tuned on a small sector are not taken in a larger one of the same
    cluster, nor are those of a file without kernel generation and size."""
    small, large = block("ring20_C", 14, 0), block("ring20_C", 0, 0)
    P.autotune_clear()
    want = {id(b): lanes_used(b, 1) for b in (small, large)}
    best, _, _ = small.autotune(1, P.F64)
    assert lanes_used(large, 1) == want[id(large)] != want[id(small)]
    f = tmp_path / "tune.txt"
    n = P.autotune_save(f)
    lines = f.read_text().split("\n")[:-1]
    # an odd choice under the same key is used, the same line without its last two fields is not
    odd = [" ".join(ln.split()[:11] + ["4"] + ln.split()[12:]) for ln in lines]
    for text, lanes in ((odd, 4), ([" ".join(ln.split()[:12]) for ln in odd], want[id(small)])):
        P.autotune_clear()
        f.write_text("\n".join(text) + "\n")
        assert P.autotune_load(f) == n
        assert lanes_used(small, 1) == lanes
        assert P.autotune_save(f) == n and sorted(f.read_text().split("\n")[:-1]) == sorted(text)
    P.autotune_clear()

"""The orbit search's candidate sets at the sizes where they can go wrong: set
words (groups of 120, 288 and 720 elements), bits per site (1, 2, 3), sites
beyond a multiple of four, a group that does not move every site to every
other, the spin flip, sectors of one word and of several workgroups.  All
integer data: bit for bit against the oracle."""
import numpy as np
import pytest

from oracle import basis, group
from oracle.spinflip import FlipGroup
from synth import clusters

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2607_17429_amd")

CASES = [  # (cluster, generators kept, 2s, 2M, spin flip)
    ("K6", None, 1, 0, False), ("K6", None, 4, 2, False), ("K6", None, 2, 0, True), ("square6x6", None, 1, 30, False),
    ("petersen", None, 3, 4, False), ("icosahedron", [2], 1, 0, True), ("icosahedron", [0], 2, 4, False),
    ("ring7", None, 5, 7, False), ("dodecahedron", None, 1, 0, True), ("ring18", [0], 1, 0, False),
]


@pytest.mark.parametrize("name,keep,two_s,two_M,flip", CASES)
def test_orbit_search(name, keep, two_s, two_M, flip):
    cl = clusters.get(name)
    gens = cl.gens if keep is None else cl.gens[keep]
    G = group.close(gens, cl.N)
    OG = FlipGroup(G) if flip else G
    sec = basis.sector_reps(OG, cl.N, two_s, two_M)
    LG = P.Group(cl.N, gens)
    S = P.Sector(cl, LG, two_M, two_s=two_s, spin_flip=flip)
    reps, sid, ssz = S.export()
    assert np.array_equal(reps.astype(np.int64), sec.reps)
    assert np.array_equal(sid.astype(np.int64), sec.stab_id)
    assert [len(s) for s in sec.stab_sets] == list(ssz)
    labs = sec.labels[:: max(1, len(sec.labels) // 3000)]
    rep, h, idx = (t.cpu().numpy() for t in S.canonicalize(torch.from_numpy(labs.astype(np.int64)).cuda()))
    orep, oh = basis.canonicalize(OG, labs, cl.N, two_s + 1)
    assert np.array_equal(rep, orep) and np.array_equal(h, oh)
    assert np.array_equal(idx, np.searchsorted(sec.reps, orep))
    # entries (listed flips, one lane each) and flips found inside the product agree bit for bit
    O = P.Sector(cl, LG, two_M, two_s=two_s, spin_flip=flip, hv_mode=P.HV_ONTHEFLY)
    B, BO = P.Block(S, 0), P.Block(O, 0)
    X = torch.from_numpy(np.random.default_rng(3).standard_normal((B.D, 5))).cuda()
    assert torch.equal(B.apply_H(X), BO.apply_H(X))

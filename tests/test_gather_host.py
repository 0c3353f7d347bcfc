"""Addresses of the H.V gathers, on the host (no GPU): the kernels' own load
arithmetic, built into a host program from the library's header, over the
n_Gamma of the oracle's blocks.  No lane of any variant, column count, leading
dimension, lane count or row layout may load outside the vector: targets in
the last rows, representatives with fewer than d_Gamma rows (blocks of fewer
rows than d_Gamma among them), and flips without a term (a target with no
rows, the padding of the one-lane kernel), which are gathered as well.  The
fused Lanczos kernel runs the same gathers on vectors of exactly D x R."""
import functools
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import basis, group, irreps
from synth import clusters

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")

CASES = [  # (cluster, 2s, 2M): d = 1 .. 6 and 8; the 2M with few states have blocks of D < d_Gamma
    ("icosahedron", 1, 0), ("icosahedron", 1, 8), ("icosahedron", 1, 12), ("icosahedron", 2, 20),
    ("cuboctahedron", 2, 18), ("cuboctahedron", 3, 30), ("square4x4", 1, 8), ("square4x4", 1, 12), ("petersen", 3, 20),
    ("dodecahedron", 1, 14), ("square6x6", 1, 32),
]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("gather") / "gather_rows")
    subprocess.run([HIPCC, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2607_17429_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "gather_rows.cpp"), "-o", exe], check=True, timeout=300)
    return exe


@functools.lru_cache(maxsize=None)
def symmetry(name):
    cl = clusters.get(name)
    G = group.close(cl.gens, cl.N)
    return cl, G, irreps.compute_irreps(G)


@pytest.mark.parametrize("name,two_s,two_M", CASES)
def test_gathers_stay_inside_the_vectors(program, name, two_s, two_M):
    cl, G, irs = symmetry(name)
    sec = basis.sector_reps(G, cl.N, two_s, two_M)
    text = []
    for ir in irs:
        if ir.dim > 12:
            continue
        n = np.array([basis.stab_data(ir, S)[0] for S in sec.stab_sets])[sec.stab_id]
        if n.sum():
            text.append(f"{ir.dim} {len(n)}\n" + " ".join(map(str, n)))
    assert text
    out = subprocess.run([program], input="\n".join(text), capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr
    blocks, fails = out.stdout.strip().splitlines()[-2:]
    assert fails == "fails 0" and int(blocks.split()[1]) == len(text)
    counts = dict(zip(blocks.split()[4::2], map(int, blocks.split()[5::2])))
    assert all(counts[v] > 0 for v in ("general", "adjacent", "one-lane", "deep"))

"""GPU parity of the mixed path's products at the edges of their tiles: stacked
slab rows that end anywhere in a 128-row tile, factor columns around multiples
of 64 and densities that straddle them, odd and even numbers of 64 x 64 blocks
of K (pairs side by side and on top of each other), inner depths of one to a few
stages, general and symmetric densities, full squares, packed slabs and prepared
digit planes, against the oracle.

Tolerance: 1e-8 normwise for K, the mixed path's bound (31-bit rows, three of 16
digit products dropped); J is FP64, 1e-12.
"""
import numpy as np
import pytest

import oracle
from paper_2608_06536_amd import synth
from conftest import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nao,naux,nd,r", [
    (7, 5, 1, 1),        # one block, one stage, one column
    (33, 31, 1, 32),     # 64 columns of [X | Y], two stages
    (64, 2, 2, 33),      # exact blocks; keys of 33 columns straddle 64
    (65, 63, 3, 11),     # two by two blocks
    (129, 1, 1, 127),    # odd blocks (on top of each other), a tile and one row
    (150, 17, 2, 21), (193, 9, 1, 64),
    (257, 6, 5, 13),     # five by five blocks, depth under one stage per split
    (40, 700, 1, 3),     # many splits of the exchange, partial maxima of many slabs
])
@pytest.mark.parametrize("sym", [False, True])
@pytest.mark.parametrize("form", ["full", "packed", "sliced"])
def test_mixed_tiles(nao, naux, nd, r, sym, form):
    from paper_2608_06536_amd import jk
    p = synth.Problem(nao=nao, naux=naux, nd=nd, r=r, ell=10.0, tau=naux / 4.0 + 1, seed=9700 + nao)
    B, CL, CR = synth.make_problem(p)
    if sym:
        CR = CL
    i, j = np.triu_indices(nao)
    Bd = torch.from_numpy(np.ascontiguousarray(B[:, i, j]) if form == "packed" else B).cuda()
    Ld = torch.from_numpy(CL).cuda()
    Rd = Ld if sym else torch.from_numpy(np.ascontiguousarray(CR)).cuda()
    sl = jk.slice_b(Bd, nao) if form == "sliced" else None
    J, K = jk.jk_build(Bd, Ld, Rd, precision="mixed", slices=sl)
    torch.cuda.synchronize()
    Jr, Kr, _ = oracle.jk_factored(B, CL, CR)
    assert rel_err(J.cpu().numpy(), Jr) <= 1e-12
    for k in range(nd):
        assert rel_err(K[k].cpu().numpy(), Kr[k]) <= 1e-8, k
    if sym:
        assert torch.equal(K, K.transpose(1, 2))

"""GPU parity of the derivative's products over their tile shapes: basis sizes at
the edges of every shape's tiles, factor widths around multiples of 64 and 128,
inner depths that end inside a stage, with both cotangents, general and symmetric
densities, full and packed slabs, against the oracle.

Tolerance: normwise 1e-12, as for every FP64 result (rounding of sums of at
most a few thousand products).
"""
import numpy as np
import pytest

import oracle
from paper_2608_06536_amd import synth
from conftest import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("nao,naux,nd,r", [
    (3, 2, 1, 1), (48, 70, 1, 8),
    (64, 9, 2, 16), (65, 5, 1, 33),        # 64 x 64, exact and one past; 66 columns
    (79, 7, 3, 5), (80, 6, 1, 40),         # 80 x 64
    (96, 8, 2, 9), (97, 66, 1, 3),         # 96 x 64; past it, many splits
    (128, 5, 1, 64), (129, 3, 2, 17),      # 128 x 64
    (193, 4, 1, 31), (257, 5, 2, 13),      # 96 x 64 over two and three row tiles
    (380, 3, 2, 32),                       # 128 x 128
])
@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("sym", [False, True])
def test_vjp_shape(nao, naux, nd, r, packed, sym):
    from paper_2608_06536_amd import jk
    p = synth.Problem(nao=nao, naux=naux, nd=nd, r=r, ell=10.0, tau=naux / 4.0 + 1, seed=9900 + nao)
    B, CL, CR = synth.make_problem(p)
    if sym:
        CR = CL
    rng = np.random.default_rng(nao)
    W, V = rng.standard_normal((2, nd, nao, nao))
    i, j = np.triu_indices(nao)
    Bd = torch.from_numpy(np.ascontiguousarray(B[:, i, j]) if packed else B).cuda()
    Ld = torch.from_numpy(CL).cuda()
    Rd = Ld if sym else torch.from_numpy(np.ascontiguousarray(CR)).cuda()
    dB, dL, dR = jk.jk_vjp(Bd, Ld, Rd, torch.from_numpy(W).cuda(), torch.from_numpy(V).cuda())
    torch.cuda.synchronize()
    rB, rL, rR = oracle.vjp(B, CL, CR, W, V)
    if packed:
        rB = rB[:, i, j] + np.where(i == j, 0.0, rB[:, j, i])
    assert rel_err(dB.cpu().numpy(), rB) <= TOL
    assert rel_err(dL.cpu().numpy(), rL) <= TOL
    assert rel_err(dR.cpu().numpy(), rR) <= TOL

"""GPU parity of the exchange's tile shapes and splits (FP64): basis sizes at
the edges of every shape's tiles, inner depths that end inside a stage (odd
rank times slabs, at most 8 and more than 8 indices in the last stage), and
depths long enough for many splits, general and symmetric densities, against
the oracle.

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
    (16, 40, 1, 2),      # 64 x 64, one fragment
    (64, 33, 2, 7),      # 64 x 64, exact; depth 231 = 14 stages + 7
    (65, 9, 3, 5),       # one past a tile
    (79, 21, 1, 11), (80, 17, 2, 3),       # 80 x 64
    (96, 12, 2, 9), (97, 300, 1, 10),      # 96 x 64; past it, many splits
    (127, 16, 1, 12), (128, 8, 2, 16),     # 128 x 64 / 128 x 128
    (150, 90, 3, 15),    # 80 x 64 over two row tiles
    (193, 30, 1, 19), (257, 24, 2, 25),    # 96 x 64
    (255, 20, 1, 25),    # 128 x 128
    (48, 400, 1, 8),     # one tile, more splits than slabs in a stage
])
@pytest.mark.parametrize("sym", [False, True])
def test_exchange_shape(nao, naux, nd, r, sym):
    from paper_2608_06536_amd import jk
    p = synth.Problem(nao=nao, naux=naux, nd=nd, r=r, ell=10.0, tau=naux / 4.0 + 1, seed=9300 + nao)
    B, CL, CR = synth.make_problem(p)
    if sym:
        CR = CL
    Bd, Ld = torch.from_numpy(B).cuda(), torch.from_numpy(CL).cuda()
    Rd = Ld if sym else torch.from_numpy(np.ascontiguousarray(CR)).cuda()
    J, K = jk.jk_build(Bd, Ld, Rd)
    torch.cuda.synchronize()
    Jr, Kr, _ = oracle.jk_factored(B, CL, CR)
    assert rel_err(J.cpu().numpy(), Jr) <= TOL
    for k in range(nd):
        assert rel_err(K[k].cpu().numpy(), Kr[k]) <= TOL, k
    if sym:
        assert torch.equal(K, K.transpose(1, 2))

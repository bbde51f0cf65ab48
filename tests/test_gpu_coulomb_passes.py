"""GPU parity of the passes over B that give gamma, omega and J: one or several
blocks of positions per workgroup and runs of positions per wave, every group
width, slab counts that end inside a block of slabs, full squares and packed
slabs, single builds against the oracle and batched members against single
builds (bit for bit).

Tolerance: normwise 1e-12, as for every FP64 result (rounding of sums of at
most a few ten thousand products).
"""
import numpy as np
import pytest

import oracle
from paper_2608_06536_amd import synth
from conftest import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-12


def _problem(nao, naux, nd, r):
    p = synth.Problem(nao=nao, naux=naux, nd=nd, r=r, ell=10.0, tau=naux / 4.0 + 1, seed=9500 + nao + nd)
    return synth.make_problem(p)


def _pack(B):
    i, j = np.triu_indices(B.shape[1])
    return np.ascontiguousarray(B[:, i, j])


@pytest.mark.parametrize("nao,naux,nd,r", [
    (1, 1, 1, 1), (2, 17, 2, 1),
    (44, 15, 1, 2), (45, 16, 3, 4),        # 990 and 1035 positions: one block and two
    (64, 129, 5, 3), (65, 33, 9, 2),       # 64-tiles of the folded density; widths 8 and 16
    (50, 131, 17, 1),                      # two groups of 16
    (127, 40, 1, 2), (128, 40, 1, 2),      # gamma summed by the J pass: 8 partial sums, 9
    (20, 4096, 1, 1), (20, 4097, 1, 1), (24, 256, 9, 2), (24, 257, 9, 2),  # its LDS full, and past it
    (361, 20, 2, 3), (362, 37, 4, 2),      # one and four runs of positions per wave
    (370, 19, 16, 1),                      # several blocks of positions per workgroup
    (540, 11, 1, 2), (760, 7, 2, 2), (1080, 6, 1, 1),   # 4, 2, 1 slab slices
])
@pytest.mark.parametrize("packed", [False, True])
def test_coulomb_passes(nao, naux, nd, r, packed):
    from paper_2608_06536_amd import jk
    B, CL, CR = _problem(nao, naux, nd, r)
    Bd = torch.from_numpy(_pack(B) if packed else B).cuda()
    Ld, Rd = torch.from_numpy(CL).cuda(), torch.from_numpy(np.ascontiguousarray(CR)).cuda()
    J, _ = jk.jk_build(Bd, Ld, Rd, want_k=False)
    torch.cuda.synchronize()
    D = np.einsum("kmi,kni->kmn", CL, CR)
    g = np.einsum("qmn,kmn->kq", B, D)
    Jr = np.einsum("kq,qmn->kmn", g, B)
    if nao <= 65:
        assert rel_err(Jr, oracle.jk_factored(B, CL, CR)[0]) <= 1e-14
    J = J.cpu().numpy()
    for k in range(nd):
        assert rel_err(J[k], Jr[k]) <= TOL, k
    assert np.array_equal(J, J.transpose(0, 2, 1))


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("shapes", [
    [(45, 33, 1, 2), (64, 129, 3, 3), (30, 20, 8, 2)],
    [(45, 33, 2, 2), (370, 40, 17, 1), (65, 9, 9, 2)],
])
def test_batched_member_is_its_single_build(shapes, packed):
    from paper_2608_06536_amd import jk
    items = []
    for s in shapes:
        B, CL, CR = _problem(*s)
        items.append(tuple(torch.from_numpy(np.ascontiguousarray(a)).cuda()
                           for a in (_pack(B) if packed else B, CL, CR)))
    res = jk.jk_build_batched(items, want_k=False)
    torch.cuda.synchronize()
    for (B, CL, CR), (J, _) in zip(items, res):
        assert torch.equal(J, jk.jk_build(B, CL, CR, want_k=False)[0])


@pytest.mark.parametrize("nao,naux,nd,r", [(30, 20, 1, 2), (45, 33, 4, 3), (64, 17, 9, 2)])
@pytest.mark.parametrize("packed", [False, True])
def test_derivative_of_j(nao, naux, nd, r, packed):
    """dB, dC_L, dC_R of sum_k <W_k, J_k>; for packed slabs the gradient of an
    element off the diagonal is that of both of its places."""
    from paper_2608_06536_amd import jk
    B, CL, CR = _problem(nao, naux, nd, r)
    W = np.random.default_rng(nao).standard_normal((nd, nao, nao))
    Bd = torch.from_numpy(_pack(B) if packed else B).cuda()
    dB, dL, dR = jk.jk_vjp(Bd, torch.from_numpy(CL).cuda(), torch.from_numpy(np.ascontiguousarray(CR)).cuda(),
                           torch.from_numpy(W).cuda(), None)
    torch.cuda.synchronize()
    rB, rL, rR = oracle.vjp(B, CL, CR, W, None)
    assert rel_err(dL.cpu().numpy(), rL) <= TOL and rel_err(dR.cpu().numpy(), rR) <= TOL
    if packed:
        i, j = np.triu_indices(nao)
        rB = rB[:, i, j] + np.where(i == j, 0.0, rB[:, j, i])
    assert rel_err(dB.cpu().numpy(), rB) <= TOL

"""When the contraction may leave nothing out: N^-1 values that are not finite, in
every call that contracts, and kernels whose blocks overflow FP32.  A zero factor
does not give a zero product there, so every element the tile contributes to has
to come out not finite, as the full contraction gives it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1504_04653_amd as sp
from oracle import grid as G
from oracle import operators as O
from workloads import synth as S

from _parity import gate, stored_pairs

pytestmark = pytest.mark.gpu

PRECS = ["fp64", "fp32", "bf16x6", "bf16x3"]


def nans(n):
    return torch.full((int(n),), float("nan"), dtype=torch.float64, device="cuda")


def one_grid(call, cut):
    """(contract(ninv) -> blocks, npix, hit(tile)) of one of the one-grid calls."""
    g = sp.Grid(64, 8)
    b_l, R = S.gaussian_beam(64, g.npix, 2.0)
    kern, kd = sp.Kernel(g, b_l, R if cut else 0.0), sp.Kernel(g, (np.arange(65) + 1.0) ** 2)
    nptr, ncol = g.neighbours()
    bptr, bcol = g.blocks()

    def contract(ninv, prec):
        C, w = nans(g.out_len), torch.as_tensor(ninv).cuda()
        if call == "combined":
            D, want = nans(g.out_len), nans(g.out_len)
            sp.sample_D_BtNB(g, kd, kern, w, D, C, prec)
            sp.sample_D(g, kd, want)
            assert torch.equal(D, want)
        elif call == "batch":
            other = nans(g.out_len)
            batch = sp.Batch([(g, kern, w, C), (g, kern, torch.ones_like(w), other)], prec)
            batch.launch()
            torch.cuda.synchronize()
            assert torch.isfinite(other).all()
        else:
            sp.sample_BtNB(g, kern, w, C, prec)
        torch.cuda.synchronize()
        return C.view(-1, 64, 64)

    def hit(tile):
        near = np.zeros(g.ntiles, dtype=bool)
        near[ncol[nptr[tile]:nptr[tile + 1]]] = True
        return [near[J] and near[bcol[n]] for J in range(g.ntiles) for n in range(bptr[J], bptr[J + 1])]

    return contract, g.npix, hit


def two_grids(cut):
    g1, g2 = sp.Grid(40, 8), sp.Grid(100, 8)
    x = sp.Cross(g2, g1)
    b_l, R = S.gaussian_beam(40, g1.npix, 2.0)
    kern = sp.CrossKernel(x, b_l, R if cut else 0.0)
    _, rp, col, _ = x.neighbours()
    bptr, bcol = g1.blocks()

    def contract(ninv, prec):
        C = nans(x.out_len)
        sp.sample_BtNB_cross(x, kern, torch.as_tensor(ninv).cuda(), C, prec)
        torch.cuda.synchronize()
        return C.view(-1, 64, 64)

    def hit(tile):
        near = np.zeros(g1.ntiles, dtype=bool)
        near[col[rp[tile]:rp[tile + 1]]] = True
        return [near[J] and near[bcol[n]] for J in range(g1.ntiles) for n in range(bptr[J], bptr[J + 1])]

    return contract, g2.npix, hit


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("call,cut", [("alone", False), ("combined", True), ("batch", True), ("batch", False),
                                      ("two grids", True), ("two grids", False)])
def test_non_finite_noise(call, cut, prec):
    contract, npix, hit = two_grids(cut) if call == "two grids" else one_grid(call, cut)
    ninv = np.random.default_rng(11).uniform(0.5, 2.0, npix)
    good = contract(ninv, prec)
    assert torch.isfinite(good).all()
    tile = npix // 64 // 2 + 3
    for bad in (float("inf"), float("nan")):
        ninv[64 * tile + 37] = bad
        C = contract(ninv, prec)
        at = torch.as_tensor(np.array(hit(tile)), device="cuda")
        assert bool(at.any()) and not torch.isfinite(C[at]).any()
        assert torch.equal(C[~at], good[~at])


@pytest.mark.parametrize("prec", PRECS)
def test_blocks_that_overflow_fp32(prec):
    """Every value within the cut overflows FP32: each element of the FP32 and
    split forms has a term inf * 0 or inf * inf; FP64 gives the oracle's values.
    The kernel after it, in the memory it leaves, is an ordinary one again."""
    lmax = 64
    g, og = sp.Grid(lmax, 8), G.make_grid(lmax, 8)
    ninv = np.random.default_rng(5).uniform(0.5, 2.0, g.npix)
    w = torch.as_tensor(ninv).cuda()
    b_l, R = S.gaussian_beam(lmax, g.npix, 2.0)

    def contract(coef):
        kern, C = sp.Kernel(g, coef, R), nans(g.out_len)
        sp.sample_BtNB(g, kern, w, C, prec)
        torch.cuda.synchronize()
        return C.view(-1, 64, 64)

    before = contract(b_l)
    C = contract(1e60 * b_l)
    if prec == "fp64":
        pairs = stored_pairs(og)
        ref = O.sample_BtNB(og, 1e60 * b_l, ninv, R, pairs)
        assert gate(C.cpu().numpy(), ref, [J for J, _ in pairs]) <= 1e-10
    else:
        assert not torch.isfinite(C).any()
    assert torch.equal(contract(b_l), before)

"""The contraction's skipping of products that are zero by the radial cut:
beams from a fraction of a pixel (rows with next to no products) to no cut at
all (nothing skipped) against the oracle, and N^-1 values that are not finite,
which no zero factor may hide."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1504_04653_amd as sp
from oracle import grid as G
from oracle import operators as O
from workloads import synth as S

from _parity import gate, stored_pairs

pytestmark = pytest.mark.gpu

# those of the parity tests: FP64 1e-10, FP32 and BF16x6 1e-6, BF16x3 2^-15
GATE = {"fp64": 1e-10, "fp32": 1e-6, "bf16x6": 1e-6, "bf16x3": 2.0 ** -15}


def sample(g, kern, ninv, prec):
    out = torch.full((g.out_len,), float("nan"), dtype=torch.float64, device="cuda")
    sp.sample_BtNB(g, kern, torch.as_tensor(ninv).cuda(), out, prec)
    torch.cuda.synchronize()
    return out.view(g.nblocks, 64, 64)


@pytest.mark.parametrize("lmax,fwhm", [(40, 0.25), (40, 2.0), (64, 1.0), (64, 5.0), (100, 2.5), (64, 2.9), (64, 3.6), (64, None)])
def test_cut_widths(lmax, fwhm):
    """Cut radii (3 FWHM, in mean pixel spacings) from under one pixel to none."""
    g, og = sp.Grid(lmax, 8), G.make_grid(lmax, 8)
    ninv = np.random.default_rng(lmax).uniform(0.5, 2.0, g.npix)
    b_l, R = S.gaussian_beam(lmax, g.npix, fwhm if fwhm is not None else 3.0)
    R = 0.0 if fwhm is None else R
    pairs = stored_pairs(og)
    ref = O.sample_BtNB(og, b_l, ninv, R if fwhm is not None else None, pairs)
    kern = sp.Kernel(g, b_l, R)
    for prec in GATE:
        worst = gate(sample(g, kern, ninv, prec).cpu().numpy(), ref, [J for J, _ in pairs])
        print(f"[cut] lmax {lmax} fwhm {fwhm} {prec}: {worst:.2e}", flush=True)
        assert worst <= GATE[prec]


@pytest.mark.parametrize("prec", sorted(GATE))
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_non_finite_noise_reaches_every_element(prec, bad):
    """A pixel whose N^-1 is not finite leaves no element of the blocks its tile
    contributes to finite, zero products included, and no other block changed."""
    g = sp.Grid(64, 8)
    ninv = np.random.default_rng(7).uniform(0.5, 2.0, g.npix)
    kern = sp.Kernel(g, *S.gaussian_beam(64, g.npix, 2.0))
    good = sample(g, kern, ninv, prec)
    tile = g.ntiles // 2 + 3
    ninv[64 * tile + 9] = bad
    C = sample(g, kern, ninv, prec)
    nptr, ncol = g.neighbours()
    near = np.zeros(g.ntiles, dtype=bool)
    near[ncol[nptr[tile]:nptr[tile + 1]]] = True
    bptr, bcol = g.blocks()
    hit = np.array([near[J] and near[bcol[n]] for J in range(g.ntiles) for n in range(bptr[J], bptr[J + 1])])
    hit = torch.as_tensor(hit, device="cuda")
    assert not torch.isfinite(C[hit]).any()
    assert torch.equal(C[~hit], good[~hit])

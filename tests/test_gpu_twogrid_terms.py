"""Two-grid contractions whose classes have more terms than one list of steps
holds (16), than tiles of 64 members take (51) and on to 82: an auxiliary grid
of over twice the band limit, with a cut and without, every block against the
oracle, in each mode (the FP64 form alone changes its tiles with the terms)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1504_04653_amd as sp
from oracle import grid as G
from oracle import operators as O
from oracle import twogrid as X
from workloads import synth as S

from _parity import gate

pytestmark = pytest.mark.gpu

# those of the parity tests
GATE = {"fp64": 1e-10, "fp32": 1e-6, "bf16x6": 1e-6, "bf16x3": 2.0 ** -15}


@pytest.mark.parametrize("l2,l1,terms", [(120, 60, 42), (100, 40, 49), (108, 40, 63), (120, 40, 72), (140, 40, 81)])
@pytest.mark.parametrize("cut", [True, False])
def test_many_terms(l2, l1, terms, cut):
    og2, og1 = G.make_grid(l2, 8), G.make_grid(l1, 8)
    g2, g1 = sp.Grid(l2, 8), sp.Grid(l1, 8)
    x = sp.Cross(g2, g1)
    assert x.max_terms == terms
    ninv2 = np.random.default_rng(l2 + l1).uniform(0.5, 2.0, g2.npix)
    b_l, R = S.gaussian_beam(l1, g1.npix, 2.0)
    pairs = O.stored_block_list(og1)
    ref = X.sample_BtNB_cross(og2, og1, b_l, ninv2, R if cut else None, pairs)
    kern = sp.CrossKernel(x, b_l, R if cut else 0.0)
    for prec in GATE:
        out = torch.full((x.out_len,), float("nan"), dtype=torch.float64, device="cuda")
        sp.sample_BtNB_cross(x, kern, torch.as_tensor(ninv2).cuda(), out, prec)
        worst = gate(out.view(-1, 64, 64).cpu().numpy(), ref, [J for J, _ in pairs])
        print(f"[twogrid terms] {l2}/{l1} cut {cut} {prec}: {worst:.2e}", flush=True)
        assert worst <= GATE[prec]

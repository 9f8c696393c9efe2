"""Batches whose problems all have a short cut (their kernels leave products out),
all a wide one (none do) and some of each: three kernels in the split-BF16 modes.
Every problem's blocks are those of its own single call, bit for bit, launch
after launch, whichever kernel runs it; several grids, so that queues run dry at
different times."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_1504_04653_amd as sp
from workloads import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16x6", "bf16x3"])
@pytest.mark.parametrize("fwhm", [(2.0, 2.0, 2.0), (5.0, 5.0, 5.0), (2.0, 5.0, 2.0)])
def test_forms(fwhm, prec):
    problems, want = [], []
    for i, (lmax, fw) in enumerate(zip((64, 40, 128), fwhm)):
        g = sp.Grid(lmax, 8)
        kern = sp.Kernel(g, *S.gaussian_beam(lmax, g.npix, fw))
        w = torch.as_tensor(np.random.default_rng(i).uniform(0.5, 2.0, g.npix)).cuda()
        out = torch.full((g.out_len,), float("nan"), dtype=torch.float64, device="cuda")
        ref = torch.full_like(out, float("nan"))
        sp.sample_BtNB(g, kern, w, ref, prec)
        problems.append((g, kern, w, out))
        want.append(ref)
    batch = sp.Batch(problems, prec)
    for tiling in sp.TILINGS:
        for schedule in sp.SCHEDULES:
            batch.set_tiling(tiling)
            batch.set_schedule(schedule)
            for _, _, _, out in problems:
                out.fill_(float("nan"))
            batch.launch()
            torch.cuda.synchronize()
            for (_, _, _, out), ref in zip(problems, want):
                assert torch.equal(out, ref), f"{tiling} {schedule}"

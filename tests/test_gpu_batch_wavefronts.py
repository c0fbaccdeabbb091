"""Regenerated radial phases with two and with four wavefronts an order: the same uneven instances once (158 orders in the launch)
and sixteen times over (more than 1024), columns of one to eight segments of 32 degrees, against the FP64 oracle: 1e-12 normwise
as for the tables, 1e-5 for FP32."""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import rhs_scalar
from oracle.transform import Tables

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SIZES = [(16, 8), (33, 12), (65, 20), (97, 30), (128, 36), (160, 60), (193, 64), (256, 240)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("copies", [1, 16])
def test_batch_wavefronts(copies, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import MLG_FP32, Batch, mlg_grid
    print("batch wavefronts", copies, prec, flush=True)
    b = Batch([mlg_grid(nr, n, 1, 0, 0, 0, 1.0, 2 * np.pi, 1) for nr, n in SIZES * copies], prec=MLG_FP32 if prec else 0)
    b.set_config(1, 128, 8, 8)
    sin, sout = b.empty_spec(), b.empty_spec()
    sout.fill_(float("nan"))
    ref = []
    for k, (nr, n) in enumerate(SIZES):
        g = Grid(nr, n, 1, 1.0)
        S = synth.geometric_spectrum(g.M, g.nrc, 1, 1, seed=70 + k, a=0.95, b=0.9)
        if prec:
            S = S.astype(np.complex64).astype(np.complex128)
        for c in range(copies):
            o = k + c * len(SIZES)
            sin[int(b.offsets[o]):int(b.offsets[o + 1])] = torch.from_numpy(to_lib(S)[:, 0]).to(sin.dtype).cuda()
        ref.append((g, rhs_scalar(S, g, Tables(g), "kpp", 0.25)))
    b.rhs_kpp(0.25, sin, sout)
    torch.cuda.synchronize()
    got = sout.cpu().numpy().astype(np.complex128)
    for o in range(len(SIZES) * copies):
        g, want = ref[o % len(SIZES)]
        mine = from_lib(got[int(b.offsets[o]):int(b.offsets[o + 1])][:, None], g.M, g.nrc)
        assert rel(mine, want) < (1e-5 if prec else 1e-12), (o, rel(mine, want))
    b.close()

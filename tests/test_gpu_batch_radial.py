"""Radial phases of the batched term at the edges of their tiles: one node and 64, 65, 128 half nodes, odd N_r, degree
columns of 1, 64, 65, 192 and 256, truncations N_r^c and N_phi^c below and at the Nyquist order, with and without the mask,
one to four wavefronts a block.  Sums of at most 256 terms of order one: 1e-12 normwise against the FP64 oracle
with tables and with the recurrence, 1e-5 for FP32 batches (256 roundings of 6e-8)."""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import rhs_scalar
from oracle.transform import Tables

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# nr, nphi, nrc, dealias
SIZES = [(2, 2, 2, 1), (3, 4, 3, 1), (7, 6, 5, 0), (127, 12, 64, 1), (128, 10, 65, 1), (129, 8, 129, 0), (130, 18, 128, 1),
         (193, 9, 193, 1), (255, 15, 192, 1), (256, 250, 256, 1), (200, 256, 1, 1), (64, 48, 20, 0)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("cfg", [(0, 64, 1, 2), (0, 128, 8, 4), (0, 256, 8, 8), (1, 64, 8, 4), (1, 256, 2, 8)])
def test_batch_radial_edges(cfg, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import MLG_FP32, Batch, mlg_grid
    print("batch radial edges", cfg, prec, flush=True)
    b = Batch([mlg_grid(nr, nphi, 1, nrc, 0, 0, 1.0, 2 * np.pi, d) for nr, nphi, nrc, d in SIZES], prec=MLG_FP32 if prec else 0)
    b.set_config(*cfg)
    sin, sout = b.empty_spec(), b.empty_spec()
    sout.fill_(float("nan"))  # every coefficient is written, those of masked orders too
    ref = []
    for k, (nr, nphi, nrc, d) in enumerate(SIZES):
        g = Grid(nr, nphi, 1, 1.0, nrc=nrc)
        S = synth.geometric_spectrum(g.M, g.nrc, 1, 1, seed=50 + k, a=0.95, b=0.9)
        if prec:
            S = S.astype(np.complex64).astype(np.complex128)
        sin[int(b.offsets[k]):int(b.offsets[k + 1])] = torch.from_numpy(to_lib(S)[:, 0]).to(sin.dtype).cuda()
        ref.append((g, rhs_scalar(S, g, Tables(g), "kpp", 0.25, dealias=bool(d))))
    b.rhs_kpp(0.25, sin, sout)
    torch.cuda.synchronize()
    got = sout.cpu().numpy().astype(np.complex128)
    for k, (g, want) in enumerate(ref):
        mine = from_lib(got[int(b.offsets[k]):int(b.offsets[k + 1])][:, None], g.M, g.nrc)
        assert np.all(np.isfinite(mine)), SIZES[k]
        assert rel(mine, want) < (1e-5 if prec else 1e-12), (SIZES[k], rel(mine, want))
    b.close()

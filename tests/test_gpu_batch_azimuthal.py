"""Azimuthal phase of the batched term at every accepted N_phi (one to three stages of the radices 2 to 10, N_phi = 2 with the
mean alone) and at line counts that do and do not divide N_r: 1e-12 normwise against the FP64 oracle, 1e-5 for FP32."""
import numpy as np
import pytest

import synth
from helpers import from_lib, rel, to_lib
from oracle.grid import Grid
from oracle.rhs import rhs_scalar
from oracle.transform import Tables

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


SIZES = [(3 + n % 5, n) for n in range(2, 257) if _smooth(n)]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("threads, lines", [(64, 2), (128, 6), (256, 8)])
def test_batch_every_azimuthal_length(threads, lines, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_18026_amd import MLG_FP32, Batch, mlg_grid
    print("batch azimuthal", threads, lines, prec, flush=True)
    b = Batch([mlg_grid(nr, n, 1, 0, 0, 0, 1.0, 2 * np.pi, 1) for nr, n in SIZES], prec=MLG_FP32 if prec else 0)
    b.set_config(1, threads, 8, lines)
    sin, sout = b.empty_spec(), b.empty_spec()
    ref = []
    for k, (nr, n) in enumerate(SIZES):
        g = Grid(nr, n, 1, 1.0)
        S = synth.geometric_spectrum(g.M, g.nrc, 1, 1, seed=90 + k, a=0.9, b=0.9)
        if prec:
            S = S.astype(np.complex64).astype(np.complex128)
        sin[int(b.offsets[k]):int(b.offsets[k + 1])] = torch.from_numpy(to_lib(S)[:, 0]).to(sin.dtype).cuda()
        ref.append((g, rhs_scalar(S, g, Tables(g), "kpp", 0.25)))
    b.rhs_kpp(0.25, sin, sout)
    torch.cuda.synchronize()
    got = sout.cpu().numpy().astype(np.complex128)
    for k, (g, want) in enumerate(ref):
        mine = from_lib(got[int(b.offsets[k]):int(b.offsets[k + 1])][:, None], g.M, g.nrc)
        assert rel(mine, want) < (1e-5 if prec else 1e-12), (SIZES[k], rel(mine, want))
    b.close()

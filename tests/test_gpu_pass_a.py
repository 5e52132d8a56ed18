"""FFT pass A at the edges of its split into classes and blocks of image rows.

Pass A cuts a line of N' cells into classes of outputs and keeps the image rows
of each class that fall inside the image, writes the intermediate in blocks of
16 image rows, and reads the marked tiles of a row in batches of 16 per group of
threads.  The cases: image sizes N that are not a multiple of 16 or of the
number of classes (1, 2, 3, 4, 8 classes; N far below N'), and a band of
visibilities that marks every tile of a few rows of tiles (several batches).
Against the FP64 oracle, FP64 1e-10 and FP32 1e-6 as in test_gpu_parity.py.
"""
import numpy as np
import pytest
import torch

from oracle import wstack
from oracle.kernel_design import least_misfit
from oracle.plan import make_plan
from paper_2101_11172_amd import inputs
from paper_2101_11172_amd import wsgrid as wg

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def rel(a, b):
    a, b = np.ravel(a), np.ravel(b)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("N,Np,band", [(10, 64, False), (40, 128, False), (250, 1536, False), (1000, 2048, False),
                                       (1466, 3072, False), (100, 4096, True), (1992, 8192, True)])
def test_ragged_image_sizes(N, Np, band):
    L, W, x0, wmax, M = 0.1, 4, N / (2.0 * Np), 20.0, 3000
    op, lm = make_plan(N, L, W, x0, wmax), least_misfit(W, x0)
    assert op.Nprime == Np
    umax = 0.5 * Np * x0 / (0.5 * L)                     # the whole N' x N' plane
    uvw = inputs.uniform_uvw(M, 0.99 * umax, wmax, 7)
    if band:
        uvw[:, 0] *= 0.01
    vis, img = inputs.random_vis(M, 8), inputs.random_image(N, 9)
    ref_g, ref_d = wstack.grid(op, lm, uvw, vis), wstack.degrid(op, lm, uvw, img)
    plan = wg.Plan(N, L, W, x0, wmax, device=DEV)
    t_uvw = torch.from_numpy(uvw).to(DEV)
    for cdt, rdt, tol in ((torch.complex128, torch.float64, 1e-10), (torch.complex64, torch.float32, 1e-6)):
        g = plan.grid(t_uvw, torch.from_numpy(vis).to(DEV, cdt)).cpu().double().numpy()
        d = plan.degrid(t_uvw, torch.from_numpy(img).to(DEV, rdt)).cpu().to(torch.complex128).numpy()
        print(f"N={N} N'={Np} layers {op.n_layers} {rdt}: grid {rel(g, ref_g):.3e} degrid {rel(d, ref_d):.3e}", flush=True)
        assert rel(g, ref_g) <= tol and rel(d, ref_d) <= tol
    plan.close()

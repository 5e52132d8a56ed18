"""The tile kernels on clumps of visibilities: runs that share a window.

Records are taken 64 at a time and in groups of four (gridding) or 16
(degridding) of one window of 8 cells.  Clumps of 1 ... 500 visibilities a
fraction of a cell apart, some on a window's edge, among scattered ones give
runs that end inside a group, fill it exactly and span several batches, in and
across tiles.  Widths from two cells (window of seven starts) to eight (a window
per start), and a w-axis width of its own.  Plain and shared-binning calls
against the FP64 oracle, tolerances as in test_gpu_parity.py.
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


def clumps(N, L, x0, wmax, seed):
    rng = np.random.default_rng(seed)
    umax = 0.9 * N / (2 * L)
    cell = x0 / (0.5 * L)                                      # one u, v cell in wavelengths
    parts = [inputs.uniform_uvw(300, umax, wmax, seed)]
    for n in (1, 2, 3, 4, 5, 15, 16, 17, 63, 64, 65, 500):
        c = rng.uniform(-1, 1, 3) * np.array([umax, umax, 0.9 * wmax])
        parts.append(c + rng.uniform(-0.7, 0.7, (n, 3)) * np.array([cell, cell, 1.0]))
    return np.concatenate(parts)


@pytest.mark.parametrize("W,Wz", [(2, 2), (5, 5), (7, 7), (8, 8), (7, 3)])
def test_clumps(W, Wz):
    N, L, x0, wmax = 64, 0.3, 0.25, 400.0
    uvw = clumps(N, L, x0, wmax, 17)
    uvw[:, 2] = np.clip(uvw[:, 2], -wmax, wmax)
    M = uvw.shape[0]
    vis, img = inputs.random_vis(M, 18), inputs.random_image(N, 19)
    lm = least_misfit(W, x0)
    if Wz == W:
        op = make_plan(N, L, W, x0, wmax)
        ref_g, ref_d = wstack.grid(op, lm, uvw, vis), wstack.degrid(op, lm, uvw, img)
    else:
        lmz = least_misfit(Wz, x0)
        op = make_plan(N, L, W, x0, wmax, Wz=Wz, z0=x0)
        ref_g, ref_d = wstack.grid(op, lm, uvw, vis, lmz=lmz), wstack.degrid(op, lm, uvw, img, lmz=lmz)
    plan = wg.Plan(N, L, W, x0, wmax, device=DEV, Wz=Wz, z0=x0)
    t_uvw = torch.from_numpy(uvw).to(DEV)
    for cdt, rdt, tol in ((torch.complex128, torch.float64, 1e-10), (torch.complex64, torch.float32, 1e-6)):
        t_vis, t_img = torch.from_numpy(vis).to(DEV, cdt), torch.from_numpy(img).to(DEV, rdt)
        plan.prepare(t_uvw, rdt)
        got = {"prepared": (plan.grid_prepared(t_vis).cpu(), plan.degrid_prepared(t_img).cpu()),
               "plain": (plan.grid(t_uvw, t_vis).cpu(), plan.degrid(t_uvw, t_img).cpu())}
        for how, (g, d) in got.items():
            eg, ed = rel(g.double().numpy(), ref_g), rel(d.to(torch.complex128).numpy(), ref_d)
            print(f"W={W} Wz={Wz} {rdt} {how}: grid {eg:.3e} degrid {ed:.3e}", flush=True)
            assert eg <= tol and ed <= tol, (how, rdt, eg, ed)
    plan.close()

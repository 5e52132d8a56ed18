"""Kernels that take several units of work one after the other, where the count
leaves a remainder.

FFT pass A gives a block several layers of a tile layer while 4,096 blocks are
left, fewer in the last block and where a channel's padding begins; the scans of
the bin counts take one block of two rounds at 8,192 bins and three launches
above.  Sizes at which these run are asserted with the rules of the launches.
Against the FP64 oracle, FP64 1e-10 and FP32 1e-6 as in test_gpu_parity.py; in
layer passes degridding bit for bit and gridding within 1e-13 (FP64) and 1e-6
(FP32) of the call in one pass.
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
TYPES = ((torch.complex128, torch.float64, 1e-10, 1e-13), (torch.complex64, torch.float32, 1e-6, 1e-6))


def rel(a, b):
    a, b = np.ravel(a), np.ravel(b)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def layers_per_block(Np, layers, f64):
    """Rule of the launch: classes of 1,024 outputs, rows of 64 threads each in
    blocks of 256 (FP64) or 512, layers per block halved from 16."""
    classes = Np // 1024
    blocks = layers * (Np // 16) * classes * (16 // ((256 if f64 else 512) // 64))
    each = 16
    while each > 1 and blocks // each < 4096:
        each //= 2
    return each


@pytest.mark.parametrize("N,Np,wmax,counts", [(200, 2048, 600.0, [2000, 1200]),
                                              (200, 3072, 200.0, [2500])])
def test_pass_a_layers_per_block(N, Np, wmax, counts):
    L, W, x0, M, C = 0.1, 4, N / (2.0 * Np), sum(counts), len(counts)
    op, lm = make_plan(N, L, W, x0, wmax), least_misfit(W, x0)
    virtual = (C - 1) * -(-op.n_layers // 16) * 16 + op.n_layers
    each = [layers_per_block(Np, virtual, f64) for f64 in (False, True)]
    print(f"N'={Np} {C} channels of {op.n_layers} layers, per block {each}", flush=True)
    assert op.Nprime == Np and min(each) > 1 and all(op.n_layers % 16 % e for e in each)
    uvw = inputs.uniform_uvw(M, 0.99 * 0.5 * Np * x0 / (0.5 * L), wmax, 91)
    vis, off = inputs.random_vis(M, 92), np.concatenate([[0], np.cumsum(counts)])
    img = np.stack([inputs.random_image(N, 93 + c) for c in range(C)])
    part = [slice(off[c], off[c + 1]) for c in range(C)]
    ref_g = [wstack.grid(op, lm, uvw[s], vis[s]) for s in part]
    ref_d = [wstack.degrid(op, lm, uvw[s], img[c]) for c, s in enumerate(part)]
    plan = wg.Plan(N, L, W, x0, wmax, device=DEV)
    least = wg.Plan(N, L, W, x0, wmax, device=DEV, max_workspace_bytes=1)
    t_uvw = torch.from_numpy(uvw).to(DEV)
    for cdt, rdt, tol, same in TYPES:
        t_vis, t_img = torch.from_numpy(vis).to(DEV, cdt), torch.from_numpy(img).to(DEV, rdt)
        g, d = plan.grid_batch(t_uvw, counts, t_vis), plan.degrid_batch(t_uvw, counts, t_img)
        for c, s in enumerate(part):
            eg, ed = rel(g[c].cpu().double().numpy(), ref_g[c]), rel(d[s].cpu().to(torch.complex128).numpy(), ref_d[c])
            print(f"channel {c} {rdt}: grid {eg:.3e} degrid {ed:.3e}", flush=True)
            assert eg <= tol and ed <= tol, (c, rdt)
        assert torch.equal(least.degrid_batch(t_uvw, counts, t_img), d)
        assert rel(least.grid_batch(t_uvw, counts, t_vis).cpu().double().numpy(), g.cpu().double().numpy()) <= same
    plan.close()
    least.close()


@pytest.mark.parametrize("wmax,counts,bins", [(300.0, [9000], 8192), (600.0, [9000], 12288),
                                              (300.0, [5000, 4000], 16384), (300.0, [70000], 8192)])
def test_scans_of_many_bins(wmax, counts, bins):
    N, L, W, x0, M = 512, 0.3, 7, 0.25, sum(counts)
    op, lm = make_plan(N, L, W, x0, wmax), least_misfit(W, x0)
    assert len(counts) * (op.Nprime // 16) ** 2 * -(-op.n_layers // 16) == bins
    uvw = inputs.uniform_uvw(M, 0.9 * N / (2 * L), wmax, 94)
    uvw[::7, 2] = 2.0 * wmax
    keep = np.abs(uvw[:, 2]) <= wmax
    off = np.concatenate([[0], np.cumsum(counts)])
    img = np.stack([inputs.random_image(N, 95 + c) for c in range(len(counts))])
    vis = torch.from_numpy(inputs.random_vis(M, 97)).to(DEV)
    plan = wg.Plan(N, L, W, x0, wmax, device=DEV)
    t_uvw, t_img = torch.from_numpy(uvw).to(DEV), torch.from_numpy(img).to(DEV)
    out = torch.full((M,), float("nan"), dtype=torch.complex128, device=DEV)
    d = plan.degrid_batch(t_uvw, counts, t_img, out=out).cpu().numpy()
    assert plan.skipped(wg.WSG_F64) == M - keep.sum() and np.all(d[~keep] == 0)
    g = plan.grid_batch(t_uvw, counts, vis)
    for c in range(len(counts)):
        idx = np.arange(off[c], off[c + 1])
        idx = idx[keep[idx]]
        some = idx[::max(1, idx.size // 500)]
        assert rel(d[some], wstack.degrid(op, lm, uvw[some], img[c])) <= 1e-10
        assert rel(g[c].cpu().numpy(), wstack.grid(op, lm, uvw[idx], vis.cpu().numpy()[idx])) <= 1e-10
    plan.close()

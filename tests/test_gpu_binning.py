"""Binning on both sides of its rule: a thread per visibility up to 65,536
visibilities, chunks with an LDS table above; one or three scan launches (8,192
bins); skipped visibilities, whose places the degrid call must zero.

Counts at, one below and one above the rule's line, in one channel and split over
channels (one empty, one of a single visibility), every seventh visibility beyond
wmax and some not finite.  Degridding against the FP64 oracle on a subset, zero
where skipped whatever the output held before, and the skipped count; gridding
against the map of the kept visibilities alone (the same binning rule may not
apply to both, so they differ by rounding).
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


@pytest.mark.parametrize("N,counts", [(64, [65535]), (64, [65536]), (64, [65537]), (64, [40000, 0, 1, 25535]),
                                      (64, [40000, 0, 1, 25536]), (512, [65536]), (512, [70001])])
def test_binning_rule(N, counts):
    L, W, x0, wmax = 0.3, 7, 0.25, 120.0
    M = sum(counts)
    uvw = inputs.uniform_uvw(M, 0.9 * N / (2 * L), wmax, 31)
    uvw[::7, 2] = 2.0 * wmax
    uvw[3::1000, 0] = np.nan
    keep = np.isfinite(uvw).all(1) & (np.abs(uvw[:, 2]) <= wmax)
    op, lm = make_plan(N, L, W, x0, wmax), least_misfit(W, x0)
    plan = wg.Plan(N, L, W, x0, wmax, device=DEV)
    nbins = len(counts) * (op.Nprime // 16) ** 2 * -(-op.n_layers // 16)
    print(f"N={N} M={M} channels={len(counts)} bins={nbins} skipped={M - keep.sum()}", flush=True)
    t_uvw = torch.from_numpy(uvw).to(DEV)
    imgs = np.stack([inputs.random_image(N, 40 + c) for c in range(len(counts))])
    t_img = torch.from_numpy(imgs).to(DEV)
    out = torch.full((M,), float("nan"), dtype=torch.complex128, device=DEV)
    plan.degrid_batch(t_uvw, counts, t_img, out=out)
    assert plan.skipped(wg.WSG_F64) == M - keep.sum()
    d = out.cpu().numpy()
    assert np.all(d[~keep] == 0)
    off = np.concatenate([[0], np.cumsum(counts)])
    for c in range(len(counts)):
        idx = np.arange(off[c], off[c + 1])
        idx = idx[keep[idx]][:400]
        if idx.size:
            ref = wstack.degrid(op, lm, uvw[idx], imgs[c])
            assert np.linalg.norm(d[idx] - ref) <= 1e-10 * np.linalg.norm(ref), c
    vis = torch.from_numpy(inputs.random_vis(M, 50)).to(DEV)
    kept = [int(keep[off[c]:off[c + 1]].sum()) for c in range(len(counts))]
    t_keep = torch.from_numpy(keep).to(DEV)
    a = plan.grid_batch(t_uvw, counts, vis)
    b = plan.grid_batch(t_uvw[t_keep].contiguous(), kept, vis[t_keep].contiguous())
    assert float(torch.linalg.vector_norm(a - b)) <= 1e-12 * float(torch.linalg.vector_norm(b))
    plan.close()

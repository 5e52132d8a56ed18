"""Workspace of the lists of marked tiles, and lists made pass by pass.

A marked tile's record takes 128 bytes.  The smallest workspace holds the
records of one tile layer's tiles only, so that it does not grow with all the tiles of many layers or
channels: at most 64 bytes per tile of the bin tables (45, and the marks) and 8
MiB of alignment.  With that workspace the lists are made anew for each pass;
plain and shared-binning calls of several channels then agree with those in the
full workspace: degridding bit for bit, gridding but for the order in which the
passes' maps are summed (1e-13 FP64, 1e-6 FP32 as in test_gpu_prepared.py).
"""
import numpy as np
import pytest
import torch

from paper_2101_11172_amd import inputs
from paper_2101_11172_amd import wsgrid as wg

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("N,wmax,M", [(2048, 518.6, 4_000_000), (2048, 518.6, 30_000_000), (512, 4000.0, 100_000)])
def test_smallest_workspace_per_tile(N, wmax, M):
    plan = wg.Plan(N, 0.4, 7, 0.25, wmax, device=DEV)
    tiles = (plan.info["Nprime"] // 16) ** 2 * -(-plan.info["n_layers"] // 16)
    for prec in (wg.WSG_F32, wg.WSG_F64):
        one = wg.grid_workspace_bytes_batch(plan._p, prec, 1, M, True)
        for nch in (2, 16, 64):
            if nch * tiles > 1 << 25:
                continue
            more = wg.grid_workspace_bytes_batch(plan._p, prec, nch, M, True) - one
            print(f"N={N} M={M} prec={prec} channels={nch}: {more / ((nch - 1) * tiles):.1f} bytes per tile", flush=True)
            assert more <= 64 * (nch - 1) * tiles + (8 << 20)
    plan.close()


@pytest.mark.parametrize("counts", [[3000], [2000, 0, 1, 1500]])
def test_lists_pass_by_pass(counts):
    N, L, W, x0, wmax = 64, 0.8, 7, 0.25, 200.0
    M, C = sum(counts), len(counts)
    uvw = torch.from_numpy(inputs.uniform_uvw(M, 0.9 * N / (2 * L), wmax, 71)).to(DEV)
    full = wg.Plan(N, L, W, x0, wmax, device=DEV)
    least = wg.Plan(N, L, W, x0, wmax, device=DEV, max_workspace_bytes=1)
    for rdt, cdt, prec, tol in ((torch.float64, torch.complex128, wg.WSG_F64, 1e-13),
                                (torch.float32, torch.complex64, wg.WSG_F32, 1e-6)):
        ws = wg.grid_workspace_bytes_batch(least._p, prec, C, M, True)
        assert wg.grid_layers_per_pass(least._p, prec, C, M, ws) == 16 < full.info["n_layers"]
        vis = torch.from_numpy(inputs.random_vis(M, 72)).to(DEV, cdt)
        img = torch.from_numpy(np.stack([inputs.random_image(N, 73 + c) for c in range(C)])).to(DEV, rdt)
        g, d = full.grid_batch(uvw, counts, vis), full.degrid_batch(uvw, counts, img)
        got = [(least.grid_batch(uvw, counts, vis), least.degrid_batch(uvw, counts, img))]
        least.prepare(uvw, rdt, counts)
        for _ in range(2):
            got.append((least.grid_prepared(vis).view_as(g), least.degrid_prepared(img.view(-1, N, N) if C > 1 else img[0])))
        for gg, dd in got:
            assert torch.equal(dd, d)
            assert float(torch.linalg.vector_norm(gg - g)) <= tol * float(torch.linalg.vector_norm(g))
    full.close()
    least.close()

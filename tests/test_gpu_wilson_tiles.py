"""The fine stencil where a workgroup has a tile of 64 x 4 sites: from 2^15 sites, at most an
eighth of the tiles' threads outside the lattice; 2 right-hand sides per thread once input
and output exceed 256 MB.  Against the oracle's D, with the bounds of the other stencil tests
(about a dozen roundings per entry)."""
import numpy as np
import pytest

from oracle import wilson as ow
from paper_2211_15383_amd.inputs import link_angles

from _helpers import random_vectors, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Lx,Lt,nrhs,precs", [
    (256, 128, 3, "both"),   # the smallest in tiles: 32768 sites, whole tiles
    (180, 180, 3, "both"),   # 32400 sites: consecutive sites
    (184, 180, 9, "both"),   # a ragged last tile
    (60, 548, 2, "both"),    # one ragged tile across
    (68, 484, 2, "both"),    # nearly half of the tiles' threads outside: consecutive sites
    (252, 132, 121, "fp64"),  # 257.6 MB: 2 right-hand sides per thread, an odd last one
    (252, 132, 241, "mixed"),
])
def test_stencil_tiles(gpu, Lx, Lt, nrhs, precs):
    torch, dm, ctx = gpu
    theta = link_angles(Lx, Lt, 0.5, Lx * 1000 + Lt)
    m0 = -0.07
    H = dm.Hierarchy(ctx, theta, m0, [], [])
    D = ow.dirac_operator(theta, m0)
    x = random_vectors(D.shape[0], nrhs, 1)
    ref = D @ x
    g5 = np.tile([1.0, -1.0], D.shape[0] // 2)
    for name, prec, dt, tol in (("fp64", dm.FP64, torch.complex128, 1e-13),
                                ("mixed", dm.MIXED, torch.complex64, 1e-6)):
        if precs not in ("both", name):
            continue
        xd = to_dev(torch, x, dt)
        y = torch.empty_like(xd)
        H.apply(dm.OP_D, 1, xd, y, prec)
        assert rel_err(to_host(y), ref) < tol, name
        H.apply(dm.OP_GAMMA5_D, 1, xd, y, prec)
        assert rel_err(to_host(y), g5[:, None] * ref) < tol, name


def test_stencil_of_more_right_hand_sides_than_workgroup_rows(gpu):
    """70000 right-hand sides with one asked for per thread: the launch has at most 65535 rows of
    workgroups.  The first, middle and last rows are those of small blocks."""
    torch, dm, ctx = gpu
    H = dm.Hierarchy(ctx, link_angles(8, 8, 0.5, 3), -0.07, [], [])
    H.set_kernel_variant(1, dm.KV_WILSON_RB, 1)
    x = torch.randn((70000, H.n(1)), dtype=torch.complex64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    y = H.apply(dm.OP_D, 1, x, torch.full_like(x, float("nan")), dm.MIXED)
    for r in (0, 1, 34999, 65535, 65536, 69999):
        ref = H.apply(dm.OP_D, 1, x[r:r + 1], torch.empty_like(x[:1]), dm.MIXED)
        assert torch.equal(torch.view_as_real(y[r:r + 1]), torch.view_as_real(ref))


@pytest.mark.parametrize("Lx,Lt,nrhs,name", [
    (400, 300, 33, "fp64"),   # 253 MB, just within the cache
    (400, 300, 65, "fp64"),   # beyond it, ragged tiles, rows of 525 workgroups: 2 right-hand sides per thread
    (256, 132, 119, "fp64"),  # beyond it, whole tiles: 2
    (720, 512, 13, "fp64"),   # beyond it, vectors of 24 MB: 8
    (1024, 64, 130, "fp64"),  # 545 MB, both vectors beyond it: 2
])
def test_stencil_right_hand_sides_per_thread(gpu, Lx, Lt, nrhs, name):
    torch, dm, ctx = gpu
    theta = link_angles(Lx, Lt, 0.5, Lx * 1000 + Lt)
    H = dm.Hierarchy(ctx, theta, -0.07, [], [])
    D = ow.dirac_operator(theta, -0.07)
    xd = torch.randn((nrhs, H.n(1)), dtype=torch.complex128, device="cuda",
                     generator=torch.Generator("cuda").manual_seed(2))
    y = H.apply(dm.OP_D, 1, xd, torch.full_like(xd, float("nan")), dm.FP64)
    for r in (0, nrhs // 2, nrhs - 2, nrhs - 1):
        ref = D @ xd[r].cpu().numpy()
        assert np.linalg.norm(y[r].cpu().numpy() - ref) < 1e-13 * np.linalg.norm(ref), r

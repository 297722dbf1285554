"""Fixed-count GMRES of coarsest levels against numpy: one launch up to 2048 entries, split
Gram-Schmidt steps up to 16384, passes over many workgroups beyond.

dmlmc_apply(OP_VCYCLE) at the coarsest level is the coarsest solve alone: x = e0 + GMRES_m(r)
with r = b - W W^H b, e0 = X Lambda^-1 W^H b for an attached deflation (r = b, e0 = 0
without).  The reference builds the Krylov space in FP64 with the exported blocks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M, M_DEFL = 24, 8  # default iteration counts without and with a deflation

# lattice, aggregate, test vectors per chirality: sites x dofs of the coarsest level
SHAPES = {
    "8x2": ((8, 16), (4, 4), 1),       # 16 entries, the smallest level
    "16x8": ((16, 16), (4, 4), 4),     # 128: blocks in LDS
    "12x10": ((16, 12), (4, 4), 5),    # 120: in FP64 a row over two threads, summed through LDS
    "6x24": ((12, 8), (4, 4), 12),     # 144: the same over four, a site's threads in two wavefronts
    "8x12": ((16, 8), (4, 4), 6),      # 96: three columns a direction and thread
    "60x10": ((24, 40), (4, 4), 5),    # 600: dofs that are no power of two
    "64x16": ((32, 32), (4, 4), 8),    # 1024: part of the FP32 basis outside LDS
    "50x24": ((20, 40), (4, 4), 12),   # 1200: more than 16 dofs
    "128x16": ((64, 32), (4, 4), 8),   # 2048: the largest in one launch
    "rows8": ((16, 16), (4, 2), 3),    # 8, 12 and 24 rows per interpolation block: one chunk of eight,
    "rows12": ((16, 12), (4, 3), 4),   # one and a remainder, three
    "rows24": ((16, 24), (4, 6), 5),
    "2079x16": ((252, 132), (4, 4), 8),  # 66528 fine dofs: prolongation by whole rows, a ragged last block
    "132x16": ((48, 44), (4, 4), 8),   # 2112: the first in separate launches
    "1024x16": ((128, 128), (4, 4), 8),  # 16384: the largest with split Gram-Schmidt steps
    "1056x16": ((132, 128), (4, 4), 8),  # 16896: the first with the passes of long vectors
    "1064x16": ((152, 112), (4, 4), 8),  # 17024: their last workgroup half empty
}


def _blocks_apply(A, Lx, Lt, x):
    """D x for x [n, nrhs] with blocks A [sites, 5, d, d] (self, +x, -x, +t, -t)."""
    d = A.shape[-1]
    f = x.reshape(Lt, Lx, d, -1)
    nb = [f, np.roll(f, -1, 1), np.roll(f, 1, 1), np.roll(f, -1, 0), np.roll(f, 1, 0)]
    B = A.reshape(Lt, Lx, 5, d, d)
    return sum(B[:, :, k] @ nb[k] for k in range(5)).reshape(x.shape)


def _gmres(apply, b, m):
    """x in the m-step Krylov space of b with the least residual (one vector, FP64)."""
    beta = np.linalg.norm(b)
    if beta == 0.0:
        return np.zeros_like(b)
    V = np.zeros((b.size, m + 1), dtype=np.complex128)
    H = np.zeros((m + 1, m), dtype=np.complex128)
    V[:, 0] = b / beta
    for j in range(m):
        w = apply(V[:, j : j + 1])[:, 0]
        for _ in range(2):
            h = V[:, : j + 1].conj().T @ w
            w = w - V[:, : j + 1] @ h
            H[: j + 1, j] += h
        H[j + 1, j] = np.linalg.norm(w)
        V[:, j + 1] = w / H[j + 1, j]
    e1 = np.zeros(m + 1)
    e1[0] = beta
    return V[:, :m] @ np.linalg.lstsq(H, e1, rcond=None)[0]


@pytest.mark.parametrize("k", [0, 4])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("shape", sorted(SHAPES))
def test_coarsest_gmres(shape, prec, k):
    import torch

    from paper_2211_15383_amd import dmlmc

    (Lx, Lt), agg, ntv = SHAPES[shape]
    rng = np.random.default_rng(17)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[cn(2 * Lx * Lt, ntv)])
    lx, lt, d = H.level_info(2)
    n = H.n(2)
    A = H.export(2, Dc=True)["Dc"]
    m = min(M_DEFL if k else M, n // 2)
    H.solver_params(coarsest_iters=m, coarsest_iters_defl=m)
    g5 = np.tile(np.repeat([1.0, -1.0], d // 2), n // d)
    defl = None
    if k:
        X = np.linalg.qr(cn(n, k))[0]
        lam = np.array([0.3, -0.4, 0.5, -0.7])
        defl = dmlmc.Deflation(H, 2, k, import_X=X, import_lambda=lam)
        H.set_deflation(defl)
    b = cn(3, n)
    b[1] = 0.0
    mixed = prec == "mixed"
    dt = torch.complex64 if mixed else torch.complex128
    bd = torch.as_tensor(b, device="cuda").to(dt)
    x = H.apply(dmlmc.OP_VCYCLE, 2, bd, torch.full_like(bd, float("nan")),
                prec=dmlmc.MIXED if mixed else dmlmc.FP64).cpu().numpy().astype(np.complex128)
    b = bd.cpu().numpy().astype(np.complex128)
    # FP32: vectors rounded to 6e-8, operator sums of up to 5 d products, m steps, a condition
    # number of the projected matrix of order 10: 24 * 5e-7 * 10; FP64: 2^-29 of it
    tol = 2e-4 if mixed else 1e-11
    for r in range(3):
        ref, rhs = np.zeros(n, dtype=np.complex128), b[r]
        if k:
            W = g5[:, None] * X
            c = W.conj().T @ rhs
            ref, rhs = X @ (c / lam), rhs - W @ c
        ref = ref + _gmres(lambda v: _blocks_apply(A, lx, lt, v), rhs, m)
        if r == 1:
            assert np.array_equal(x[r], np.zeros(n))
        else:
            assert np.linalg.norm(x[r] - ref) <= tol * np.linalg.norm(ref), (shape, prec, k, r)


@pytest.mark.parametrize("m", [1, 9, 16, 17, 25, 31])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("shape", ["16x8", "132x16"])
def test_iteration_counts(shape, prec, m):
    """Back substitutions with room for 8, 16, 24 and 32 columns, and the one in LDS of the
    one-launch kernel beyond 8; bounds as above."""
    import torch

    from paper_2211_15383_amd import dmlmc

    (Lx, Lt), agg, ntv = SHAPES[shape]
    rng = np.random.default_rng(31)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[cn(2 * Lx * Lt, ntv)])
    lx, lt, _ = H.level_info(2)
    A = H.export(2, Dc=True)["Dc"]
    H.solver_params(coarsest_iters=m)
    mixed = prec == "mixed"
    bd = torch.as_tensor(cn(2, H.n(2)), device="cuda").to(torch.complex64 if mixed else torch.complex128)
    x = H.apply(dmlmc.OP_VCYCLE, 2, bd, torch.empty_like(bd),
                prec=dmlmc.MIXED if mixed else dmlmc.FP64).cpu().numpy()
    b = bd.cpu().numpy().astype(np.complex128)
    for r in range(2):
        ref = _gmres(lambda v: _blocks_apply(A, lx, lt, v), b[r], m)
        assert np.linalg.norm(x[r] - ref) <= (2e-4 if mixed else 1e-11) * np.linalg.norm(ref), (shape, prec, m, r)


@pytest.mark.parametrize("nrhs", [1, 3, 8, 17, 33])
@pytest.mark.parametrize("shape", ["8x2", "16x8", "8x12", "60x10", "64x16", "50x24", "132x16", "rows8", "rows12", "rows24",
                                   "2079x16"])
def test_coarse_operator_and_transfers(shape, nrhs):
    """D, P^H and P of small levels: one right-hand side, the remainders of the groups of 4
    and 16, FP64 (a matrix-core tile per wavefront from 8 on at 16 dofs) and complex FP32."""
    import torch

    from paper_2211_15383_amd import dmlmc

    (Lx, Lt), agg, ntv = SHAPES[shape]
    rng = np.random.default_rng(23)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[cn(2 * Lx * Lt, ntv)])
    lx, lt, _ = H.level_info(2)
    P, A = H.export(1, P=True)["P"], H.export(2, Dc=True)["Dc"]
    xf, xc = cn(nrhs, H.n(1)), cn(nrhs, H.n(2))
    for prec, dt, tol in ((dmlmc.FP64, torch.complex128, 1e-13), (dmlmc.MIXED, torch.complex64, 1e-6)):
        f, c = (torch.as_tensor(v, device="cuda").to(dt) for v in (xf, xc))
        hf, hc = (t.cpu().numpy().astype(np.complex128) for t in (f, c))
        for op, lv, src, ref in ((dmlmc.OP_D, 2, c, _blocks_apply(A, lx, lt, hc.T).T),
                                 (dmlmc.OP_RESTRICT, 1, f, hf @ P.conj()),
                                 (dmlmc.OP_PROLONG, 1, c, hc @ P.T)):
            out = H.apply(op, lv, src, torch.full(ref.shape, float("nan"), dtype=dt, device="cuda"), prec=prec)
            err = np.linalg.norm(out.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
            assert err.max() <= tol, (shape, nrhs, prec, op, err.max())


@pytest.mark.parametrize("nrhs", [1, 5])
@pytest.mark.parametrize("Lx,Lt,ntv", [(16, 16, 4), (16, 16, 5), (16, 24, 6), (16, 16, 8), (16, 16, 3)])
def test_coarse_gauss_seidel(Lx, Lt, ntv, nrhs):
    """Two red/black sweeps on the second of three levels: 8, 10, 12 and 16 dofs and any other
    count."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(29)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.3, [(4, 4), (2, 2)],
                        [ntv, 2], import_tv=[cn(2 * Lx * Lt, ntv), cn(Lx * Lt // 16 * 2 * ntv, 2)])
    lx, lt, d = H.level_info(2)
    A = H.export(2, Dc=True)["Dc"]
    Ainv = np.linalg.inv(A[:, 0])
    t, x = np.divmod(np.arange(lx * lt), lx)
    b = cn(nrhs, H.n(2))
    # sums of up to 6 d products, inverse blocks with condition numbers of order 10
    for prec, dt, tol in ((dmlmc.FP64, torch.complex128, 1e-12), (dmlmc.MIXED, torch.complex64, 1e-4)):
        H.solver_params(smoother_half=0)
        bd = torch.as_tensor(b, device="cuda").to(dt)
        out = H.apply(dmlmc.OP_SMOOTH, 2, bd, torch.zeros_like(bd), prec=prec, arg=2).cpu().numpy()
        bh = bd.cpu().numpy().astype(np.complex128).T
        y = np.zeros_like(bh)
        for _ in range(2):
            for color in (0, 1):
                r = (bh - _blocks_apply(A, lx, lt, y)).reshape(lx * lt, d, nrhs)
                on = (x + t) % 2 == color
                y.reshape(lx * lt, d, nrhs)[on] += (Ainv @ r)[on]
        assert np.linalg.norm(out.T - y) <= tol * np.linalg.norm(y), (prec, nrhs)


@pytest.mark.parametrize("shape,k,m", [("16x8", 32, 24), ("64x16", 32, 8), ("64x16", 64, 8), ("64x16", 65, 24),
                                       ("64x16", 256, 8), ("60x10", 109, 8), ("60x10", 110, 8), ("50x24", 300, 8),
                                       ("128x16", 17, 24), ("128x16", 512, 8)])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_deflation_of_many_vectors(shape, prec, k, m):
    """Deflation inside the one-launch solve (up to 512 KB of vectors, more of them than its 16
    wavefronts) and in launches of its own beyond; bounds as above (the k terms are FP64 sums)."""
    import torch

    from paper_2211_15383_amd import dmlmc

    (Lx, Lt), agg, ntv = SHAPES[shape]
    rng = np.random.default_rng(37)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[cn(2 * Lx * Lt, ntv)])
    lx, lt, d = H.level_info(2)
    n = H.n(2)
    A = H.export(2, Dc=True)["Dc"]
    H.solver_params(coarsest_iters_defl=m)
    X = np.linalg.qr(cn(n, k))[0]
    lam = np.linspace(0.3, 2.0, k) * (-1.0) ** np.arange(k)
    defl = dmlmc.Deflation(H, 2, k, import_X=X, import_lambda=lam)  # (the hierarchy keeps no reference)
    H.set_deflation(defl)
    W = np.tile(np.repeat([1.0, -1.0], d // 2), n // d)[:, None] * X
    mixed = prec == "mixed"
    bd = torch.as_tensor(cn(2, n), device="cuda").to(torch.complex64 if mixed else torch.complex128)
    x = H.apply(dmlmc.OP_VCYCLE, 2, bd, torch.empty_like(bd),
                prec=dmlmc.MIXED if mixed else dmlmc.FP64).cpu().numpy()
    for r, b in enumerate(bd.cpu().numpy().astype(np.complex128)):
        c = W.conj().T @ b
        ref = X @ (c / lam) + _gmres(lambda v: _blocks_apply(A, lx, lt, v), b - W @ c, m)
        assert np.linalg.norm(x[r] - ref) <= (2e-4 if mixed else 1e-11) * np.linalg.norm(ref), (shape, prec, k, r)


@pytest.mark.parametrize("Lx,Lt,agg,ntv,nrhs", [
    (16, 16, (4, 4), 2, 1), (16, 16, (4, 4), 2, 2), (16, 16, (4, 4), 2, 5), (24, 16, (4, 4), 7, 1), (24, 16, (4, 4), 7, 2),
    (24, 16, (4, 4), 7, 6), (16, 16, (4, 4), 9, 1), (16, 16, (4, 4), 9, 2), (16, 16, (4, 4), 9, 5),  # 4, 14, 18 dofs
    (16, 16, (4, 4), 1, 2), (16, 16, (4, 4), 3, 2), (16, 16, (4, 4), 8, 2), (16, 16, (2, 2), 4, 7),
    (16, 16, (4, 4), 16, 3), (16, 16, (4, 4), 11, 6),  # 32 and 22 dofs: remainders of the chunks of 0 and 6
    (256, 256, (4, 4), 6, 30), (256, 256, (4, 4), 7, 16),  # restriction by half chunks in FP64
    (256, 256, (4, 4), 16, 16),  # blocks of 335 MB in FP64, entry by entry
])
def test_coarse_operator_and_transfers_by_dofs(Lx, Lt, agg, ntv, nrhs):
    """D, P^H and P for any number of test vectors, incomplete groups of four right-hand sides
    included; the references on three of them."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(53)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    (ax, at), lx, lt = agg, Lx // agg[0], Lt // agg[1]
    # test vectors orthonormal on each (aggregate, chirality) block: the blocks of P
    B = np.linalg.qr(cn(lt * lx * 2, ax * at, ntv))[0]
    tv = B.reshape(lt, lx, 2, at, ax, ntv).transpose(0, 3, 1, 4, 2, 5).reshape(-1, ntv)
    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[np.ascontiguousarray(tv)])
    A = H.export(2, Dc=True)["Dc"]
    xf, xc = cn(nrhs, H.n(1)), cn(nrhs, H.n(2))
    rows = sorted({0, nrhs // 2, nrhs - 1})

    def aggregated(x):
        return x.reshape(-1, lt, at, lx, ax, 2).transpose(0, 1, 3, 5, 2, 4).reshape(-1, lt * lx * 2, ax * at)

    for prec, dt, tol in ((dmlmc.FP64, torch.complex128, 1e-13), (dmlmc.MIXED, torch.complex64, 1e-6)):
        f, c = (torch.as_tensor(v, device="cuda").to(dt) for v in (xf, xc))
        hf, hc = (t[rows].cpu().numpy().astype(np.complex128) for t in (f, c))
        for op, lv, src, shape, ref in (
                (dmlmc.OP_D, 2, c, c.shape, _blocks_apply(A, lx, lt, hc.T).T),
                (dmlmc.OP_RESTRICT, 1, f, c.shape, np.einsum("bri,qbr->qbi", B.conj(), aggregated(hf)).reshape(len(rows), -1)),
                (dmlmc.OP_PROLONG, 1, c, f.shape, np.einsum("bri,qbi->qbr", B, hc.reshape(len(rows), -1, ntv)))):
            out = H.apply(op, lv, src, torch.full(shape, float("nan"), dtype=dt, device="cuda"), prec=prec)
            assert torch.isfinite(torch.view_as_real(out)).all()
            out = out[rows].cpu().numpy()
            if op == dmlmc.OP_PROLONG:
                out = aggregated(out)
            err = [np.linalg.norm(o - r) / np.linalg.norm(r) for o, r in zip(out, ref)]
            assert max(err) <= tol, (prec, op, err)


@pytest.mark.parametrize("Lx,Lt,ntv,nrhs", [
    (16, 16, 1, 3), (16, 24, 2, 3), (24, 16, 7, 3), (16, 16, 9, 2),  # 2, 4 and 14 dofs prefetching, 18 in chunks
    (64, 64, 2, 257), (64, 64, 3, 257), (64, 64, 4, 160),  # 4, 6 and 8 dofs, many groups of right-hand sides
    (32, 32, 7, 321), (32, 32, 8, 300),  # 14 and 16 dofs, FP64 by directions
    (128, 128, 5, 65), (128, 128, 6, 48),  # 10 and 12 dofs, FP64 of the latter by directions
    (512, 512, 4, 3), (288, 288, 8, 5),  # FP64 entry by entry: 16384 sites of 8 dofs, 5184 of 16
    (160, 160, 16, 21), (256, 256, 16, 6),  # 32 dofs in chunks of 64 threads and entry by entry
    # rows of workgroups that are no multiple of 8 in number, several groups of right-hand sides
    (88, 24, 4, 34), (120, 72, 12, 40), (168, 104, 7, 34), (208, 248, 4, 12),
])
def test_coarse_gauss_seidel_forms(Lx, Lt, ntv, nrhs):
    """The forms of the sweep by dofs, sites and right-hand sides; bounds as above."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(47)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.3, [(4, 4), (2, 2)], [ntv, 1],
                        import_tv=[cn(2 * Lx * Lt, ntv), cn(Lx * Lt // 16 * 2 * ntv, 1)])
    H.solver_params(smoother_half=0)
    lx, lt, d = H.level_info(2)
    A = H.export(2, Dc=True)["Dc"]
    Ainv = np.linalg.inv(A[:, 0])
    t, x = np.divmod(np.arange(lx * lt), lx)
    b = cn(nrhs, H.n(2))
    for prec, dt, tol in ((dmlmc.FP64, torch.complex128, 1e-12), (dmlmc.MIXED, torch.complex64, 1e-4)):
        bd = torch.as_tensor(b, device="cuda").to(dt)
        out = H.apply(dmlmc.OP_SMOOTH, 2, bd, torch.zeros_like(bd), prec=prec, arg=1).cpu().numpy()
        bh = bd.cpu().numpy().astype(np.complex128).T
        y = np.zeros_like(bh)
        for color in (0, 1):
            r = (bh - _blocks_apply(A, lx, lt, y)).reshape(lx * lt, d, nrhs)
            on = (x + t) % 2 == color
            y.reshape(lx * lt, d, nrhs)[on] += (Ainv @ r)[on]
        err = np.linalg.norm(out.T - y, axis=0) / np.linalg.norm(y, axis=0)
        assert err.max() <= tol, (prec, err.max())


@pytest.mark.parametrize("k", [0, 4, 65])
@pytest.mark.parametrize("Lx,Lt,ntv,few", [(64, 64, 4, 1), (64, 40, 5, 1), (56, 48, 6, 1), (48, 48, 7, 1), (64, 32, 8, 3),
                                           (40, 32, 12, 1), (32, 32, 16, 2)])
def test_one_launch_and_separate_launches_agree(Lx, Lt, ntv, few, k):
    """Levels of 1600 to 2048 entries, 8 to 32 dofs, 24 steps: a few right-hand sides take the
    separate launches, a block of 64 the one launch, and in complex FP32 both give the same bits
    (set-ups depend on the order of the sums), inside and outside deflations included."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(41)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    ctx = dmlmc.Context(0)
    H = dmlmc.Hierarchy(ctx, rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [(4, 4)], [ntv], import_tv=[cn(2 * Lx * Lt, ntv)])
    n = H.n(2)
    H.solver_params(coarsest_iters=24, coarsest_iters_defl=24)
    if k:
        X = np.linalg.qr(cn(n, k))[0]
        defl = dmlmc.Deflation(H, 2, k, import_X=X, import_lambda=np.linspace(0.3, 2.0, k))
        H.set_deflation(defl)
    b = torch.as_tensor(cn(64, n), device="cuda").to(torch.complex64)
    ctx.timing(True)
    out = {}
    for name, x in (("few", b[:few]), ("block", b)):
        ctx.timing_reset()
        out[name] = H.apply(dmlmc.OP_VCYCLE, 2, x, torch.empty_like(x), prec=dmlmc.MIXED)
        assert ctx.timing_get("coarsest")[0] == (1 if name == "block" else 0)
    assert torch.equal(torch.view_as_real(out["few"]), torch.view_as_real(out["block"][:few]))


def test_fp64_basis_outside_lds():
    """1600 entries in complex FP64: a block of 64 takes the one launch, no basis vector of which
    fits into LDS, one vector the separate launches; both to 1e-11 as above, so 2e-11 apart."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(43)
    ctx = dmlmc.Context(0)
    tv = rng.standard_normal((2 * 64 * 40, 5)) + 1j * rng.standard_normal((2 * 64 * 40, 5))
    H = dmlmc.Hierarchy(ctx, rng.normal(0.0, 0.3, (2, 40, 64)), 0.1, [(4, 4)], [5], import_tv=[tv])
    H.solver_params(coarsest_iters=8)
    n = H.n(2)
    b = torch.as_tensor(rng.standard_normal((64, n)) + 1j * rng.standard_normal((64, n)), device="cuda")
    ctx.timing(True)
    x = H.apply(dmlmc.OP_VCYCLE, 2, b, torch.empty_like(b))
    assert ctx.timing_get("coarsest")[0] == 1
    for r in (0, 63):
        y = H.apply(dmlmc.OP_VCYCLE, 2, b[r:r + 1], torch.empty_like(b[:1]))
        assert float((x[r] - y[0]).norm() / y[0].norm()) <= 2e-11
    assert ctx.timing_get("coarsest")[0] == 1


@pytest.mark.parametrize("k", [0, 4])
@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("shape", ["16x8", "64x16"])
def test_nan_and_infinity_stay_in_their_right_hand_side(shape, prec, k):
    """The one-launch solve of a block with a NaN and an infinite entry: those two come out not
    finite, the others as without them."""
    import torch

    from paper_2211_15383_amd import dmlmc

    (Lx, Lt), agg, ntv = SHAPES[shape]
    rng = np.random.default_rng(59)

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.1, [agg], [ntv],
                        import_tv=[cn(2 * Lx * Lt, ntv)])
    n = H.n(2)
    H.solver_params(coarsest_iters=8)
    if k:
        defl = dmlmc.Deflation(H, 2, k, import_X=np.linalg.qr(cn(n, k))[0], import_lambda=np.linspace(0.3, 2.0, k))
        H.set_deflation(defl)
    p, dt = (dmlmc.MIXED, torch.complex64) if prec == "mixed" else (dmlmc.FP64, torch.complex128)
    b = torch.as_tensor(cn(5, n), device="cuda").to(dt)
    ref = H.apply(dmlmc.OP_VCYCLE, 2, b, torch.empty_like(b), prec=p)
    b[1, n // 3] = float("nan")
    b[3, n - 1] = float("inf")
    x = H.apply(dmlmc.OP_VCYCLE, 2, b, torch.empty_like(b), prec=p)
    finite = torch.isfinite(torch.view_as_real(x)).reshape(5, -1).all(1).tolist()
    assert finite == [True, False, True, False, True]
    assert torch.equal(torch.view_as_real(x[::2]), torch.view_as_real(ref[::2]))


def _to_blocks(x, lx, lt, d, agg):
    """[rows, n] of a level by (aggregate, chirality) blocks: [rows, blocks, entries of a block]."""
    ax, at = agg
    x = x.reshape(-1, lt // at, at, lx // ax, ax, 2, d // 2).transpose(0, 1, 3, 5, 2, 4, 6)
    return x.reshape(x.shape[0], lx * lt // (ax * at) * 2, -1)


def _from_blocks(x, lx, lt, d, agg):
    ax, at = agg
    x = x.reshape(-1, lt // at, lx // ax, 2, at, ax, d // 2).transpose(0, 1, 4, 2, 5, 3, 6)
    return x.reshape(x.shape[0], -1)


def _three_levels(rng, Lx, Lt, ntv, agg):
    """A hierarchy of imported test vectors, those of the second level orthonormal on their blocks;
    also the blocks."""
    from paper_2211_15383_amd import dmlmc

    def cn(*s):
        return rng.standard_normal(s) + 1j * rng.standard_normal(s)

    lx, lt, d = Lx // 4, Lt // 4, 2 * ntv[0]
    B = np.linalg.qr(cn(lx * lt // (agg[0] * agg[1]) * 2, agg[0] * agg[1] * ntv[0], ntv[1]))[0]
    tv2 = _from_blocks(B.transpose(2, 0, 1), lx, lt, d, agg).T
    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, Lt, Lx)), 0.3, [(4, 4), agg], list(ntv),
                        import_tv=[cn(2 * Lx * Lt, ntv[0]), np.ascontiguousarray(tv2)])
    return H, B


@pytest.mark.parametrize("Lx,Lt,ntv,agg,nrhs", [
    (64, 64, (5, 4), (4, 4), 5),   # 4 test vectors, an incomplete group of right-hand sides
    (64, 64, (4, 12), (4, 4), 3),  # 12: by chunks
    (64, 64, (7, 8), (2, 4), 4),   # 8 in the straight-line form
    (264, 264, (8, 8), (6, 6), 3),  # 8 by whole rows through LDS, a ragged last workgroup
])
def test_vcycle_with_presmoothing(Lx, Lt, ntv, agg, nrhs):
    """A V-cycle of the second of three levels, whose prolongation adds to the smoothed vector."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(61)
    H, B = _three_levels(rng, Lx, Lt, ntv, agg)
    m = 6
    H.solver_params(nu_pre=1, nu_post_coarse=1, smoother_half=0, coarsest_iters=m)
    lx, lt, d = H.level_info(2)
    lx3, lt3, _ = H.level_info(3)
    A, A3 = H.export(2, Dc=True)["Dc"], H.export(3, Dc=True)["Dc"]
    Ainv = np.linalg.inv(A[:, 0])
    t, x = np.divmod(np.arange(lx * lt), lx)
    b = rng.standard_normal((nrhs, H.n(2))) + 1j * rng.standard_normal((nrhs, H.n(2)))

    def sweep(y, bh):
        for color in (0, 1):
            r = (bh - _blocks_apply(A, lx, lt, y)).reshape(lx * lt, d, -1)
            on = (x + t) % 2 == color
            y.reshape(lx * lt, d, -1)[on] += (Ainv @ r)[on]

    # bounds of the coarsest solve, which is the least accurate part
    for prec, dt, tol in ((dmlmc.FP64, torch.complex128, 1e-11), (dmlmc.MIXED, torch.complex64, 2e-4)):
        bd = torch.as_tensor(b, device="cuda").to(dt)
        out = H.apply(dmlmc.OP_VCYCLE, 2, bd, torch.full_like(bd, float("nan")), prec=prec).cpu().numpy()
        bh = bd.cpu().numpy().astype(np.complex128).T
        y = np.zeros_like(bh)
        sweep(y, bh)
        r = _to_blocks((bh - _blocks_apply(A, lx, lt, y)).T, lx, lt, d, agg)
        bc = (r[:, :, None, :] @ B.conj()[None]).reshape(nrhs, -1)
        xc = np.stack([_gmres(lambda v: _blocks_apply(A3, lx3, lt3, v), v, m) for v in bc])
        y += _from_blocks((B[None] @ xc.reshape(nrhs, -1, ntv[1], 1))[..., 0], lx, lt, d, agg).T
        sweep(y, bh)
        err = np.linalg.norm(out.T - y, axis=0) / np.linalg.norm(y, axis=0)
        assert err.max() <= tol, (prec, err.max())


@pytest.mark.parametrize("Lx,Lt,ntv,nrhs", [
    (32, 32, 8, 9),     # 16 dofs, 64 sites: a wavefront per tile, through LDS
    (128, 128, 8, 8), (128, 128, 8, 20),  # 1024 sites, padded work vectors, one tile and two
    (256, 256, 8, 9),   # 4096 sites, one tile: straight from memory
    (256, 256, 8, 17),  # two tiles: both in one wavefront
    (128, 128, 8, 1), (128, 128, 8, 2), (128, 128, 8, 7),  # the scalar kernel
    (64, 64, 5, 1), (64, 64, 5, 2), (64, 64, 7, 6), (64, 64, 12, 2), (64, 64, 12, 5), (128, 128, 4, 5),
])
def test_refinement_residual(Lx, Lt, ntv, nrhs):
    """The relative residual that a solve of the second level reports is that of its solution (the
    residual form of the FP64 stencils, stored in FP32 at padded strides by mixed solves)."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(67)
    H, _ = _three_levels(rng, Lx, Lt, (ntv, 2), (2, 2))
    lx, lt, _ = H.level_info(2)
    A = H.export(2, Dc=True)["Dc"]
    b = torch.as_tensor(rng.standard_normal((nrhs, H.n(2))) + 1j * rng.standard_normal((nrhs, H.n(2))), device="cuda")
    # FP64: residuals of size 0.1 from sums rounded at 1e-15; mixed: each entry rounded to FP32
    for prec, tol in ((dmlmc.FP64, 1e-11), (dmlmc.MIXED, 1e-6)):
        X, st = H.solve(2, b, prec=prec, rtol=0.2)
        r = b.cpu().numpy() - _blocks_apply(A, lx, lt, X.cpu().numpy().T).T
        rel = np.linalg.norm(r, axis=1) / np.linalg.norm(b.cpu().numpy(), axis=1)
        assert st.converged and st.ir_steps >= 1 and rel.max() > 1e-4
        assert abs(st.relres_max - rel.max()) <= tol * rel.max(), (prec, st.relres_max, rel.max())


def test_block_larger_than_the_readback_buffer():
    """8200 right-hand sides: their norms (8 bytes each) exceed the pinned staging buffer."""
    import torch

    from paper_2211_15383_amd import dmlmc

    rng = np.random.default_rng(5)
    H = dmlmc.Hierarchy(dmlmc.Context(0), rng.normal(0.0, 0.3, (2, 8, 8)), 0.1, [(4, 4)], [2])
    n = H.n(1)
    b = torch.as_tensor(rng.standard_normal((8200, n)) + 0j, device="cuda")
    x, st = H.solve(1, b, prec=dmlmc.FP64, rtol=1e-10)
    r = b - H.apply(dmlmc.OP_D, 1, x, torch.empty_like(x))
    assert st.converged and float((r.norm(dim=1) / b.norm(dim=1)).max()) <= 1.01e-10

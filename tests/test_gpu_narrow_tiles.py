"""Queries in 32-query tiles (launches with at most one such tile per compute unit)
against the 64-query tiles, bit for bit, and against the FP64 oracle.

A query's arithmetic and the order of its sums do not depend on the tile, so the
first points of a large call, which runs in 64-query tiles, give the same bits as a
small call over them.  Sizes sit at the edges of a tile (1, 31, 32, 33, 64, 65), and
at the largest narrow launch.  Oracle tolerances are those of the precisions (see
test_gpu_parity.py)."""
import numpy as np
import pytest

from paper_2601_18548_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp32": (5e-5, 5e-5), "bf16x2": (1e-3, 1e-2), "bf16x2_f16": (1e-3, 1e-2), "bf16": (0.07, 0.08)}


@pytest.fixture(scope="module")
def gcdf():
    import paper_2601_18548_amd as g

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g.library()
    return g


@pytest.mark.parametrize("spheres", [False, True])
@pytest.mark.parametrize("width", [256, 512])
@pytest.mark.parametrize("precision", ["fp32", "bf16x2", "bf16x2_f16", "bf16"])
def test_narrow_tiles_match_wide_tiles_and_oracle(gcdf, oracle_mod, precision, width, spheres):
    w = wl.weights(width, 3, in_dim=wl.IN_DIM_SPHERE if spheres else wl.IN_DIM)
    big = 20000  # more 32-query tiles than compute units, whatever the knots
    p = wl.spheres(big, 5) if spheres else wl.points_patches(big, 5)
    k = wl.knots(3, 4)
    ctx = gcdf.Context(w.to_blob(), width, precision)
    kt, pt = torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda()
    dw, Jw = ctx.eval_grad(kt, pt)
    for Np in (1, 31, 32, 33, 64, 65, 1000):
        print("narrow %s W=%d spheres=%d Np=%d" % (precision, width, spheres, Np), flush=True)
        pn = pt[:Np].contiguous()
        d, J = ctx.eval_grad(kt, pn)
        assert torch.equal(d, dw[:, :Np]) and torch.equal(J, Jw[:, :Np])
        assert torch.equal(ctx.eval(kt, pn), d)
        dmin, am, Jm = ctx.knot_min(kt, pn, with_jacobian=True)
        assert torch.equal(dmin, d.min(dim=1).values)
        assert torch.equal(am.long(), torch.from_numpy(d.cpu().numpy().argmin(1)).cuda())
        # (pair lists of the pure BF16 point network of width 256, the training
        # configuration, take the input layer from split BF16 products)
        if precision != "bf16" or width != 256 or spheres:
            assert torch.equal(Jm, J[torch.arange(3, device="cuda"), am.long()])
    dr, Jr = oracle_mod.eval_grad(w.to_blob(), k, p[:65])
    d, J = (t.cpu().numpy().astype(np.float64) for t in ctx.eval_grad(kt, pt[:65].contiguous()))
    nr = np.linalg.norm(Jr.reshape(-1, 9), axis=1)
    rj = np.linalg.norm((J - Jr).reshape(-1, 9), axis=1) / np.maximum(nr, 1e-3 * np.median(nr))
    assert np.abs(d - dr).max() <= TOL[precision][0] and rj.max() <= TOL[precision][1]
    ctx.close()


@pytest.mark.parametrize("N,Np,radius", [(1, 1, 9.0), (5, 33, 9.0), (40, 100, 0.7), (120, 40, 9.0)])
def test_narrow_csr_rows_match_dense(gcdf, N, Np, radius):
    w = wl.weights(256, 8)
    ctx = gcdf.Context(w.to_blob(), 256, "bf16x2_f16")
    kt = torch.from_numpy(wl.trajectory(max(N, 2), 2)[:N].copy()).cuda()
    pt = torch.from_numpy(wl.points_uniform(Np, 3)).cuda()
    off, idx = ctx.partition(kt, pt, radius)
    c, J = ctx.eval_grad_csr(kt, pt, off, idx)
    big = torch.from_numpy(np.concatenate([wl.points_uniform(Np, 3), wl.points_uniform(20000, 4)])).cuda()
    d, Jd = ctx.eval_grad(kt, big)  # 64-query tiles
    knot = torch.repeat_interleave(torch.arange(N, device="cuda"), off[1:] - off[:-1])
    assert torch.equal(c, d[knot, idx.long()]) and torch.equal(J, Jd[knot, idx.long()])
    ctx.close()


@pytest.mark.parametrize("B", [1, 32, 33, 5001])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_narrow_pair_lists_match_the_training_tiles(gcdf, precision, B):
    """The separate forward of a small batch (32-sample tiles) gives the distances of
    the fused loss (64-sample training tiles)."""
    from paper_2601_18548_amd import train

    tr = train.Trainer(256, precision, 8192)
    params = train.flat_params(wl.weights(256, 4, bf16_hidden=False))
    k, p, noise = wl.training_batch(B, 6)
    kt, pt, y = torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda(), torch.from_numpy(noise).cuda()
    d = tr.forward(params, kt, pt)
    d2 = torch.empty_like(d)
    tr.mse(params, kt, pt, y, d=d2)
    torch.cuda.synchronize()
    assert torch.equal(d, d2)
    tr.close()


@pytest.mark.parametrize("spheres", [False, True])
@pytest.mark.parametrize("precision", ["bf16x2", "bf16x2_f16"])
def test_one_round_workgroups_match_larger_launches(gcdf, precision, spheres):
    """Width 256, split modes: launches of up to one 64-query tile per compute unit (129
    to 256 of them here) run 8-wave workgroups, larger ones two 4-wave ones per compute
    unit.  The sums' order does not depend on the waves, so the bits agree."""
    w = wl.weights(256, 3, in_dim=wl.IN_DIM_SPHERE if spheres else wl.IN_DIM)
    p = wl.spheres(20000, 5) if spheres else wl.points_patches(20000, 5)
    ctx = gcdf.Context(w.to_blob(), 256, precision)
    kt, pt = torch.from_numpy(wl.knots(3, 4)).cuda(), torch.from_numpy(p).cuda()
    dw, Jw = ctx.eval_grad(kt, pt)
    for Np in (2753, 3841, 5408, 5440):
        print("one round %s spheres=%d Np=%d" % (precision, spheres, Np), flush=True)
        pn = pt[:Np].contiguous()
        d, J = ctx.eval_grad(kt, pn)
        assert torch.equal(d, dw[:, :Np]) and torch.equal(J, Jw[:, :Np])
        assert torch.equal(ctx.eval(kt, pn), d)
        dmin, am, Jm = ctx.knot_min(kt, pn, with_jacobian=True)
        assert torch.equal(dmin, d.min(dim=1).values)
        assert torch.equal(Jm, J[torch.arange(3, device="cuda"), am.long()])
    off, idx = ctx.partition(kt, pt[:5000].contiguous(), 1e3)  # every point in range: 237 gathered tiles at most
    c, Jc = ctx.eval_grad_csr(kt, pt[:5000].contiguous(), off, idx)
    assert torch.equal(c, dw[:, :5000].reshape(-1)) and torch.equal(Jc, Jw[:, :5000].reshape(-1, 9))
    ctx.close()


@pytest.mark.parametrize("N,M", [(128, 1025), (150, 700), (250, 300)])
def test_csr_tiles_near_one_round_match_dense(gcdf, N, M):
    """Width 256, split modes: CSR queries whose likely number of tiles and its bound lie
    on either side of the compute units' number, also with more tiles than one round."""
    w = wl.weights(256, 9)
    ctx = gcdf.Context(w.to_blob(), 256, "bf16x2_f16")
    kt, pt = torch.from_numpy(wl.trajectory(N, 1)).cuda(), torch.from_numpy(wl.points_patches(M, 2)).cuda()
    off, idx = ctx.partition(kt, pt, 1.0)
    print("csr %d x %d: %d rows" % (N, M, idx.shape[0]), flush=True)
    c, J = ctx.eval_grad_csr(kt, pt, off, idx)
    d, Jd = ctx.eval_grad(kt, pt)
    knot = torch.repeat_interleave(torch.arange(N, device="cuda"), off[1:] - off[:-1])
    assert torch.equal(c, d[knot, idx.long()]) and torch.equal(J, Jd[knot, idx.long()])
    ctx.close()

"""Per-knot minimum (the constraint f - delta >= 0 of eq. optimization-in-general,
Sec. IV-A, holds for every point of a knot iff it holds for the minimum) against
the FP64 oracle's minimum, through gcdf_knot_min and gcdf_query.

The oracle's d goes through oracle.knot_min (plain loop, lowest index on ties).
For every knot:
  * |dmin - m_ref| <= tol_d (the precision's value bar);
  * argmin equals the oracle's, unless the oracle's best-vs-second gap is below
    2 tol_d, where another point is an equally valid answer at the GPU's
    precision; then d_ref at the GPU's argmin is within 2 tol_d of m_ref;
  * Jmin is within the Jacobian bar of the oracle's J at the GPU's argmin.
Tolerances as the parity tests: FP32 (5e-5, 5e-5), split modes (1e-3, 1e-2).
"""
import numpy as np
import pytest

from paper_2601_18548_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp32": (5e-5, 5e-5), "bf16x2": (1e-3, 1e-2), "bf16x2_f16": (1e-3, 1e-2)}


@pytest.fixture(scope="module")
def gcdf():
    import paper_2601_18548_amd as g

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g.library()
    return g


def rel_j_err(J, Jr, scale):
    J = J.reshape(-1, 9).astype(np.float64)
    Jr = Jr.reshape(-1, 9)
    return np.linalg.norm(J - Jr, axis=1) / np.maximum(np.linalg.norm(Jr, axis=1), 1e-3 * scale)


def check_min(oracle_mod, name, dr, Jr, dmin, am, Jm, tol_d, tol_j):
    """dr (K, Np), Jr (K, Np, 9): the oracle's; dmin, am, Jm: the GPU's."""
    K, Np = dr.shape
    m_ref, a_ref = oracle_mod.knot_min(dr)
    srt = np.sort(dr, axis=1)
    gap = srt[:, 1] - srt[:, 0] if Np > 1 else np.full(K, np.inf)
    assert am.dtype == np.int32 and np.all((am >= 0) & (am < Np))
    dm_err = np.abs(dmin - m_ref)
    same = am == a_ref
    near = gap < 2 * tol_d
    print("%s: |dmin - m_ref| max %.3e, argmin equal on %d of %d knots (%d near-ties)"
          % (name, dm_err.max(), same.sum(), K, near.sum()), flush=True)
    assert dm_err.max() <= tol_d
    assert np.all(same | near), np.nonzero(~(same | near))[0]
    kk = np.arange(K)
    assert np.all(dr[kk, am] <= m_ref + 2 * tol_d)
    if Jm is not None:
        nr = np.linalg.norm(Jr.reshape(-1, 9), axis=1)
        rj = rel_j_err(Jm, Jr[kk, am], np.median(nr))
        print("%s: Jmin rel err max %.3e" % (name, rj.max()), flush=True)
        assert np.all(np.isfinite(Jm)) and rj.max() <= tol_j


def gpu_min(g, ctx, kt, pt, via):
    K = kt.shape[0]
    if via == "knot_min":
        dmin, am, Jm = ctx.knot_min(kt, pt, with_jacobian=True)
    else:  # gcdf_query with only the minimum outputs
        dmin = torch.empty(K, dtype=torch.float32, device="cuda")
        am = torch.empty(K, dtype=torch.int32, device="cuda")
        Jm = torch.empty((K, 9), dtype=torch.float32, device="cuda")
        ctx.query(kt, pt, dmin=dmin, argmin=am, Jmin=Jm)
    torch.cuda.synchronize()
    return dmin.cpu().numpy(), am.cpu().numpy(), Jm.cpu().numpy()


@pytest.mark.parametrize("precision", ["fp32", "bf16x2", "bf16x2_f16"])
@pytest.mark.parametrize("width", [256, 512])
def test_knot_min_matches_oracle_small(gcdf, oracle_mod, precision, width):
    """16 x 64 (the small workload's sizes) and a ragged 3 x 100 case."""
    w = wl.weights(width, seed=41)
    tol_d, tol_j = TOL[precision]
    ctx = gcdf.Context(w.to_blob(), width, precision)
    for K, Np, seed in [(16, 64, 1), (3, 100, 7)]:
        k = wl.knots(K, seed)
        p = wl.points_uniform(Np, seed + 1)
        print("case width=%d precision=%s K=%d Np=%d" % (width, precision, K, Np), flush=True)
        dr, Jr = oracle_mod.eval_grad(w.to_blob(), k, p)
        kt, pt = torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda()
        for via in ("knot_min", "query"):
            dmin, am, Jm = gpu_min(gcdf, ctx, kt, pt, via)
            check_min(oracle_mod, "w%d %s %dx%d %s" % (width, precision, K, Np, via), dr, Jr, dmin, am, Jm, tol_d, tol_j)
    ctx.close()


def test_knot_min_exact_ties_match_oracle_rule(gcdf, oracle_mod):
    """Each point three times over: the oracle's d ties exactly across the copies
    and its loop keeps the first copy; the GPU must return an index in the first
    copy, the oracle's whenever the distinct points are not near-tied."""
    w = wl.weights(256, seed=42)
    k = wl.knots(6, 4)
    base = wl.points_uniform(70, 5)
    p = np.concatenate([base, base, base], 0)
    dr, Jr = oracle_mod.eval_grad(w.to_blob(), k, p)
    m_ref, a_ref = oracle_mod.knot_min(dr)
    assert np.all(a_ref < 70)
    ctx = gcdf.Context(w.to_blob(), 256, "bf16x2")
    kt, pt = torch.from_numpy(k).cuda(), torch.from_numpy(p).cuda()
    dmin, am, Jm = gpu_min(gcdf, ctx, kt, pt, "knot_min")
    assert np.all(am < 70)
    check_min(oracle_mod, "ties", dr[:, :70], Jr[:, :70], dmin, am, Jm, *TOL["bf16x2"])


def test_knot_min_benchmark_workload_slice(gcdf, oracle_mod):
    """4 knots x all 16,384 patch points of the 128 x 16,384 W=512 benchmark
    workload, in the benchmark precision (65,536 oracle pairs), through both
    entry points; the minimum is also the one of the full 128-knot launch."""
    wk = wl.workload("bf16")
    sel = np.array([0, 41, 87, wk.K - 1])
    k = np.ascontiguousarray(wk.knots[sel])
    print("case benchmark slice: K=%d Np=%d width=%d %s" % (len(k), wk.Np, wk.width, wk.precision), flush=True)
    dr, Jr = oracle_mod.eval_grad(wk.weights.to_blob(), k, wk.points)
    ctx = gcdf.Context(wk.weights.to_blob(), wk.width, wk.precision)
    kt, pt = torch.from_numpy(k).cuda(), torch.from_numpy(wk.points).cuda()
    tol_d, tol_j = TOL[wk.precision]
    for via in ("knot_min", "query"):
        dmin, am, Jm = gpu_min(gcdf, ctx, kt, pt, via)
        check_min(oracle_mod, "benchmark slice %s" % via, dr, Jr, dmin, am, Jm, tol_d, tol_j)
    full_t = torch.from_numpy(wk.knots).cuda()
    fmin, fam, fJm = gpu_min(gcdf, ctx, full_t, pt, "query")
    assert np.array_equal(fmin[sel], dmin) and np.array_equal(fam[sel], am) and np.array_equal(fJm[sel], Jm)
    ctx.close()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("with_jacobian", [False, True])
def test_minimum_keys_start_afresh(noalloc, with_jacobian):
    """The minimum's keys are set back by the call that used them: a call over a subset
    of the points (whose minimum is higher) sees nothing of a call over all of them,
    also with other knot counts in between."""
    import paper_2601_18548_amd as g

    w = wl.weights(256, 11)
    ctx = g.Context(w.to_blob(), 256, "bf16x2_f16")
    pt = torch.from_numpy(wl.points_patches(3000, 12)).cuda()
    kt = torch.from_numpy(wl.knots(300, 13)).cuda()
    for K, Np in ((300, 3000), (7, 1), (300, 40), (33, 3000), (300, 1), (1, 65)):
        k, p = kt[:K].contiguous(), pt[:Np].contiguous()
        d, J = ctx.eval_grad(k, p)
        dmin = torch.empty(K, device="cuda")
        am = torch.empty(K, dtype=torch.int32, device="cuda")
        Jm = torch.empty((K, 9), device="cuda") if with_jacobian else None
        ctx.query(k, p, dmin=dmin, argmin=am, Jmin=Jm, noalloc=noalloc)
        assert torch.equal(dmin, d.min(dim=1).values)
        assert np.array_equal(am.cpu().numpy(), d.cpu().numpy().argmin(axis=1))
        if with_jacobian:
            assert torch.equal(Jm, J[torch.arange(K, device="cuda"), am.long()])
    ctx.close()

"""Table I training loss on the GPU (gcdf_train_table1) against the FP64 oracle.

FP32 trainer: loss terms within 1e-4 relative, weight gradient per parameter array
within 1e-5 relative (norm-wise), printed; with only the value term switched on the
gradient equals the MSE trainer's; two calls agree bitwise; Adam on the loss
lowers it.
"""
import numpy as np
import pytest

from paper_2601_18548_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NAMES = ["W1", "b1", "W2", "b2", "W3", "b3", "W4", "b4", "w_out", "b_out"]
M_DIAG = [4.0, 4.0, 1.0, 1.0, 1.0, 1.0, 1.0, 1.0, 1.0]


@pytest.fixture(scope="module")
def tr_mod():
    import paper_2601_18548_amd as g
    from paper_2601_18548_amd import train

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g.library()
    return train


def _split(flat, w):
    out, off = [], 0
    for a in w.flat_params():
        out.append(flat[off:off + a.size].reshape(a.shape))
        off += a.size
    return out


def _case(B, seed):
    k, p, _ = wl.training_batch(B, seed)
    r = np.random.default_rng(seed + 1)
    return k, p, r.normal(size=B).astype(np.float32), r.normal(size=(B, 9)).astype(np.float32)


def _cuda(*arrs):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]


def test_loss_and_gradient_match_oracle(tr_mod, oracle_mod):
    w = wl.weights(256, seed=81, bf16_hidden=False)
    B = 300
    k, p, fs, Js = _case(B, 4)
    tr = tr_mod.Trainer(256, "fp32", max_batch=B)
    params = tr_mod.flat_params(w)
    kt, pt, ft, Jt = _cuda(k, p, fs, Js)
    losses, g = tr.table1(params, kt, pt, ft, Jt, M_DIAG)
    torch.cuda.synchronize()
    total, L, gref = oracle_mod.table1_grad(w.to_blob(), k, p, fs, Js, M_DIAG)
    lg = losses.cpu().numpy()
    print("losses gpu", lg, "oracle", L, total, flush=True)
    np.testing.assert_allclose(lg[:4], L, rtol=1e-4)
    assert lg[4] == pytest.approx(total, rel=1e-4)
    for name, a, b in zip(NAMES, _split(g.cpu().numpy(), w), gref):
        err = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
        print("%-5s rel err %.2e" % (name, err), flush=True)
        assert err <= 1e-5, name


def test_loss_and_gradient_match_oracle_multi_chunk(tr_mod, oracle_mod):
    """6,181 samples: 20 weight-gradient GEMM chunks of 320 on 256 compute units
    (the second product accumulated into the first), the sums of 97 workgroups, a ragged last
    tile; against the oracle's straight sums, then central differences of the
    GPU's own loss."""
    w = wl.weights(256, seed=86, bf16_hidden=False)
    B = 6181
    k, p, fs, Js = _case(B, 9)
    tr = tr_mod.Trainer(256, "fp32", max_batch=B)
    params = tr_mod.flat_params(w)
    kt, pt, ft, Jt = _cuda(k, p, fs, Js)
    print("case Table I multi-chunk B=%d" % B, flush=True)
    losses, g = tr.table1(params, kt, pt, ft, Jt, M_DIAG)
    torch.cuda.synchronize()
    total, L, gref = oracle_mod.table1_grad(w.to_blob(), k, p, fs, Js, M_DIAG)
    lg = losses.cpu().numpy()
    print("losses gpu", lg, "oracle", L, total, flush=True)
    np.testing.assert_allclose(lg[:4], L, rtol=1e-4)
    assert lg[4] == pytest.approx(total, rel=1e-4)
    gn = g.cpu().numpy()
    for name, a, b in zip(NAMES, _split(gn, w), gref):
        err = np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)
        print("B=%d %-5s rel err %.2e" % (B, name, err), flush=True)
        assert err <= 1e-5, name
    # central differences of the device loss (FP32 sums over 6,181 samples)
    picks, off = [], 0
    for a in w.flat_params():
        seg = np.abs(gn[off:off + a.size])
        picks.append(off + int(np.argmax(seg)))
        off += a.size
    h = 2e-3
    for i in picks:
        pp, pm = params.clone(), params.clone()
        pp[i] += h
        pm[i] -= h
        lp = float(tr.table1(pp, kt, pt, ft, Jt, M_DIAG)[0][4])
        lm = float(tr.table1(pm, kt, pt, ft, Jt, M_DIAG)[0][4])
        fd = (lp - lm) / (2 * h)
        print("FD param %d: fd %.6e grad %.6e" % (i, fd, gn[i]), flush=True)
        assert abs(fd - gn[i]) <= 5e-3 * abs(gn[i]) + 2e-6 * abs(float(lg[4])) / h, (i, fd, gn[i])


def test_value_term_alone_equals_mse_gradient(tr_mod):
    w = wl.weights(256, seed=82, bf16_hidden=False)
    B = 1000
    k, p, fs, Js = _case(B, 5)
    tr = tr_mod.Trainer(256, "fp32", max_batch=B)
    params = tr_mod.flat_params(w)
    kt, pt, ft, Jt = _cuda(k, p, fs, Js)
    _, g1 = tr.table1(params, kt, pt, ft, Jt, M_DIAG, lam=(1.0, 0.0, 0.0, 0.0))
    d = tr.forward(params, kt, pt)
    g2 = tr.backward(params, kt, pt, (2.0 * (d - ft) / B).contiguous())
    torch.cuda.synchronize()
    a, b = g1.cpu().numpy(), g2.cpu().numpy()
    assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b)


def test_deterministic_and_descends(tr_mod):
    teacher = wl.weights(256, seed=83, bf16_hidden=False)
    student = wl.weights(256, seed=84, bf16_hidden=False)
    B = 2048
    k, p, _, _ = _case(B, 6)
    tr = tr_mod.Trainer(256, "fp32", max_batch=B)
    kt, pt = _cuda(k, p)
    # targets: the teacher's distances and configuration gradients (one query per sample)
    import paper_2601_18548_amd as g

    ctx = g.Context(teacher.to_blob(), 256, "fp32")
    ki = torch.arange(B, dtype=torch.int64, device="cuda")
    d, J = [], []
    for i in range(0, B, 256):  # pairs (knot i, point i) as 1 x 1 queries in blocks
        kk, pp = kt[i:i + 256], pt[i:i + 256]
        dd, JJ = ctx.eval_grad(kk, pp)
        d.append(torch.diagonal(dd))
        J.append(JJ[torch.arange(len(kk)), torch.arange(len(kk))])
    ft, Jt = torch.cat(d).contiguous(), torch.cat(J).contiguous()
    params = tr_mod.flat_params(student).requires_grad_(True)
    l1, g1 = tr.table1(params.detach(), kt, pt, ft, Jt, M_DIAG)
    l2, g2 = tr.table1(params.detach(), kt, pt, ft, Jt, M_DIAG)
    assert torch.equal(g1, g2) and torch.equal(l1, l2)
    opt = tr_mod.Adam(params, lr=2e-3)
    first = None
    for _ in range(40):
        losses, gr = tr.table1(params.detach(), kt, pt, ft, Jt, M_DIAG)
        params.grad = gr
        opt.step()
        first = float(losses[4]) if first is None else first
    last = float(tr.table1(params.detach(), kt, pt, ft, Jt, M_DIAG)[0][4])
    print("Table I loss %.4f -> %.4f" % (first, last), flush=True)
    assert last < 0.7 * first


def test_bf16_trainer_is_rejected(tr_mod):
    import paper_2601_18548_amd as g

    tr = tr_mod.Trainer(256, "bf16", max_batch=64)
    w = wl.weights(256, seed=85)
    k, p, fs, Js = _case(64, 7)
    kt, pt, ft, Jt = _cuda(k, p, fs, Js)
    with pytest.raises(g.GcdfError):
        tr.table1(tr_mod.flat_params(w), kt, pt, ft, Jt, M_DIAG)


def test_small_trainer_needs_little_memory(tr_mod):
    """The workspaces follow the largest batch, not the device: one tile's worth of Table I
    scratch (0.7 MiB) and sums, not every compute unit's (360 MiB)."""
    params, args = tr_mod.flat_params(wl.weights(256, seed=82, bf16_hidden=False)), _cuda(*_case(64, 5))

    def used():
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        tr = tr_mod.Trainer(256, "fp32", max_batch=64)
        tr.table1(params, *args, M_DIAG)
        torch.cuda.synchronize()
        after = torch.cuda.mem_get_info()[0]
        tr.close()
        return before - after

    used()  # the kernels' own first-use allocations
    assert used() <= 32 << 20  # a dozen small allocations of at most 2 MiB granularity each

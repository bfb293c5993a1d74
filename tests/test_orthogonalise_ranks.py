"""P_hat of the Cholesky-QR route against 64 bits at every rank that has its own code: panels around the height of a workgroup's
rows, shorter than the rank allows, of several workgroups, with a zero column, factorised in the sums' launch and in one of its own."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

SHAPES = [(255, 65), (256, 66), (257, 68), (5, 65), (8, 67), (3001, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 6, 7, 8])
def test_p_hat(rank, fused):
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    plan = B.Plan(SHAPES, rank, 2)
    for key, value in (("one_sweep", 0), ("ortho_rows", 0), ("gram_fused", fused)):
        plan.set_tuning(key, value)
    s = plan.sizes
    gen = torch.Generator(device=dev)
    gen.manual_seed(rank)
    grad = torch.randn(2 * s.grad_stride, generator=gen, device=dev)
    err = torch.randn(2 * s.err_stride, generator=gen, device=dev)
    q = torch.randn(s.q_elems, generator=gen, device=dev)
    dead = 1 if rank > 2 else None   # a column of Q, and so of P, that is zero
    qs = []
    for t, (n, m) in enumerate(SHAPES):
        _, _, q_off, r = plan.offsets(t)
        Q = q[q_off: q_off + m * r].view(m, r)
        if dead is not None:
            Q[:, dead] = 0.0
        qs.append(Q.double().cpu().numpy())
    mats = [np.stack([(grad[w * s.grad_stride + plan.offsets(t)[0]:][: n * m] + err[w * s.err_stride + plan.offsets(t)[0]:][: n * m])
                      .double().cpu().numpy().reshape(n, m) for w in range(2)]) for t, (n, m) in enumerate(SHAPES)]
    p = torch.full((s.p_elems,), float("nan"), device=dev)
    ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
    plan.compress(grad, err, q, p, ws, stream)
    plan.check(stream)
    torch.cuda.synchronize()
    for t, (n, m) in enumerate(SHAPES):
        _, p_off, _, r = plan.offsets(t)
        got = p[p_off: p_off + n * r].double().cpu().numpy().reshape(n, r)
        live = [c for c in range(r) if c != dead]
        if dead is not None:
            assert (got[:, dead] == 0.0).all()
        # orthonormal to the rounding of P_hat's own entries: sum |x_i| |y_i| 2^-24 on either side, at most 2^-23 by Cauchy-Schwarz, and as
        # much again for the fp64 rounding, which a well conditioned panel does not reach
        gram = got[:, live].T @ got[:, live]
        panel = mats[t].mean(0) @ qs[t][:, live]
        cond = np.linalg.cond(panel)
        assert np.abs(gram - np.eye(len(live))).max() <= 2.0 ** -22 + cond ** 2 * 2.0 ** -50, (t, n, m)
        # P is summed in fp32 (m addends of two workers, in some order, from an M rounded once): at most (m + 4) 2^-24 of the sum of
        # the absolute values; a QR factor moves by at most 2 cond times the panel's relative change
        change = (m + 4) * 2.0 ** -24 * np.linalg.norm(np.abs(mats[t]).mean(0) @ np.abs(qs[t][:, live])) / np.linalg.norm(panel, 2)
        want, R = np.linalg.qr(panel)
        want = want * np.sign(np.diag(R))
        assert np.linalg.norm(got[:, live] - want) <= 2 * cond * change + 2.0 ** -23 * np.sqrt(len(live)), (t, n, m)

"""The one walk over M on the GPU: distance from 64 bits on the matrix-core plans, infinities and NaN, the widest rows with many workers
and several iterations."""
import pytest

torch = pytest.importorskip("torch")


def _plan(shapes, rank, workers, bf16, keys):
    from paper_1905_13727_amd import binding as B
    plan = B.Plan(shapes, rank, workers, B.PSGD_BF16 if bf16 else B.PSGD_F32, B.PSGD_F32)
    for key, value in keys.items():
        plan.set_tuning(key, value)
    return plan


def _gen(seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    return gen


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3000, 1024), (700, 8192), (2000, 2052), (4000, 260)])
def test_matrix_core_walk_is_no_further_from_64_bits_than_three(shape):
    """P, Q and Delta' of one psgd_step of a matrix-core plan, in the one walk and in the three, against torch's own products in 64 bits
    on a planted spectrum.  Room of a tenth: the rounding errors of one draw.  Both sum their products in fp64, so what is left are the
    roundings of P, Q and Delta' to fp32 (6e-8 each at most, a third of it on average) and of M: under 1.5e-7 for P and Q; Q of the three
    walks is a sum in fp32."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev, (n, m), rank = torch.device("cuda:0"), shape, 4
    stream = torch.cuda.current_stream(dev).cuda_stream
    gen = _gen(9)
    U, V = (torch.randn(k, 8, generator=gen, device=dev) / k ** 0.5 for k in shape)
    grad = ((U / torch.arange(1, 9, device=dev)) @ V.T + 0.01 / m ** 0.5 * torch.randn(n, m, generator=gen, device=dev)).to(torch.bfloat16)
    err0 = 0.017 / m ** 0.5 * torch.randn(n, m, generator=gen, device=dev)
    q0 = (V[:, :rank] / torch.arange(1, rank + 1, device=dev) + 0.01 / m ** 0.5 * torch.randn(m, rank, generator=gen, device=dev)).contiguous()
    M = grad.double() + err0.double()
    P = M @ q0.double()
    for k in range(rank):
        for j in range(k):
            P[:, k] -= (P[:, j] @ P[:, k]) * P[:, j]
        P[:, k] /= P[:, k].norm()
    Q = M.T @ P
    far = {}
    for one in (1, 0):
        plan = _plan([shape], rank, 1, True, {"bf16_valu": 0, "one_sweep": one})
        s = plan.sizes
        assert plan.path() == "matrix cores" and plan.one_sweep()[0] == bool(one)
        g, e = torch.zeros(s.grad_stride, dtype=torch.bfloat16, device=dev), torch.zeros(s.err_stride, device=dev)
        g[: n * m], e[: n * m] = grad.view(-1), err0.view(-1)
        q, p, out = q0.clone().view(-1), torch.zeros(s.p_elems, device=dev), torch.zeros(s.out_elems, device=dev)
        ws = torch.empty(s.workspace_bytes // 4 + 64, device=dev)
        plan.step(g, e, q, p, out, ws, stream)
        plan.check(stream)
        rel = lambda x, y: float((x.double().view(-1) - y.reshape(-1)).norm() / y.norm())
        far[one] = (rel(p[: n * rank], P), rel(q[: m * rank], Q), rel(out[: n * m], P @ Q.T))
    assert all(a <= 1.1 * b for a, b in zip(far[1], far[0])), far
    assert max(far[1][:2]) <= 1.5e-7, far


@pytest.mark.gpu
@pytest.mark.parametrize("wide,workers,rank", [(False, 1, 2), (False, 3, 4), (False, 1, 4), (True, 1, 4)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan"), 3.0e38])
def test_non_finite_gradients(wide, workers, rank, value):
    """An element that is not finite makes the same outputs non-finite as in the walks of the other route, and touches no other matrix:
    those are what they are without it, bit for bit.  Where only products overflow (3e38), what the other route gives finite is finite: the
    one walk's products of the mean, and its fp64 sums, overflow later."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    shapes = [(40, 1024), (130, 300), (9, 772), (64, 36)]
    got = {}
    for one in (1, 0):
        for bad in (True, False):
            plan = _plan(shapes, rank, workers, wide, {"one_sweep": one, **({"bf16_valu": 0} if wide else {"resident": 0})})
            s, gen = plan.sizes, _gen(4)
            grad = torch.randn(workers * s.grad_stride, generator=gen, device=dev)
            if bad:
                grad[(workers - 1) * s.grad_stride + plan.offsets(1)[0] + 7 * 300 + 5] = value
            grad = grad.to(torch.bfloat16 if wide else torch.float32)
            err, q = 0.5 * torch.randn(workers * s.err_stride, generator=gen, device=dev), torch.randn(s.q_elems, generator=gen, device=dev)
            p, out = torch.zeros(s.p_elems, device=dev), torch.zeros(s.out_elems, device=dev)
            ws = torch.empty(s.workspace_bytes // 4 + 64, device=dev)
            plan.step(grad, err, q, p, out, ws, stream)
            plan.check(stream)
            assert plan.one_sweep()[0] == bool(one)
            got[one, bad] = (plan, err, q, p, out)
    for t, (n, m) in enumerate(shapes):
        off, p_off, q_off, r = got[1, True][0].offsets(t)
        at = [(1, w * s.err_stride + off, n * m) for w in range(workers)] + [(2, q_off, m * r), (3, p_off, n * r), (4, off, n * m)]
        for i, a, size in at:
            x, y, clean = (got[k][i][a: a + size] for k in ((1, True), (0, True), (1, False)))
            if t == 1:
                x, y = torch.isfinite(x), torch.isfinite(y)
                assert torch.equal(x, y) if value != 3.0e38 else bool((x | ~y).all()), (t, i)
            else:
                assert torch.equal(x, clean) and torch.isfinite(x).all(), (t, i)


@pytest.mark.gpu
@pytest.mark.parametrize("shapes,rank,workers,its", [([(70, 4096), (33, 3000), (9, 2052)], 4, 5, 3), ([(41, 3072), (130, 4095), (5, 3070)], 2, 9, 4),
                                                     ([(300, 2304)], 3, 17, 2)])
def test_widest_rows_with_many_workers_and_iterations(shapes, rank, workers, its):
    """Rows of eight wavefronts, products of the mean over many workers, several iterations: the one walk against the two.  fp32 sums of at
    most 4096 products in other orders, times the condition of random panels, which every iteration brings down."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    got = []
    for one in (1, 0):
        plan = _plan(shapes, rank, workers, False, {"one_sweep": one})
        s, gen = plan.sizes, _gen(2)
        grad, err = torch.randn(workers * s.grad_stride, generator=gen, device=dev), 0.5 * torch.randn(workers * s.err_stride, generator=gen, device=dev)
        q, p, out = torch.randn(s.q_elems, generator=gen, device=dev), torch.zeros(s.p_elems, device=dev), torch.zeros(s.out_elems, device=dev)
        ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
        for _ in range(2):
            plan.step_iterations(grad, err, q, p, out, ws, its, stream)
        plan.check(stream)
        assert plan.one_sweep()[0] == bool(one)
        got.append((plan, q, p, out))
    for t, (n, m) in enumerate(shapes):
        off, p_off, q_off, r = got[0][0].offsets(t)
        for i, a, size in ((1, q_off, m * r), (2, p_off, n * r), (3, off, n * m)):
            x, y = got[0][i][a: a + size], got[1][i][a: a + size]
            assert torch.isfinite(x).all() and float((x - y).norm()) <= 2e-5 * float(y.norm()), (t, i)

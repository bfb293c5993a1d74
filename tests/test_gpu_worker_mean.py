"""Several workers on the streaming kernels: the products are taken of the mean over the workers' M (one mean matrix,
plan-owned).  Compared with the general path, which multiplies every worker's M by itself: the same plan with the
one-launch orthogonalisation switched off takes it."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# every access width (rows of a multiple of 4, of 2, odd), rows shorter and longer than a column chunk, one and two
# rows, fewer rows than a tile and one more than one, a vector
SHAPES = [(64, 576), (17, 1028), (33, 650), (2, 130), (65, 257), (1, 3), (130, 63), (77,), (300, 5)]


@pytest.mark.parametrize("rank,workers,grad_bf16,call", [
    (1, 3, False, "step"), (2, 3, False, "split"), (3, 16, False, "step"), (4, 4, True, "iterations"),
    (5, 5, False, "iterate"), (8, 3, True, "step"), (8, 4, False, "iterations"), (2, 4, False, "update"),
    (3, 3, False, "hints"), (2, 2, False, "step"),
])
def test_mean_route_equals_general_route(rank, workers, grad_bf16, call):
    _mean_route_equals_general_route(SHAPES, rank, workers, grad_bf16, call)


@pytest.mark.parametrize("rank,workers,grad_bf16,call", [
    (4, 9, True, "step"), (2, 16, False, "iterate"), (3, 12, False, "iterations"), (8, 9, True, "hints"),
    (2, 11, True, "iterate"), (1, 10, False, "hints iterate"), (5, 16, True, "hints iterations"),
    (3, 9, False, "ortho step"), (8, 4, False, "ortho iterations"),
])
def test_mean_route_equals_general_route_above_eight_workers_and_with_short_panels_apart(rank, workers, grad_bf16, call):
    _mean_route_equals_general_route(SHAPES, rank, workers, grad_bf16, call)


# 33 column chunks at each access width: the partial P are reduced before the orthogonalisation; 32: they are not
WIDE = [(40, 8448), (40, 4162), (40, 2081), (40, 8192)]


@pytest.mark.parametrize("shapes,rank,workers,grad_bf16,call", [
    (WIDE, 2, 4, False, "step"), (WIDE, 8, 5, True, "iterations"), (WIDE[3:], 4, 4, False, "split"), (WIDE[:1], 1, 16, False, "iterate"),
])
def test_mean_route_equals_general_route_on_long_rows(shapes, rank, workers, grad_bf16, call):
    _mean_route_equals_general_route(shapes, rank, workers, grad_bf16, call)


def _mean_route_equals_general_route(SHAPES, rank, workers, grad_bf16, call):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    outs = []
    for fused in (1, 0):
        plan = B.Plan(SHAPES, rank, workers, B.PSGD_BF16 if grad_bf16 else B.PSGD_F32, B.PSGD_F32)
        plan.set_tuning("resident", 0)
        plan.set_tuning("gram_fused", fused)
        plan.set_tuning("worker_mean", fused)   # small sets and odd rows do not take it by themselves
        if "ortho" in call:   # panels of at most 64 rows by one workgroup, the others over row blocks
            plan.set_tuning("ortho_rows", 64)
        if "hints" in call:
            plan.set_tuning("stream_hints", 1)
        s = plan.sizes
        gen = torch.Generator(device=dev)
        gen.manual_seed(rank * 100 + workers)
        grad = torch.randn(workers * s.grad_stride, generator=gen, device=dev).to(
            torch.bfloat16 if grad_bf16 else torch.float32)
        err = 0.5 * torch.randn(workers * s.err_stride, generator=gen, device=dev)
        q = torch.randn(s.q_elems, generator=gen, device=dev)
        live = torch.zeros(s.err_stride, dtype=torch.bool, device=dev)
        for t, shape in enumerate(SHAPES):
            if len(shape) == 2:
                live[plan.offsets(t)[0]: plan.offsets(t)[0] + shape[0] * shape[1]] = True
        err0 = err.clone()
        p = torch.zeros(s.p_elems, device=dev)
        out = torch.zeros(s.out_elems, device=dev)
        ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
        if "iterations" in call:
            plan.step_iterations(grad, err, q, p, out, ws, 3, stream)
        elif call == "update":
            param = torch.zeros(s.out_elems, device=dev)
            plan.step_update(grad, err, q, p, out, param, 0.1, 0.9, ws, stream)
        elif call == "split" or "iterate" in call:
            plan.compress(grad, err, q, p, ws, stream)
            M = grad.view(workers, -1)[:, : s.n_mat_elems].float() + err0.view(workers, -1)
            assert torch.equal(err.view(workers, -1)[:, live], M[:, live])   # M_w itself is left for the next call
            if "iterate" in call:   # on whatever M the caller holds by then
                scale = torch.linspace(0.5, 1.5, workers, device=dev).repeat_interleave(s.err_stride)
                err, err0 = err * scale, err0 * scale
                ws.fill_(float("nan"))
                plan.iterate(err, q, p, ws, stream)
            plan.decompress(p, q, err, grad, out, ws, stream)
        else:
            plan.step(grad, err, q, p, out, ws, stream)
        plan.check(stream)
        assert plan.worker_mean() == (bool(fused), 4 * s.n_mat_elems if fused else 0)   # the route that is meant
        assert torch.equal(err.view(workers, -1)[:, ~live], err0.view(workers, -1)[:, ~live])   # gaps are not touched
        outs.append((plan, q, p, out, err.view(workers, -1)[:, live]))
    a, b = outs
    # Per matrix: both are fp32 sums over at most 8448 terms in different orders, far below 1e-6 of the largest entry;
    # the orthogonalisation multiplies by the panels' condition (random 1 x 3 ... 300 x 5 matrices at full rank: up to a few hundred).
    for t, shape in enumerate(SHAPES):
        off, p_off, q_off, r = a[0].offsets(t)
        size = shape[0] * (shape[1] if len(shape) == 2 else 1)
        pairs = [(a[3][off: off + size], b[3][off: off + size])]
        if r:
            pairs += [(a[1][q_off: q_off + shape[1] * r], b[1][q_off: q_off + shape[1] * r]),
                      (a[2][p_off: p_off + shape[0] * r], b[2][p_off: p_off + shape[0] * r])]
        for x, y in pairs:
            assert torch.isfinite(x).all() and float((x - y).norm()) <= 1e-5 * float(y.norm()) + 1e-30, (t, shape)
    assert float((a[4] - b[4]).norm()) <= 1e-6 * float(b[4].norm())


@pytest.mark.parametrize("rank,workers", [(2, 3), (8, 9)])
def test_without_room_for_the_one_launch_orthogonalisation_each_worker_is_multiplied_by_itself(rank, workers):
    """2200 panels of one row block each: more than the device holds at once, so gram_fused does not hold and the mean is not
    taken.  The plan then runs exactly what it runs with the mean switched off (rows of 65 vectors: one chunk of two
    vectors per lane, two chunks of one)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    outs = []
    for mean in (1, 0):
        plan = B.Plan([(9, 260)] * 2200, rank, workers)
        plan.set_tuning("worker_mean", mean)
        s = plan.sizes
        gen = torch.Generator(device=dev)
        gen.manual_seed(3)
        grad = torch.randn(workers * s.grad_stride, generator=gen, device=dev)
        err = torch.randn(workers * s.err_stride, generator=gen, device=dev)
        q = torch.randn(s.q_elems, generator=gen, device=dev)
        p, out = torch.zeros(s.p_elems, device=dev), torch.zeros(s.out_elems, device=dev)
        ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
        plan.step(grad, err, q, p, out, ws, stream)
        plan.check(stream)
        assert plan.worker_mean() == (False, 0) and torch.isfinite(out).all()
        outs.append((q, p, out, err))
        plan.destroy()
    for a, b in zip(*outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("shape,rank,workers", [
    ((512, 4608), 1, 4), ((512, 4608), 4, 16), ((512, 4608), 8, 4), ((256, 2304), 2, 4), ((256, 8196), 3, 4), ((256, 4608), 5, 9),
])
def test_p_is_no_further_from_64_bits_than_with_each_worker_by_itself(shape, rank, workers):
    """The roundings of the workers' own products average out over the workers, those of the mean's one product do not: its
    column chunks (9 to 18 here, 33 of 8196 columns) are added in several chains."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    n, m = shape
    dist = []
    for mean in (1, 0):
        plan = B.Plan([shape], rank, workers)
        plan.set_tuning("worker_mean", mean)
        s = plan.sizes
        gen = torch.Generator(device=dev)
        gen.manual_seed(7)
        u, v = (torch.randn(k, rank, generator=gen, device=dev) / k ** 0.5 for k in (n, m))
        noise = torch.randn(workers, n * m, generator=gen, device=dev)
        grad = ((u @ v.T).reshape(1, -1) + 0.01 * noise).contiguous()
        err = 0.017 * torch.randn(workers, n * m, generator=gen, device=dev)
        assert s.grad_stride == s.err_stride == n * m
        want = (grad.double() + err.double()).mean(0).view(n, m) @ v.double()
        for k in range(rank):
            for j in range(k):
                want[:, k] -= (want[:, j] @ want[:, k]) * want[:, j]
            want[:, k] /= want[:, k].norm()
        q, p = v.reshape(-1).clone(), torch.zeros(s.p_elems, device=dev)
        ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
        plan.compress(grad, err, q, p, ws, stream)
        plan.check(stream)
        dist.append(float((p[:n * rank].double() - want.reshape(-1)).norm()))
    # two sets of at least 512 rounding errors: their 2-norms scatter by 1 / sqrt(2 * 512) = 3 % each
    assert dist[0] <= 1.05 * dist[1], dist
    assert dist[1] < 2e-7 * rank ** 0.5, dist


@pytest.mark.parametrize("size,workers", [(64, 4), (66, 5), (65, 13)])
def test_large_values_do_not_overflow_in_the_mean(size, workers):
    """Every M_w is 2e38 times the identity: the sum over the workers is beyond fp32's 3.4e38, the mean and all that follows are
    not (P = 2e38 q, Q = 2e38 / sqrt(n), which also the sum of the workers' own Q stays below while W <= 1.7 sqrt(n))."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    assert workers <= 3.4 / 2 * size ** 0.5
    outs = []
    for mean in (1, 0):
        plan = B.Plan([(size, size)], 1, workers)
        plan.set_tuning("worker_mean", mean)
        s = plan.sizes
        grad = torch.zeros(workers, s.grad_stride, device=dev)
        grad[:, : size * size] = 2e38 * torch.eye(size, device=dev).reshape(-1)
        err = torch.zeros(workers * s.err_stride, device=dev)
        q, p = torch.full((s.q_elems,), 1e-3, device=dev), torch.zeros(s.p_elems, device=dev)
        out = torch.zeros(s.out_elems, device=dev)
        ws = torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev)
        plan.step(grad, err, q, p, out, ws, stream)
        plan.check(stream)
        outs.append((q, p, out, err))
    for a, b in zip(*outs):
        assert torch.isfinite(a).all() and torch.isfinite(b).all()
        assert float((a.double() - b.double()).norm()) <= 1e-6 * float(b.double().norm())


@pytest.mark.parametrize("workers,rank,grad_bf16", [(4, 2, False), (8, 8, False), (5, 3, True)])
def test_default_rule_against_the_oracle(workers, rank, grad_bf16):
    """A set that takes the mean by the planner's own rule, three steps with error feedback, to the parity bar (1e-5)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    from paper_1905_13727_amd import workloads as WL
    from gpu_harness import GpuRun, OracleRun, compare
    shapes = [(512, 1152), (64, 27), (128, 4608), (33,)]
    wl = WL.Workload("mean", shapes, WL.tiny().planted_rank, WL.tiny().singular_values, WL.tiny().sigma)
    factors, q0 = WL.planted_factors(wl, 0), WL.initial_q(wl, rank, 0)
    gpu = GpuRun(shapes, rank, workers, q0, grad_bf16=grad_bf16)
    ora = OracleRun(shapes, rank, workers, q0)
    for t in range(3):
        grads = [WL.gradients(wl, factors, 0, t, w) for w in range(workers)]
        if grad_bf16:
            grads = [[torch.from_numpy(np.asarray(g, dtype=np.float32)).bfloat16().float().numpy() for g in gw] for gw in grads]
        prev = ora.errs
        rg, ro = gpu.step(grads), ora.step(grads)
        worst = compare(rg, ro, shapes, workers, rank, grads, prev)
        assert max(worst.values()) <= 1e-5, (t, worst)
    assert gpu.plan.worker_mean()[0]


@pytest.mark.parametrize("iterations,workers,grad_bf16", [(1, 4, False), (3, 9, True)])
def test_mean_route_replayed_from_a_hip_graph(iterations, workers, grad_bf16):
    """Captured once, replayed with new gradients and other work in between: the bits of the same steps launched directly."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    plan = B.Plan(SHAPES, 2, workers, B.PSGD_BF16 if grad_bf16 else B.PSGD_F32, B.PSGD_F32)
    plan.set_tuning("worker_mean", 1)
    plan.check(None)
    s = plan.sizes
    assert plan.worker_mean() == (True, 4 * s.n_mat_elems)
    gen = torch.Generator(device=dev)
    gen.manual_seed(9)
    dt = torch.bfloat16 if grad_bf16 else torch.float32
    grads = [torch.randn(workers * s.grad_stride, generator=gen, device=dev).to(dt) for _ in range(4)]
    q0 = torch.randn(s.q_elems, generator=gen, device=dev)
    g_in, q, p = torch.zeros_like(grads[0]), q0.clone(), torch.zeros(s.p_elems, device=dev)
    err, out = torch.zeros(workers * s.err_stride, device=dev), torch.zeros(s.out_elems, device=dev)
    ws = torch.zeros(s.workspace_bytes // 4 + 64, device=dev)

    def step():
        plan.step_iterations(g_in, err, q, p, out, ws, iterations, torch.cuda.current_stream().cuda_stream)

    def snapshot():
        torch.cuda.synchronize()
        return [x.clone() for x in (err, q, p, out)]

    want = []
    for g in grads:
        g_in.copy_(g)
        step()
        want.append(snapshot())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    err.zero_(), out.zero_(), ws.fill_(float("nan")), q.copy_(q0)
    for g, w in zip(grads, want):
        g_in.copy_(g)
        graph.replay()
        noise = torch.randn(1 << 20, device=dev).mul_(2)   # unrelated work between the replays
        got = snapshot()
        assert torch.isfinite(noise).all() and all(torch.isfinite(x).all() for x in got)
        for a, b in zip(got, w):
            assert torch.equal(a, b)
    plan.check(None)

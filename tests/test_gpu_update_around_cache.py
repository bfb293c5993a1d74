"""The update fused into the decompression on a set whose M fits the memory-side cache and whose M, momentum and
parameters together do not (28 M elements and more, one worker): momentum and parameters go around the cache."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shapes,rank,grad_bf16", [
    ([(5003, 5700), (7, 33), (31,)], 2, False), ([(5003, 5701)], 8, False), ([(4000, 7002), (9,)], 1, True),
])
def test_update_equals_step_and_elementwise_update(shapes, rank, grad_bf16):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    dt, code = (torch.bfloat16, B.PSGD_BF16) if grad_bf16 else (torch.float32, B.PSGD_F32)
    plan = B.Plan(shapes, rank, 1, code, B.PSGD_F32)
    s = plan.sizes
    assert 12 * s.n_mat_elems > 320 << 20 >= 4 * s.n_mat_elems
    gen = torch.Generator(device=dev)
    gen.manual_seed(5)
    grad = torch.randn(s.grad_stride, generator=gen, device=dev).to(dt)
    state = [torch.randn(n, generator=gen, device=dev) for n in (s.err_stride, s.q_elems)]
    mom, param = torch.randn(s.out_elems, generator=gen, device=dev), torch.randn(s.out_elems, generator=gen, device=dev)
    out, p = torch.zeros(s.out_elems, device=dev), torch.zeros(s.p_elems, device=dev)
    ws = torch.empty(s.workspace_bytes // 4 + 64, device=dev)
    e1, q1 = (x.clone() for x in state)
    plan.step(grad, e1, q1, p, out, ws, stream)
    e2, q2 = (x.clone() for x in state)
    m2, x2, p2 = mom.clone(), param.clone(), torch.zeros_like(p)
    plan.step_update(grad, e2, q2, p2, m2, x2, 0.1, 0.9, ws, stream)
    plan.check(stream)
    assert torch.equal(e1, e2) and torch.equal(q1, q2) and torch.equal(p, p2)   # the step itself is the same
    live = torch.zeros(s.out_elems, dtype=torch.bool, device=dev)
    for t, shape in enumerate(shapes):
        off = plan.offsets(t)[0]
        live[off: off + shape[0] * (shape[1] if len(shape) == 2 else 1)] = True
    assert torch.equal(m2[~live], mom[~live]) and torch.equal(x2[~live], param[~live])
    wm = 0.9 * mom.double() + out.double()
    wx = param.double() - 0.1 * (out.double() + wm)
    # three fp32 roundings of values below |x| + |mom| + 2 |out| each
    bound = 2.0 ** -22 * (param.double().abs() + mom.double().abs() + 2 * out.double().abs())
    for got, want in ((m2, wm), (x2, wx)):
        assert ((got.double() - want).abs() <= bound)[live].all()

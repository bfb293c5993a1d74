"""The resident step fused with the momentum / parameter update: rows requested ahead through strip descriptors, around the caches
on large sets, against the same step on the streaming kernels."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# every access width; strips that end inside a set of four rows and after one row, lanes without columns, one and two rows, a vector
SMALL = [(64, 576), (17, 1028), (33, 650), (2, 130), (65, 257), (1, 3), (512, 9), (77,)]
LARGE = SMALL + [(512, 4608), (500, 3100), (301, 1023)]   # 4.3 M elements: around the caches


@pytest.mark.parametrize("shapes,rank,around", [(SMALL, 1, False), (SMALL, 4, False), (LARGE, 2, True), (LARGE, 3, True),
                                                (LARGE, 4, True), (LARGE, 1, False)])
def test_resident_update_equals_streaming_update(shapes, rank, around):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13727_amd import binding as B
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev).cuda_stream
    got = []
    for resident in (1, 0):
        plan = B.Plan(shapes, rank, 1)
        plan.set_tuning("resident", resident)
        if not around and resident:
            plan.set_tuning("stream_hints", 0)
        s = plan.sizes
        gen = torch.Generator(device=dev)
        gen.manual_seed(rank)
        err = 0.5 * torch.randn(s.err_stride, generator=gen, device=dev)
        q = torch.randn(s.q_elems, generator=gen, device=dev)
        p = torch.zeros(s.p_elems, device=dev)
        mom, param = torch.randn(s.out_elems, generator=gen, device=dev), torch.randn(s.out_elems, generator=gen, device=dev)
        before = mom.clone(), param.clone(), err.clone()
        ws = torch.empty(s.workspace_bytes // 4 + 64, device=dev)
        for _ in range(2):
            grad = torch.randn(s.grad_stride, generator=gen, device=dev)
            plan.step_update(grad, err, q, p, mom, param, 0.1, 0.9, ws, stream)
        assert plan.check(stream) is bool(resident)
        live = torch.zeros(s.out_elems, dtype=torch.bool, device=dev)
        for t, shape in enumerate(shapes):
            off = plan.offsets(t)[0]
            live[off: off + shape[0] * (shape[1] if len(shape) == 2 else 1)] = True
        n = s.err_stride
        for x, y, at in ((mom, before[0], live), (param, before[1], live), (err, before[2], live[:n])):
            assert torch.equal(x[~at], y[~at])   # gaps between matrices are not touched
        got.append((mom[live], param[live], err[live[:n]]))
    # fp32 sums of at most 4608 terms in different orders, times the panels' condition (random matrices: below a hundred)
    for x, y in zip(*got):
        assert torch.isfinite(x).all() and float((x - y).norm()) <= 1e-5 * float(y.norm())

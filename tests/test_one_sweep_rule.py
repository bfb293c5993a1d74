"""Which sets go through one walk over M before the decompression, and how it divides them: the planner's choices (CPU, under the
sanitizers), and the kernels on what those choices hand them (GPU)."""
import os
import subprocess

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_rule_and_division(tmp_path):
    exe = str(tmp_path / "one_sweep_rule_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_1905_13727_amd", "csrc"),
           os.path.join(ROOT, "tests", "one_sweep_rule_check.cpp"),
           os.path.join(ROOT, "paper_1905_13727_amd", "csrc", "psgd_plan.cpp"), "-o", exe]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    res = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0 and "OK" in res.stdout, res.stdout


def _plans(shapes, rank, workers, keys, bf16=False):
    from paper_1905_13727_amd import binding as B
    plans = []
    for k in keys:
        plan = B.Plan(shapes, rank, workers, B.PSGD_BF16 if bf16 else B.PSGD_F32, B.PSGD_F32)
        for key, value in k.items():
            plan.set_tuning(key, value)
        plans.append(plan)
    return plans


def _state(plan, workers, seed, bf16=False):
    s, dev = plan.sizes, torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    draw = lambda n: torch.randn(n, generator=gen, device=dev)
    return dict(grad=draw(workers * s.grad_stride).to(torch.bfloat16 if bf16 else torch.float32), err=0.5 * draw(workers * s.err_stride),
                q=draw(s.q_elems), p=torch.zeros(s.p_elems, device=dev), out=torch.zeros(s.out_elems, device=dev),
                ws=torch.full((s.workspace_bytes // 4 + 64,), float("nan"), device=dev))


@pytest.mark.gpu
@pytest.mark.parametrize("shapes,workers", [([(64, 9)] * 600 + [(300, 2560)], 3), ([(32, 9)] * 400 + [(512, 1000)] * 20, 1)])
def test_many_matrices_equal_the_two_walks(shapes, workers):
    """More blocks than workgroups at once, dealt largest first.  Sums of at most 2560 fp32 products in other orders, times the condition
    of random panels of two columns."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = torch.cuda.current_stream().cuda_stream
    got = []
    for plan in _plans(shapes, 2, workers, ({"resident": 0}, {"resident": 0, "one_sweep": 0})):
        x = _state(plan, workers, 3)
        plan.step(x["grad"], x["err"], x["q"], x["p"], x["out"], x["ws"], stream)
        plan.check(stream)
        got.append((plan, x))
    assert got[0][0].one_sweep()[0] and not got[1][0].one_sweep()[0]
    for t, (n, m) in enumerate(shapes):
        off, p_off, q_off, r = got[0][0].offsets(t)
        for key, at, size in (("out", off, n * m), ("p", p_off, n * r), ("q", q_off, m * r)):
            a, b = got[0][1][key][at: at + size], got[1][1][key][at: at + size]
            assert torch.isfinite(a).all() and float((a - b).norm()) <= 2e-5 * float(b.norm()), (t, key)


@pytest.mark.gpu
@pytest.mark.parametrize("bf16", [False, True])
def test_several_iterations_go_over_the_stored_mean(bf16):
    """One call of two and of three iterations on a plan that takes the one walk: bit for bit what the two walks over the mean give, and
    within rounding what the calls apart give (fp32 sums of 1200 products in other orders, times the condition of random panels); one
    iteration, and the calls apart, are the one walk."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = torch.cuda.current_stream().cuda_stream
    shapes, workers = [(1200, 1200)], 16
    plan, walks, never = _plans(shapes, 2, workers, ({}, {"one_sweep": 0}, {"one_sweep": 1}), bf16)

    def run(pl, its, split=False):
        x = _state(plan, workers, 7, bf16)
        for _ in range(2):
            if split:
                pl.compress(x["grad"], x["err"], x["q"], x["p"], x["ws"], stream)
                for _ in range(its - 1):
                    pl.iterate(x["err"], x["q"], x["p"], x["ws"], stream)
                pl.decompress(x["p"], x["q"], x["err"], x["grad"], x["out"], x["ws"], stream)
            elif its == 1:
                pl.step(x["grad"], x["err"], x["q"], x["p"], x["out"], x["ws"], stream)
            else:
                pl.step_iterations(x["grad"], x["err"], x["q"], x["p"], x["out"], x["ws"], its, stream)
        pl.check(stream)
        return [x[k] for k in ("err", "q", "p", "out")]

    for its in (2, 3):
        a, b, c, d = run(plan, its), run(walks, its), run(plan, its, split=True), run(never, its, split=True)
        assert all(torch.equal(x, y) for x, y in zip(a, b))
        assert all(torch.equal(x, y) for x, y in zip(c, d))
        assert all(float((x - y).norm()) <= 2e-5 * float(y.norm()) for x, y in zip(a, c))
    assert all(torch.equal(x, y) for x, y in zip(run(plan, 1), run(never, 1)))
    assert plan.one_sweep()[0] and plan.worker_mean() == (True, 4 * 1200 * 1200) and walks.worker_mean() == (True, 4 * 1200 * 1200)
    assert never.worker_mean() == (True, 0)

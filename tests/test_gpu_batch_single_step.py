"""GPU tests of batched steps of one iteration, whose phases run beside the
iteration: how many kernels such a step launches, and that steps of one and of
several iterations may follow each other in any order, with solves joining in
between, without a solve's bits or counts changing."""

import os

import pytest
import torch

import workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2606_12650_amd as sem
    from paper_2606_12650_amd.batch import SemBatch

DEV = "cuda:0"
ORDERS = (3, 5, 7, 9, 11)


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-test] {os.environ.get('PYTEST_CURRENT_TEST', '')}", flush=True)


def _solve(i, mesh, N, prec, amp=0.04):
    A = sem.SemOperator(*mesh, N, amp, lowprec=None if prec == "f64" else prec, device=DEV)
    return A, torch.from_numpy(workload.continuous_rhs(90 + i, *mesh, N)).to(DEV)


def _launches(batch, iters):
    """Kernels on the device during one step."""
    from torch.profiler import ProfilerActivity, profile

    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA], acc_events=True) as prof:
        batch.step(iters)
        torch.cuda.synchronize()
    return sum(e.device_type == torch.autograd.DeviceType.CUDA and "batch_" in e.name for e in prof.events())


# One launch each for the lists, alpha, beta, the finishing lists, a finishing
# pass per family and the phases; per order an operator and an update launch; a
# mixed batch has the outer operators and one residual launch besides.
@pytest.mark.parametrize("families,most", [(("f64",), 6 + 10), (("f32",), 6 + 10 + 5 + 1), (("bf16",), 6 + 10 + 5 + 1),
                                           (("f64", "f32"), 7 + 20 + 5 + 1)])
def test_launches_of_a_short_step(families, most):
    batch, keep = SemBatch(16, device=DEV), []
    for prec in families:
        for i, N in enumerate(ORDERS):
            A, b = _solve(i, (3, 2, 2), N, prec)
            keep.append((A, b))
            batch.add(A, b, rtol=1e-12, mixed=prec != "f64")
    batch.step(1)  # takes the inner starts of the solves that joined
    one, two = _launches(batch, 1), _launches(batch, 2)
    assert 0 < one <= most
    assert 0 < two <= 2 * most
    batch.close()


@pytest.mark.parametrize("steps", [(1,), (1, 2), (1, 12, 1, 1, 3), (11, 1)])
@pytest.mark.parametrize("captured", [False, True])
def test_steps_of_any_length_in_any_order(steps, captured):
    jobs = []
    for i, (mesh, N) in enumerate((((1, 1, 1), 5), ((3, 2, 2), 7), ((2, 2, 2), 8), ((2, 2, 2), 9), ((2, 1, 2), 11))):
        for prec in ("f64", "f32", "bf16"):
            A, b = _solve(i, mesh, N, prec)
            x, r = A.cg(b, rtol=1e-8, mixed=prec != "f64")
            jobs.append((A, b, x.clone(), r, prec != "f64"))
    torch.cuda.synchronize()
    stream = torch.cuda.Stream(device=DEV) if captured else torch.cuda.default_stream(torch.device(DEV))
    with torch.cuda.stream(stream):
        batch, running, waiting = SemBatch(len(jobs), device=DEV), {}, list(jobs)
        for turn in range(4000):
            if waiting:
                job = waiting.pop()
                running[batch.add(job[0], job[1], mixed=job[4])] = job
            batch.step(steps[turn % len(steps)])
            for slot, got in batch.poll()[0]:
                _, _, x, r, _ = running.pop(slot)
                assert (got.status, got.iters, got.outer_iters, got.rel_res) == (0, r.iters, r.outer_iters, r.rel_res)
                assert torch.equal(batch.solution(slot), x)
                batch.remove(slot)
            if not waiting and not running:
                break
        assert not running and not waiting
        batch.close()
    torch.cuda.synchronize()

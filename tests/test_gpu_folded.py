"""GPU tests of the CG iterations whose scalar steps run inside the operator and
update kernels (solves with at most 1024 partials per reduction).

A batched solve takes the same steps in launches of their own and sums the
same partials in the same order, so the bar is bitwise equality with it, on
both sides of the limit (1024 elements: the operator's partials) and at the
edges of a wave of partials.  Where a run of iterations ends (check_every) must
not change a bit either, whether the solve stops inside a run, at its end or
at an iteration cap.
"""

import os

import pytest
import torch

import workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2606_12650_amd as sem
    from paper_2606_12650_amd import _lib as L
    from paper_2606_12650_amd.batch import SemBatch

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-test] {os.environ.get('PYTEST_CURRENT_TEST', '')}", flush=True)


def _case(mesh, N, lowprec=None):
    A = sem.SemOperator(*mesh, N, 0.05, lowprec=lowprec, device=DEV)
    return A, torch.from_numpy(workload.continuous_rhs(31 + N, *mesh, N)).to(DEV)


# 1, 63, 64, 65, 1023, 1024 and 1025 elements
MESHES = [(1, 1, 1), (9, 7, 1), (4, 4, 4), (13, 5, 1), (31, 11, 3), (16, 8, 8), (41, 5, 5)]


@pytest.mark.parametrize("N", [2, 5])
@pytest.mark.parametrize("mesh", MESHES)
def test_folded_equals_batched(mesh, N):
    A, b = _case(mesh, N)
    x, r = A.cg(b, rtol=1e-8)
    x = x.clone()
    B = SemBatch(1, device=DEV)
    s = B.add(A, b)
    rb = B.run_all(iters_per_step=9)[s]
    assert rb.status == r.status == 0 and rb.iters == r.iters and rb.rel_res == r.rel_res
    assert torch.equal(B.solution(s), x)
    B.remove(s)


@pytest.mark.parametrize("N,lowprec", [(3, "f32"), (7, "f32"), (7, "bf16"), (9, "f32"), (11, "f32")])
def test_folded_inner_solve_equals_batched(N, lowprec):
    A, b = _case((3, 4, 3), N, lowprec)
    x, r = A.cg(b, rtol=1e-8, mixed=True)
    x = x.clone()
    B = SemBatch(1, device=DEV)
    s = B.add(A, b, mixed=True)
    rb = B.run_all(iters_per_step=9)[s]
    assert rb.status == r.status == 0 and (rb.iters, rb.outer_iters) == (r.iters, r.outer_iters)
    assert torch.equal(B.solution(s), x)
    B.remove(s)


@pytest.mark.parametrize("precond", [True, False])
@pytest.mark.parametrize("N", [4, 7, 10])
def test_run_length_does_not_change_bits(N, precond):
    A, b = _case((4, 3, 3), N)
    x0, r0 = A.cg(b, rtol=1e-9, check_every=25, precond=precond)
    x0 = x0.clone()
    f0, _ = A.cg(b, fixed_iter=23, check_every=23, precond=precond)
    f0 = f0.clone()
    side = torch.cuda.Stream(device=DEV)
    for every in (1, 7, 64):
        for stream in (torch.cuda.current_stream(), side):  # direct launches, a captured graph
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                x, r = A.cg(b, rtol=1e-9, check_every=every, precond=precond)
                assert r.iters == r0.iters and r.rel_res == r0.rel_res and torch.equal(x, x0)
                f, rf = A.cg(b, fixed_iter=23, check_every=every, precond=precond)
                assert rf.iters == 23 and torch.equal(f, f0)
                _, rm = A.cg(b, rtol=1e-14, max_iter=5, check_every=every, precond=precond, raise_on_fail=False)
                assert rm.iters == 5 and rm.status == L.SEM_ERR_NOTCONV
            torch.cuda.synchronize()

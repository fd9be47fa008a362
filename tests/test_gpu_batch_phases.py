"""GPU tests of where a batched step advances the phases of its solves (after
every tenth iteration and after the last) and of launches bounded by the
batch's own work: whatever the length of the steps, every solve has the bits and
the counts of its solve alone, also when solves join and leave so that the
bounds grow and shrink."""

import os

import pytest
import torch

import workload

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2606_12650_amd as sem
    from paper_2606_12650_amd.batch import SemBatch

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-test] {os.environ.get('PYTEST_CURRENT_TEST', '')}", flush=True)


def _solves(prec):
    out = []
    for i, (mesh, N) in enumerate((((1, 1, 1), 5), ((3, 2, 2), 7), ((4, 3, 3), 3), ((2, 2, 2), 9), ((2, 1, 2), 11))):
        A = sem.SemOperator(*mesh, N, 0.04, lowprec=None if prec == "f64" else prec, device=DEV)
        b = torch.from_numpy(workload.continuous_rhs(70 + i, *mesh, N)).to(DEV)
        x, r = A.cg(b, rtol=1e-8, mixed=prec != "f64")
        out.append((A, b, x.clone(), r))
    return out


@pytest.mark.parametrize("steps", [1, 9, 10, 11, 23])
@pytest.mark.parametrize("prec", ["f64", "f32", "bf16"])
def test_step_length_does_not_change_a_solve(prec, steps):
    solves = _solves(prec)
    side = torch.cuda.Stream(device=DEV)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):  # captured steps
        B = SemBatch(8, device=DEV)
        slots = [B.add(A, b, mixed=prec != "f64") for A, b, _, _ in solves]
        res = B.run_all(iters_per_step=steps)
        for s, (_, _, x, r) in zip(slots, solves):
            got = res[s]
            assert (got.status, got.iters, got.outer_iters, got.rel_res) == (0, r.iters, r.outer_iters, r.rel_res)
            assert torch.equal(B.solution(s), x)
        for s in slots:
            B.remove(s)
    side.synchronize()


def test_joins_and_leaves_move_the_bounds():
    f64, f32 = _solves("f64"), _solves("f32")
    side = torch.cuda.Stream(device=DEV)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        B = SemBatch(10, device=DEV)
        waiting = [(s, False) for s in f64] + [(s, True) for s in f32]
        running = {}
        for _ in range(2000):
            if waiting:  # one more each step
                solve, mixed = waiting.pop()
                running[B.add(solve[0], solve[1], mixed=mixed)] = solve
            B.step(4)
            for slot, got in B.poll()[0]:
                _, _, x, r = running.pop(slot)
                assert (got.status, got.iters, got.outer_iters) == (0, r.iters, r.outer_iters)
                assert torch.equal(B.solution(slot), x)
                B.remove(slot)
            if not waiting and not running:
                break
        assert not running and not waiting
    side.synchronize()

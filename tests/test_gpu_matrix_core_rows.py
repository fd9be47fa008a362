"""GPU tests of the matrix-core operator at every number of rows in its last
group of four (N + 1 = 1, 2, 3, 0 mod 4), of the BF16 solves of order 8, whose
CG runs the matrix-core tile while the bare operator keeps the vector one, and
of the CG update that streams z against the one that does not.

Bounds of the low-precision operator, componentwise with B = |D|^T |G| |D| |u|
(rounded operands, assembled like the result): FP32 (4 (N + 1) + 8) 2^-24 B, BF16
2^-7 B.
"""

import math
import os

import numpy as np
import pytest
import torch

import workload
from oracle import operator as op
from oracle import pcg as opcg
from oracle.mixed import ax_local_abs_bound, ax_local_rounded

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


@pytest.mark.parametrize("mfma", [None, False, True], ids=["default", "valu", "mfma"])
@pytest.mark.parametrize("prec", ["f32", "bf16"])
@pytest.mark.parametrize("N", [2, 4, 6, 8, 10])
def test_even_orders_componentwise(N, prec, mfma):
    mesh, amp = (3, 2, 2), 0.05
    pr = op.Problem(*mesh, N, amp)
    A = sem.SemOperator(*mesh, N, amp, lowprec=prec, device=DEV, mfma=mfma)
    u = workload.iid_lvector(300 + N, pr.L).astype(np.float32).astype(np.float64)
    ug = torch.from_numpy(u.astype(np.float32)).to(DEV)
    ref, B = ax_local_rounded(pr, u, prec), ax_local_abs_bound(pr, u, prec)
    tol = (4 * (N + 1) + 8) * 2.0 ** -24 if prec == "f32" else 2.0 ** -7
    w = A.ax_lowp(ug, sem.LOCAL).cpu().numpy().astype(np.float64).reshape(ref.shape)
    assert np.all(np.abs(w - ref) <= tol * B + 1e-30)
    wm = A.ax_lowp(ug, sem.MASKED).cpu().numpy().astype(np.float64).reshape(ref.shape)
    assert np.all(np.abs(wm - pr.mask * pr.dssum(ref)) <= tol * pr.dssum(B) + 1e-30)


def test_bf16_order_8_bare_operator_on_the_solver_tile():
    """The default bare operator is the vector tile; OP_TILE 1 gives the one the
    inner CG runs, which is that of a matrix-core operator."""
    mesh, N = (3, 2, 2), 8
    u = torch.from_numpy(workload.iid_lvector(5, 12 * 9 ** 3).astype(np.float32)).to(DEV)
    w = {m: sem.SemOperator(*mesh, N, 0.05, lowprec="bf16", device=DEV, mfma=m).ax_lowp(u, sem.LOCAL)
         for m in (None, False, True)}
    A = sem.SemOperator(*mesh, N, 0.05, lowprec="bf16", device=DEV)
    A.set_knob(sem.OP_TILE, 1, "bf16")
    assert torch.equal(w[None], w[False])
    assert torch.equal(A.ax_lowp(u, sem.LOCAL), w[True])


@pytest.mark.parametrize("mesh", [(1, 1, 1), (2, 1, 3), (5, 4, 3)])
def test_bf16_order_8_solves(mesh):
    """Against the oracle's FP64 solution, the default solve bit for bit the one
    on a matrix-core operator, and the same in a batch with either tile."""
    N = 8
    pr = op.Problem(*mesh, N, 0.05)
    bnp = workload.continuous_rhs(48, *mesh, N)
    xr, _ = opcg.pcg(pr.ax, pr.shape4(bnp), pr.minv, pr.c, rtol=1e-12)
    b = torch.from_numpy(bnp).to(DEV)
    A = sem.SemOperator(*mesh, N, 0.05, lowprec="bf16", device=DEV)
    x, r = A.cg(b, rtol=1e-8, mixed=True)
    x = x.clone()
    assert r.status == 0 and r.rel_res <= 1e-8
    xv, c = x.cpu().numpy(), pr.c.reshape(-1)
    assert math.sqrt(np.sum(c * (xv - xr.reshape(-1)) ** 2) / np.sum(c * xr.reshape(-1) ** 2)) <= 1e-5
    assert opcg.true_rel_residual(pr.ax, pr.shape4(bnp), pr.shape4(xv), pr.c) <= 1e-8 * (1 + 1e-3)
    forced = sem.SemOperator(*mesh, N, 0.05, lowprec="bf16", device=DEV, mfma=True)
    xm, rm = forced.cg(b, rtol=1e-8, mixed=True)
    assert (rm.iters, rm.outer_iters) == (r.iters, r.outer_iters) and torch.equal(xm, x)
    for epb in (1, 2):
        batch = SemBatch(1, device=DEV)
        batch.set_tile(N, epb, "bf16")
        slot = batch.add(A, b, mixed=True)
        rb = batch.run_all(iters_per_step=9)[slot]
        assert (rb.status, rb.iters, rb.outer_iters) == (0, r.iters, r.outer_iters)
        assert torch.equal(batch.solution(slot), x)
        batch.remove(slot)


# 303, 303 and 276 MB a vector
@pytest.mark.parametrize("N,n,prec", [(7, 42, "f64"), (11, 28, "f64"), (9, 41, "f32")])
def test_streaming_update_equals_plain_update(N, n, prec):
    """Three iterations with the default tile, whose update streams z on these
    vectors, against another tile shape, which does not.  An iteration rounds
    each value of x and z some 20 times (eight copies, three products and sums)
    and the scalars by much less, and three iterations on a rough right-hand
    side cancel little: 1e3 roundings bound the difference against max|x|."""
    A = sem.SemOperator(n, n, n, N, 0.05, lowprec=None if prec == "f64" else prec, device=DEV)
    assert A.L * (8 if prec == "f64" else 4) > 256 << 20
    b = workload.continuous_rhs_device(9, n, n, n, N, DEV)
    out = []
    for shape in (0, 1):
        A.set_knob(sem.UPDATE_TILE, shape, prec)
        if prec == "f64":
            x, r = A.cg(b, fixed_iter=3)
        else:  # one outer step of three inner iterations
            x, r = A.cg(b, rtol=1e-30, mixed=True, max_iter=1, inner_rtol=1e-30, inner_max=3, raise_on_fail=False)
        assert r.iters == 3
        out.append((x.clone(), r.rel_res))
    (x0, r0), (x1, r1) = out
    tol = 1e3 * (2.0 ** -53 if prec == "f64" else 2.0 ** -24)
    assert float((x0 - x1).abs().max()) <= tol * float(x1.abs().max())
    assert abs(r0 - r1) <= tol * r1

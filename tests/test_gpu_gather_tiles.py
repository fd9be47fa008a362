"""GPU tests of the gathers of sem_ax and of the CG update on meshes that reach
every branch of their tiles: the gather's own tile shapes (orders 9..12) with
partial last tiles, slab and single-element meshes, both tile orders (one
range per XCD, and chunks walked backwards from 4096 tiles on), and the
update that streams r (vectors above 256 MB).

Tolerances as for the existing parity tests: max|w - w_ref| <= 1e-12 max|w_ref|
in FP64; assembled results are bitwise equal on all copies of a node.  On the
large meshes the reference is the element-local result, assembled by torch.
"""

import os

import numpy as np
import pytest
import torch

import workload
from oracle import operator as op

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2606_12650_amd as sem

DEV = "cuda:0"


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-test] {os.environ.get('PYTEST_CURRENT_TEST', '')}", flush=True)


@pytest.mark.parametrize("mesh", [(1, 1, 1), (2, 1, 1), (7, 1, 1), (1, 5, 2), (5, 3, 2), (4, 4, 3)])
@pytest.mark.parametrize("N", [8, 9, 10, 11, 12])
def test_gather_tiles_match_oracle(N, mesh):
    pr = op.Problem(*mesh, N, 0.05)
    A = sem.SemOperator(*mesh, N, 0.05, lowprec="f32", device=DEV)
    u = workload.iid_lvector(3, pr.L)
    ug = torch.from_numpy(u).to(DEV)
    for mode, ref in ((sem.ASSEMBLED, pr.ax_assembled(u)), (sem.MASKED, pr.ax(u))):
        ref = ref.reshape(-1)
        w = A.ax(ug, mode).cpu().numpy()
        assert np.max(np.abs(w - ref)) <= 1e-12 * max(np.max(np.abs(ref)), np.max(np.abs(pr.ax_local(u))))
        # FP32: the sum of the FP32 copies, accumulated in FP64 and rounded once
        loc = A.ax_lowp(ug.float(), sem.LOCAL).double().cpu().numpy()
        ref32 = pr.dssum(loc) * (pr.mask if mode == sem.MASKED else 1.0)
        w32 = A.ax_lowp(ug.float(), mode).double().cpu().numpy()
        scale = pr.dssum(np.abs(loc)).reshape(-1)
        assert np.all(np.abs(w32 - ref32.reshape(-1)) <= (2.0 ** -23) * scale)


def _assemble(v, nx, ny, nz, N):
    v = v.reshape(nz, ny, nx, N + 1, N + 1, N + 1).clone()
    for axis, m in ((0, nz), (1, ny), (2, nx)):
        hi = v.narrow(axis, 0, m - 1).select(axis + 3, N)
        lo = v.narrow(axis, 1, m - 1).select(axis + 3, 0)
        s = hi + lo
        hi.copy_(s)
        lo.copy_(s)
    return v.reshape(-1)


# 4094, 4096 and 4100 gather tiles of 10 elements at N = 4, and column and
# linear tiles of higher orders well above 4096
@pytest.mark.parametrize("mesh,N", [((46, 89, 10), 4), ((64, 64, 10), 4), ((41, 100, 10), 4), ((29, 27, 23), 7),
                                    ((22, 21, 20), 10)])
def test_large_gather_equals_assembled_local(mesh, N):
    A = sem.SemOperator(*mesh, N, 0.05, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    u = torch.rand(A.L, generator=gen, device=DEV, dtype=torch.float64) * 2 - 1
    ref = _assemble(A.ax(u, sem.LOCAL), *mesh, N)
    w = A.ax(u, sem.ASSEMBLED)
    # at most eight copies, each side one rounding per addition
    scale = _assemble(A.ax(u, sem.LOCAL).abs(), *mesh, N)
    assert bool(torch.all((w - ref).abs() <= 16 * 2.0 ** -53 * scale))


@pytest.mark.parametrize("N,n,lowprec", [(7, 42, None), (11, 28, None), (9, 41, "f32")])
def test_streaming_update_matches_small_run_length(N, n, lowprec):
    """Vectors above 256 MB (37.9, 37.9 and 68.9 M points, 303, 303 and 276 MB):
    CG iterates stay continuous and the true residual follows the recursive one."""
    A = sem.SemOperator(n, n, n, N, 0.05, lowprec=lowprec, device=DEV)
    b = workload.continuous_rhs_device(9, n, n, n, N, DEV)
    if lowprec is None:
        x, res = A.cg(b, fixed_iter=30)
        r = b - A.ax(x)
        c = A.export(sem._lib.SEM_FIELD_C)
        rel = float(((c * r * r).sum() / (c * b * b).sum()).sqrt())
        assert abs(rel - res.rel_res) <= 1e-8 * res.rel_res
    else:
        x, res = A.cg(b, rtol=1e-2, mixed=True, max_iter=1, inner_max=30, raise_on_fail=False)
        assert res.iters <= 30 and 0.0 < res.rel_res < 1.0
    v = x.reshape(n, n, n, N + 1, N + 1, N + 1)
    for axis in range(3):
        hi = v.narrow(axis, 0, n - 1).select(axis + 3, N)
        lo = v.narrow(axis, 1, n - 1).select(axis + 3, 0)
        assert torch.equal(hi, lo)

"""The two tile orders of the gathers of sem_ax: one contiguous range of tiles
per XCD, and from 4096 tiles on large vectors chunks walked backwards (FP64
from 128 MiB, FP32 from 160 MiB; the Jacobi set-up at any size).

On the CPU: which order each mesh takes.  On the GPU: on either side of every
limit, assembled and masked results against the element-local result assembled
by torch, and the Jacobi inverse against the diagonal formed by torch from the
exported metric.  The tile counts are no multiples of 256, so that the last
chunk has tiles without work.
"""

import os
import shutil
import subprocess

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_12650_amd", "csrc")
DEV = "cuda:0"

if torch.cuda.is_available():
    import paper_2606_12650_amd as sem
    from paper_2606_12650_amd import _lib as L

# mesh, N, precision, in chunks
MESHES = [
    ((60, 59, 37), 4, "f64", False),   # 130980 elements, 125.0 MiB
    ((64, 47, 45), 4, "f64", True),    # 135360 elements, 129.1 MiB
    ((37, 31, 29), 7, "f64", True),    # 33263 elements, 129.9 MiB
    ((29, 23, 21), 10, "f64", True),   # 14007 elements, 142.2 MiB, tiles of plane ranges
    ((17, 15, 13), 15, "f64", False),  # compiled at run time, linear tiles: 103.6 MiB
    ((19, 19, 18), 13, "f64", True),   # the same, 136.0 MiB
    ((67, 65, 64), 4, "f32", False),   # 132.9 MiB
    ((73, 71, 67), 4, "f32", True),    # 165.6 MiB
    ((45, 43, 41), 7, "f32", False),   # 154.9 MiB
    ((45, 44, 43), 7, "f32", True),    # 166.3 MiB
    ((31, 30, 28), 11, "f32", True),   # 171.6 MiB, tiles of plane ranges
]
IDS = [f"{'x'.join(map(str, m))}-N{n}-{p}" for m, n, p, _ in MESHES]


def _hipcc():
    for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    return None


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_which_order_each_mesh_takes(tmp_path):
    exe = str(tmp_path / "gather_order")
    cmd = [_hipcc(), "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", os.path.join(ROOT, "include"),
           "-I", CSRC, os.path.join(ROOT, "tests", "host", "gather_order.cpp"), "-o", exe]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    for mesh, N, prec, chunked in MESHES:
        args = [str(v) for v in (*mesh, N, 8 if prec == "f64" else 4)]
        out = subprocess.run([exe, *args], stdout=subprocess.PIPE, text=True, timeout=60, check=True).stdout.split()
        assert int(out[0]) >= 4096 and int(out[0]) % 256 != 0, (mesh, N, prec, out)
        assert bool(int(out[1])) == chunked, (mesh, N, prec, out)


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu-test] {os.environ.get('PYTEST_CURRENT_TEST', '')}", flush=True)


def _assemble(v, nx, ny, nz, N):
    v = v.reshape(nz, ny, nx, N + 1, N + 1, N + 1).clone()
    for axis, m in ((0, nz), (1, ny), (2, nx)):
        hi = v.narrow(axis, 0, m - 1).select(axis + 3, N)
        lo = v.narrow(axis, 1, m - 1).select(axis + 3, 0)
        s = hi + lo
        hi.copy_(s)
        lo.copy_(s)
    return v.reshape(-1)


def _mask(v, nx, ny, nz, N):
    v = v.reshape(nz, ny, nx, N + 1, N + 1, N + 1)
    for axis, m in ((0, nz), (1, ny), (2, nx)):
        v.select(axis, 0).select(axis + 2, 0).zero_()
        v.select(axis, m - 1).select(axis + 2, N).zero_()
    return v.reshape(-1)


@pytest.mark.gpu
@pytest.mark.parametrize("mesh,N,prec,chunked", MESHES, ids=IDS)
def test_gather_equals_assembled_local(mesh, N, prec, chunked):
    """At most eight copies, one rounding per addition on either side (FP64);
    FP32 copies are added in FP64 and rounded once."""
    _need_gpu()
    A = sem.SemOperator(*mesh, N, 0.05, lowprec=None if prec == "f64" else prec, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    u = torch.rand(A.L, generator=gen, device=DEV, dtype=torch.float64) * 2 - 1
    f = A.ax if prec == "f64" else A.ax_lowp
    u = u if prec == "f64" else u.float()
    loc = f(u, sem.LOCAL).double()
    ref, scale = _assemble(loc, *mesh, N), _assemble(loc.abs(), *mesh, N)
    del loc
    bound = (16 * 2.0 ** -53 if prec == "f64" else 2.0 ** -23) * scale
    del scale
    w = f(u, sem.ASSEMBLED).double()
    assert bool(torch.all((w - ref).abs() <= bound))
    w = f(u, sem.MASKED).double()
    assert bool(torch.all((w - _mask(ref, *mesh, N)).abs() <= bound))


# 4094, 4096 and 4100 tiles of 10 elements; linear tiles; linear tiles of an
# order compiled at run time
@pytest.mark.gpu
@pytest.mark.parametrize("mesh,N", [((46, 89, 10), 4), ((64, 64, 10), 4), ((41, 100, 10), 4), ((22, 21, 20), 10),
                                    ((17, 16, 13), 13)])
def test_jacobi_inverse_equals_assembled_diagonal(mesh, N):
    """1 / Minv against diag of the element operator, assembled: 3 (N + 1) + 3
    terms of at most four factors and seven additions per node, so at most
    (3 (N + 1) + 16) roundings a side of the sum of their magnitudes."""
    _need_gpu()
    n = N + 1
    A = sem.SemOperator(*mesh, N, 0.05, device=DEV)
    G = A.export(L.SEM_FIELD_G).reshape(-1, 6, n, n, n)
    D = A.export(L.SEM_FIELD_D).reshape(n, n)
    D2 = D * D  # D2[l, i]: node i's weight in the sum over l
    rr, rs, rt, ss, st, tt = (G[:, q] for q in range(6))
    diag = torch.matmul(rr, D2)
    diag += torch.matmul(D2.t().contiguous(), ss)
    diag += torch.matmul(D2.t().contiguous(), tt.reshape(-1, n, n * n)).reshape(-1, n, n, n)
    dd = torch.diagonal(D)
    di, dj, dk = dd.view(1, 1, 1, n), dd.view(1, 1, n, 1), dd.view(1, n, 1, 1)
    cross = [2 * di * dj * rs, 2 * di * dk * rt, 2 * dj * dk * st]
    mag = _assemble(diag + sum(c.abs() for c in cross), *mesh, N)
    ref = _assemble(diag + sum(cross), *mesh, N)
    minv = A.export(L.SEM_FIELD_MINV)
    inside = _mask(torch.ones_like(ref), *mesh, N)
    assert bool(torch.all(minv[inside == 0] == 0))
    err = ((minv * ref - 1).abs() * inside)
    assert bool(torch.all(err <= 2 * (3 * n + 16) * 2.0 ** -53 * mag / ref.abs()))

"""End-to-end parity of the batched solves against the CPU oracle (needs an MI355X).

The oracle's dense LU solution is the reference. FP64 paths must match it to 1e-6 relative error
with relative residual below the requested tolerance; mixed-precision paths (FP32 or BF16 T
inside FP64 refinement) must reach the same FP64 residual and the same 1e-6 error. Properties
that hold at any size (charge conservation, reciprocity, passivity) are checked on the GPU result.
"""

import numpy as np
import pytest

from oracle import wfq_oracle as O
from helpers import GRAPHENE, ragged_tube
import wfq_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2103_00438_amd import wfq
    wfq.load()
    return wfq


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def test_disk600_fp64_gmres50(lib):
    wl = wi.workload("disk600")
    P = O.Problem(wl.xyz, wl.params)
    h = lib.wfq_build(wl.xyz, wl.params)
    out = lib.wfq_solve(h, wl.omegas_eV, wl.dirs, wl.tol, restart=wl.restart, precision="fp64")
    assert out["status"] == 0
    info = out["info"][0]
    assert info["relres"] <= wl.tol
    q = out["q"][0, 0]
    q_lu = P.solve_lu(wl.omegas_eV[0], wl.dirs[0])
    assert rel(q, q_lu) <= 1e-6
    assert P.residual(wl.omegas_eV[0], wl.dirs[0], q) <= 2 * wl.tol     # oracle's own FP64 residual
    a = O.polarisability(P.xyz, q[:, None])[:, 0]
    assert np.allclose(out["alpha"][0, 0], a, rtol=1e-9, atol=1e-9 * np.abs(a).max())
    assert abs(q.sum()) <= 1e-9 * np.linalg.norm(q)
    h.close()


@pytest.fixture(scope="module")
def tube_case():
    xyz = ragged_tube()
    P = O.Problem(xyz, GRAPHENE)
    om = np.array([0.05, 0.31, 0.77, 1.0])
    dirs = np.eye(3)
    ref = {(a, k): P.solve_lu(om[a], dirs[k]) for a in range(len(om)) for k in range(3)}
    return xyz, P, om, dirs, ref


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_batched_mixed_precision(lib, tube_case, prec):
    xyz, P, om, dirs, ref = tube_case
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp64", "fp32", "bf16"))
    tol = 1e-8
    out = lib.wfq_solve(h, om, dirs, tol, restart=30, precision=prec)
    assert out["status"] == 0, out["info"]
    for a in range(len(om)):
        for k in range(3):
            info = out["info"][a * 3 + k]
            assert info["status"] == 0 and info["relres"] <= tol
            q = out["q"][a, k]
            assert rel(q, ref[(a, k)]) <= 1e-6, (prec, a, k, rel(q, ref[(a, k)]))
    al = out["alpha"]
    for a in range(len(om)):
        A = al[a].T                     # A[l, k]
        assert abs(A[0, 1] - A[1, 0]) <= 1e-6 * abs(A[0, 0])     # reciprocity (no conjugation)
        assert A[0, 0].imag > 0 and A[2, 2].imag > 0                # passivity
    h.close()


def test_restart_one_and_iteration_cap(lib, tube_case):
    xyz, P, om, dirs, ref = tube_case
    h = lib.wfq_build(xyz, GRAPHENE)
    out = lib.wfq_solve(h, om[:1], dirs[:1], 1e-8, restart=50, max_iter=5, precision="fp64")
    assert out["status"] == lib.WFQ_ENOCONV
    assert out["info"][0]["status"] == lib.WFQ_ENOCONV and out["info"][0]["iters"] == 5
    out1 = lib.wfq_solve(h, om[3:], dirs[:1], 1e-6, restart=1, max_iter=2000, precision="fp64")
    assert out1["info"][0]["relres"] <= 1e-6 or out1["info"][0]["status"] == lib.WFQ_ENOCONV
    h.close()


def test_errors(lib, tube_case):
    xyz, P, om, dirs, ref = tube_case
    h = lib.wfq_build(xyz, GRAPHENE)
    with pytest.raises(lib.WfqError) as e:
        lib.wfq_solve(h, [0.0], dirs[:1], 1e-8)
    assert e.value.code == lib.WFQ_ESINGULAR
    with pytest.raises(lib.WfqError) as e:
        lib.wfq_solve(h, [0.3], [[1.0, 1.0, 0.0]], 1e-8)
    assert e.value.code == lib.WFQ_EINVAL
    with pytest.raises(lib.WfqError) as e:
        lib.wfq_solve(h, [0.3], dirs[:1], 1e-8, precision="bf16")     # BF16 copy not built
    assert e.value.code == lib.WFQ_EINVAL
    h.close()


def test_dimer_solve(lib):
    xyz = np.array([[0.0, 0.0, 0.0], [1.7, 0.0, 0.0]])
    P = O.Problem(xyz, GRAPHENE)
    h = lib.wfq_build(xyz, GRAPHENE)
    out = lib.wfq_solve(h, [0.1, 0.7, 3.0], [[1.0, 0.0, 0.0]], 1e-12, restart=5, precision="fp64")
    for a, om in enumerate((0.1, 0.7, 3.0)):
        assert rel(out["q"][a, 0], P.solve_lu(om, [1, 0, 0])) <= 1e-10
    h.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n,n_omega,restart", [(5, 1, 6), (511, 1, 30), (512, 9, 30), (513, 20, 256), (1300, 30, 50),
                                               (2900, 20, 40), (8192, 1, 30), (8193, 2, 30)])
def test_gmres_steps_over_chunks_columns_and_restarts(lib, n, n_omega, restart, prec):
    # the step's kernels at the edges of their 512-row chunks and of the longest restart, with the norm formed in the
    # pack (up to 16 chunks) and by its own launch, and the products of 2 to 60 columns of a small T: every
    # system must satisfy the oracle's equations to the tolerance
    xyz = wi.geometry.jitter(wi.geometry.nanotube(8, 8, n // 32 + 1)[:n], 0.01, seed=n)
    om, tol, e = np.linspace(0.15, 1.1, n_omega), 1e-9, np.array([[0.0, 0.6, 0.8]])
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp64", "fp32"))
    out = lib.wfq_solve(h, om, e, tol, algorithm="gmres", restart=restart, precision=prec, max_iter=5000)
    h.close()
    assert out["status"] == 0, out["info"]
    P = O.Problem(xyz, GRAPHENE)
    for a in (0, n_omega // 2, n_omega - 1):
        assert P.residual(om[a], e[0], out["q"][a, 0]) <= 1.01 * tol + 1e-13, (a, out["info"][a])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("radius,fermi_d,entries,nsys", [
    (14.5, 20.0, 87, 3), (14.5, 14.0, 201, 5), (14.5, 12.0, 321, 1), (14.5, 12.0, 321, 9), (14.5, 6.0, 767, 9),
    (33.0, 12.0, 321, 2)])
def test_solves_with_long_neighbour_lists(lib, radius, fermi_d, entries, nsys, prec):
    # lists that leave the sparse product 32, 16 or 8 rows a work-group, or too long for its LDS, and the lanes beyond the
    # rows to further systems (fewer of them than there are, and as many); two systems above 8 192 rows
    xyz = wi.geometry.jitter(wi.geometry.fcc_sphere(radius), 0.01, 22)
    par = dict(wi.workloads.FCC_METAL, fermi_d=fermi_d)
    P = O.Problem(xyz, par)
    assert np.bincount(P.L.nonzero()[0]).max() == entries
    om, tol = np.linspace(2.0, 4.0, nsys), 1e-8
    h = lib.wfq_build(xyz, par)
    out = lib.wfq_solve(h, om, [[0.0, 0.6, 0.8]], tol, restart=60, precision=prec)
    h.close()
    assert out["status"] == 0, out["info"]
    for a in range(nsys):
        assert P.residual(om[a], np.array([0.0, 0.6, 0.8]), out["q"][a, 0]) <= 1.01 * tol + 1e-13, (a, out["info"][a])

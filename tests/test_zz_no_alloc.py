"""The allocation-free operator entry point wfq_apply_op_noalloc (device buffers, static scratch)
against the existing entry point wfq_apply_op on the same inputs, and both against the oracle's
operator with the same element-wise bound as the operator test (needs an MI355X). Two calls in a row
share the scratch; the second has a smaller input, so anything the first left behind would show."""

import numpy as np
import pytest

from oracle import wfq_oracle as O
from helpers import GRAPHENE, UNIT, ragged_tube, round_to
from wfq_inputs import geometry as geo

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2103_00438_amd import wfq
    wfq.load()
    return wfq


def run_noalloc(lib, torch, h, prec, z, X):
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(dev)
    zr, zi, xr, xi = t(z.real), t(z.imag), t(X.real), t(X.imag)
    yr = torch.full_like(xr, float("nan"))
    yi = torch.full_like(xi, float("nan"))
    stream = torch.cuda.Stream(dev)
    torch.cuda.synchronize()
    lib.wfq_apply_op_noalloc(h, prec, zr, zi, xr, xi, yr, yi, stream=stream.cuda_stream)
    stream.synchronize()
    return yr.cpu().numpy() + 1j * yi.cpu().numpy()


def oracle_bound_ok(P, prec, z, X, Y):
    L = P.L
    for s in range(X.shape[0]):
        if prec == "fp64":
            ref = L @ (P.T @ X[s]) + z[s] * X[s]
            scale = np.abs(L) @ (np.abs(P.T) @ np.abs(X[s])) + np.abs(z[s] * X[s])
            if not np.all(np.abs(Y[s] - ref) <= 1e-12 * scale):
                return False
        else:
            Tq = round_to(prec, P.T)
            xr, xi = round_to(prec, X[s].real), round_to(prec, X[s].imag)
            ref = L @ (Tq @ xr + 1j * (Tq @ xi)) + z[s] * X[s]
            scale = np.abs(L) @ (np.abs(Tq) @ (np.abs(xr) + np.abs(xi))) + np.abs(z[s] * X[s])
            if not np.all(np.abs(Y[s] - ref) <= 2 * P.n * UNIT["fp32"] * scale):
                return False
    return True


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_noalloc_matches_apply_op_on_two_calls(lib, prec):
    import torch
    cases = [(ragged_tube(), 7, 11), (geo.jitter(geo.graphene_disk(9.0), 0.01, 12), 2, 13)]   # second is smaller
    for xyz, nsys, seed in cases:
        P = O.Problem(xyz, GRAPHENE)
        h = lib.wfq_build(xyz, GRAPHENE, store=("fp64", "fp32", "bf16"))
        rng = np.random.default_rng(seed)
        X = rng.standard_normal((nsys, P.n)) + 1j * rng.standard_normal((nsys, P.n))
        z = np.array([P.z(om) for om in np.linspace(0.05, 1.0, nsys)])
        y_ref = lib.wfq_apply_op(h, prec, z, X)
        y = run_noalloc(lib, torch, h, prec, z, X)
        assert np.all(np.isfinite(y))
        # the same kernels; only the split of the block product's k range may differ
        tol = {"fp64": 1e-13, "fp32": 1e-5, "bf16": 1e-5}[prec]
        assert np.linalg.norm(y - y_ref) <= tol * np.linalg.norm(y_ref)
        assert oracle_bound_ok(P, prec, z, X, y)
        h.close()


def test_noalloc_rejects_what_does_not_fit(lib):
    import torch
    xyz = ragged_tube()
    h = lib.wfq_build(xyz, GRAPHENE)
    n = len(xyz)
    cap = lib.wfq_noalloc_scratch_bytes()
    assert cap == 256 << 20
    nsys = cap // (16 * 1280) + 1          # the systems' vectors alone exceed the scratch
    dev = torch.device("cuda:0")
    z = torch.zeros(nsys, dtype=torch.float64, device=dev)
    X = torch.zeros((nsys, n), dtype=torch.float64, device=dev)
    Y = torch.zeros_like(X)
    with pytest.raises(lib.WfqError) as e:
        lib.wfq_apply_op_noalloc(h, "fp64", z, z, X, X, Y, Y)
    assert e.value.code == lib.WFQ_ENOMEM
    with pytest.raises(lib.WfqError) as e:
        lib.wfq_apply_op_noalloc(h, "bf16", z[:1], z[:1], X[:1], X[:1], Y[:1], Y[:1])   # no BF16 copy built
    assert e.value.code == lib.WFQ_EINVAL
    h.close()


def _pieces(shape):
    import wfq_inputs as wi
    if shape == "tube":
        return geo.jitter(geo.nanotube(6, 6, 12), 0.01, 21), GRAPHENE
    metal = dict(wi.workloads.FCC_METAL)
    if shape == "long":   # neighbour lists beyond the 426 entries that the sparse product stages
        return geo.jitter(geo.fcc_sphere(14.5), 0.01, 22), dict(metal, fermi_d=6.0)
    return geo.jitter(geo.fcc_sphere(14.5), 0.01, 22), metal


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nsys", [1, 2, 3, 4, 5, 8, 9, 17, 40])
@pytest.mark.parametrize("shape", ["tube", "sphere", "long"])
def test_noalloc_sparse_product_forms(lib, shape, nsys, prec):
    # one to several systems per lane group, planes and row pairs, staged and unstaged neighbour lists
    import torch
    xyz, par = _pieces(shape)
    P = O.Problem(xyz, par)
    if shape == "long":
        assert np.bincount(P.L.nonzero()[0]).max() > 426
    h = lib.wfq_build(xyz, par, store=(prec,))
    rng = np.random.default_rng(nsys)
    X = rng.standard_normal((nsys, P.n)) + 1j * rng.standard_normal((nsys, P.n))
    z = rng.standard_normal(nsys) + 1j * rng.standard_normal(nsys)
    y = run_noalloc(lib, torch, h, prec, z, X)
    h.close()
    assert oracle_bound_ok(P, prec, z, X, y)


@pytest.mark.parametrize("nsys", [2, 5])
def test_noalloc_in_place_and_overlapping_vectors(lib, nsys):
    # the result may replace the vectors, or overlap them anywhere
    import torch
    xyz, par = _pieces("tube")
    h = lib.wfq_build(xyz, par)
    n = xyz.shape[0]
    rng = np.random.default_rng(5)
    X = rng.standard_normal((nsys, n)) + 1j * rng.standard_normal((nsys, n))
    z = rng.standard_normal(nsys) + 1j * rng.standard_normal(nsys)
    ref = run_noalloc(lib, torch, h, "fp64", z, X)
    dev = torch.device("cuda:0")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(dev)
    zr, zi = t(z.real), t(z.imag)
    for shift, swap in ((0, False), (0, True), (1, False), (n, False), (n + 3, True)):
        re = torch.zeros(nsys * n + shift, dtype=torch.float64, device=dev)
        im = torch.zeros_like(re)
        view = lambda b, o: b[o:o + nsys * n].view(nsys, n)
        xr, xi = view(re, 0), view(im, 0)
        xr.copy_(t(X.real))
        xi.copy_(t(X.imag))
        yr, yi = (view(im, shift), view(re, shift)) if swap else (view(re, shift), view(im, shift))
        torch.cuda.synchronize()
        lib.wfq_apply_op_noalloc(h, "fp64", zr, zi, xr, xi, yr, yi, stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        y = yr.cpu().numpy() + 1j * yi.cpu().numpy()
        assert np.array_equal(y, ref), (shift, swap)
    h.close()


@pytest.mark.parametrize("n,nsys", [(45600, 12), (48640, 7), (50000, 6), (50000, 16), (52000, 32), (58000, 1), (60000, 8),
                                    (64000, 1)])
def test_noalloc_matrix_free_fp64_up_to_the_scratch_limit(lib, n, nsys):
    # The recomputed FP64 product needs work space for its partial sums: what the call's own vectors leave of the scratch
    # goes from more than the symmetric form needs to less than one part of the one-sided form. Sampled rows
    # against the oracle's elements, with the bound of the operator test.
    import torch
    from oracle.cpp_oracle import CppProblem
    xyz = geo.jitter(geo.nanotube(10, 10, n // 40), 0.01, 23)
    P = CppProblem(xyz, GRAPHENE, dense_T=False, build_L=True)
    rng = np.random.default_rng(nsys)
    X = rng.standard_normal((nsys, n)) + 1j * rng.standard_normal((nsys, n))
    z = rng.standard_normal(nsys) + 1j * rng.standard_normal(nsys)
    h = lib.wfq_build(xyz, GRAPHENE, t_mode="otf")
    print(f"n={n} nsys={nsys}", flush=True)
    Y = run_noalloc(lib, torch, h, "fp64", z, X)
    h.close()
    rows = np.r_[0, rng.choice(n, 6, replace=False), n - 1]
    L = P.L[rows]
    near = np.unique(L.indices)
    parts = np.concatenate([X.real, X.imag]).T
    TX, TA = (P.apply_T_rows(near, v) for v in (parts, np.abs(parts)))
    TX, TA = TX[:, :nsys] + 1j * TX[:, nsys:], TA[:, :nsys] + TA[:, nsys:]
    zX = z * X.T[rows]
    assert np.all(np.abs(Y.T[rows] - (L[:, near] @ TX + zX)) <= 1e-12 * (abs(L[:, near]) @ TA + np.abs(zX)))


def test_noalloc_product_has_the_scratch_that_the_vectors_leave(lib):
    # 24 columns of 45 600 atoms: X and Y leave 77 MiB of the 256, the symmetric narrow product's sums take 65, so that the
    # product is the one of wfq_apply_op, bit by bit (no shift: the sparse product then adds nothing after its sums)
    import torch
    xyz = geo.jitter(geo.nanotube(10, 10, 1140), 0.01, 24)
    n, nsys = len(xyz), 12
    rng = np.random.default_rng(9)
    X = rng.standard_normal((nsys, n)) + 1j * rng.standard_normal((nsys, n))
    h = lib.wfq_build(xyz, GRAPHENE, t_mode="otf")
    y = run_noalloc(lib, torch, h, "fp64", np.zeros(nsys, complex), X)
    ref = lib.wfq_apply_op(h, "fp64", np.zeros(nsys, complex), X)
    h.close()
    assert np.array_equal(y, ref)


@pytest.mark.parametrize("prec,nsys,shift", [("fp64", 1, None), ("fp64", 5, 0), ("fp64", 5, 3), ("fp32", 9, 3), ("bf16", 2, 3)])
def test_noalloc_enqueues_kernels_only(lib, prec, nsys, shift):
    # a captured call (results apart, in place, overlapping the inputs) holds kernel nodes alone: no copies or memsets
    import ctypes as C
    import torch
    xyz, par = _pieces("tube")
    n = xyz.shape[0]
    h = lib.wfq_build(xyz, par, store=tuple({"fp64", prec}))
    re = torch.zeros(2 * nsys * n + 8, dtype=torch.float64, device="cuda:0")
    im = torch.zeros_like(re)
    z = torch.ones(nsys, dtype=torch.float64, device="cuda:0")
    view = lambda b, o: b[o:o + nsys * n].view(nsys, n)
    off = nsys * n if shift is None else shift
    call = lambda: lib.wfq_apply_op_noalloc(h, prec, z, z, view(re, 0), view(im, 0), view(re, off), view(im, off),
                                            stream=torch.cuda.current_stream().cuda_stream)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    with open("/proc/self/maps") as f:
        hip = C.CDLL(next(line.split()[-1] for line in f if "libamdhip64.so" in line))
    graph, count = C.c_void_p(g.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(graph, None, C.byref(count)) == 0 and count.value >= 3
    nodes = (C.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(count)) == 0
    kinds = []
    for node in nodes:
        kind = C.c_int(-1)
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0
        kinds.append(kind.value)
    h.close()
    assert set(kinds) == {0}, kinds   # hipGraphNodeTypeKernel

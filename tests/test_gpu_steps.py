"""Step-by-step parity of the HIP path against the CPU oracle (needs an MI355X).

Each stage of the hot path is called through the C interface and compared element by element
with the oracle on the same seeded structure: the damped Coulomb matrix in each storage precision,
the Drude Laplacian, the right-hand sides, the block product T X in each precision and every tile
variant, and the full operator (L T + z I) X.
"""

import numpy as np
import pytest

from oracle import wfq_oracle as O
from helpers import GRAPHENE, UNIT, ragged_tube, round_to
import wfq_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2103_00438_amd import wfq
    wfq.load()
    return wfq


@pytest.fixture(scope="module")
def tube():
    xyz = ragged_tube()                      # 1200 atoms: 4 full 256-tiles and a ragged tail
    return xyz, O.Problem(xyz, GRAPHENE)


@pytest.fixture(scope="module")
def handle(lib, tube):
    xyz, _ = tube
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp64", "fp32", "bf16"))
    yield h
    h.close()


def test_T_elements_all_precisions(lib, handle, tube):
    _, P = tube
    n = P.n
    i, j = np.meshgrid(np.arange(n), np.arange(n), indexing="ij")
    i, j = i.ravel(), j.ravel()
    ref = P.T[i, j]
    t64 = lib.wfq_sample_T(handle, "fp64", i, j)
    assert np.max(np.abs(t64 - ref) / np.abs(ref)) < 4e-16 * 8      # a few ulps (erf implementations)
    for prec in ("fp32", "bf16"):
        tp = lib.wfq_sample_T(handle, prec, i, j)
        # stored copy = FP64 value rounded to nearest; allow the FP64 ulps to flip a tie
        assert np.max(np.abs(tp - ref) / np.abs(ref)) <= UNIT[prec] * (1 + 1e-6)
        exact = tp == round_to(prec, ref)
        assert exact.mean() > 0.9999


def test_laplacian_structure_and_values(lib, handle, tube):
    _, P = tube
    r, c, v = lib.wfq_export_L(handle)
    L = P.L.tocoo()
    got = {(a, b): x for a, b, x in zip(r, c, v)}
    want = {(a, b): x for a, b, x in zip(L.row, L.col, L.data)}
    assert set(got) == set(want)                                     # same sparsity pattern, exactly
    keys = list(want)
    g = np.array([got[k] for k in keys])
    w = np.array([want[k] for k in keys])
    assert np.allclose(g, w, rtol=1e-13, atol=1e-16)
    rows = np.zeros(P.n)
    np.add.at(rows, r, v)
    assert np.max(np.abs(rows)) < 1e-14 * np.max(np.abs(v))


@pytest.mark.parametrize("case", ["pair", "cells of more than 64 atoms", "empty cells between"])
def test_neighbour_searches_over_full_and_empty_cells(lib, case):
    # a wave visits the cells around its atom 64 at a time and their atoms 64 at a time: the rows of L (27 cells) and,
    # through the narrow recomputed product, the near-field rows (up to 125)
    from wfq_inputs import geometry as geo
    par = wi.workloads.FCC_METAL
    xyz = geo.jitter(geo.fcc_sphere(20.0), 0.02, 5)
    if case == "pair":
        xyz = np.array([[0.0, 0.0, 0.0], [2.9, 0.0, 0.0]])
    elif case == "empty cells between":
        xyz = xyz[(xyz[:, 0] < 0.0) | (np.abs(xyz[:, 1]) > 11.5)]
    P = O.Problem(xyz, par)
    h = lib.wfq_build(xyz, par, t_mode="otf")
    r, c, v = lib.wfq_export_L(h)
    X = np.random.default_rng(2).standard_normal((2, P.n))
    Y = lib.wfq_apply_T(h, "fp64", X)
    h.close()
    L = P.L.tocoo()
    want = {(i, j): x for i, j, x in zip(L.row, L.col, L.data)}
    got = {(i, j): x for i, j, x in zip(r, c, v)}
    assert set(got) == set(want)
    k = list(want)
    assert np.allclose([got[q] for q in k], [want[q] for q in k], rtol=1e-13, atol=1e-16)
    assert np.all(np.abs(Y - X @ P.T.T) <= 1e-13 * (np.abs(X) @ np.abs(P.T).T))


def test_rhs(lib, handle, tube):
    _, P = tube
    dirs = np.eye(3)
    b = lib.wfq_rhs(handle, dirs, E0=1.0)
    for k in range(3):
        ref = P.rhs(dirs[k])
        # b is a short sum of large terms (positions times L): bound the rounding by |L| |r . k|
        scale = np.abs(P.L) @ np.abs(P.xyz @ dirs[k])
        assert np.all(np.abs(b[k] - ref) <= 64 * UNIT["fp64"] * scale)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("ncol", [1, 2, 5, 8, 9, 24, 32, 33, 64, 65, 130])
def test_block_product(lib, handle, tube, prec, ncol):
    _, P = tube
    rng = np.random.default_rng(100 + ncol)
    X = rng.standard_normal((ncol, P.n))
    Y = lib.wfq_apply_T(handle, prec, X)
    Tq = round_to(prec, P.T)
    Xq = round_to(prec, X)
    ref = Xq @ Tq                     # T symmetric: row c of Y is T x_c
    bound = np.abs(Xq) @ np.abs(Tq)
    # accumulation error of an n-term sum in the accumulator precision (FP64 or FP32)
    u_acc = UNIT["fp64"] if prec == "fp64" else UNIT["fp32"]
    assert np.all(np.abs(Y - ref) <= 2 * P.n * u_acc * bound + 1e-300)


def test_block_product_larger_than_staging_chunk(lib, handle, tube):
    # 3500 columns: X and Y are 35.8 MB each, more than the 32 MiB pinned staging chunk through which
    # host arrays are copied, so both copy directions take more than one chunk
    _, P = tube
    rng = np.random.default_rng(77)
    X = rng.standard_normal((3500, P.n))
    Y = lib.wfq_apply_T(handle, "fp64", X)
    ref = X @ P.T
    bound = np.abs(X) @ np.abs(P.T)
    # element by element within the accumulation bound: a chunk copied to a wrong offset (or not at
    # all) would put whole rows of Y far outside it
    assert np.all(np.abs(Y - ref) <= 2 * P.n * UNIT["fp64"] * bound + 1e-300)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_every_block_product_variant(lib, handle, tube, prec):
    # each shape the autotuner may choose, at ragged widths (partial column tiles, split k parts)
    _, P = tube
    Tq = round_to(prec, P.T)
    u_acc = UNIT["fp64"] if prec == "fp64" else UNIT["fp32"]
    rng = np.random.default_rng(31)
    for name, max_ncol in lib.wfq_tx_variants(prec):
        widths = [max_ncol, max_ncol - 1] if max_ncol < 64 else [3, 97, 200]
        for ncol in widths:
            if ncol < 1:
                continue
            X = rng.standard_normal((ncol, P.n))
            Y = lib.wfq_apply_T_variant(handle, prec, name, X)
            Xq = round_to(prec, X)
            ref = Xq @ Tq
            bound = np.abs(Xq) @ np.abs(Tq)
            assert np.all(np.abs(Y - ref) <= 2 * P.n * u_acc * bound + 1e-300), (name, ncol)


@pytest.mark.parametrize("n", [240, 760, 1020, 5880, 6140, 12020, 12040])
def test_narrow_products_where_their_rows_per_wave_change(lib, n):
    # 1, 2 and 4 rows a wave, one and several loads ahead, with and without a last step of fewer: padded sizes 256, 1 024
    # (760 and 1 020 atoms), 6 144 and 12 288. Rows against the oracle's elements; the bound is n roundings of the
    # accumulator and one each of T's and X's elements.
    from oracle.cpp_oracle import CppProblem
    from wfq_inputs import geometry as geo
    xyz = geo.jitter(geo.nanotube(5, 5, n // 20), 0.01, 3)
    n = len(xyz)
    P = CppProblem(xyz, GRAPHENE, dense_T=False, build_L=False)
    rows = np.unique(np.r_[np.arange(0, n, max(1, n // 24)), n - 1])
    X = np.random.default_rng(n).standard_normal((8, n))
    ref, bound = P.apply_T_rows(rows, X.T).T, P.apply_T_rows(rows, np.abs(X).T).T
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp64", "fp32", "bf16"))
    for prec in ("fp64", "fp32", "bf16"):
        tol = 2 * n * UNIT["fp64" if prec == "fp64" else "fp32"] + (0 if prec == "fp64" else 3 * UNIT[prec])
        for name, ncol in (("skinny2", 1), ("skinny2", 2), ("skinny4", 3), ("skinny4", 4), ("skinny8", 5), ("skinny8", 8)):
            Y = lib.wfq_apply_T_variant(h, prec, name, X[:ncol])[:, rows]
            assert np.all(np.abs(Y - ref[:ncol]) <= tol * bound[:ncol]), (prec, name, ncol)
    h.close()


def test_variant_entry_point_rejects(lib, handle):
    X = np.ones((5, handle.n))
    with pytest.raises(lib.WfqError):
        lib.wfq_apply_T_variant(handle, "fp32", "skinny4", X)       # 5 columns > 4
    with pytest.raises(lib.WfqError):
        lib.wfq_apply_T_variant(handle, "fp32", 10 ** 6, X)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_operator_apply(lib, handle, tube, prec):
    _, P = tube
    rng = np.random.default_rng(7)
    S = 5
    X = rng.standard_normal((S, P.n)) + 1j * rng.standard_normal((S, P.n))
    z = np.array([P.z(om) for om in (0.05, 0.2, 0.4, 0.7, 1.0)])
    Y = lib.wfq_apply_op(handle, prec, z, X)
    L = P.L
    for s in range(S):
        if prec == "fp64":
            ref = L @ (P.T @ X[s]) + z[s] * X[s]
            scale = np.abs(L) @ (np.abs(P.T) @ np.abs(X[s])) + np.abs(z[s] * X[s])
            assert np.all(np.abs(Y[s] - ref) <= 1e-12 * scale)
        else:
            Tq = round_to(prec, P.T)
            xr, xi = round_to(prec, X[s].real), round_to(prec, X[s].imag)
            ty = Tq @ xr + 1j * (Tq @ xi)
            ref = L @ ty + z[s] * X[s]
            scale = np.abs(L) @ (np.abs(Tq) @ (np.abs(xr) + np.abs(xi))) + np.abs(z[s] * X[s])
            assert np.all(np.abs(Y[s] - ref) <= 2 * P.n * UNIT["fp32"] * scale)


def test_small_structure_dimer(lib):
    # N = 2: one 256-tile of padding around two atoms
    xyz = np.array([[0.0, 0.0, 0.0], [1.7, 0.0, 0.0]])
    P = O.Problem(xyz, GRAPHENE)
    h = lib.wfq_build(xyz, GRAPHENE)
    t = lib.wfq_sample_T(h, "fp64", [0, 0, 1, 1], [0, 1, 0, 1])
    assert np.allclose(t, P.T.ravel(), rtol=1e-15)
    Y = lib.wfq_apply_T(h, "fp64", np.array([[1.0, -2.0]]))
    assert np.allclose(Y[0], P.T @ np.array([1.0, -2.0]), rtol=1e-14)
    h.close()


@pytest.mark.parametrize("ncol", [1, 31, 33, 64, 65, 129, 193, 260])
@pytest.mark.parametrize("name", ["s32n256k32", "s64n256k32", "s96n256k32", "s128n256k32", "s64n128k64", "s96n128k64",
                                  "s128n128k64", "s192n128k32"])
def test_fp16_split_product_scales_and_edges(lib, handle, tube, name, ncol):
    # FP32 products through the FP16 matrix cores: columns of very different scales (each has its own
    # exponent), entries spread over 20 orders of magnitude within a column, an empty column; one tile
    # and its remainders. The bound is the accumulation bound of the FP32 products.
    _, P = tube
    rng = np.random.default_rng(1000 + ncol)
    X = rng.standard_normal((ncol, P.n)) * 2.0 ** rng.integers(-100, 100, (ncol, 1))
    X[0] *= 10.0 ** (-20 * rng.random(P.n))
    X[ncol // 2] = 0.0
    Y = lib.wfq_apply_T_variant(handle, "fp32", name, X)
    Xq, Tq = round_to("fp32", X), round_to("fp32", P.T)
    assert np.all(np.abs(Y - Xq @ Tq) <= 2 * P.n * UNIT["fp32"] * (np.abs(Xq) @ np.abs(Tq)))
    assert np.all(Y[ncol // 2] == 0.0)


def test_fp16_split_product_keeps_infinities_and_nan(lib, handle, tube):
    # T's elements are positive: an infinite entry gives that infinity in its column, a NaN or both
    # signs NaN; the other columns are untouched
    _, P = tube
    X = np.random.default_rng(5).standard_normal((40, P.n))
    ref = lib.wfq_apply_T_variant(handle, "fp32", "s64n128k64", X)
    X[3, 7], X[4, 100], X[5, 0], X[6, 1], X[6, 2] = np.inf, -np.inf, np.nan, np.inf, -np.inf
    Y = lib.wfq_apply_T_variant(handle, "fp32", "s64n128k64", X)
    assert np.all(Y[3] == np.inf) and np.all(Y[4] == -np.inf) and np.all(np.isnan(Y[5])) and np.all(np.isnan(Y[6]))
    keep = [c for c in range(40) if c not in (3, 4, 5, 6)]
    assert np.array_equal(Y[keep], ref[keep])


@pytest.mark.parametrize("ncol", [5, 8, 9, 16, 17, 33, 48, 49, 65, 80, 81, 96, 97, 129, 145, 160, 161, 177, 257])
def test_fragment_product_column_edges(lib, handle, tube, ncol):
    # the default FP64 product at each number of 16-column fragments and passes, with partial last fragments
    _, P = tube
    rng = np.random.default_rng(ncol)
    X = rng.standard_normal((ncol, P.n))
    Y = lib.wfq_apply_T(handle, "fp64", X)
    assert np.all(np.abs(Y - X @ P.T) <= 2 * P.n * UNIT["fp64"] * (np.abs(X) @ P.T) + 1e-300)
    for name in ("f16n64", "f32n64", "f48n32", "f48n64", "f64n32", "f80n32"):
        Y = lib.wfq_apply_T_variant(handle, "fp64", name, X)
        assert np.all(np.abs(Y - X @ P.T) <= 2 * P.n * UNIT["fp64"] * (np.abs(X) @ P.T) + 1e-300), name


@pytest.mark.parametrize("n,ncol", [(1281, 8), (1537, 8), (4352, 4), (4353, 3), (9985, 8), (10240, 6), (10240, 9)])
def test_default_fp64_product_at_its_size_limits(lib, n, ncol):
    # where another kernel takes over by default: the result is that of the LDS-tile shape to rounding
    xyz = wi.geometry.jitter(wi.geometry.nanotube(8, 8, n // 32 + 1)[:n], 0.01, seed=n)
    h = lib.wfq_build(xyz, GRAPHENE)
    X = np.random.default_rng(n).standard_normal((ncol, n))
    Y, ref = lib.wfq_apply_T(h, "fp64", X), lib.wfq_apply_T_variant(h, "fp64", "m32n128", X)
    h.close()
    # each sum of n products is within n u of sum |T||X| <= n max|T| max|X|: two of them
    assert np.abs(Y - ref).max() <= 2 * n * UNIT["fp64"] * np.abs(X).sum(axis=1).max() * GRAPHENE["eta"]


def test_tuned_narrow_products_run_the_kernel_that_was_timed(lib):
    # 5 000 atoms, the two columns of one system: recomputed, they take about 22 us with both rows of a pair at once, 53
    # with each row by itself, streamed 31. A solve runs the second form, so that streaming is what tuning has
    # to choose for it; a row's sums are the same in every streaming shape, and with them the solve's results.
    xyz = wi.geometry.jitter(wi.geometry.nanotube(10, 10, 125), 0.01, 5)
    n = len(xyz)
    h = lib.wfq_build(xyz, GRAPHENE)
    X = np.random.default_rng(2).standard_normal((2, n))
    solve = lambda: lib.wfq_solve(h, [0.4], [[0.0, 0.0, 1.0]], 1e-8, restart=30, precision="fp64")
    ref = solve()
    tune = lib.wfq_tune(h, "fp64", [2], reps=20)
    name = dict(zip(tune["variants"], tune["ms"][0]))
    assert tune["chosen"][0] == min((k for k in name if name[k] > 0), key=name.get)
    assert not tune["chosen"][0].startswith("otfn"), name
    out = solve()
    if tune["chosen"][0].startswith("skinny"):
        assert np.array_equal(out["q"], ref["q"])
    # the operator takes the recomputed product with both rows of a pair at once, the faster one there
    assert np.array_equal(lib.wfq_apply_T(h, "fp64", X), lib.wfq_apply_T_variant(h, "fp64", "otfn2", X))
    h.close()


def test_tuned_fp32_solves_keep_the_fp32_instruction(lib):
    # at 6 000 atoms and 128 columns an FP16-split shape is fastest: tuning keeps it for the operator entry points only
    xyz = wi.geometry.jitter(wi.geometry.nanotube(10, 10, 150), 0.01, 6)
    h = lib.wfq_build(xyz, GRAPHENE)
    X = np.random.default_rng(3).standard_normal((128, len(xyz)))
    tune = lib.wfq_tune(h, "fp32", [128], reps=5)
    name = dict(zip(tune["variants"], tune["ms"][0]))
    split = [k for k in name if k[0] == "s" and k[1].isdigit()]
    assert split and all(name[k] > 0 for k in split)
    assert tune["chosen"][0] not in split
    assert tune["chosen"][0] == min((k for k in name if name[k] > 0 and k not in split), key=name.get)
    best = min((k for k in name if name[k] > 0), key=name.get)
    assert np.array_equal(lib.wfq_apply_T(h, "fp32", X), lib.wfq_apply_T_variant(h, "fp32", best, X))
    h.close()


@pytest.mark.parametrize("ncol", [1, 33])
def test_fp16_split_product_is_as_accurate_as_claimed(lib, handle, tube, ncol):
    # Columns of one scale. Of each product of two elements at most 2^-22 is lost, of either sign, and the 3 n / 32 roundings of
    # the running sum add at most 2^-24 (3 n / 64)^(1/2): below 7e-7 of a column's norm in all. Without one of the two cross
    # terms the error is 1.1e-4 and more (the same inputs in numpy); 2e-6 tells them apart.
    _, P = tube
    X = np.random.default_rng(2000 + ncol).standard_normal((ncol, P.n))
    ref = round_to("fp32", X) @ round_to("fp32", P.T)
    for name in [v[0] for v in lib.wfq_tx_variants("fp32") if v[0][0] == "s" and v[0][1].isdigit()]:
        Y = lib.wfq_apply_T_variant(handle, "fp32", name, X)
        err = np.linalg.norm(Y - ref, axis=1) / np.linalg.norm(ref, axis=1)
        assert err.max() <= 2e-6, (name, err.max())


@pytest.mark.parametrize("n,ncol,tile", [(1289, 256, "m128n256w8k64"), (1289, 128, "m96n256w8"), (1721, 40, "m64n128k256i"),
                                         (1721, 64, "m64n128k256i"), (2315, 48, "m64n128k256i"), (1289, 384, "m128n256w8k64")])
def test_small_fp32_products_are_no_less_accurate_than_a_large_tile(lib, n, ncol, tile):
    # the operator's FP32 products of small structures run in smaller tiles than a large structure's; after L, which takes the
    # slowly varying part away, the result is as close to the 64-bit one (2 % for the order of the sums)
    geo = wi.geometry
    xyz = geo.jitter(geo.fcc_sphere(geo.A_FCC * (3 * n / (16 * np.pi)) ** (1 / 3)), 0.02, 5)
    assert len(xyz) == n
    par = wi.workloads.FCC_METAL
    P = O.Problem(xyz, par)
    X = np.random.default_rng(n).standard_normal((ncol, n))
    X = 2 * X - np.roll(X, 1, axis=1) - np.roll(X, -1, axis=1)
    h = lib.wfq_build(xyz, par, store=("fp32",))
    exact = P.L @ (X @ P.T).T
    err = [np.linalg.norm(P.L @ Y.T - exact) for Y in (lib.wfq_apply_T(h, "fp32", X), lib.wfq_apply_T_variant(h, "fp32", tile, X))]
    h.close()
    print(n, ncol, tile, err[0] / err[1], flush=True)
    assert err[0] <= 1.02 * err[1], err


@pytest.mark.parametrize("ncol", [3, 4])
def test_large_narrow_fp32_product_keeps_its_sums(lib, ncol):
    # 4 rows a wave where there were 8: the same result, bit by bit
    xyz = wi.geometry.jitter(wi.geometry.nanotube(10, 10, 411), 0.01, 9)
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp32",))
    X = np.random.default_rng(ncol).standard_normal((ncol, len(xyz)))
    assert np.array_equal(lib.wfq_apply_T(h, "fp32", X), lib.wfq_apply_T_variant(h, "fp32", "skinny4r8", X))
    h.close()


@pytest.mark.parametrize("n,ncol,tile", [(16380, 24, "f32n64"), (16400, 24, "m32n128"), (16400, 32, "m32n128"), (16400, 33, "f48n64")])
def test_fp64_product_where_the_tile_takes_over_again(lib, n, ncol, tile):
    # up to 32 columns beyond 16 384 rows run in the LDS tile, the others in the fragment layout: rows against the oracle
    from oracle.cpp_oracle import CppProblem
    xyz = wi.geometry.jitter(wi.geometry.nanotube(10, 10, n // 40 + 1)[:n], 0.01, seed=n)
    X = np.random.default_rng(n).standard_normal((ncol, n))
    h = lib.wfq_build(xyz, GRAPHENE, store=("fp64",))
    Y, ref = lib.wfq_apply_T(h, "fp64", X), lib.wfq_apply_T_variant(h, "fp64", tile, X)
    h.close()
    assert np.array_equal(Y, ref)
    P = CppProblem(xyz, GRAPHENE, dense_T=False, build_L=False)
    rows = np.r_[np.arange(0, n, 997), n - 1]
    assert np.all(np.abs(Y[:, rows].T - P.apply_T_rows(rows, X.T)) <= 2 * n * UNIT["fp64"] * P.apply_T_rows(rows, np.abs(X).T))

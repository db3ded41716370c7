"""Kernels on full tiles at the edges of their ranges against the oracle
(MI355X only; every call goes through the C ABI)."""
import sys

import numpy as np
import pytest

import floquet_inputs as fin
import oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2111_08044_amd as fl  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _random_context(L, dtype, seed, variant="plain"):
    hs = 2.0 * fin.gue_bond_sample(L, seed=seed)
    ctx = fl.fl_create(L, dtype, variant)
    fl.fl_set_bonds(ctx, hs, 0.7)
    psi = fl.new_state(ctx)
    ref = torch.from_numpy(fin.random_state(L, seed)).to(psi.dtype)
    psi.copy_(ref)
    return ctx, hs, psi, ref.to(torch.complex128).numpy()


# 2 tiles (the shortest chains of the tiled kernel), one bond left over for a
# second or third pass, more tiles than workgroups
@pytest.mark.parametrize("dtype,L", [("c64", 14), ("c64", 15), ("c64", 22), ("c64", 23),
                                     ("c128", 13), ("c128", 14), ("c128", 19), ("c128", 21)])
def test_h0_psi_and_its_sums(dtype, L):
    """Every amplitude of H0 psi for distinct random bond terms.  A row sums
    8 entries a window and at most 13 windows: about 100 roundings of random
    sign, 10 units in the last place of the norm."""
    say(f"case: H0 psi {dtype} L={L}")
    ctx, hs, psi, ref = _random_context(L, dtype, 70 + L)
    ws = torch.full_like(psi, float("nan"))
    E, E2, N = fl.fl_energy_spread(ctx, psi, ws)
    want = O.apply_h0(ref, L, hs)
    got = ws.cpu().numpy().astype(np.complex128)
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    assert np.linalg.norm(got - want) < 10 * ulp * np.linalg.norm(want)
    # the sums are FP64 sums over the stored values
    assert abs(E - np.vdot(ref, got).real) < 1e-12 * np.linalg.norm(ref) * np.linalg.norm(got)
    assert abs(E2 - np.vdot(got, got).real) < 1e-12 * E2
    assert abs(N - np.vdot(ref, ref).real) < 1e-12 * N
    assert np.array_equal(psi.cpu().numpy(), ref.astype(psi.cpu().numpy().dtype))


# one workgroup (L <= 10), then each tile size of the short chains at its
# shortest chain (two or more tiles) and its longest, and the first chain on
# full tiles; a call of 2 periods and one of 3 (another geometry in complex128)
@pytest.mark.parametrize("dagger", [False, True])
@pytest.mark.parametrize("dtype,L,n", [("c64", 3, 5), ("c64", 10, 5), ("c64", 11, 5), ("c64", 18, 3), ("c64", 19, 3),
                                       ("c64", 20, 3), ("c64", 21, 2), ("c128", 3, 5), ("c128", 10, 5), ("c128", 11, 5),
                                       ("c128", 17, 3), ("c128", 18, 3), ("c128", 19, 3), ("c128", 20, 2),
                                       ("c128", 20, 3), ("c128", 21, 18)])
def test_sweep_at_the_edges_of_its_tile_sizes(dtype, L, n, dagger):
    """Every amplitude after n periods of distinct Haar-random gates.  An
    amplitude passes n (L-1) gates: a rounding of a gate's entries shifts the
    state by up to one unit in the last place each (they add up in line at
    worst), the FMAs by random ones."""
    say(f"case: sweep {dtype} L={L} n={n} dagger={dagger}")
    G = fin.random_unitaries(L - 1, 4, 500 + L)
    ctx = fl.fl_create(L, dtype)
    fl.fl_set_gates(ctx, G)
    psi = fl.new_state(ctx)
    psi.copy_(torch.from_numpy(fin.random_state(L, L)).to(psi.dtype))
    ref = psi.cpu().numpy().astype(np.complex128)
    want = O.evolve(ref, L, G, n, dagger=dagger)
    fl.fl_apply_period(ctx, psi, n, dagger=dagger)
    got = psi.cpu().numpy().astype(np.complex128)
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    assert np.linalg.norm(got - want) < n * (L - 1) * ulp * np.linalg.norm(want)


# one workgroup: a lone quad, then each number of threads per quad (4 in one
# wave, 4, 2) at its shortest and longest chain; two threads per quad on 9- and
# 10-bit tiles between the chains above, with a remainder after a block
@pytest.mark.parametrize("dagger", [False, True])
@pytest.mark.parametrize("dtype,L,n", [(d, L, n) for d in ("c64", "c128") for L, n in
                                       ((2, 5), (3, 19), (4, 5), (6, 5), (7, 5), (8, 19), (9, 5), (10, 17),
                                        (12, 17), (14, 3))])
def test_sweep_with_several_threads_per_quad(dtype, L, n, dagger):
    """As test_sweep_at_the_edges_of_its_tile_sizes, with its tolerance."""
    test_sweep_at_the_edges_of_its_tile_sizes(dtype, L, n, dagger)


# one tile of each size; 2 tiles; window shares of 1, 2 and 3 bonds, one and two bonds
# left for a last pass, the 16 tiles a workgroup sums between two flushes
@pytest.mark.parametrize("dtype,L", [("c64", 10), ("c64", 11), ("c64", 12), ("c128", 10), ("c128", 11),
                                     ("c64", 13), ("c64", 15), ("c64", 20), ("c64", 22), ("c64", 23), ("c64", 26),
                                     ("c128", 12), ("c128", 13), ("c128", 17), ("c128", 20), ("c128", 23)])
def test_bond_density_matrices_in_windows(dtype, L):
    """Every bond density matrix and the norm of a random state, against plain
    torch FP64 sums over the same stored amplitudes.  FP64 chains of at most
    16 tiles x 8 parts x 8 terms a lane, and trees above them: 1e-13 of the
    norm."""
    say(f"case: rdm windows {dtype} L={L}")
    ctx = fl.fl_create(L, dtype)
    fl.fl_set_bonds(ctx, 2.0 * fin.gue_bond_sample(L, seed=3), 0.7)
    gen = torch.Generator(device="cuda").manual_seed(L)
    psi = torch.randn(1 << L, dtype=ctx.torch_dtype, device="cuda", generator=gen)
    E, N, rho = fl.fl_expect_energy(ctx, psi, rdm=True)
    v = psi.to(torch.complex128)
    norm = v.abs().square().sum().item()
    assert abs(N - norm) < 1e-13 * norm
    for b in range(L - 1):
        x = v.view(1 << b, 4, 1 << (L - 2 - b))
        for i in range(4):
            for j in range(i, 4):
                want = (x[:, i] * x[:, j].conj()).sum().item()
                assert abs(rho[b, i, j] - want) < 1e-13 * norm, (b, i, j)
                assert rho[b, j, i] == np.conj(rho[b, i, j])


# one workgroup, then each tile size of the reverse pass at its shortest and
# longest chains, and the first chain on 12-bit tiles with 4-bit groups
@pytest.mark.parametrize("dtype,L,n,K", [("c64", 3, 4, 2), ("c64", 10, 4, 2), ("c64", 11, 4, 0), ("c64", 17, 2, 1),
                                         ("c64", 18, 2, 0), ("c64", 19, 2, 0), ("c64", 20, 2, 1), ("c64", 21, 2, 0),
                                         ("c128", 2, 3, 1), ("c128", 10, 4, 2), ("c128", 11, 4, 0), ("c128", 17, 2, 1),
                                         ("c128", 18, 2, 0), ("c128", 19, 2, 0), ("c128", 20, 2, 1)])
def test_gradient_at_the_edges_of_its_tile_sizes(dtype, L, n, K):
    """Every component against the oracle adjoint.  The replayed states are off
    by at most n (L-1) units in the last place (as the sweep's), the gradient by
    that times ||H0|| <= 4 (L-1) and the generators' norms, times two."""
    say(f"case: grad {dtype} L={L} n={n} K={K}")
    w = fin.xyz_workload(L, seed=800 + L)
    hs = O.xyz_bond_hamiltonians(L, w["J"], w["fields"])
    gens = O.xyz_coupling_generators(L)
    ref, _ = O.adjoint_gradient(L, hs, gens, w["T"], O.product_state(w["spinors"]), n)
    ctx = fl.fl_create(L, dtype)
    fl.fl_set_bonds(ctx, hs, w["T"])
    psi = fl.new_state(ctx)
    fl.fl_init_state(ctx, psi, w["spinors"])
    ck = []
    for _ in range(n // K if K else 0):
        ck.append(psi.clone())
        fl.fl_apply_period(ctx, psi, K)
    if not K:
        fl.fl_apply_period(ctx, psi, n)
    g = fl.fl_grad(ctx, psi, ck, n, K, gens, torch.empty_like(psi))
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    assert np.max(np.abs(g - ref)) < 2 * n * (L - 1) * ulp * 4 * (L - 1)


# the reverse pass in one workgroup of one wave, of four with idle lanes and
# with none; tiles between the chains above
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("L,n,K", [(2, 5, 0), (4, 3, 0), (7, 18, 0), (8, 4, 2), (9, 18, 9), (12, 17, 0), (14, 4, 2)])
def test_gradient_with_two_threads_per_quad(dtype, L, n, K):
    """As test_gradient_at_the_edges_of_its_tile_sizes, with its tolerance."""
    test_gradient_at_the_edges_of_its_tile_sizes(dtype, L, n, K)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("L", [2, 4, 8])
def test_more_periods_than_one_launch_of_a_short_chain(dtype, L):
    """300 periods in one workgroup are two launches, of 256 and 44: the sweep
    against the oracle (tolerance as above), and the gradient's replay back to
    the initial state, off by the forward's and its own n (L-1) units."""
    n = 300
    test_sweep_at_the_edges_of_its_tile_sizes(dtype, L, n, False)
    ctx, hs, psi, ref = _random_context(L, dtype, 90 + L)
    fl.fl_apply_period(ctx, psi, n)
    fl.fl_grad(ctx, psi, [], n, 0, O.xyz_coupling_generators(L), torch.empty_like(psi))
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    assert np.linalg.norm(psi.cpu().numpy() - ref) < 2 * n * (L - 1) * ulp * np.linalg.norm(ref)


# both sides of the window tables: terms Hermitian to rounding, and terms that
# are Hermitian only within what fl_set_bonds accepts (1e-12 of max(1, |h|))
@pytest.mark.parametrize("dtype,L", [("c64", 12), ("c64", 14), ("c64", 22), ("c128", 12), ("c128", 13), ("c128", 19)])
@pytest.mark.parametrize("size,asym", [(1.0, 0.0), (1.0, 2e-16), (1.0, 5e-13), (3e-13, 3e-13)])
def test_h0_psi_takes_every_entry_of_its_terms(dtype, L, size, asym):
    """H0 psi applies the matrices as given, with the tolerance of
    test_h0_psi_and_its_sums."""
    say(f"case: H0 psi {dtype} L={L} size={size} asym={asym}")
    rng = np.random.default_rng(40 + L)
    hs = size * fin.gue_bond_sample(L, seed=40 + L)
    hs = hs + asym * (rng.uniform(-0.5, 0.5, hs.shape) + 0.5j * rng.uniform(-0.5, 0.5, hs.shape))
    ctx = fl.fl_create(L, dtype)
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    # Hermitian terms before and after them: the two forms follow each other on one context
    for h in (2.0 * fin.gue_bond_sample(L, seed=L), hs, 2.0 * fin.gue_bond_sample(L, seed=L + 1)):
        fl.fl_set_bonds(ctx, h, 0.7)
        psi = fl.new_state(ctx)
        psi.copy_(torch.from_numpy(fin.random_state(L, L)).to(psi.dtype))
        ref = psi.cpu().numpy().astype(np.complex128)
        ws = torch.full_like(psi, float("nan"))
        E, E2, N = fl.fl_energy_spread(ctx, psi, ws)
        want = O.apply_h0(ref, L, h)
        got = ws.cpu().numpy().astype(np.complex128)
        assert np.linalg.norm(got - want) < 10 * ulp * np.linalg.norm(want)
        assert abs(E - np.vdot(ref, got).real) < 1e-12 * np.linalg.norm(ref) * np.linalg.norm(got)
        assert abs(E2 - np.vdot(got, got).real) < 1e-12 * E2
        assert abs(N - np.vdot(ref, ref).real) < 1e-12 * N


def test_bond_density_matrices_over_several_flushes():
    """As test_bond_density_matrices_in_windows, with its tolerance: 16384 tiles
    on 512 workgroups, so that sums go on after a flush (every 16 tiles).  A lane
    sums at most 16 tiles x 8 parts x 8 terms between two flushes: 1024 roundings
    of 1.1e-16, of sums that are at most a quarter of the norm."""
    test_bond_density_matrices_in_windows("c64", 27)


def test_gradient_with_several_tiles_per_workgroup():
    """As test_gradient_at_the_edges_of_its_tile_sizes, with its tolerance: 1024
    tiles on 512 workgroups, the second with the gate table and the sums of the
    first.  Both precisions against one run of the oracle."""
    L, n = 22, 1
    w = fin.xyz_workload(L, seed=800 + L)
    hs = O.xyz_bond_hamiltonians(L, w["J"], w["fields"])
    gens = O.xyz_coupling_generators(L)
    say(f"case: grad oracle L={L} n={n}")
    ref, _ = O.adjoint_gradient(L, hs, gens, w["T"], O.product_state(w["spinors"]), n)
    for dtype, ulp in (("c64", 6e-8), ("c128", 1.2e-16)):
        say(f"case: grad {dtype} L={L} n={n}")
        ctx = fl.fl_create(L, dtype)
        fl.fl_set_bonds(ctx, hs, w["T"])
        psi = fl.new_state(ctx)
        fl.fl_init_state(ctx, psi, w["spinors"])
        fl.fl_apply_period(ctx, psi, n)
        g = fl.fl_grad(ctx, psi, [], n, 0, gens, torch.empty_like(psi))
        assert np.max(np.abs(g - ref)) < 2 * n * (L - 1) * ulp * 4 * (L - 1)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("L", [2, 4, 8])
def test_gradient_over_two_launches_of_a_short_chain(dtype, L):
    """300 periods in one segment are two launches, of 256 and 44, that add to
    the same sums.  Each of the 300 terms of a component is off by as much as
    test_gradient_at_the_edges_of_its_tile_sizes allows the whole: n times its
    tolerance.  Without the 44 periods' terms the gradient would be off by 0.8
    at L = 2, 9.8 at L = 4 and 5.7 at L = 8 (tolerances in complex64: 0.04, 0.4, 2.1)."""
    n = 300
    say(f"case: grad {dtype} L={L} n={n}")
    w = fin.xyz_workload(L, seed=800 + L)
    hs = O.xyz_bond_hamiltonians(L, w["J"], w["fields"])
    gens = O.xyz_coupling_generators(L)
    ref, _ = O.adjoint_gradient(L, hs, gens, w["T"], O.product_state(w["spinors"]), n)
    ctx = fl.fl_create(L, dtype)
    fl.fl_set_bonds(ctx, hs, w["T"])
    psi = fl.new_state(ctx)
    fl.fl_init_state(ctx, psi, w["spinors"])
    fl.fl_apply_period(ctx, psi, n)
    g = fl.fl_grad(ctx, psi, [], n, 0, gens, torch.empty_like(psi))
    ulp = 6e-8 if dtype == "c64" else 1.2e-16
    assert np.max(np.abs(g - ref)) < n * 2 * n * (L - 1) * ulp * 4 * (L - 1)

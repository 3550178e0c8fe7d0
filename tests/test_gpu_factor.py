"""Spin-factorized phase evaluation (Section 2.4: Eqs. svd_weights,
precomp_alpha, precomp_beta, svd_sreverse_sum, dot_product; Algorithm
grouped_hvec) against the oracle's plain scatter and against the
unfactored evaluation of the same kernel.

The factored path changes only the order and grouping of floating-point
operations (each phase sum becomes a rank-R dot product of folded alpha
factors and precomputed beta factors), so it must meet the same bars as the
plain path: 1e-12 relative 2-norm in float64, 1e-6 for complex64 storage on
the same FP32-rounded input, and energies to float64 accumulation error.
The ranks the plan finds pin the structure of Table svd_rank_dist: the
diagonal group has rank n_o + 2, same-spin hopping groups rank 2 and
double-excitation groups rank 1."""

import numpy as np
import pytest
import torch

import synth
from oracle import apply as oapply
from oracle import jw as ojw
from oracle import space as ospace
from tests.conftest import rel_err

pytestmark = pytest.mark.gpu


def _api():
    from paper_2606_28952_amd import api

    return api


CASES = [(6, 3, 3, 1001), (8, 3, 5, 41), (7, 2, 4, 42), (10, 5, 5, 43), (9, 5, 4, 44)]


@pytest.mark.parametrize("n_o,na,nb,seed", CASES)
def test_factored_matches_oracle_and_plain(dev, n_o, na, nb, seed):
    api = _api()
    h1, h2 = synth.molecular_spin_integrals(n_o, seed)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n_o, na, nb)
    psi_np = synth.random_state(sp.dim, seed + 7)
    ref = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n_o, na, nb), psi_np)
    psi = torch.from_numpy(psi_np).to(dev)
    plain = api.apply_pauli_sum(G, sp, psi)
    assert G.factor_info()["present"] == 0
    G.factor(sp)
    info = G.factor_info()
    assert info["present"] == 1 and info["n_beta"] == nb
    assert info["alpha_lists"] == 1 and info["n_alpha"] == na and info["alpha_images"] == 1
    assert info["zero_max_rank"] == n_o + 2, info
    # every non-simple class: X_alpha = 0 (diagonal, rank n_o + 2) and the
    # C(n_o, 2) same-spin alpha hops (rank 2)
    assert info["zero_groups"] == 1 + n_o * (n_o - 1) // 2, info
    assert info["pair_groups"] == n_o * (n_o - 1) // 2 and info["pair_rank"] == 2, info
    assert info["quad_groups"] == n_o * (n_o - 1) * (n_o - 2) * (n_o - 3) // 24 and info["quad_rank"] == 1, info
    # each part alone (mode 1: X_beta = 0 groups; 2: the X_alpha = 0 class's
    # move tables; 4: the simple classes' alpha lists), then all
    errs = {}
    for mode in (1, 2, 4, 7):
        G.set_factored(mode)
        errs[mode] = rel_err(api.apply_pauli_sum(G, sp, psi).cpu().numpy(), ref)
    assert max(errs.values()) < 1e-12, errs
    fact = api.apply_pauli_sum(G, sp, psi)
    out = fact.cpu().numpy()
    assert rel_err(out, plain.cpu().numpy()) < 1e-12
    # fused energy on the factored path
    e = api.expval(G, sp, psi).cpu().numpy()
    e_ref = np.vdot(psi_np, ref)
    assert abs(e[0] - e_ref.real) < 1e-12 * max(1.0, abs(e_ref))
    # complex64 storage against the oracle on the same FP32-rounded input
    psi32_np = psi_np.astype(np.complex64)
    ref32 = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n_o, na, nb), psi32_np.astype(np.complex128))
    out32 = api.apply_pauli_sum(G, sp, torch.from_numpy(psi32_np).to(dev)).cpu().numpy()
    assert rel_err(out32, ref32) < 1e-6
    # switched off: the unfactored evaluation, bit for bit as before
    G.set_factored(0)
    again = api.apply_pauli_sum(G, sp, psi)
    assert torch.equal(torch.view_as_real(again), torch.view_as_real(plain))
    G.set_factored(7)
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(fact))


def test_factor_tables_follow_their_beta_sector(dev):
    # tables built for N_beta = 3 serve (2, 3) but not (3, 2), which falls
    # back to the unfactored evaluation; both stay correct
    api = _api()
    n_o, seed = 6, 51
    h1, h2 = synth.molecular_spin_integrals(n_o, seed)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    op = ojw.jw_sum(h1, h2)
    G.factor(api.Space.sector(n_o, 3, 3))
    for na, nb in [(2, 3), (3, 2), (4, 3)]:
        sp = api.Space.sector(n_o, na, nb)
        psi_np = synth.random_state(sp.dim, 60 + na + nb)
        ref = oapply.apply_scatter(op, ospace.SectorSpace(n_o, na, nb), psi_np)
        out = api.apply_pauli_sum(G, sp, torch.from_numpy(psi_np).to(dev)).cpu().numpy()
        assert rel_err(out, ref) < 1e-12, (na, nb)


def test_factor_refuses_complex_and_full_space(dev):
    api = _api()
    from paper_2606_28952_amd._abi import PbsError

    h1, h2 = synth.molecular_spin_integrals(4, 3)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    with pytest.raises(PbsError, match="spin-sector"):
        G.factor(api.Space.full(8))
    x = np.array([0b11], np.uint64)
    z = np.array([0b01], np.uint64)
    Gc = api.PauliSum.create(8, x, z, np.array([0.5 + 0.25j])).canonicalize().group()
    with pytest.raises(PbsError, match="real"):
        Gc.factor(api.Space.sector(4, 2, 2))


def test_rows_kernel_hubbard_long_rows(dev):
    """Rows too long to stage (complex128, 6,435 beta strings) with alpha
    lists: the barrier-free rows kernel, against the oracle and against the
    unfactored evaluation, apply and fused energy."""
    api = _api()
    h1, h2 = synth.hubbard_spin_integrals(3, 5)
    n_o, na, nb = 15, 2, 7
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n_o, na, nb)
    psi_np = synth.random_state(sp.dim, 71)
    ref = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n_o, na, nb), psi_np)
    psi = torch.from_numpy(psi_np).to(dev)
    plain = api.apply_pauli_sum(G, sp, psi).cpu().numpy()
    G.factor(sp)
    assert G.factor_info()["alpha_lists"] == 1
    out = torch.empty_like(psi)
    e = api.expval(G, sp, psi, out=out).cpu().numpy()
    got = out.cpu().numpy()
    assert rel_err(got, ref) < 1e-12
    assert rel_err(got, plain) < 1e-12
    e_ref = np.vdot(psi_np, ref)
    assert abs(e[0] - e_ref.real) < 1e-12 * max(1.0, abs(e_ref))
    assert abs(e[2] - 1.0) < 1e-13
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(out))
    # the energy alone (no stored product) and the fixed-workspace entry point
    # give the same bits
    assert np.array_equal(api.expval(G, sp, psi).cpu().numpy(), e)
    res = torch.empty(3, dtype=torch.float64, device=dev)
    assert np.array_equal(api.expval_noalloc(G, sp, psi, res).cpu().numpy(), e)
    # complex64 storage: against the oracle on the same FP32-rounded input
    psi32_np = psi_np.astype(np.complex64)
    ref32 = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n_o, na, nb), psi32_np.astype(np.complex128))
    psi32 = torch.from_numpy(psi32_np).to(dev)
    out32 = torch.empty_like(psi32)
    e32 = api.expval(G, sp, psi32, out=out32).cpu().numpy()
    assert rel_err(out32.cpu().numpy().astype(np.complex128), ref32) < 1e-6
    e32_ref = np.vdot(psi32_np.astype(np.complex128), ref32)
    assert abs(e32[0] - e32_ref.real) < 1e-12 * max(1.0, abs(e32_ref))
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi32)), torch.view_as_real(out32))


def _chain_integrals(n, kind, rng):
    """Nearest-neighbour hops on a ring and density-density terms, per kind:
    equal hops with on-site terms, random hops with terms of all ranges and
    spins (diagonal masks across both bytes), hops alone."""
    h1, h2 = np.zeros((2 * n, 2 * n)), np.zeros((2 * n,) * 4)
    for spin in (0, n):
        for p in range(n):
            q = (p + 1) % n
            t = -1.0 if kind != "random" else rng.standard_normal()
            h1[spin + p, spin + q] = h1[spin + q, spin + p] = t
    if kind == "equal":
        pairs = [(p, n + p, 4.0) for p in range(n)]
    elif kind == "random":
        pairs = [(p, q, rng.standard_normal()) for p in range(2 * n) for q in range(p) if rng.random() < 0.3]
    else:
        pairs = []
    for p, q, v in pairs:
        h2[p, q, q, p] = h2[q, p, p, q] = v
    return h1, h2


@pytest.mark.parametrize("n,na,nb,dtype,kind", [(15, 1, 6, "c128", "random"), (16, 2, 5, "c128", "equal"),
                                                (16, 1, 6, "c128", "random"), (16, 1, 7, "c64", "hops"),
                                                (16, 1, 8, "c64", "equal"), (16, 1, 8, "c64", "random"),
                                                (16, 1, 7, "c128", "equal")])
def test_lists_kernel_long_rows(dev, n, na, nb, dtype, kind):
    """Column lists over rows staged in LDS: the shortest and longest rows of
    each storage type (and one too long, which stays with the rows kernel),
    one and many magnitudes, no diagonal group, a last group of 64 columns that
    is not full; against the oracle and the evaluation without move tables.
    Every target sums some forty float64 products of one sign each, so 1e-12;
    single-precision storage rounds inputs exactly and outputs to 2^-24."""
    api = _api()
    rng = np.random.default_rng(n * nb)
    h1, h2 = _chain_integrals(n, kind, rng)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n, na, nb)
    psi_np = synth.random_state(sp.dim, 5)
    if dtype == "c64":
        psi_np = psi_np.astype(np.complex64).astype(np.complex128)
    tol = 1e-12 if dtype == "c128" else 2.0 ** -23
    ref = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n, na, nb), psi_np)
    psi = torch.from_numpy(psi_np).to(dev).to(torch.complex128 if dtype == "c128" else torch.complex64)
    G.factor(sp)
    out = torch.empty_like(psi)
    e = api.expval(G, sp, psi, out=out).cpu().numpy()
    assert rel_err(out.cpu().numpy().astype(np.complex128), ref) < tol
    e_ref = np.vdot(psi_np, ref)
    assert abs(e[0] - e_ref.real) < 1e-12 * max(1.0, abs(e_ref))
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(out))
    rows = sp.shape()[3]
    parts = [api.apply_pauli_sum_rows(G, sp, psi, a, b) for a, b in ((0, 1), (1, rows - 1), (rows - 1, rows))]
    assert torch.equal(torch.view_as_real(torch.cat(parts)), torch.view_as_real(out))
    G.set_factored(5)  # without the move tables
    assert rel_err(api.apply_pauli_sum(G, sp, psi).cpu().numpy().astype(np.complex128), ref) < tol


@pytest.mark.parametrize("n,na,nb,dtype", [(16, 1, 7, "c64"), (16, 2, 7, "c64"), (16, 2, 5, "c128")])
def test_lists_kernel_infinite_amplitude(dev, n, na, nb, dtype):
    """Rows of the lists kernel are summed from their own sources alone: where a
    large amplitude gives a large sum, an infinite one gives that infinity, and
    the other sums stay as they are."""
    api = _api()
    h1, h2 = _chain_integrals(n, "equal", np.random.default_rng(1))
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n, na, nb)
    G.factor(sp)
    da, db = sp.shape()[3:5]
    psi = torch.from_numpy(synth.random_state(sp.dim, 5)).to(dev)
    psi = psi.to(torch.complex128 if dtype == "c128" else torch.complex64)
    for row in range(min(da, 16)):
        col = (37 * row) % db
        outs = []
        for value in (1e30, float("inf")):
            torch.view_as_real(psi)[row * db + col, 0] = value
            outs.append(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)).reshape(da, db, 2))
        torch.view_as_real(psi)[row * db + col, 0] = 0.25
        others = torch.arange(da, device=dev) != row
        big, inf = outs[0][others], outs[1][others]
        large = big.abs() > 1e20
        assert bool(large.any())
        assert torch.equal(torch.where(large, big.sign() * float("inf"), big), inf), row

"""Panel kernel (matrix-core evaluation of factored two-body sectors) against
the oracle where it is quick enough and against the unfactored evaluation of
the sector kernel everywhere, at the edges of its tiles: beta columns around
its 64-column tiles and its 512-column widths, class counts that do and do not
fill a step of four, one to four target rows per workgroup.

Both evaluations sum the same float64 products in another order, so the bars
are those of every factored path: 1e-12 relative 2-norm in float64, 1e-6 for
complex64 storage on the same FP32-rounded input."""

import numpy as np
import pytest
import torch

import synth
from oracle import apply as oapply
from oracle import jw as ojw
from oracle import space as ospace
from tests.conftest import rel_err
from tests.panel_sizes import BATCHES, SINGLE

pytestmark = pytest.mark.gpu

# (n_orb, N_alpha, N_beta): 5 classes per row = one step and one more; 6 and
# 10 columns; 56 and 70; 210; rows and columns on both sides of 256 and 512;
# 715 (ten steps), 924, 1,001, 1,287 and 1,716 columns; 3,432 columns
CASES = [(4, 2, 2), (5, 1, 2), (5, 4, 3), (8, 3, 5), (8, 4, 4), (10, 3, 6), (10, 5, 4), (11, 4, 6), (11, 6, 5),
         (12, 2, 6), (12, 3, 5), (13, 2, 9), (13, 3, 8), (13, 2, 7), (14, 2, 4), (14, 2, 7)]


@pytest.mark.parametrize("n_o,na,nb", CASES)
def test_panel_matches_oracle_and_plain(dev, n_o, na, nb):
    from paper_2606_28952_amd import api

    seed = 900 + 17 * n_o + 5 * na + nb
    h1, h2 = synth.molecular_spin_integrals(n_o, seed)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n_o, na, nb)
    psi_np = synth.random_state(sp.dim, seed + 1)
    psi = torch.from_numpy(psi_np).to(dev)
    plain = api.apply_pauli_sum(G, sp, psi)
    psi32 = psi.to(torch.complex64)
    plain32 = api.apply_pauli_sum(G, sp, psi32.to(torch.complex128))
    G.factor(sp)
    out = torch.empty_like(psi)
    e = api.expval(G, sp, psi, out=out).cpu().numpy()
    got = out.cpu().numpy()
    assert rel_err(got, plain.cpu().numpy()) < 1e-12
    if sp.dim <= 60000:
        ref = oapply.apply_scatter(ojw.jw_sum(h1, h2), ospace.SectorSpace(n_o, na, nb), psi_np)
        assert rel_err(got, ref) < 1e-12
    e_ref = np.vdot(psi_np, plain.cpu().numpy())
    assert abs(e[0] - e_ref.real) < 1e-12 * max(1.0, abs(e_ref)) and abs(e[2] - 1.0) < 1e-13
    # the product alone gives the same bits, twice; the energy alone too
    for _ in range(2):
        assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(out))
    assert np.array_equal(api.expval(G, sp, psi).cpu().numpy(), e)
    # a share of the rows that starts and ends inside row blocks
    a, b = sp.shape()[3] // 3, sp.shape()[3] - sp.shape()[3] // 5
    part = api.apply_pauli_sum_rows(G, sp, psi, a, b)
    db = sp.shape()[4]
    assert torch.equal(torch.view_as_real(part), torch.view_as_real(out[a * db:b * db]))
    out32 = torch.empty_like(psi32)
    e32 = api.expval(G, sp, psi32, out=out32).cpu().numpy()
    assert rel_err(out32.cpu().numpy().astype(np.complex128), plain32.cpu().numpy()) < 1e-6
    p64 = psi32.cpu().numpy().astype(np.complex128)
    e32_ref = np.vdot(p64, plain32.cpu().numpy())
    assert abs(e32[0] - e32_ref.real) < 1e-12 * max(1.0, abs(e32_ref))
    # switched off, the evaluation is the unfactored one, bit for bit
    G.set_factored(0)
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(plain))


def test_panel_reads_an_unaligned_state(dev):
    """A complex64 state that starts 8 bytes past a 16-byte boundary."""
    from paper_2606_28952_amd import api

    h1, h2 = synth.molecular_spin_integrals(8, 77)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(8, 4, 3)
    G.factor(sp)
    psi = torch.from_numpy(synth.random_state(sp.dim, 78)).to(dev).to(torch.complex64)
    base = torch.zeros(sp.dim + 1, dtype=torch.complex64, device=dev)
    base[1:] = psi
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, base[1:])),
                       torch.view_as_real(api.apply_pauli_sum(G, sp, psi)))


def test_panel_needs_its_operator_structure(dev):
    """Operators whose X_alpha = 0 pair groups do not split (a term with an
    alpha Z-mask and another beta parity), or that have other classes, keep
    the sector kernel: same results as unfactored."""
    from paper_2606_28952_amd import api

    n_o = 5
    h1, h2 = synth.molecular_spin_integrals(n_o, 79)
    H = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev))
    x, z, c = H.read()
    # X_0 X_1 on the beta half with a Z on an alpha and on another beta orbital (and its
    # Y Y partner, so that the pair conserves the number)
    bx = (0b11 << n_o)
    extra_z = 0b100 | (0b1000 << n_o)
    xs = np.concatenate([x.reshape(-1), np.array([bx, bx], np.uint64)])
    zs = np.concatenate([z.reshape(-1), np.array([extra_z, extra_z | bx], np.uint64)])
    G = api.PauliSum.create(2 * n_o, xs, zs, np.concatenate([c, [0.3, 0.3]])).canonicalize().group()
    sp = api.Space.sector(n_o, 2, 3)
    psi = torch.from_numpy(synth.random_state(sp.dim, 80)).to(dev)
    plain = api.apply_pauli_sum(G, sp, psi).cpu().numpy()
    G.factor(sp)
    assert rel_err(api.apply_pauli_sum(G, sp, psi).cpu().numpy(), plain) < 1e-12


@pytest.mark.parametrize("n_o,na,nb", [(4, 2, 2), (6, 3, 2), (6, 2, 4), (8, 4, 4)])
def test_panel_without_diagonal_factors(dev, n_o, na, nb):
    """No class has an X_beta = 0 group but the simple ones: the diagonal and
    the single hops of alpha alone are left out, so there is no F row at all."""
    from oracle import pauli as opauli
    from paper_2606_28952_amd import api

    seed = 700 + 10 * n_o + nb
    h1, h2 = synth.molecular_spin_integrals(n_o, seed)
    op = ojw.jw_sum(h1, h2)
    flips = (op.letters == opauli.X) | (op.letters == opauli.Y)
    keep = flips[:, n_o:].any(axis=1) | (flips[:, :n_o].sum(axis=1) == 4)
    op = opauli.PauliSum(2 * n_o, op.letters[keep], op.coeff[keep])
    x, z = op.xz()
    G = api.PauliSum.create(2 * n_o, x, z, op.coeff).canonicalize().group()
    sp = api.Space.sector(n_o, na, nb)
    psi_np = synth.random_state(sp.dim, seed + 1)
    ref = oapply.apply_scatter(op, ospace.SectorSpace(n_o, na, nb), psi_np)
    G.factor(sp)
    psi = torch.from_numpy(psi_np).to(dev)
    out = torch.empty_like(psi)
    e = api.expval(G, sp, psi, out=out).cpu().numpy()
    assert rel_err(out.cpu().numpy(), ref) < 1e-12
    e_ref = np.vdot(psi_np, ref)
    assert abs(e[0] - e_ref.real) < 1e-12 * max(1.0, abs(e_ref))


@pytest.mark.parametrize("n_o,na,nb", [(12, 6, 6), (13, 5, 4), (13, 4, 6), (14, 5, 5), (14, 4, 7)])
@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
def test_panel_shares_of_few_rows(dev, n_o, na, nb, dtype):
    """Shares of few rows give several workgroups to a row: every count of parts
    (one or two groups of 512 columns each, the last one not full) and the sizes
    at which it changes give the whole sector's bits, and energies that add up."""
    from paper_2606_28952_amd import api

    h1, h2 = synth.molecular_spin_integrals(n_o, 501)
    G = api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()
    sp = api.Space.sector(n_o, na, nb)
    G.factor(sp)
    psi = torch.from_numpy(synth.random_state(sp.dim, 502)).to(dev).to(dtype)
    da, db = sp.shape()[3:5]
    whole = torch.view_as_real(api.apply_pauli_sum(G, sp, psi)).reshape(da, db, 2)
    groups = (db + 511) // 512
    for rows in sorted({1, 256 // groups, 256 // groups + 1, 512 // (groups + 1), 512 // groups + 1, 257}):
        a = (da - rows) // 2
        out = torch.empty(rows * db, dtype=dtype, device=dev)
        e = api.expval_rows(G, sp, psi, a, a + rows, out=out).cpu().numpy()
        assert torch.equal(torch.view_as_real(out).reshape(rows, db, 2), whole[a:a + rows]), rows
        part = api.apply_pauli_sum_rows(G, sp, psi, a, a + rows)
        assert torch.equal(torch.view_as_real(part), torch.view_as_real(out)), rows
        p = psi.reshape(da, db)[a:a + rows].to(torch.complex128)
        ref = torch.sum(p.conj() * torch.view_as_complex(whole[a:a + rows].to(torch.float64))).cpu().numpy()
        # the energy sums float64 products, the reference those rounded to storage
        tol = 1e-12 if dtype == torch.complex128 else 1e-6
        assert abs(e[0] - ref.real) < tol * max(1.0, abs(ref)) and abs(e[1] - ref.imag) < tol * max(1.0, abs(ref))
        assert abs(e[2] - float(p.abs().square().sum())) < 1e-12


def _operator(dev, n_o, seed):
    from paper_2606_28952_amd import api

    h1, h2 = synth.molecular_spin_integrals(n_o, seed)
    return api.jw_transform(torch.from_numpy(h1).to(dev), torch.from_numpy(h2).to(dev)).group()


@pytest.mark.parametrize("n_o,na,nb", list(SINGLE))
def test_panel_variants_match_plain(dev, n_o, na, nb):
    """Every variant with its full number of rows per workgroup (the host test of
    the same sizes says that they do), both storage types, against the unfactored
    evaluation."""
    from paper_2606_28952_amd import api

    G = _operator(dev, n_o, 800 + n_o + na)
    sp = api.Space.sector(n_o, na, nb)
    psi = torch.from_numpy(synth.random_state(sp.dim, 801)).to(dev)
    psi32 = psi.to(torch.complex64)
    plain = api.apply_pauli_sum(G, sp, psi)
    plain32 = api.apply_pauli_sum(G, sp, psi32.to(torch.complex128))
    G.factor(sp)
    out, out32 = torch.empty_like(psi), torch.empty_like(psi32)
    e = api.expval(G, sp, psi, out=out).cpu().numpy()
    e32 = api.expval(G, sp, psi32, out=out32).cpu().numpy()

    def off(a, b):
        return float((a - b).abs().square().sum().sqrt() / b.abs().square().sum().sqrt())

    assert off(out, plain) < 1e-12
    assert off(out32.to(torch.complex128), plain32) < 1e-6
    for got, p, h in ((e, psi, plain), (e32, psi32.to(torch.complex128), plain32)):
        ref = float(torch.sum(p.conj() * h).real)
        assert abs(got[0] - ref) < 1e-12 * max(1.0, abs(ref))
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi)), torch.view_as_real(out))
    assert torch.equal(torch.view_as_real(api.apply_pauli_sum(G, sp, psi32)), torch.view_as_real(out32))


@pytest.mark.parametrize("sector,n_jobs", list(BATCHES))
def test_panel_batches_equal_single_launches(dev, sector, n_jobs):
    """A batch's workgroups take three or four rows of a job, a single launch of it
    one or two: same outputs, bit for bit, and energies to rounding."""
    from paper_2606_28952_amd import api

    sp = api.Space.sector(*sector)
    jobs, energies = [], torch.zeros(3 * n_jobs, dtype=torch.float64, device=dev)
    operators = []
    for k in range(n_jobs):
        if k < 3:
            G = _operator(dev, sector[0], 850 + k)
            G.factor(sp)
            operators.append(G)
        psi = torch.from_numpy(synth.random_state(sp.dim, 860 + k)).to(dev)
        jobs.append((operators[k % 3], sp, psi, torch.empty_like(psi)))
    api.Batch(jobs).run(energies)
    e = energies.cpu().numpy().reshape(-1, 3)
    for (G, _, psi, out), got in zip(jobs, e):
        single = torch.empty_like(psi)
        want = api.expval(G, sp, psi, out=single).cpu().numpy()
        assert torch.equal(torch.view_as_real(out), torch.view_as_real(single))
        assert np.abs(got - want).max() < 1e-12 * max(1.0, abs(want[0]))

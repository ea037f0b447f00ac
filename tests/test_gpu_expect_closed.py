"""Photon-number expectations without the Fock space (the default for the full
space) against the oracle's sum over all outputs and its gradient: arbitrary
matrices (the identity holds off the unitary group), bunched inputs, the
vacuum, every photon number it serves, and the recursion beyond."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import rel_err, say, to_dev_c64, widen  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402


@pytest.mark.parametrize("m,n,unitary", [(1, 1, True), (2, 8, True), (3, 7, False), (5, 4, False), (20, 2, True),
                                         (6, 5, False), (32, 1, False), (7, 3, True), (4, 6, True)])
def test_expectations_and_adjoint_against_oracle(m, n, unitary):
    rng = np.random.default_rng(31 * m + n)
    Bn = 4
    U = W.haar_unitaries(rng, Bn, m)
    if not unitary:
        U = U + 0.3 * (rng.standard_normal(U.shape) + 1j * rng.standard_normal(U.shape))
    U = U.astype(np.complex64)
    occ = np.zeros((Bn, m), dtype=np.int32)
    for b in range(Bn - 1):
        np.add.at(occ[b], rng.choice(m, size=max(1, n - b), replace=True), 1)  # the last sample is the vacuum
    say("expectations closed form", m, n)
    batch = B.Batch(B.Plan(m, n), occ)
    w = rng.standard_normal((Bn, m)).astype(np.float32)
    Ud = to_dev_c64(U)
    e = B.fock_mode_expectations(batch, Ud).cpu().numpy()
    g = B.fock_mode_expectations_backward(batch, Ud, torch.from_numpy(w).to(Ud.device)).cpu().numpy()
    for b in range(Bn):
        ref = O.mode_expectations(widen(U[b]), occ[b])
        # FP64 sums rounded once
        assert np.abs(e[b] - ref).max() <= 2.0 ** -23 * max(1.0, np.abs(ref).max())
        if occ[b].sum() == 0:
            assert not g[b].any()
            continue
        basis = O.fock_basis(m, int(occ[b].sum()))
        ref_g = O.probs_grad(widen(U[b]), occ[b], np.asarray(basis) @ w[b].astype(np.float64))
        assert rel_err(g[b], ref_g) <= 1e-6


def test_photon_numbers_beyond_take_the_recursion():
    m, n = 3, 9
    rng = np.random.default_rng(2)
    U = W.haar_unitaries(rng, 2, m).astype(np.complex64)
    occ = np.array([[5, 4, 0], [1, 0, 1]], dtype=np.int32)
    batch = B.Batch(B.Plan(m, n), occ)
    e = B.fock_mode_expectations(batch, to_dev_c64(U)).cpu().numpy()
    for b in range(2):
        assert np.abs(e[b] - O.mode_expectations(widen(U[b]), occ[b])).max() <= 2e-5


@pytest.mark.parametrize("m,n", [(32, 3), (9, 6), (9, 7), (6, 8), (1, 8), (17, 4), (8, 1)])
def test_every_photon_number_below_in_one_batch(m, n):
    # one thread per column subset, 64 of them up to 6 photons and 256 above: samples
    # of every photon number up to n at both widths, modes up to and past a
    # workgroup's rows of eight
    rng = np.random.default_rng(5 * m + n)
    occ = np.zeros((n + 1, m), dtype=np.int32)
    for b in range(n + 1):
        np.add.at(occ[b], rng.choice(m, size=b, replace=True), 1)
    U = (W.haar_unitaries(rng, n + 1, m) * 1.05).astype(np.complex64)
    say("expectations, photon numbers up to", n, "modes", m)
    batch = B.Batch(B.Plan(m, n), occ)
    w = rng.standard_normal((n + 1, m)).astype(np.float32)
    Ud = to_dev_c64(U)
    e = B.fock_mode_expectations(batch, Ud).cpu().numpy()
    g = B.fock_mode_expectations_backward(batch, Ud, torch.from_numpy(w).to(Ud.device)).cpu().numpy()
    for b in range(n + 1):
        ref = O.mode_expectations(widen(U[b]), occ[b])
        # FP64 sums rounded once
        assert np.abs(e[b] - ref).max() <= 2.0 ** -23 * max(1.0, np.abs(ref).max())
        if b == 0:
            assert not g[b].any()
            continue
        basis = O.fock_basis(m, b)
        ref_g = O.probs_grad(widen(U[b]), occ[b], np.asarray(basis) @ w[b].astype(np.float64))
        assert rel_err(g[b], ref_g) <= 2.0 ** -23

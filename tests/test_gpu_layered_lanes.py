"""Layered kernels: one, two and up to eight samples per group, lone samples in a
pair of lanes, pairs of lanes with different photon numbers, every register
class of the adjoint's modes with uneven shares, more than two groups of
predecessors, grids below and above one block per XCD, and restricted spaces."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle as O
from paper_2602_11092_amd import _binding as B
from tests.gpu_util import DEV, G_RTOL, rel_err, say, to_dev_c64, widen

pytestmark = pytest.mark.gpu

# amplitudes of at most 1: n levels of n products in FP32, 12 * 12 * 2^-24 = 9e-6 at
# the largest n here, as random signs 7e-7
ATOL = 2e-6


def _case(m, ns, seed, unbunched=False):
    rng = np.random.default_rng(seed)
    U = W.haar_unitaries(rng, len(ns), m).astype(np.complex64)
    occ = np.zeros((len(ns), m), dtype=np.int32)
    for b, n in enumerate(ns):
        np.add.at(occ[b], rng.choice(m, size=n, replace=not unbunched and (b % 2 == 1 or n > m)), 1)
    batch = B.Batch(B.Plan(m, max(ns), unbunched=unbunched), occ)
    g = rng.uniform(0, 1, batch.out_len).astype(np.float32)
    h = (rng.standard_normal(batch.out_len) + 1j * rng.standard_normal(batch.out_len)).astype(np.complex64)
    return U, occ, batch, g, h


def _run(batch, U, g, h, variant):
    for op in (B.OP_AMPLITUDES, B.OP_PROBS, B.OP_AMPLITUDES_BACKWARD, B.OP_PROBS_BACKWARD):
        batch.set_config(op, variant)
    Ud, gd, hd = to_dev_c64(U), torch.from_numpy(g).to(DEV), torch.from_numpy(h).to(DEV)
    r = [B.fock_amplitudes(batch, Ud), B.fock_probs(batch, Ud), B.fock_amplitudes_backward(batch, Ud, hd),
         B.fock_probs_backward(batch, Ud, gd)]
    torch.cuda.synchronize()
    return [x.cpu().numpy() for x in r]


@pytest.mark.parametrize("m,ns", [
    (3, [2]), (4, [12, 9, 5]), (5, [3, 3]), (8, [1, 4, 4]), (9, [4, 2, 0, 3, 1]), (12, [3] * 7), (13, [4]),
    (17, [3, 2, 3, 3, 1, 3, 3, 2, 3]), (20, [4, 3]), (24, [4]), (24, [3, 4, 4]), (32, [3, 1, 3]), (32, [3]),
])
def test_layered_lanes_against_the_oracle(m, ns):
    say("layered lanes", m, ns)
    U, occ, batch, g, h = _case(m, ns, 31 * m + len(ns))
    a, p, ga, gp = _run(batch, U, g, h, B.VARIANT_LAYERED)
    for b in range(len(ns)):
        o = slice(batch.offsets[b], batch.offsets[b + 1])
        ref = O.amplitudes(widen(U[b]), occ[b])
        assert np.abs(a[o] - ref).max() <= ATOL, b
        assert np.abs(p[o] - np.abs(ref) ** 2).max() <= ATOL, b
        if ns[b] == 0:
            assert np.abs(ga[b]).max() == 0 and np.abs(gp[b]).max() == 0
            continue
        assert rel_err(ga[b], O.amplitude_grad(widen(U[b]), occ[b], h[o].astype(np.complex128))) <= G_RTOL, b
        assert rel_err(gp[b], O.probs_grad(widen(U[b]), occ[b], g[o].astype(np.float64))) <= G_RTOL, b


@pytest.mark.parametrize("m,ns", [(9, [4]), (14, [5, 3, 4]), (22, [4, 4, 2, 4, 4, 4, 1, 4, 4])])
def test_layered_lanes_of_restricted_spaces(m, ns):
    say("layered lanes, restricted", m, ns)
    U, occ, batch, g, h = _case(m, ns, 17 * m, unbunched=True)
    got = _run(batch, U, g, h, B.VARIANT_LAYERED)
    ref = _run(batch, U, g, h, B.VARIANT_FUSED)
    for x, y in zip(got[:2], ref[:2]):
        assert np.abs(x - y).max() <= ATOL
    for x, y in zip(got[2:], ref[2:]):
        assert rel_err(x.astype(np.complex128), y.astype(np.complex128)) <= G_RTOL

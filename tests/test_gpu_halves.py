"""Spaces beyond on-chip memory by the two halves of the modes (the default
there) against the layer-by-layer recursion, every output: each compiled photon
number, odd mode counts (unequal halves), the smallest batches that take it,
bunched inputs, a batch evaluated in two passes; and the batches that keep the
recursion."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import rel_err, say, to_dev_c64  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402

# FP32 on both sides: sums of up to 32 products per rounding chain, and n levels:
# 2^-24 sqrt(32 + 2 n^2) = 8e-7 on either
REL = 2e-6


def _batch(m, n, Bn, seed):
    rng = np.random.default_rng(seed)
    U = W.haar_unitaries(rng, Bn, m).astype(np.complex64)
    occ = np.zeros((Bn, m), dtype=np.int32)
    for b in range(Bn):
        np.add.at(occ[b], rng.choice(m, size=n, replace=b % 2 == 1), 1)
    return to_dev_c64(U), occ


@pytest.mark.parametrize("m,n,Bn", [(28, 6, 8), (31, 6, 5), (26, 7, 5), (28, 7, 1), (23, 8, 1), (24, 8, 2), (24, 8, 33)])
def test_two_halves_match_the_recursion(m, n, Bn):
    U, occ = _batch(m, n, Bn, 7 * m + n)
    say("two halves", m, n, Bn)
    batch = B.Batch(B.Plan(m, n), occ)
    ref = B.Batch(batch.plan, occ)
    for op in (B.OP_PROBS, B.OP_AMPLITUDES):
        assert batch.get_config(op)[0] == B.VARIANT_LAYERED
        ref.set_config(op, B.VARIANT_LAYERED, 256)
    a, p = B.fock_amplitudes(batch, U), B.fock_probs(batch, U)
    ra, rp = B.fock_amplitudes(ref, U), B.fock_probs(ref, U)
    torch.cuda.synchronize()
    assert not torch.equal(a, ra)  # two routes
    for b in sorted({0, Bn // 2, (Bn - 1) // 2, Bn - 1}):
        o = slice(batch.offsets[b], batch.offsets[b + 1])
        assert rel_err(a[o].cpu().numpy(), ra[o].cpu().numpy()) <= REL, b
        assert rel_err(p[o].cpu().numpy(), rp[o].cpu().numpy()) <= REL, b
        assert (p[o] - a[o].abs().square()).abs().max().item() <= 1e-6


@pytest.mark.parametrize("few", [False, True])
def test_mixed_photon_numbers_and_small_batches_keep_the_recursion(few):
    m = 28
    U, occ = _batch(m, 6, 9, 5)
    occ[1] = 0
    occ[1, :5] = 1
    if few:
        U, occ = U[:2].contiguous(), np.tile(occ[:1], (2, 1))
    batch = B.Batch(B.Plan(m, 6), occ)
    ref = B.Batch(batch.plan, occ)
    ref.set_config(B.OP_PROBS, B.VARIANT_LAYERED, 0)
    assert torch.equal(B.fock_probs(batch, U), B.fock_probs(ref, U))


def test_two_halves_graph_replays():
    m, n = 28, 6
    U, occ = _batch(m, n, 8, 9)
    batch = B.Batch(B.Plan(m, n), occ)
    out = torch.empty(batch.out_len, dtype=torch.float32, device=U.device)
    ws = batch.workspace(B.OP_PROBS, U.device)
    B.fock_probs(batch, U, out=out, ws=ws)
    torch.cuda.synchronize()
    want = out.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.fock_probs(batch, U, out=out, ws=ws)
    for _ in range(3):
        out.zero_()
        ws.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


@pytest.mark.parametrize("m,n,Bn", [(28, 6, 8), (29, 6, 7), (28, 7, 2), (23, 8, 2)])
def test_two_halves_against_64_bit_permanents(m, n, Bn):
    """A sample of the outputs, each cut of the photons between the halves among
    them, and the first and the last state."""
    from oracle import oracle as O
    U, occ = _batch(m, n, Bn, m + n)
    batch = B.Batch(B.Plan(m, n), occ)
    say("two halves against permanents", m, n, Bn)
    a, p = B.fock_amplitudes(batch, U).cpu().numpy(), B.fock_probs(batch, U).cpu().numpy()
    rng = np.random.default_rng(1)
    ref = B.Batch(batch.plan, occ)
    ref.set_config(B.OP_PROBS, B.VARIANT_LAYERED, 256)
    assert not np.array_equal(p, B.fock_probs(ref, U).cpu().numpy())  # the two halves ran
    states = []
    for k in range(n + 1):  # k photons in the low half
        for _ in range(20):
            t = np.zeros(m, dtype=np.int32)
            np.add.at(t, rng.integers(0, m // 2, size=k), 1)
            np.add.at(t, rng.integers(m // 2, m, size=n - k), 1)
            states.append(t)
    for j in (0, m - 1):
        states.append((np.arange(m) == j).astype(np.int32) * n)
    ranks = np.array([O.fock_rank(m, n, t) for t in states])
    for b in (0, Bn - 1):
        want = O.amplitudes(U[b].cpu().numpy().astype(np.complex128), occ[b], outputs=np.asarray(states))
        at = batch.offsets[b] + ranks
        assert rel_err(a[at], want) <= REL, b
        assert rel_err(p[at], np.abs(want) ** 2) <= 2 * REL, b

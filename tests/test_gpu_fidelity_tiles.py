"""The tiled fidelity kernels at the edges of their 16 x 16 (n <= 7) and 8 x 8
(n = 8) tiles, for every compiled n: against 64-bit permanents, and a Gram
matrix (formed above the diagonal, mirrored) against the same matrix as a
product of two batches."""
import itertools

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import say, to_dev_c64, widen  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402

# FP64 sums rounded to FP32 once: half an ulp of values up to 1
TOL = 2.0 ** -24 + 1e-12


def _perm(M):
    n = M.shape[0]
    level = {0: 1.0 + 0j}
    for r in range(n):
        nxt = {}
        for s, v in level.items():
            for i in range(n):
                if not s >> i & 1:
                    nxt[s | 1 << i] = nxt.get(s | 1 << i, 0) + v * M[r, i]
        level = nxt
    return level[(1 << n) - 1]


@pytest.mark.parametrize("n", range(1, 9))
@pytest.mark.parametrize("B1,B2", [(1, 1), (17, 5), (9, 33)])
def test_tiles_against_64_bit_permanents(n, B1, B2):
    rng = np.random.default_rng(100 * n + B1)
    m = max(3, n)
    U1 = W.haar_unitaries(rng, B1, m).astype(np.complex64)
    U2 = W.haar_unitaries(rng, B2, m).astype(np.complex64)
    occ = np.zeros(m, dtype=np.int32)
    np.add.at(occ, rng.choice(m, size=n, replace=n > 2), 1)
    C = np.repeat(np.arange(m), occ)
    fact = np.prod([float(np.prod(np.arange(1, v + 1))) for v in occ])
    say("fidelity tiles", n, B1, B2)
    K = B.fock_fidelity_kernel(occ, to_dev_c64(U1), to_dev_c64(U2)).cpu().numpy()
    pairs = list(itertools.product(range(B1), range(B2)))
    for i in rng.permutation(len(pairs))[:40].tolist() + [len(pairs) - 1]:
        a, b = pairs[i]
        M = widen(U1[a])[:, C].conj().T @ widen(U2[b])[:, C]
        assert abs(K[a, b] - abs(_perm(M) / fact) ** 2) <= TOL, (a, b)


@pytest.mark.parametrize("n,Bn", [(2, 16), (3, 31), (5, 33), (7, 18), (8, 19)])
def test_gram_matrix_is_the_mirrored_product(n, Bn):
    rng = np.random.default_rng(n)
    m = 9
    U = to_dev_c64(W.haar_unitaries(rng, Bn, m))
    occ = (np.arange(m) < n).astype(np.int32)
    G = B.fock_fidelity_kernel(occ, U)
    K = B.fock_fidelity_kernel(occ, U, U.clone())
    torch.cuda.synchronize()
    assert torch.equal(G, G.t())
    iu = torch.triu_indices(Bn, Bn)
    assert torch.equal(G[iu[0], iu[1]], K[iu[0], iu[1]])
    assert (G.diagonal() - 1).abs().max().item() <= 1e-6  # complex64 unitaries: n rounding errors of 6e-8


@pytest.mark.parametrize("n,rows,length", [(3, 1, 16385), (4, 2, 16385), (5, 2, 16400), (6, 2, 16385), (6, 1, 16385),
                                           (7, 6, 4097), (7, 7, 4097), (8, 1, 4097), (8, 2, 100), (5, 3, 40), (2, 12, 40)])
def test_few_rows_or_columns_against_64_bit_permanents(n, rows, length):
    # a thread per pair, and tiles with waves that have no pairs, both ways round
    rng = np.random.default_rng(10 * n + rows)
    m = 8
    U1 = W.haar_unitaries(rng, rows, m).astype(np.complex64)
    U2 = np.tile(W.haar_unitaries(rng, 37, m), (-(-length // 37), 1, 1))[:length].astype(np.complex64)
    occ = np.zeros(m, dtype=np.int32)
    np.add.at(occ, rng.choice(m, size=n, replace=True), 1)
    C = np.repeat(np.arange(m), occ)
    fact = np.prod([float(np.prod(np.arange(1, v + 1))) for v in occ])
    say("fidelity, few rows", n, rows, length)
    K = B.fock_fidelity_kernel(occ, to_dev_c64(U1), to_dev_c64(U2))
    Kt = B.fock_fidelity_kernel(occ, to_dev_c64(U2), to_dev_c64(U1))
    assert K.shape == (rows, length) and Kt.shape == (length, rows)
    K, Kt = K.cpu().numpy(), Kt.cpu().numpy()
    for a in range(rows):
        for b in (0, 1, 15, 16, 36):
            want = abs(_perm(widen(U1[a])[:, C].conj().T @ widen(U2[b])[:, C]) / fact) ** 2
            # U2 repeats every 37 matrices
            assert np.abs(K[a, b::37] - want).max() <= TOL and np.abs(Kt[b::37, a] - want).max() <= TOL, (a, b)

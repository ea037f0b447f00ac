"""The shot search that keeps the cumulative sums on chip: sample lengths
around its runs of 16 states, few samples with many shots (several workgroups
per sample), targets on and past the last state."""
import math

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import DEV, say, to_dev_c64  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402


@pytest.mark.parametrize("m,n,Bn,S", [(1, 3, 2, 5), (15, 1, 3, 64), (16, 1, 3, 64), (17, 1, 2, 1025), (5, 3, 1, 5000),
                                      (14, 6, 2, 3000)])
def test_shots_follow_the_cumulative_sums(m, n, Bn, S):
    rng = np.random.default_rng(m + n)
    U = W.haar_unitaries(rng, Bn, m).astype(np.complex64)
    occ = np.zeros((Bn, m), dtype=np.int32)
    for b in range(Bn):
        np.add.at(occ[b], rng.choice(m, size=n, replace=True), 1)
    occ[-1, :] = 0  # one vacuum sample beside the others
    u = rng.random((Bn, S)).astype(np.float32)
    u[:, 0] = 0.0
    u[:, 1] = np.nextafter(np.float32(1), np.float32(0))
    say("sample direct", m, n, Bn, S)
    batch = B.Batch(B.Plan(m, n), occ)
    Ud = to_dev_c64(U)
    for op in (B.OP_SAMPLE, B.OP_PROBS):
        batch.set_config(op, B.VARIANT_FUSED, 256)
    shots = B.fock_sample(batch, Ud, torch.from_numpy(u).to(DEV)).cpu().numpy()
    p = B.fock_probs(batch, Ud).cpu().numpy().astype(np.float64)
    for b in range(Bn):
        cdf = np.cumsum(p[batch.offsets[b]:batch.offsets[b + 1]])
        target = u[b].astype(np.float64) * cdf[-1]
        want = np.minimum(np.searchsorted(cdf, target, side="right"), cdf.size - 1)
        # the sums' order differs by FP64 rounding: 2^-53 N of a total of 1
        close = np.abs(cdf[want] - target) <= cdf.size * 2.0 ** -52
        assert np.all((shots[b] == want) | close), b
        assert cdf.size == math.comb(m + int(occ[b].sum()) - 1, int(occ[b].sum()))


# batches that take 256 threads a sample, samples at the edges of a run of 16 states,
# and the longest sample that does (8192 states at most) beside the first that does not
@pytest.mark.parametrize("m,n,Bn,S", [(2, 1, 1024, 3), (17, 1, 1030, 300), (31, 1, 1024, 40), (16, 2, 1024, 20),
                                      (20, 4, 1024, 9), (22, 4, 1024, 5)])
def test_shots_of_many_samples_follow_the_cumulative_sums(m, n, Bn, S):
    rng = np.random.default_rng(m + n)
    U = np.tile(W.haar_unitaries(rng, 16, m), (-(-Bn // 16), 1, 1))[:Bn].astype(np.complex64)
    occ = np.zeros((Bn, m), dtype=np.int32)
    for b in range(Bn):
        np.add.at(occ[b], rng.choice(m, size=n, replace=True), 1)
    occ[-1, :] = 0
    u = rng.random((Bn, S)).astype(np.float32)
    u[:, 0] = 0.0
    u[:, 1] = np.nextafter(np.float32(1), np.float32(0))
    say("sample direct, many samples", m, n, Bn, S)
    batch = B.Batch(B.Plan(m, n), occ)
    Ud = to_dev_c64(U)
    for op in (B.OP_SAMPLE, B.OP_PROBS):
        batch.set_config(op, B.VARIANT_FUSED, 256)
    shots = B.fock_sample(batch, Ud, torch.from_numpy(u).to(DEV)).cpu().numpy()
    p = B.fock_probs(batch, Ud).cpu().numpy().astype(np.float64)
    for b in [0, 1, Bn // 2, Bn - 2, Bn - 1]:
        cdf = np.cumsum(p[batch.offsets[b]:batch.offsets[b + 1]])
        target = u[b].astype(np.float64) * cdf[-1]
        want = np.minimum(np.searchsorted(cdf, target, side="right"), cdf.size - 1)
        # the sums' order differs by FP64 rounding: 2^-53 N of a total of 1
        close = np.abs(cdf[want] - target) <= cdf.size * 2.0 ** -52
        assert np.all((shots[b] == want) | close), b

"""The fused adjoint reading click-pattern gradients: each workgroup size and mode
class, n from 1 up, mixed photon numbers and a restricted plan (whose gradients
are expanded first), against the probability adjoint on gradients expanded by
the oracle's pattern list."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle as O
from paper_2602_11092_amd import _binding as B
from tests.gpu_util import DEV, rel_err, say, to_dev_c64

pytestmark = pytest.mark.gpu

# the same kernel body on the same values: contraction may differ between the
# instances, one FP32 rounding per term
REL = 1e-6


@pytest.mark.parametrize("m,ns,block,unbunched", [
    (6, [1, 3, 0, 2, 1], 256, False), (9, [4, 4, 2], 512, False), (14, [3, 4, 1], 256, False),
    (18, [4, 4], 768, False), (20, [4, 4, 3], 1024, False), (23, [3, 2], 512, False), (27, [3, 1], 256, False),
    (8, [3, 3, 1], 256, True),
])
def test_click_adjoint_reads_the_pattern_gradients(m, ns, block, unbunched):
    rng = np.random.default_rng(13 * m)
    U = to_dev_c64(W.haar_unitaries(rng, len(ns), m).astype(np.complex64))
    occ = np.zeros((len(ns), m), dtype=np.int32)
    for b, n in enumerate(ns):
        np.add.at(occ[b], rng.choice(m, size=n, replace=not unbunched), 1)
    batch = B.Batch(B.Plan(m, max(ns), threshold=True, unbunched=unbunched), occ)
    try:
        for op in (B.OP_THRESHOLD_PROBS_BACKWARD, B.OP_PROBS_BACKWARD):
            batch.set_config(op, B.VARIANT_FUSED, block)
    except B.SlosError:
        assert block >= 768  # not offered for this shape
        pytest.skip("workgroup size not offered for this shape")
    gP = rng.standard_normal(batch.threshold_len).astype(np.float32)
    gp = np.zeros(batch.out_len, dtype=np.float32)
    for b, n in enumerate(ns):
        index = {c: i for i, c in enumerate(O.click_patterns(m, n))}
        basis = [t for t in O.fock_basis(m, n) if not unbunched or t.max(initial=0) <= 1]
        g = gP[batch.threshold_offsets[b]:batch.threshold_offsets[b + 1]]
        gp[batch.offsets[b]:batch.offsets[b + 1]] = [g[index[tuple(int(j) for j in np.nonzero(t)[0])]] for t in basis]
    say("click adjoint", m, ns, block, unbunched)
    got = B.fock_threshold_probs_backward(batch, U, torch.from_numpy(gP).to(DEV))
    want = B.fock_probs_backward(batch, U, torch.from_numpy(gp).to(DEV))
    torch.cuda.synchronize()
    got, want = got.cpu().numpy().astype(np.complex128), want.cpu().numpy().astype(np.complex128)
    for b, n in enumerate(ns):
        assert rel_err(got[b], want[b]) <= REL if n else not got[b].any(), b

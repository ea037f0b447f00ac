"""Workspaces: a route that keeps everything on chip asks for none and runs
without one; the routes beside it ask for theirs and are refused without."""
import numpy as np
import pytest

from oracle import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

from gpu_util import DEV, say, to_dev_c64  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402


def _refused(fn):
    with pytest.raises(B.SlosError) as e:
        fn()
    assert e.value.code == B.SLOS_EWORKSPACE


def _raw(name, *args):
    B._check(name, getattr(B.lib(), name)(*args, B._stream_ptr(torch.device(DEV))))


def _batch(m, n, Bn, **plan):
    rng = np.random.default_rng(m + n)
    occ = np.zeros((Bn, m), dtype=np.int32)
    occ[:, :n] = 1
    return B.Batch(B.Plan(m, n, **plan), occ), to_dev_c64(W.haar_unitaries(rng, Bn, m))


def test_closed_expectations_need_no_workspace():
    batch, U = _batch(8, 4, 3)
    say("expectations without a workspace")
    w = torch.randn((3, 8), device=DEV)
    e, g = torch.empty((3, 8), device=DEV), torch.empty_like(U)
    for op in (B.OP_MODE_EXPECTATIONS, B.OP_MODE_EXPECTATIONS_BACKWARD):
        assert batch.workspace_bytes(op, B.DETECTOR_PNR) == 0
    _raw("fock_mode_expectations", batch.handle, U.data_ptr(), e.data_ptr(), None, 0)
    _raw("fock_mode_expectations_backward", batch.handle, U.data_ptr(), w.data_ptr(), g.data_ptr(), None, 0)
    assert torch.equal(e, B.fock_mode_expectations(batch, U))
    assert torch.equal(g, B.fock_mode_expectations_backward(batch, U, w))
    # click detectors take the recursion's adjoint, and its workspace
    op = B.OP_MODE_EXPECTATIONS_BACKWARD
    assert batch.workspace_bytes(op, B.DETECTOR_THRESHOLD) == batch.workspace_bytes(op) >= 4 * batch.out_len
    _refused(lambda: _raw("fock_mode_expectations_backward_ex", batch.handle, U.data_ptr(), w.data_ptr(), g.data_ptr(),
                          B.DETECTOR_THRESHOLD, None, 0))
    batch.set_config(op, B.VARIANT_FUSED)
    assert batch.workspace_bytes(op, B.DETECTOR_PNR) == batch.workspace_bytes(op) >= 4 * batch.out_len
    _refused(lambda: _raw("fock_mode_expectations_backward", batch.handle, U.data_ptr(), w.data_ptr(), g.data_ptr(),
                          None, 0))


def test_dense_superpositions_need_no_workspace():
    m, n = 6, 3
    occ = np.asarray(O.fock_basis(m, n), dtype=np.int32)
    batch = B.Batch(B.Plan(m, n), occ)
    sup = B.Superposition(batch, [0, len(occ)])
    U = to_dev_c64(W.haar_unitaries(np.random.default_rng(1), 1, m))
    x = torch.randn(len(occ), dtype=torch.complex64, device=DEV)
    y, gU, gx = torch.empty_like(x), torch.empty_like(U), torch.empty_like(x)

    def forward():
        _raw("fock_superposition_amplitudes", sup.handle, U.data_ptr(), x.data_ptr(), y.data_ptr(), None, 0)

    def backward():
        _raw("fock_superposition_amplitudes_backward", sup.handle, U.data_ptr(), x.data_ptr(), x.data_ptr(),
             gU.data_ptr(), gx.data_ptr(), None, 0)

    say("dense superpositions without a workspace")
    forward()
    backward()
    assert torch.equal(y, B.fock_superposition_amplitudes(sup, U, x))
    assert all(map(torch.equal, (gU, gx), B.fock_superposition_amplitudes_backward(sup, U, x, x)))
    batch.set_config(B.OP_AMPLITUDES, B.VARIANT_FUSED)
    _refused(forward)
    backward()
    batch.set_config(B.OP_AMPLITUDES_BACKWARD, B.VARIANT_FUSED)
    _refused(backward)


# 131072 states at most per sample on chip: C(19 + 5, 6) = 134596 are too many
@pytest.mark.parametrize("m,n,kept", [(8, 4, False), (18, 6, False), (19, 6, True)])
def test_shots_ask_for_sums_only_beyond_the_chip(m, n, kept):
    batch, U = _batch(m, n, 2)
    say("shots' workspace", m, n)
    batch.set_config(B.OP_SAMPLE, B.VARIANT_LAYERED if m > 8 else B.VARIANT_FUSED)
    batch.set_config(B.OP_PROBS, *batch.get_config(B.OP_SAMPLE))
    p = 4 * batch.out_len
    need = batch.workspace_bytes(B.OP_SAMPLE) - batch.workspace_bytes(B.OP_PROBS)
    assert (need >= 3 * p) if kept else (p <= need < p + 256)
    ws = torch.full((batch.workspace_bytes(B.OP_SAMPLE) + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    u = torch.rand((2, 700), device=DEV)
    u[:, 0], u[:, 1] = 0.0, 1 - 2.0 ** -24
    shots = B.fock_sample(batch, U, u, ws=ws[:-4096])
    assert bool((ws[-4096:] == 0xA5).all())  # nothing beyond what was asked for
    _refused(lambda: B.fock_sample(batch, U, u, ws=ws[:256]))
    probs = B.fock_probs(batch, U).cpu().numpy().astype(np.float64).reshape(2, -1)
    for b in range(2):
        cdf = np.cumsum(probs[b])
        target = u[b].cpu().numpy().astype(np.float64) * cdf[-1]
        want = np.minimum(np.searchsorted(cdf, target, side="right"), cdf.size - 1)
        # the sums' order differs by FP64 rounding: 2^-53 N of a total of 1
        assert np.all((shots[b].cpu().numpy() == want) | (np.abs(cdf[want] - target) <= cdf.size * 2.0 ** -52))


@pytest.mark.parametrize("unbunched", [False, True])
def test_click_adjoint_workspace(unbunched):
    batch, U = _batch(8, 3, 4, threshold=True, unbunched=unbunched)
    op = B.OP_THRESHOLD_PROBS_BACKWARD
    say("click adjoint's workspace", unbunched)
    assert batch.get_config(op)[0] == B.VARIANT_FUSED
    g, gU = torch.randn(batch.threshold_len, device=DEV), torch.empty_like(U)

    def bare():
        _raw("fock_threshold_probs_backward", batch.handle, U.data_ptr(), g.data_ptr(), gU.data_ptr(), None, 0)

    if unbunched:
        assert batch.workspace_bytes(op) >= 4 * batch.out_len
        _refused(bare)
    else:
        assert batch.workspace_bytes(op) == 0
        bare()
        assert torch.equal(gU, B.fock_threshold_probs_backward(batch, U, g))
        batch.set_config(op, B.VARIANT_LAYERED)
        _refused(bare)


def test_layers_in_a_workspace_of_any_alignment():
    # the layers are read two complex values at a time; a workspace carved from a
    # larger one need not begin on 16 bytes
    batch, U = _batch(20, 5, 12)
    say("layered workspace at 8 bytes past an allocation")
    g = torch.randn(batch.out_len, device=DEV)
    for op in (B.OP_PROBS, B.OP_PROBS_BACKWARD):
        batch.set_config(op, B.VARIANT_LAYERED)
    want = B.fock_probs(batch, U), B.fock_probs_backward(batch, U, g)

    def off(op):
        return torch.empty(batch.workspace_bytes(op) + 8, dtype=torch.uint8, device=DEV)[8:]

    assert torch.equal(want[0], B.fock_probs(batch, U, ws=off(B.OP_PROBS)))
    assert torch.equal(want[1], B.fock_probs_backward(batch, U, g, ws=off(B.OP_PROBS_BACKWARD)))

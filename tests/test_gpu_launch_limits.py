"""Batches of 2^32 threads and more along one dimension of a launch, which the
runtime refuses or takes modulo 2^32: the kernels with one workgroup per tile or
per sample spread over a second dimension."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import DEV, say  # noqa: E402
import torch  # noqa: E402
from paper_2602_11092_amd import _binding as B  # noqa: E402


def _columns(Bn, seed):
    """Bn 1 x 1 'interferometers', complex numbers of modulus about 1."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    phase = torch.rand(Bn, device=DEV, generator=g) * 6.0
    return torch.polar(0.9 + 0.1 * torch.cos(phase), phase).reshape(Bn, 1, 1)


# tiles of 16 rows (n <= 7) and 8 (n = 8), two of them: 2^24 tiles of 256 threads
@pytest.mark.parametrize("n,B1,B2", [(1, 17, (1 << 27) + 16), (8, 9, (1 << 26) + 8)])
def test_fidelity_of_more_tiles_than_a_launch_takes(n, B1, B2):
    say("fidelity tiles past the launch limit", n, B1, B2)
    U1, U2 = _columns(B1, 1), _columns(B2, 2)
    K = B.fock_fidelity_kernel(np.array([n], dtype=np.int32), U1, U2)
    torch.cuda.synchronize()
    # one mode: Perm(conj(u) v in every place) = n! (conj(u) v)^n, so K = |u v|^(2 n)
    at = torch.cat([torch.arange(100), torch.arange(B2 - 100, B2), torch.randint(0, B2, (800,))]).to(DEV)
    u, v = U1.reshape(B1, 1).to(torch.complex128).abs(), U2.reshape(-1)[at].to(torch.complex128).abs()
    # FP64 arithmetic, rounded to FP32 once (values up to 1)
    assert (K[:, at].double() - (u * v) ** (2 * n)).abs().max().item() <= 2.0 ** -24 + 1e-12


def test_shots_of_more_samples_than_a_launch_takes():
    # one workgroup of 1024 threads per sample: 2^22 of them are too many
    Bn = (1 << 22) + 2
    say("samples past the launch limit", Bn)
    g = torch.Generator(device=DEV).manual_seed(3)
    angle = torch.rand(Bn, device=DEV, generator=g) * 6.0
    c, s = torch.cos(angle), torch.sin(angle)
    U = torch.stack([c, -s, s, c], dim=1).reshape(Bn, 2, 2).to(torch.complex64)
    batch = B.Batch(B.Plan(2, 1), np.tile(np.array([[1, 0]], dtype=np.int32), (Bn, 1)))
    u = torch.rand((Bn, 1), device=DEV, generator=g)
    shots = B.fock_sample(batch, U, u)
    torch.cuda.synchronize()
    # state 0 (the photon in mode 0) while u (p_0 + p_1) < p_0
    p = B.fock_probs(batch, U).reshape(Bn, 2).double()
    want = (u[:, 0].double() * p.sum(dim=1) >= p[:, 0]).to(torch.int32)
    assert torch.equal(shots[:, 0], want)

"""The work whose speed counts: calls of this framework's public entry points
as a program makes them, with the sizes of its own workloads.

Every case runs with the library's own choice of kernels (no autotuning), the
plan, batch or layer built beforehand, as a program that calls repeatedly
keeps them.  Kinds:

  layer    a QuantumLayer training step: mesh -> U -> outputs (probabilities,
           per-mode expectations or click probabilities, in the full or the
           unbunched space), and the gradients of its phases and features
           for a given output gradient
  probs    fock_probs on given unitaries (inference, or a scan over circuits)
  mesh     mesh_to_unitary, then fock_probs, on a batch of mixed photon numbers
  grad     fock_probs and its adjoint on given unitaries
  amps     fock_amplitudes and its adjoint (complex outputs and gradients),
           bunched inputs among them
  sample   fock_sample: shots from given uniforms
  gram     fock_fidelity_kernel: the Gram matrix of a kernel method
  super    amplitude-encoded inputs, a circuit of its own per input, with the
           gradients of the circuit and of the input amplitudes

`exact` computes the same in 64 bits with torch alone: the photon-by-photon
recursion over index tables made here, and the mesh as products of 2x2 blocks.
"""
import functools
import itertools
import math

import numpy as np
import torch

import paper_2602_11092_amd as slos

DEV = "cuda"


def listed():
    return [
        # the smallest layer step, the example of the readme: latency and launches
        dict(name="layer_m6_n3_b64", kind="layer", out="probs", space="fock", m=6, n=3, B=64),
        # inference over a batch of interferometers
        dict(name="probs_m16_n6_b256", kind="probs", m=16, n=6, B=256),
        # angle-encoded features through one mesh, inputs of 2 to 6 photons in one call
        dict(name="mesh_m12_n2to6_b4096", kind="mesh", m=12, lo=2, n=6, B=4096),
        # the headline training step: 42504 outputs per sample
        dict(name="layer_m20_n5_b512", kind="layer", out="probs", space="fock", m=20, n=5, B=512),
        # the largest Fock space: 7.9 million outputs per sample, beyond on-chip memory
        dict(name="grad_m24_n8_b16", kind="grad", m=24, n=8, B=16),
        # complex outputs and gradients, an odd size, bunched inputs
        dict(name="amps_m13_n4_b77", kind="amps", m=13, n=4, B=77),
        # measurement strategies of the layer
        dict(name="expect_m20_n5_b512", kind="layer", out="mode_expectations", space="fock", m=20, n=5, B=512),
        dict(name="clicks_m20_n5_b512", kind="layer", out="threshold_probs", space="fock", m=20, n=5, B=512),
        # training in the collision-free space
        dict(name="unbunched_m20_n5_b512", kind="layer", out="probs", space="unbunched", m=20, n=5, B=512),
        # shots, as hardware returns them
        dict(name="sample_m20_n5_b512_s1024", kind="sample", m=20, n=5, B=512, S=1024),
        # a kernel method's Gram matrix
        dict(name="gram_m10_n7_b512", kind="gram", m=10, n=7, B=512),
        # amplitude encoding: 56 components per input
        dict(name="super_m6_n3_g1024", kind="super", m=6, n=3, B=1024),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)) - 1e-9)))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "probs", "mesh", "grad", "amps", "sample", "gram", "super"])
    if kind == "layer":
        out = rng.choice(["probs", "probs", "mode_expectations", "threshold_probs"])
        space = rng.choice(["fock", "fock", "unbunched"])
        m, n = rng.randint(5, 20), rng.randint(2, 5)
        B = _log(rng, 16, min(1024, max(17, 22_000_000 // _dim(m, n))))
        return dict(kind=kind, out=out, space=space, m=m, n=n, B=B)
    if kind in ("probs", "sample"):
        m, n = rng.randint(5, 20), rng.randint(2, 6)
        while _dim(m, n) > 60_000:
            n -= 1
        B = _log(rng, 8, min(1024, max(9, 20_000_000 // _dim(m, n))))
        return dict(kind=kind, m=m, n=n, B=B, **({"S": _log(rng, 50, 5000)} if kind == "sample" else {}))
    if kind == "mesh":
        m, n = rng.randint(6, 14), rng.randint(3, 6)
        return dict(kind=kind, m=m, lo=rng.randint(1, n - 1), n=n, B=_log(rng, 64, 4096 if _dim(m, n) <= 12_376 else 1024))
    if kind == "grad":
        m, n = rng.randint(12, 24), rng.randint(5, 8)
        while _dim(m, n) > 7_900_000:
            n -= 1
        return dict(kind=kind, m=m, n=n, B=_log(rng, 2, min(64, max(3, 80_000_000 // _dim(m, n)))))
    if kind == "amps":
        m, n = rng.randint(5, 17), rng.randint(2, 5)
        return dict(kind=kind, m=m, n=n, B=_log(rng, 8, min(512, max(9, 8_000_000 // _dim(m, n)))))
    if kind == "gram":
        m, n = rng.randint(6, 20), rng.randint(2, 8)
        return dict(kind=kind, m=m, n=min(n, m), B=_log(rng, 32, 1024 if n <= 5 else 512))
    m, n = rng.randint(4, 8), rng.randint(2, 3)
    return dict(kind=kind, m=m, n=n, B=_log(rng, 32, 1024))


def _dim(m, n, space="fock"):
    return math.comb(m, n) if space == "unbunched" else math.comb(m + n - 1, n)


# ------------------------------------------------------------------ inputs

def _haar(rng, B, m):
    z = rng.standard_normal((B, m, m)) + 1j * rng.standard_normal((B, m, m))
    q, r = np.linalg.qr(z)
    d = np.diagonal(r, axis1=1, axis2=2)
    return (q * (d / np.abs(d))[:, None, :]).astype(np.complex64)


def _inputs(case, seed):
    """The case's numbers, from the seed alone: numpy arrays, and on the GPU what is large."""
    kind, m, n, B = case["kind"], case["m"], case["n"], case["B"]
    rng = np.random.default_rng([seed, m, n, B])
    gen = torch.Generator(device=DEV).manual_seed(seed * 7919 + m * 101 + n)
    d = {}
    if kind in ("layer", "mesh"):
        d["x"] = rng.standard_normal((B, m)).astype(np.float32)
        d["theta"] = rng.uniform(0, 2 * math.pi, m * (m - 1)).astype(np.float32)
    else:
        d["U"] = _haar(rng, B, m)
    if kind == "mesh":
        # which samples hold how many photons is part of the plan: the same for every seed
        photons = np.random.default_rng([m, n, B]).integers(case["lo"], n + 1, size=B)
        photons[0] = n
        d["occ"] = (np.arange(m)[None, :] < photons[:, None]).astype(np.int32)
    elif kind == "super":
        d["occ"] = np.tile(_occupations(m, n), (B, 1)).astype(np.int32)
    elif kind == "amps":
        d["occ"] = np.stack([np.bincount(rng.integers(0, m, n), minlength=m) for _ in range(B)]).astype(np.int32)
    elif kind == "layer":
        occ = np.zeros(m, np.int32)
        occ[[(j * m) // n for j in range(n)]] = 1
        d["occ"] = np.tile(occ, (B, 1))
    else:
        d["occ"] = np.tile((np.arange(m) < n).astype(np.int32), (B, 1))
    if kind == "layer":
        cols = {"probs": _dim(m, n, case["space"]), "mode_expectations": m,
                "threshold_probs": sum(math.comb(m, k) for k in range(1, min(m, n) + 1))}[case["out"]]
        # a mean loss behind a readout: both signs, every output
        d["g"] = torch.randn(B, cols, generator=gen, device=DEV) / B
    if kind == "grad":
        d["g"] = torch.rand(B * _dim(m, n), generator=gen, device=DEV)
    if kind == "amps":
        d["g"] = torch.randn(B * _dim(m, n), generator=gen, device=DEV, dtype=torch.complex64)
    if kind == "sample":
        d["u"] = torch.rand(B, case["S"], generator=gen, device=DEV)
    if kind == "super":
        N = _dim(m, n)
        a = torch.randn(B, N, generator=gen, device=DEV, dtype=torch.complex64)
        d["a"] = (a / a.abs().square().sum(1, keepdim=True).sqrt()).reshape(-1)
        d["g"] = torch.randn(B * N, generator=gen, device=DEV, dtype=torch.complex64)
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    kind, m, n, B = case["kind"], case["m"], case["n"], case["B"]
    s = dict(case=case)
    if kind == "layer":
        layer = slos.QuantumLayer(m, d["occ"][0], measurement=case["out"], computation_space=case["space"])
        with torch.no_grad():
            layer.theta.copy_(torch.from_numpy(d["theta"]))
        s["layer"] = layer.to(DEV)
        s["x"] = torch.from_numpy(d["x"]).to(DEV).requires_grad_(True)
        s["g"] = d["g"]
        with torch.no_grad():
            s["layer"](s["x"])  # builds the layer's plan, as a program's earlier steps have
        return s
    if kind == "mesh":
        s["theta"], s["x"] = torch.from_numpy(d["theta"]).to(DEV), torch.from_numpy(d["x"]).to(DEV)
    else:
        s["U"] = torch.from_numpy(d["U"]).to(DEV)
    if kind == "gram":
        s["occ"] = d["occ"][0]
        return s
    plan = slos.Plan(m, n, forward_only=kind in ("probs", "mesh", "sample"))
    s["batch"] = slos.Batch(plan, d["occ"])
    if kind == "super":
        N = _dim(m, n)
        s["sup"] = slos.Superposition(s["batch"], np.arange(B + 1) * N)
        s["U"].requires_grad_(True)
        s["a"] = d["a"].requires_grad_(True)
    s.update((k, d[k]) for k in ("g", "u") if k in d)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "layer":
        y = s["layer"](s["x"])
        gt, gx = torch.autograd.grad(y, (s["layer"].theta, s["x"]), s["g"])
        return {"y": y.detach(), "grad_theta": gt, "grad_x": gx}
    if kind == "probs":
        return slos.fock_probs(s["batch"], s["U"])
    if kind == "mesh":
        U = slos.mesh_to_unitary(s["theta"], s["x"], math.pi)
        return slos.fock_probs(s["batch"], U)
    if kind == "grad":
        p = slos.fock_probs(s["batch"], s["U"])
        return {"p": p, "grad_U": slos.fock_probs_backward(s["batch"], s["U"], s["g"])}
    if kind == "amps":
        a = slos.fock_amplitudes(s["batch"], s["U"])
        return {"a": a, "grad_U": slos.fock_amplitudes_backward(s["batch"], s["U"], s["g"])}
    if kind == "sample":
        return slos.fock_sample(s["batch"], s["U"], s["u"])
    if kind == "gram":
        return slos.fock_fidelity_kernel(s["occ"], s["U"])
    out = slos.autograd.fock_superposition_amplitudes(s["U"], s["a"], s["sup"])
    gU, ga = torch.autograd.grad(out, (s["U"], s["a"]), s["g"])
    return {"out": out.detach(), "grad_U": gU, "grad_a": ga}


# ------------------------------------------------------------------ what a pass cannot do without

def work(case):
    """Each input read and each output written once; the edges of the photon
    recursion once per direction and product (8 flops each)."""
    kind, m, n, B = case["kind"], case["m"], case["n"], case["B"]
    space = case.get("space", "fock")
    U = 8.0 * m * m
    N = _dim(m, n, space)
    edges = sum(k * _dim(m, k, space) for k in range(1, n + 1))
    if kind == "layer":
        cols = {"probs": N, "mode_expectations": m,
                "threshold_probs": sum(math.comb(m, k) for k in range(1, min(m, n) + 1))}[case["out"]]
        return {"bytes": B * (2 * 4.0 * cols + 3 * 4.0 * m) + 8.0 * m * m, "flops": B * 8.0 * 4 * edges}
    if kind in ("probs", "sample"):
        out = 4.0 * N if kind == "probs" else 8.0 * case["S"]
        return {"bytes": B * (U + out), "flops": B * 8.0 * edges}
    if kind == "mesh":
        span = range(case["lo"], n + 1)
        each = [(_dim(m, k), sum(i * _dim(m, i) for i in range(1, k + 1))) for k in span]
        return {"bytes": B * (4.0 * m + 4.0 * sum(a for a, _ in each) / len(each)),
                "flops": B * 8.0 * sum(b for _, b in each) / len(each)}
    if kind in ("grad", "amps"):
        return {"bytes": B * (2 * U + (8.0 if kind == "grad" else 16.0) * N), "flops": B * 8.0 * 4 * edges}
    if kind == "gram":
        pairs = B * (B + 1) / 2
        return {"bytes": B * U + 4.0 * B * B, "flops": pairs * 8.0 * (n * n * m + n * 2 ** (n - 1))}
    swap = sum(_dim(m, k) * _dim(m, n - k) * m for k in range(1, n + 1))
    return {"bytes": B * (2 * U + 4 * 8.0 * N), "flops": B * 8.0 * 3 * swap}


# ------------------------------------------------------------------ 64 bits, without this framework

@functools.lru_cache(maxsize=4)
def _lists(m, n, unbunched=False):
    """Sorted mode lists of n photons, lexicographic: [N, n]."""
    L = np.zeros((1, 0), np.int16)
    for _ in range(n):
        lo = (L[:, -1] + (1 if unbunched else 0)) if L.shape[1] else np.zeros(1, np.int16)
        reps = np.maximum(m - lo, 0).astype(np.int64)
        start = np.repeat(np.cumsum(reps) - reps, reps)
        nxt = (np.arange(int(reps.sum())) - start + np.repeat(lo, reps)).astype(np.int16)
        L = np.concatenate([np.repeat(L, reps, axis=0), nxt[:, None]], axis=1)
    return L


def _occupations(m, n):
    return np.stack([np.bincount(row, minlength=m) for row in _lists(m, n)])


def _keys(T, m):
    key = torch.zeros(T.shape[0], dtype=torch.int64, device=T.device)
    for p in range(T.shape[1]):
        key = key * (m + 1) + T[:, p] + 1
    return key


def _steps(m, n, unbunched):
    """Per layer k: the size N_k and, for every mode j, which layer k-1 states take a photon in j and to which state."""
    layers = [torch.from_numpy(_lists(m, k, unbunched).astype(np.int64)).to(DEV) for k in range(n + 1)]
    out = []
    for k in range(1, n + 1):
        keys = _keys(layers[k], m)
        moves = []
        for j in range(m):
            src = layers[k - 1]
            idx = torch.arange(src.shape[0], device=DEV)
            if unbunched and k > 1:
                idx = idx[~(src == j).any(1)]
                src = src[idx]
            T = torch.sort(torch.cat([src, torch.full((src.shape[0], 1), j, device=DEV)], 1), 1).values
            moves.append((idx, torch.searchsorted(keys, _keys(T, m))))
        out.append((layers[k].shape[0], moves))
    occ = torch.zeros(layers[n].shape[0], m, dtype=torch.float64, device=DEV)
    occ.scatter_add_(1, layers[n], torch.ones_like(layers[n], dtype=torch.float64))
    return out, occ, torch.exp(0.5 * torch.lgamma(occ + 1).sum(1))


def _amplitudes(U, occ, steps, norm):
    """U [b, m, m] complex128, occ [b, m], all of the same photon number: [b, N]."""
    b, m, _ = U.shape
    modes = torch.from_numpy(np.stack([np.repeat(np.arange(m), o) for o in occ])).to(DEV)
    d = torch.ones(b, 1, dtype=torch.complex128, device=DEV)
    for k, (N, moves) in enumerate(steps):
        col = torch.gather(U, 2, modes[:, k][:, None, None].expand(b, m, 1))[:, :, 0]
        nxt = torch.zeros(b, N, dtype=torch.complex128, device=DEV)
        for j, (idx, to) in enumerate(moves):
            nxt = nxt.index_add(1, to, col[:, j: j + 1] * d[:, idx])
        d = nxt
    fac = np.array([math.prod(math.factorial(int(v)) for v in o) for o in occ], np.float64)
    return d * norm[None, :] / torch.from_numpy(np.sqrt(fac)).to(DEV)[:, None]


def _mesh(theta, x, m):
    """The rectangular mesh with the angle encoding between its halves, complex128 [B, m, m]."""
    U = torch.eye(m, dtype=torch.complex128, device=DEV)
    bs = torch.tensor([[1, 1j], [1j, 1]], dtype=torch.complex128, device=DEV) / math.sqrt(2)
    q, halves = 0, []
    for c in range(m):
        if c == m // 2:
            halves.append(U)
            U = torch.eye(m, dtype=torch.complex128, device=DEV)
        for k in range(c % 2, m - 1, 2):
            t, f = torch.exp(1j * theta[2 * q]), torch.exp(1j * theta[2 * q + 1])
            one = torch.ones((), dtype=torch.complex128, device=DEV)
            T = bs @ torch.diag(torch.stack([t, one])) @ bs @ torch.diag(torch.stack([f, one]))
            U = torch.cat([U[:k], T @ U[k: k + 2], U[k + 2:]])
            q += 1
    return U[None] @ (torch.exp(1j * math.pi * x)[:, :, None] * halves[0][None])


def _clicks(p, m, n, unbunched):
    """Click probabilities of p [b, N]: patterns by click count, then lexicographic."""
    where = {}
    for k in range(1, min(m, n) + 1):
        for c in itertools.combinations(range(m), k):
            where[c] = len(where)
    to = [where[tuple(sorted(set(map(int, row))))] for row in _lists(m, n, unbunched)]
    out = torch.zeros(p.shape[0], len(where), dtype=p.dtype, device=DEV)
    return out.index_add(1, torch.tensor(to, device=DEV), p)


def _permanents(M):
    """Permanents of [..., n, n] by subsets of columns, one row at a time."""
    n = M.shape[-1]
    level = {0: torch.ones(M.shape[:-2], dtype=M.dtype, device=M.device)}
    for r in range(n):
        nxt = {}
        for s, v in level.items():
            for i in range(n):
                if not s >> i & 1:
                    t = s | 1 << i
                    w = v * M[..., r, i]
                    nxt[t] = nxt[t] + w if t in nxt else w
        level = nxt
    return level[(1 << n) - 1]


def exact(case, seed):
    kind, m, n, B = case["kind"], case["m"], case["n"], case["B"]
    if kind == "sample":
        return None
    d = _inputs(case, seed)
    c128 = functools.partial(torch.as_tensor, dtype=torch.complex128, device=DEV)
    f64 = functools.partial(torch.as_tensor, dtype=torch.float64, device=DEV)
    if kind == "gram":
        V = c128(d["U"])[:, :, :n]
        rows = [_permanents(torch.einsum("ki,bkj->bij", V[a].conj(), V)).abs().square() for a in range(B)]
        return torch.stack(rows)
    unb = case.get("space") == "unbunched"
    if kind == "layer":
        theta, x = f64(d["theta"]).requires_grad_(True), f64(d["x"]).requires_grad_(True)
        U = _mesh(theta, x, m)
        Ud = U.detach()
        steps, occ, norm = _steps(m, n, unb)
        ys, gU = [], torch.zeros_like(Ud)
        for b0 in range(0, B, 128):
            Ub = Ud[b0: b0 + 128].clone().requires_grad_(True)
            p = _amplitudes(Ub, d["occ"][b0: b0 + 128], steps, norm)
            p = p.real.square() + p.imag.square()
            y = p if case["out"] == "probs" else p @ occ if case["out"] == "mode_expectations" else _clicks(p, m, n, unb)
            (g,) = torch.autograd.grad(y, Ub, d["g"][b0: b0 + 128].double())
            gU[b0: b0 + 128] = g
            ys.append(y.detach())
        gt, gx = torch.autograd.grad(U, (theta, x), gU)
        return {"y": torch.cat(ys), "grad_theta": gt, "grad_x": gx}
    if kind == "mesh":
        U = _mesh(f64(d["theta"]), f64(d["x"]), m)
        photons = d["occ"].sum(1)
        rows = [None] * B
        for k in sorted(set(photons.tolist())):
            steps, _, norm = _steps(m, k, False)
            at = np.flatnonzero(photons == k)
            for i in range(0, at.size, 256):
                pick = at[i: i + 256]
                a = _amplitudes(U[torch.from_numpy(pick).to(DEV)], d["occ"][pick], steps, norm).abs().square()
                for r, b in enumerate(pick):
                    rows[b] = a[r]
        return torch.cat(rows)
    steps, _, norm = _steps(m, n, False)
    U = c128(d["U"])
    N = _dim(m, n)
    if kind == "super":
        Ug, a = U.requires_grad_(True), c128(d["a"]).requires_grad_(True)
        out = torch.zeros(B, N, dtype=torch.complex128, device=DEV)
        for c in range(N):
            col = _amplitudes(Ug, np.tile(d["occ"][c], (B, 1)), steps, norm)
            out = out + a.view(B, N)[:, c: c + 1] * col
        gU, ga = torch.autograd.grad(out, (Ug, a), c128(d["g"]).view(B, N))
        return {"out": out.detach().reshape(-1), "grad_U": gU, "grad_a": ga}
    outs, gU = [], torch.zeros_like(U)
    step = max(1, min(B, 4_000_000 // N))
    for b0 in range(0, B, step):
        Ub = U[b0: b0 + step].clone().requires_grad_(kind != "probs")
        a = _amplitudes(Ub, d["occ"][b0: b0 + step], steps, norm)
        y = a if kind == "amps" else a.real.square() + a.imag.square()
        if kind != "probs":
            g = d["g"].view(B, N)[b0: b0 + step]
            (gU[b0: b0 + step],) = torch.autograd.grad(y, Ub, g.to(y.dtype))
        outs.append(y.detach().reshape(-1))
    y = torch.cat(outs)
    return y if kind == "probs" else {"p" if kind == "grad" else "a": y, "grad_U": gU}

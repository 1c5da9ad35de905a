"""The split-FP16 step products of FP32 chains (d >= 192) against FP64 chains
of the same steps on the CPU: every tile and accumulator form, and starts that
keep FP32 products.  Relative Frobenius error <= 1e-5, the chains' bound."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1707_02162_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-5


def R():
    from paper_1707_02162_amd import redo
    return redo


def dense(d, B, N, n_drift, seed, drift_diag=True):
    """One signed channel with a dense Hermitian generator at any d."""
    gen = np.random.default_rng(seed)
    A = gen.normal(size=(d, d)) + 1j * gen.normal(size=(d, d))
    S = ((A + A.conj().T) / (2.0 * np.sqrt(d)))[None]
    H = gen.uniform(-2e4, 2e4, (n_drift, d))
    if not drift_diag:
        H = np.stack([np.diag(h) + 2e3 * S[0] for h in H])
    u = (gen.uniform(-1, 1, (B, N, 1)) * 3e4).astype(np.float32)
    return W.Problem("dense", d, 1, False, H, drift_diag, S, None, 1e-6, 3e4 / (16 ** 2 - 1), 16, 2, u, u_scale=3e4)


def steps_of(p, b):
    """FP64 step propagators of instance b from the oracle's eigenbasis exponentials."""
    q = np.clip(np.floor(np.abs(p.u[b, :, 0].astype(np.float64)) / p.eps + 0.5), 0, p.base ** p.digits - 1)
    lam, V = np.linalg.eigh(p.S[0])
    Vd = O.drift_propagator(p.H0[b % len(p.H0)], p.dt, p.drift_is_diag)
    Vd = np.diag(Vd) if Vd.ndim == 1 else Vd
    sg = np.sign(p.u[b, :, 0])
    return [(V * np.exp(-1j * p.dt * p.eps * s * k * lam)) @ V.conj().T @ Vd for s, k in zip(sg, q)]


def relerr(X, ref):
    return float(np.linalg.norm(X.cpu().numpy() - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("d,B,cached,diag", [
    (192, 1, False, True), (192, 3, True, False), (256, 2, True, True),   # 64 x 64 tiles, with and without the tail
    (256, 66, False, True), (256, 66, True, True),    # 128 x 64 tiles (512 or more of them)
    (320, 2, False, True), (512, 17, False, True),    # 64 x 64 past d = 256; 128 x 128 tiles
    (576, 1, True, True), (1024, 4, True, True)])
@pytest.mark.parametrize("precision", ["f32", "f32_3m"])
def test_chain_vs_fp64(d, B, cached, diag, precision):
    N = 3
    p = dense(d, B, N, min(B, 2), d + B, diag)
    t = R().RedoTable.from_problem(p)
    if cached:
        t.cache_levels()
    prec = R().PREC_F32 if precision == "f32" else R().PREC_F32_3M
    U, _, _ = t.chain(torch.tensor(p.u).cuda(), precision=prec, reproject_every=2)
    for b in {0, B // 2, B - 1}:
        assert relerr(U[b], O.chain(steps_of(p, b))) < TOL


@pytest.mark.parametrize("kind", ["unitary", "zero columns", "1e-9", "1e30", "one large column"])
def test_starts_given_by_the_caller(kind):
    """A unit-column start takes the split products, any other one FP32 products: the error stays
    relative to each column, at any scale, and instances do not touch each other."""
    d, B, N = 256, 3, 4
    p = dense(d, B, N, 1, 77)
    t = R().RedoTable.from_problem(p)
    gen = np.random.default_rng(3)
    Q, _ = np.linalg.qr(gen.normal(size=(d, d)) + 1j * gen.normal(size=(d, d)))
    X0 = np.repeat(Q[None], B, 0)
    scale = np.ones(d)
    if kind == "zero columns":
        scale[5::7] = 0.0
    elif kind == "one large column":
        scale[9] = 1e20
    elif kind != "unitary":
        scale[:] = float(kind)
    X0[1] = X0[1] * scale
    X0 = X0.astype(np.complex64)
    U, _, _ = t.chain(torch.tensor(p.u).cuda(), X0=torch.tensor(X0).cuda())
    for b in range(B):
        ref = O.chain(steps_of(p, b)) @ X0[b].astype(np.complex128)
        n = np.linalg.norm(ref, axis=0)
        e = np.linalg.norm(U[b].cpu().numpy() - ref, axis=0)
        assert (e <= TOL * n).all()


def spins(n, B, N, kinds, seed):
    """A collective signed drive, x or y on each spin: real and imaginary entries in one generator,
    real factors in a diagonal gauge."""
    d = 2 ** n
    S = np.zeros((d, d), complex)
    for q, k in enumerate(kinds):
        i = np.arange(d)
        j = i ^ (1 << q)
        S[i, j] += 0.5 if k == "x" else np.where(i >> q & 1, 0.5j, -0.5j)
    gen = np.random.default_rng(seed)
    u = (gen.uniform(-1, 1, (B, N, 1)) * 3e5).astype(np.float32)
    u[:, 1] = 0.0   # a step without a factor
    return W.Problem("spins", d, 1, False, gen.uniform(-2e4, 2e4, (1, d)), True, S[None], None, 1e-6,
                     3e5 / (16 ** 2 - 1), 16, 2, u, u_scale=3e5)


@pytest.mark.parametrize("n,B,cached", [(8, 1, True), (8, 2, False), (8, 65, True), (8, 64, False), (9, 17, True),
                                        (9, 16, False), (10, 5, True)])
@pytest.mark.parametrize("kinds", ["x", "y", "xy"])
def test_real_factors_vs_fp64(n, B, cached, kinds):
    p = spins(n, B, 4, (kinds * n)[:n], 10 * n + B)
    t = R().RedoTable.from_problem(p)
    if cached:
        t.cache_levels()
    u = torch.tensor(p.u).cuda()
    U, _, _ = t.chain(u, precision=R().PREC_F32, reproject_every=3)
    V, _, _ = t.chain(u, X0=torch.eye(p.d, dtype=torch.complex64, device="cuda").repeat(B, 1, 1) * 3.0)   # FP32 products
    for b in {0, B // 2, B - 1}:
        ref = O.chain(steps_of(p, b))
        assert relerr(U[b], ref) < TOL and relerr(V[b], 3.0 * ref) < TOL


@pytest.mark.parametrize("n,B", [(7, 300), (8, 64), (8, 3), (9, 17)])
@pytest.mark.parametrize("kinds", ["x", "xy"])
def test_real_factors_bf16_panels_vs_fp64(n, B, kinds):
    """Split BF16 with and without panels (real factors need panels, 128-row tiles and symmetric
    levels): 2^-16 per product, of which there are 4."""
    p = spins(n, B, 4, (kinds * n)[:n], 20 * n + B)
    t = R().RedoTable.from_problem(p)
    t.cache_levels()
    u = torch.tensor(p.u).cuda()
    U, _, _ = t.chain(u, precision=R().PREC_BF16X3)
    t.cache_split_bf16()
    V, _, _ = t.chain(u, precision=R().PREC_BF16X3)
    for b in {0, B // 2, B - 1}:
        ref = O.chain(steps_of(p, b))
        assert relerr(U[b], ref) < 4 * 2.0 ** -16 and relerr(V[b], ref) < 4 * 2.0 ** -16

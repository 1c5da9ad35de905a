"""The register-resident kernels of d = 2 .. 64 at the edges of their shapes: batches that leave
a wave partly filled or hold one instance per wave (lane groups), lengths around a header batch
and a round of the factor ring, one to sixteen channels, every kind of step (signed, phased,
phase generators that are not half-integers, dense drift), the level cache on and off, and both
forms of GRAPE, against the FP64 oracle.  Tolerances as for the small path: ||dU||_F / sqrt(d)
<= 1e-5, |dF| <= 1e-6, gradient relative L2 <= 1e-4."""
import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_1707_02162_amd import workloads as W

pytestmark = pytest.mark.gpu

FROB_TOL, FID_TOL, GRAD_TOL = 1e-5, 1e-6, 1e-4


def R():
    from paper_1707_02162_amd import redo
    return redo


def problem(n, kind, K, B, N, seed, ragged):
    """kind: phased (collective or per spin), general (phase generators that are not half-integers),
    signed (dense random generators), dense (a dense drift)."""
    d = 2 ** n
    gen = np.random.default_rng(seed)
    lens = gen.integers(1, N + 1, B).astype(np.int32) if ragged else None
    if ragged:
        lens[0] = N
    if kind in ("phased", "general", "dense"):
        p = W.nmr_chain(n, B, N, 2e-6, 16, 2, seed, per_spin=K > 1, lengths=lens, n_drift=min(B, 3))
        if kind == "general":
            p.g = p.g * 0.7 + 0.1
        if kind == "dense":
            H = gen.normal(size=(1, d, d)) + 1j * gen.normal(size=(1, d, d))
            p.H0 = 2e3 * (H + H.conj().transpose(0, 2, 1))
            p.drift_is_diag = False
        return p
    S = gen.normal(size=(K, d, d)) + 1j * gen.normal(size=(K, d, d))
    S = (S + S.conj().transpose(0, 2, 1)) / (2 * math.sqrt(d))
    u = (gen.uniform(-1, 1, (B, N, K)) * 3e4).astype(np.float32)
    u[gen.uniform(size=u.shape) < 0.1] = 0.0     # identity factors
    H0 = gen.uniform(-2e4, 2e4, (2, d))
    Uf = np.stack([W.haar_unitary(d, gen) for _ in range(B)])
    return W.Problem("signed", d, K, False, H0, True, S, None, 1e-6, 3e4 / 255, 16, 2, u, lens, Uf, None, u_scale=3e4)


@pytest.mark.parametrize("n,kind,K,B,N", [
    (1, "phased", 1, 1, 1), (1, "signed", 9, 33, 9), (2, "phased", 2, 17, 33), (2, "signed", 16, 5, 6),
    (2, "signed", 1, 65, 65), (3, "signed", 1, 9, 17), (3, "phased", 3, 1, 40), (3, "general", 1, 3, 20),
    (4, "phased", 1, 5, 31), (4, "signed", 5, 2, 9), (4, "dense", 1, 3, 12), (5, "signed", 2, 2, 9),
    (5, "phased", 5, 1, 17), (6, "signed", 1, 2, 10), (6, "general", 1, 2, 9), (6, "dense", 1, 1, 5)])
@pytest.mark.parametrize("cached", [False, True])
def test_chain_shapes_vs_oracle(n, kind, K, B, N, cached):
    p = problem(n, kind, K, B, N, 900 + 10 * n + K, ragged=B > 1)
    t = R().RedoTable.from_problem(p)
    if cached:
        t.cache_levels()
    ns = None if p.n_steps is None else torch.tensor(p.n_steps)
    u = torch.tensor(p.u).cuda()
    U, _, _ = t.chain(u, n_steps=ns)
    U2, Xp, _ = t.chain(u, n_steps=ns, prefix=True, reproject_every=N + 1)   # the kernel with prefix states
    steps = t.compose(u)
    tab = O.DiscreteTable(p.S, p.dt, p.eps, p.base, p.digits)
    for b in range(p.B):
        nb = int(p.lengths()[b])
        us = O.compose_all_redo(p, tab, b, n_steps=nb)
        pref = O.chain(us, keep=True)
        scale = math.sqrt(p.d)
        assert np.linalg.norm(U[b].cpu().numpy() - pref[-1]) / scale < FROB_TOL
        assert np.linalg.norm(U2[b].cpu().numpy() - pref[-1]) / scale < FROB_TOL
        for m in {1, (nb + 1) // 2, nb}:
            assert np.linalg.norm(Xp[b, m - 1].cpu().numpy() - pref[m]) / scale < FROB_TOL
            assert np.linalg.norm(steps[b, m - 1].cpu().numpy() - us[m - 1]) / scale < FROB_TOL


@pytest.mark.parametrize("n,kind,K,B,N", [
    (1, "phased", 1, 3, 9), (2, "phased", 2, 18, 21), (3, "phased", 3, 9, 33), (3, "general", 1, 2, 12),
    (4, "phased", 4, 5, 18), (4, "signed", 1, 3, 9), (5, "phased", 5, 2, 10), (5, "signed", 1, 2, 9),
    (6, "signed", 1, 1, 6), (6, "phased", 1, 2, 11), (4, "dense", 1, 2, 7)])
@pytest.mark.parametrize("form", ["scan", "fused", "checkpointed"])
def test_grape_shapes_vs_oracle(n, kind, K, B, N, form):
    if kind == "dense":     # the adjoint needs phase generators that commute with the drift
        p = problem(n, "signed", K, B, N, 950 + n, ragged=True)
        H = np.random.default_rng(n).normal(size=(1, p.d, p.d))
        p.H0, p.drift_is_diag = 2e3 * (H + H.transpose(0, 2, 1)).astype(complex), False
    else:
        p = problem(n, kind, K, B, N, 950 + 10 * n + K, ragged=B > 1)
    t = R().RedoTable.from_problem(p)
    if n % 2:
        t.cache_levels()
    ns = None if p.n_steps is None else torch.tensor(p.n_steps)
    F, ov, grad = t.grape(torch.tensor(p.u).cuda(), torch.tensor(p.U_target).cuda(), n_steps=ns,
                          checkpoint_every=4 if form == "checkpointed" else 0, precompose=form == "scan")
    tab = O.DiscreteTable(p.S, p.dt, p.eps, p.base, p.digits)
    for b in range(p.B):
        Fo, go, gr = O.fidelity_and_gradient(p, b, model="redo", table=tab)
        assert abs(F[b].item() - Fo) < FID_TOL and abs(ov[b].item() - go) < FID_TOL
        nb, g = int(p.lengths()[b]), grad[b].cpu().numpy()
        assert np.linalg.norm(g[:nb] - gr[:nb]) <= GRAD_TOL * np.linalg.norm(gr[:nb]) and not g[nb:].any()


def test_grape_large_batch_d8_fused_equals_scan_form():
    """Past 4096 instances at d = 8 the library takes the fused form: the same gradients as the
    scan form's for the same instances, to FP32 rounding (the factors meet the state one by one
    there, as a composed step here)."""
    p = W.nmr_chain(3, 3, 12, 2e-6, 16, 2, 77, per_spin=True)
    t = R().RedoTable.from_problem(p)
    t.cache_levels()
    u, Uf = torch.tensor(p.u).cuda(), torch.tensor(p.U_target).cuda().to(torch.complex64)
    F1, _, g1 = t.grape(u, Uf)
    rep = 1400
    F2, _, g2 = t.grape(u.repeat(rep, 1, 1, 1), Uf.repeat(rep, 1, 1))
    assert torch.equal(F2[:3], F2[-3:]) and torch.equal(g2[:3], g2[-3:])
    assert torch.allclose(F2[:3], F1, atol=FID_TOL)
    assert torch.linalg.norm(g2[:3] - g1) <= GRAD_TOL * torch.linalg.norm(g1)

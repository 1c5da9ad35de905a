"""The workloads this framework's speed is judged on, through its public entry points.

A case is a control problem (``system``: how many spins, which controls), a call
(``op``), the size of the batch, the number of time segments and the options of
the call.  Every case is one that the repository's workloads, tests or benchmark
run, at their sizes or between them:

    listed()            the cases
    draw(rng)           one more of the same ranges
    prepare(case, seed) table, level cache and inputs on the GPU
    run(state)          one call as a program makes it, and everything it returns
    work(case)          the bytes and operations the result cannot do without
    exact(case, seed)   the same outputs in FP64, in plain torch

Fidelities, overlaps and observables come back from the library as FP64 sums over
FP32 states; a program that goes on with them keeps them as FP32, and so does run().
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1707_02162_amd import redo
from paper_1707_02162_amd import workloads as W

PRECISION = {"f32": redo.PREC_F32, "f32_3m": redo.PREC_F32_3M, "bf16x3": redo.PREC_BF16X3}
TWO_PI = 2.0 * math.pi


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(name, op, system, spins, batch, steps, **options):
    case = {"name": name, "op": op, "system": system, "spins": spins, "batch": batch, "steps": steps,
            "min_steps": steps, "base": 32, "cached": True, "precision": "f32", "observable": "none",
            "reproject": 0, "offset": 0}
    case.update(options)
    return case


def listed():
    return [
        # the smallest call: the propagator of one short pulse on one spin pair, as an interactive user evaluates it
        _case("pair_single", "chain", "pair", 2, 1, 50, base=16),
        # 65,536 noise replicas or restarts of a spin pair, objective and gradient of one optimiser iteration
        _case("pair_grape", "grape", "pair", 2, 65536, 200, base=16),
        # a slice of the freezing sweep of Sec. IV: three spins, the magnetisation after every segment and its time
        # average, re-projected every 64 segments
        _case("sweep", "chain", "sweep", 3, 16384, 2000, base=100, observable="lists", reproject=64),
        # four qubits, two species: a training iteration over 256 targets through the autograd function
        _case("species_training", "train", "species", 4, 256, 500),
        # 64 five-qubit registers with their own drift, target and pulse length, controls on every spin
        _case("register_grape", "grape", "register", 5, 64, 1500, min_steps=250),
        # the propagators of 256 pulses of 1,000 segments on a six-qubit chain
        _case("six_qubit_chain", "chain", "collective", 6, 256, 1000),
        # eight qubits, ragged pulse lengths, plain FP32 products of the digit operators (no level cache)
        _case("eight_qubit_ragged", "chain", "collective", 8, 32, 100, min_steps=40, cached=False),
        # the noisy transverse drive on nine spins in split BF16 from pre-split levels, magnetisation every segment
        _case("ising_split_bf16", "chain", "ising", 9, 256, 32, precision="bf16x3", observable="walsh", reproject=64,
              offset=48),
        # the noisy transverse drive on ten spins, FP32 three-product form: the framework's largest products
        _case("ising_ten_spins", "chain", "ising", 10, 512, 16, precision="f32_3m", observable="walsh", reproject=64,
              offset=56),
        # one ten-qubit control problem: objective and gradient of a 250-segment pulse
        _case("ten_qubit_grape", "grape", "collective", 10, 1, 250, precision="f32_3m"),
        # one ten-qubit state transfer: objective and gradient of a 500-segment pulse
        _case("ten_qubit_state", "state", "collective", 10, 1, 500),
        # the structure-aware chain on the ten-spin drive, magnetisation every segment
        _case("ising_spin_factors", "kron", "ising", 10, 512, 32, observable="walsh", reproject=64, offset=48),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.randrange(10)
    if kind == 0:      # spin pairs, chain or gradient, one to many
        b = _log(rng, 1, 65536)
        c = _case("", rng.choice(["chain", "grape"]), "pair", 2, b, _log(rng, 16, 200 if b >= 16 else 64), base=16,
                  cached=rng.random() < 0.75)
    elif kind == 1:    # sweeps
        c = _case("", "chain", "sweep", 3, _log(rng, 64, 16384), _log(rng, 100, 2000), base=100, observable="lists",
                  reproject=64, cached=rng.random() < 0.75)
    elif kind == 2:    # species training
        c = _case("", "train", "species", 4, _log(rng, 8, 256), _log(rng, 33, 500), cached=rng.random() < 0.75)
    elif kind == 3:    # registers of three to five qubits, ragged
        n = _log(rng, 50, 1500)
        c = _case("", "grape", "register", rng.choice([3, 4, 5]), _log(rng, 8, 64), n, min_steps=max(1, n // 6),
                  cached=rng.random() < 0.75)
    elif kind == 4:    # chains of one to six qubits, collective control
        n = _log(rng, 50, 1000)
        c = _case("", "chain", "collective", rng.choice([1, 4, 5, 6]), _log(rng, 16, 256), n,
                  min_steps=rng.choice([n, max(1, n // 3)]), cached=rng.random() < 0.75)
    elif kind == 5:    # seven and eight qubits, or dimensions between them, ragged, digit products or levels
        n = _log(rng, 10, 100)
        c = _case("", "chain", rng.choice(["collective", "generic"]), rng.choice([7, 8]), _log(rng, 1, 32), n,
                  min_steps=max(1, n // 3), cached=rng.random() < 0.5, precision=rng.choice(["f32", "f32_3m"]))
    elif kind == 6:    # the Ising drive on seven to ten spins, each product form
        n = rng.choice([7, 8, 9, 10])
        c = _case("", "chain", "ising", n, _log(rng, 4, 256), _log(rng, 4, 16),
                  precision=rng.choice(["f32", "f32_3m", "bf16x3"]), observable=rng.choice(["walsh", "lists", "none"]),
                  reproject=64, offset=56)
    elif kind == 7:    # gradients of seven to ten qubits
        c = _case("", "grape", "collective", rng.choice([7, 8, 9, 10]), rng.choice([1, 2, 3]), _log(rng, 20, 160),
                  precision=rng.choice(["f32", "f32_3m"]))
    elif kind == 8:    # state transfers
        c = _case("", "state", "collective", rng.choice([4, 6, 8, 10]), rng.choice([1, 2, 5]), _log(rng, 20, 500))
    else:              # structure-aware chains
        c = _case("", "kron", "ising", rng.choice([7, 8, 9, 10]), _log(rng, 8, 512), _log(rng, 4, 32),
                  observable="walsh", reproject=64, offset=48)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _problem(case):
    """The system of a case (generators, drift, quantum) as a one-instance problem."""
    n, kind, digits = case["spins"], case["system"], 2
    if kind == "pair":
        return W.c1_two_spin(B=1, N=1)
    if kind == "sweep":
        return W.freezing_sweep([1.0], [0.0], n=n, N=10000, count=1, base=case["base"], digits=digits)
    if kind == "ising":
        return W.ising_freezing(n=n, B=1, N=1, base=case["base"], digits=digits)
    if kind == "generic":   # a dimension between two powers of two, dense generator, signed channel
        d = 192 if n == 7 else 320
        gen = np.random.default_rng(d)
        A = gen.normal(size=(d, d)) + 1j * gen.normal(size=(d, d))
        S = ((A + A.conj().T) / (2.0 * math.sqrt(d)))[None]
        scale = 3e4
        return W.Problem("generic", d, 1, False, gen.uniform(-2e4, 2e4, (1, d)), True, S, None, 1e-6,
                         scale / (case["base"] ** digits - 1), case["base"], digits,
                         np.zeros((1, 1, 1), np.float32), u_scale=scale)
    species = {"species": [list(range(n // 2)), list(range(n // 2, n))]}.get(kind)
    return W.nmr_chain(n, 1, 1, 2e-6, case["base"], digits, 40 + n, per_spin=kind == "register", species=species,
                       n_drift=case["batch"] if kind == "register" else 1, targets=False)


def _haar(d, count, gen):
    z = gen.standard_normal((count, d, d)) + 1j * gen.standard_normal((count, d, d))
    q, r = np.linalg.qr(z)
    ph = np.diagonal(r, axis1=1, axis2=2)
    return (q * (ph / np.abs(ph))[:, None, :]).astype(np.complex64)


def _inputs(case, p, seed):
    """Amplitudes, lengths, targets and states of a case on the GPU, from the seed alone."""
    B, N, K = case["batch"], case["steps"], p.K
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    gen = np.random.default_rng([seed, B, N])
    new = dict(device="cuda", generator=g)
    kind = case["system"]
    if kind in ("pair", "generic"):
        shape = (B, N, K, 2) if p.phased else (B, N, K)
        u = (torch.rand(shape, **new) * 2.0 - 1.0) * p.u_scale
    elif kind == "ising":     # -h0 (cos(omega t) + 0.05 xi)
        h0, omega = p.meta["h0"], p.meta["omega"]
        t = (torch.arange(N, device="cuda", dtype=torch.float64) + case["offset"] + 0.5) * p.dt
        u = (-h0 * (torch.cos(omega * t)[None, :] + 0.05 * torch.randn((B, N), **new))).float().unsqueeze(-1)
    elif kind == "sweep":     # -h0 ((1 - lambda) cos(omega t) + lambda eta), one (omega, lambda) per instance
        h0 = p.meta["h0"]
        om = 1.0 + 24.0 * torch.rand((B, 1), **new)
        la = torch.rand((B, 1), **new)
        t = (torch.arange(N, device="cuda") + 0.5) * p.dt
        eta = torch.rand((B, N), **new) * 2.0 - 1.0
        u = (-h0 * ((1.0 - la) * torch.cos(om * t[None, :]) + la * eta)).unsqueeze(-1)
    else:                     # smooth pulses: eight sinusoids per Cartesian component, clipped
        T = N * p.dt
        t = (torch.arange(N, device="cuda") + 0.5) * p.dt
        u = torch.zeros((B, N, K, 2), device="cuda")
        for _ in range(8):
            a = torch.rand((B, 1, K, 2), **new) - 0.5
            f = torch.rand((B, 1, K, 2), **new) * (20.0 / T)
            th = torch.rand((B, 1, K, 2), **new) * TWO_PI
            u += a * torch.sin(TWO_PI * f * t[None, :, None, None] + th)
        u = u.clamp(-1.0, 1.0) * p.u_scale
    out = {"u": u.float().contiguous(), "n_steps": None}
    if case["min_steps"] < N:
        ns = gen.integers(case["min_steps"], N + 1, B).astype(np.int32)
        ns[0] = N
        out["n_steps"] = torch.from_numpy(ns).cuda()
    if case["op"] in ("grape", "train"):
        if kind == "collective":   # a gate that the controls can reach, from a neighbouring pulse (F well below 1)
            near = dict(out, u=out["u"] + 0.01 * p.u_scale * torch.cos(
                TWO_PI * torch.rand((B, 1, K, 2), **new) + math.pi * (t / T)[None, :, None, None]))
            e = _Exact(case, p, near)
            X = torch.eye(p.d, dtype=torch.complex128, device="cuda")[:, None, :].expand(p.d, B, p.d).contiguous()
            for n in range(N):
                X = e.forward(X, n)
            out["target"] = X.permute(1, 0, 2).to(torch.complex64).contiguous()
        else:
            out["target"] = torch.from_numpy(_haar(p.d, B, gen)).cuda()
    if case["op"] == "state":   # from the ground state to random superpositions
        psi0 = np.zeros((B, p.d), np.complex64)
        psi0[:, 0] = 1.0
        f = gen.standard_normal((B, p.d)) + 1j * gen.standard_normal((B, p.d))
        f /= np.linalg.norm(f, axis=1, keepdims=True)
        out["psi0"], out["psi_f"] = torch.from_numpy(psi0).cuda(), torch.from_numpy(f.astype(np.complex64)).cuda()
    return out


def prepare(case, seed):
    p = _problem(case)
    state = dict(case=case, **_inputs(case, p, seed))
    table = redo.RedoTable.from_problem(p)
    if case["cached"]:
        table.cache_levels()
        if case["precision"] == "bf16x3" and p.d >= 128:
            table.cache_split_bf16()
    state["table"] = table
    cols, vals = W.observable_ell(p.M) if case["observable"] != "none" else (None, None)
    if case["observable"] == "lists":
        state["lists"] = (torch.from_numpy(cols).cuda(), torch.from_numpy(vals.astype(np.complex64)).cuda())
    if case["observable"] == "walsh":
        state["walsh"] = redo.walsh_observable(cols, vals)
    if case["op"] == "train":
        state["u"].requires_grad_(True)
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    case, table, u, ns = state["case"], state["table"], state["u"], state["n_steps"]
    prec = PRECISION[case["precision"]]
    if case["op"] == "grape":
        F, overlap, grad = table.grape(u, state["target"], n_steps=ns, precision=prec)
        return {"fidelity": F.float(), "overlap": overlap.to(torch.complex64), "grad": grad}
    if case["op"] == "train":
        F = redo.GrapeFidelity.apply(u, table, state["target"], ns, 0, prec)
        (grad,) = torch.autograd.grad(F.sum(), u)
        return {"fidelity": F.detach().float(), "grad": grad}
    if case["op"] == "state":
        F, overlap, grad = table.state_grape(u, state["psi0"], state["psi_f"], n_steps=ns)
        return {"fidelity": F.float(), "overlap": overlap.to(torch.complex64), "grad": grad}
    walsh = state.get("walsh")
    options = dict(n_steps=ns, reproject_every=case["reproject"], step_offset=case["offset"],
                   observable=state.get("lists"), walsh=walsh)
    if case["op"] == "kron":
        X, m = table.kron_chain(u, **options)
    else:
        X, _, m = table.chain(u, precision=prec, **options)
    if walsh is not None:
        X = redo.walsh_right(X)      # out of the Walsh frame
        # the frame's start is X_0 = H / sqrt(d), so this is the propagator itself
    out = {"propagator": X}
    if m is not None:
        out["magnetisation"] = m.float()
        if case["system"] == "sweep":
            out["order_parameter"] = redo.time_average(m).float()
    return out


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _dimension(case):
    if case["system"] == "generic":
        return 192 if case["spins"] == 7 else 320
    return 2 ** case["spins"]


def work(case):
    d, B, N, n = _dimension(case), case["batch"], (case["steps"] + case["min_steps"]) / 2.0, case["spins"]
    K = {"pair": 2, "species": 2, "register": n}.get(case["system"], 1)
    phased = case["system"] in ("pair", "species", "register", "collective")
    amplitudes = 4.0 * (2 if phased else 1) * B * N * K
    products = 1.0 if case["cached"] else 2.0          # per channel and step
    op = case["op"]
    if op in ("grape", "train"):
        # forward and backward products, and the traces' rows of Y = X L at the generators' entries
        flops = B * N * (2.0 * K * products * 8.0 * d ** 3 + K * (n + 1.0) * 8.0 * d * d)
        return {"bytes": 2.0 * amplitudes + 8.0 * d * d * B, "flops": flops}
    if op == "state":
        # every factor read once, applied to one vector forward and one backward
        return {"bytes": 2.0 * amplitudes + 8.0 * d * d * B * N * K * products + 16.0 * d * B,
                "flops": B * N * K * products * 2.0 * 8.0 * d * d}
    observable = 0.0 if case["observable"] == "none" else 8.0 * n * d * d
    series = 0.0 if case["observable"] == "none" else 4.0 * B * N
    per_step = 16.0 * n * d * d if op == "kron" else K * products * 8.0 * d ** 3
    return {"bytes": amplitudes + series + 8.0 * d * d * B, "flops": B * N * (per_step + observable)}


# ---------------------------------------------------------------------------
# the same in FP64
# ---------------------------------------------------------------------------
class _Exact:
    """The split step at the quantised amplitudes, applied to states [d, B, m] in complex128."""

    def __init__(self, case, p, x):
        self.p, self.N, self.B = p, case["steps"], case["batch"]
        dev = "cuda"
        u = x["u"].detach().double()
        if p.phased:
            om = torch.sqrt(u[..., 0] * u[..., 0] + u[..., 1] * u[..., 1])
            self.phi = torch.atan2(u[..., 1], u[..., 0])
        else:
            om, self.phi = u.abs(), None
        q = torch.clamp(torch.floor(om / p.eps + 0.5), max=float(p.base ** p.digits - 1))
        self.q = q if p.phased else torch.where(u < 0, -q, q)
        self.S = torch.from_numpy(np.ascontiguousarray(p.S, np.complex128)).to(dev)
        eig = [np.linalg.eigh(s) for s in p.S]
        self.lam = [torch.from_numpy(e[0]).to(dev) for e in eig]
        self.W = [torch.from_numpy(np.ascontiguousarray(e[1])).to(dev) for e in eig]
        self.WH = [w.conj().T.contiguous() for w in self.W]
        self.g = torch.from_numpy(np.ascontiguousarray(p.g)).to(dev) if p.phased else None
        drift = torch.from_numpy(np.ascontiguousarray(p.H0)).to(dev)
        idx = torch.arange(self.B, device=dev) % p.n_drift
        self.V = torch.exp(-1j * p.dt * drift).T[:, idx].unsqueeze(-1)     # [d, B or 1, 1]
        ns = x["n_steps"]
        self.live = None if ns is None else torch.arange(self.N, device=dev)[:, None] < ns[None, :].long()

    def product(self, A, X):
        return (A @ X.reshape(X.shape[0], -1)).reshape(X.shape)

    def turn(self, n):
        """Z of step n, [d, B, 1]: exp(-i sum_k phi_k g_k)."""
        return torch.exp(-1j * (self.phi[:, n] @ self.g).T).unsqueeze(-1)

    def controls(self, X, n, sign):
        Z = self.turn(n) if self.p.phased else None
        if Z is not None:
            X = Z.conj() * X
        for k in (range(self.p.K) if sign > 0 else reversed(range(self.p.K))):
            e = torch.exp(-1j * sign * self.p.eps * self.p.dt * self.lam[k][:, None] * self.q[:, n, k][None, :])
            X = self.product(self.W[k], e.unsqueeze(-1) * self.product(self.WH[k], X))
        return X if Z is None else Z * X

    def forward(self, X, n):
        Y = self.controls(self.V * X, n, 1.0)
        return Y if self.live is None else torch.where(self.live[n][None, :, None], Y, X)

    def adjoint(self, X, n):
        Y = self.V.conj() * self.controls(X, n, -1.0)
        return Y if self.live is None else torch.where(self.live[n][None, :, None], Y, X)

    def gradient(self, X, L, g, nu):
        """dF/du from the last state X and the last co-state L = U_f (or psi_f), both [d, B, m]; nu [B]."""
        p = self.p
        shape = (self.B, self.N, p.K, 2) if p.phased else (self.B, self.N, p.K)
        grad = torch.zeros(shape, dtype=torch.float64, device="cuda")

        def slope(t):     # dF of dg = t / nu
            return 2.0 * (g.conj() * t / nu).real

        def inner(A):     # Tr(A' Y) = <L, A' X> per instance
            return (L.conj() * A).sum(dim=(0, 2))

        after = None
        if p.phased:
            after = [inner(p_g[:, None, None] * X) for p_g in self.g]
        for n in reversed(range(self.N)):
            omega = []
            for k in range(p.K):
                if not p.phased:
                    omega.append((-1j * p.dt * inner(self.product(self.S[k], X)),))
                    continue
                z = torch.exp(-1j * self.g[k][:, None] * self.phi[:, n, k][None, :]).unsqueeze(-1)
                zero = (self.q[:, n, k] == 0)[None, :, None]
                z0 = torch.where(zero, torch.ones_like(z), z)
                z1 = torch.exp(-0.5j * math.pi * self.g[k])[:, None, None]
                first = -1j * p.dt * inner(z0 * self.product(self.S[k], z0.conj() * X))
                second = None
                if bool(zero.any()):
                    second = -1j * p.dt * inner(z1 * self.product(self.S[k], z1.conj() * X))
                omega.append((first, second))
            X, L = self.adjoint(X, n), self.adjoint(L, n)
            for k in range(p.K):
                if not p.phased:
                    grad[:, n, k] = slope(omega[k][0])
                    continue
                before = inner(self.g[k][:, None, None] * X)
                dO = slope(omega[k][0])
                dP = slope(-1j * (after[k] - before))
                after[k] = before
                q = self.q[:, n, k]
                r = torch.where(q == 0, torch.ones_like(q), q * p.eps)
                c, s = torch.cos(self.phi[:, n, k]), torch.sin(self.phi[:, n, k])
                gx, gy = c * dO - s * dP / r, s * dO + c * dP / r
                if omega[k][1] is not None:
                    gx = torch.where(q == 0, dO, gx)
                    gy = torch.where(q == 0, slope(omega[k][1]), gy)
                grad[:, n, k, 0], grad[:, n, k, 1] = gx, gy
            if self.live is not None:
                grad[:, n] *= self.live[n].reshape((self.B,) + (1,) * (grad.dim() - 2))
        return grad


def exact(case, seed):
    p = _problem(case)
    x = _inputs(case, p, seed)
    e = _Exact(case, p, x)
    d, B, N = p.d, case["batch"], case["steps"]
    if case["op"] == "state":
        X = x["psi0"].to(torch.complex128).T.unsqueeze(-1).contiguous()
        L = x["psi_f"].to(torch.complex128).T.unsqueeze(-1).contiguous()
        nu = torch.ones(B, dtype=torch.float64, device="cuda")
    else:
        X = torch.eye(d, dtype=torch.complex128, device="cuda")[:, None, :].expand(d, B, d).contiguous()
    M = None
    if case["observable"] != "none":
        M = torch.from_numpy(np.ascontiguousarray(p.M, np.complex128)).cuda()
        norm = (M.abs() ** 2).sum()
        m = torch.zeros((B, N), dtype=torch.float64, device="cuda")
    for n in range(N):
        X = e.forward(X, n)
        if M is not None:
            for b0 in range(0, B, 256 if d >= 512 else B):
                Y = X[:, b0:b0 + (256 if d >= 512 else B)].contiguous()
                XM = (Y.reshape(-1, d) @ M).reshape(Y.shape)
                m[b0:b0 + Y.shape[1], n] = (e.product(M, Y).conj() * XM).sum(dim=(0, 2)).real / norm
    if case["op"] in ("chain", "kron"):
        out = {"propagator": X.permute(1, 0, 2).contiguous()}
        if M is not None:
            out["magnetisation"] = m
            if case["system"] == "sweep":
                out["order_parameter"] = m.mean(dim=1)
        return out
    if case["op"] != "state":
        L = x["target"].to(torch.complex128).permute(1, 0, 2).contiguous()
        nu = (L.abs() ** 2).sum(dim=(0, 2))
    g = (L.conj() * X).sum(dim=(0, 2)) / nu
    out = {"fidelity": g.abs() ** 2, "overlap": g, "grad": e.gradient(X, L, g, nu)}
    if case["op"] == "train":
        del out["overlap"]
    return out

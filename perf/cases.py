"""Measured cases: the work that users of this engine have it do, through its
public entry points, from the smallest chains to the 8 GiB state.

A case is a dict of plain values:

  kind     evolve   psi <- U_F^n psi (or its inverse), in place
           step     n periods, then the energy density: one record interval
           energy   <H0>, the norm and every bond density matrix of a state
           spread   sigma_E, <H0>, <H0^2> of a state (H0 psi in the workspace)
           overlap  <phi|psi> and both norms of two states
           grad     one training step's energy and gradient (FloquetEnergy)
  L        sites (the state has 2^L amplitudes)
  dtype    c64 or c128: the engine's precision
  variant  plain, dense4_fp32, dense6_fp32 or dense6_bf16x3
  model    xyz (XYZ couplings and site fields, T = 0.25) or gue (random GUE
           bond terms, drive frequency 8)
  n        periods;  dagger: the inverse evolution;  K: checkpoint interval
  noalloc  energy: the readout that leaves its results on the device
  other    overlap: precision of the second state

Contexts, bonds and states are what a program holds before the call, so
prepare() makes them; windows that a dense variant fuses on first use belong
to the first pass.
"""
import math

import numpy as np
import torch

import paper_2111_08044_amd as fl

PAULI = (np.array([[0, 1], [1, 0]], dtype=np.complex128),
         np.array([[0, -1j], [1j, 0]], dtype=np.complex128),
         np.array([[1, 0], [0, -1]], dtype=np.complex128))
TORCH = {"c64": torch.complex64, "c128": torch.complex128}
REAL = {"c64": torch.float32, "c128": torch.float64}
COUPLINGS = (1.0, 0.8, 0.6)
T_XYZ = 0.25
OMEGA_GUE = 8.0


def _case(name, kind, L, dtype="c64", variant="plain", model="xyz", n=0, dagger=False, K=0, noalloc=False, other=""):
    c = {"name": name, "kind": kind, "L": L, "dtype": dtype, "variant": variant, "model": model, "n": n,
         "dagger": dagger, "K": K, "noalloc": noalloc, "other": other}
    return c


def listed():
    return [
        # a record interval of a chain small enough to compare with exact methods
        _case("step_L12", "step", 12, n=10),
        # the same in double precision, at the depth such references are run to
        _case("evolve_L12_c128", "evolve", 12, dtype="c128", n=100),
        # a short chain of odd length: parameter scans run thousands of these
        _case("evolve_L17", "evolve", 17, n=16),
        # the backward half of an echo of the random-bond model, ragged depth
        _case("echo_back_L21_gue", "evolve", 21, model="gue", n=25, dagger=True),
        # a double-precision reference run next to a single-precision one
        _case("evolve_L23_c128", "evolve", 23, dtype="c128", n=16),
        # the benchmark's step: 10 periods and one energy readout at L = 30
        _case("step_L30", "step", 30, n=10),
        # a record with every bond's density matrix
        _case("energy_rdm_L27", "energy", 27),
        # a record of the heating study: the energy and its spread
        _case("spread_L25_gue", "spread", 25, model="gue"),
        # one training step at the size that the adjoint benchmark is quoted on
        _case("grad_L24", "grad", 24, n=100, K=25),
        # a training step of a small chain in double precision
        _case("grad_L14_c128", "grad", 14, dtype="c128", n=20, K=5),
        # the fused-window variants: the fast one for short depths, and FP32 windows
        _case("evolve_L28_bf16x3", "evolve", 28, variant="dense6_bf16x3", n=16),
        _case("evolve_L26_dense4", "evolve", 26, variant="dense4_fp32", n=10),
    ]


def draw(rng):
    kind = rng.choice(["evolve", "evolve", "evolve", "evolve", "step", "step", "energy", "spread", "overlap", "grad"])
    model = rng.choice(["xyz", "xyz", "gue"])
    dtype = rng.choice(["c64", "c64", "c64", "c128"])
    c = _case("", kind, rng.randint(10, 28 if dtype == "c64" else 26), dtype=dtype, model=model)
    if kind in ("evolve", "step"):
        # depth over its logarithm: a single period up to a few record intervals
        c["n"] = int(round(math.exp(rng.uniform(0.0, math.log(64.0 if c["L"] < 22 else 16.0)))))
        c["dagger"] = kind == "evolve" and rng.random() < 0.33
        if dtype == "c64" and c["L"] >= 13 and rng.random() < 0.4:
            c["variant"] = rng.choice(["dense4_fp32", "dense6_fp32", "dense6_bf16x3"])
    elif kind == "energy":
        c["noalloc"] = rng.random() < 0.33
    elif kind == "overlap":
        c["other"] = rng.choice(["c64", "c128"])
    elif kind == "grad":
        c["model"] = "xyz"
        c["L"] = rng.randint(8, 22)
        c["K"] = rng.randint(1, 12)
        c["n"] = c["K"] * rng.randint(1, 6)
    del c["name"]
    return c


# ------------------------------------------------------------------- inputs

def _bonds(case, rng):
    """(h, T) of the chain: (L-1, 4, 4) bond Hamiltonians of the half-period gates, and the period."""
    L = case["L"]
    if case["model"] == "gue":
        A = rng.standard_normal((L - 1, 4, 4)) + 1j * rng.standard_normal((L - 1, 4, 4))
        H = 0.5 * (A + np.conj(np.swapaxes(A, 1, 2)))
        H = H - np.trace(H, axis1=1, axis2=2)[:, None, None] / 4.0 * np.eye(4)
        H = H * (math.sqrt(2.0) / np.sqrt(np.sum(np.abs(H) ** 2, axis=(1, 2))))[:, None, None]
        return 2.0 * H, 2.0 * math.pi / OMEGA_GUE
    return _xyz(np.tile(COUPLINGS, (L - 1, 1)), rng.uniform(-1.0, 1.0, (L, 3))), T_XYZ


def _xyz(J, fields):
    one = np.eye(2)
    h = np.zeros((len(J), 4, 4), dtype=np.complex128)
    for b in range(len(J)):
        for a, s in enumerate(PAULI):
            h[b] += J[b, a] * np.kron(s, s) + 0.5 * fields[b, a] * np.kron(s, one) + 0.5 * fields[b + 1, a] * np.kron(one, s)
    return h


def _spinors(L, rng):
    z = rng.standard_normal((L, 2)) + 1j * rng.standard_normal((L, 2))
    return z / np.linalg.norm(z, axis=1, keepdims=True)


def _product(spinors):
    """The product state of single-site spinors, site 0 leading, in double precision on the GPU."""
    v = torch.ones(1, dtype=torch.complex128, device="cuda")
    for s in spinors:
        v = (v[:, None] * torch.tensor(s, dtype=torch.complex128, device="cuda")[None, :]).reshape(-1)
    return v


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    L = case["L"]
    d = {}
    if case["kind"] == "grad":
        d["fields"] = rng.uniform(-1.0, 1.0, (L, 3))
        d["spinors"] = _spinors(L, rng)
        J = np.tile(COUPLINGS, (L - 1, 1)) + 0.1 * rng.standard_normal((L - 1, 3))
        d["theta"] = torch.tensor(np.append(J.reshape(-1), T_XYZ), dtype=REAL[case["dtype"]])
        return d
    d["h"], d["T"] = _bonds(case, rng)
    d["psi"] = _product(_spinors(L, rng)).to(TORCH[case["dtype"]])
    if case["kind"] == "overlap":
        # a second state close to the first, as two precisions of one run are
        v = _product(_spinors(L, rng))
        d["phi"] = (0.01 * v + d["psi"].to(torch.complex128)).to(TORCH[case["other"]])
        del v
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    eng = fl.FloquetEngine(case["L"], case["dtype"], case["variant"])
    s = {"case": case, "engine": eng}
    if case["kind"] == "grad":
        s["theta"] = d["theta"].requires_grad_(True)
        s["fields"], s["spinors"] = d["fields"], d["spinors"]
        return s
    eng.set_bonds(d["h"], d["T"])
    s["psi"] = d["psi"]
    if case["kind"] == "spread":
        s["ws"] = eng.new_state()
    elif case["kind"] == "overlap":
        s["phi"] = d["phi"]
    elif case["kind"] == "energy" and case["noalloc"]:
        s["out"] = torch.empty(2, dtype=torch.float64, device="cuda")
        s["rdm"] = torch.empty((case["L"] - 1) * 32, dtype=torch.float64, device="cuda")
    return s


def run(state):
    case, eng = state["case"], state["engine"]
    kind = case["kind"]
    if kind == "grad":
        theta = state["theta"]
        theta.grad = None
        J, T = theta[:-1].view(case["L"] - 1, 3), theta[-1]
        E = fl.FloquetEnergy.apply(J, T, eng, state["fields"], state["spinors"], case["n"], case["K"])
        loss = E.to(theta.dtype) / case["L"]
        loss.backward()
        return {"loss": loss.detach(), "grad": theta.grad}
    psi = state["psi"]
    if kind == "evolve":
        eng.step(psi, case["n"], case["dagger"])
        return {"psi": psi}
    if kind == "step":
        eng.step(psi, case["n"])
        return {"psi": psi, "e": float(eng.energy_density(psi))}
    if kind == "energy":
        if case["noalloc"]:
            fl.fl_expect_energy_noalloc(eng.ctx, psi, state["out"], state["rdm"])
            return {"E_N": state["out"], "rdm": state["rdm"]}
        E, N, rdm = fl.fl_expect_energy(eng.ctx, psi, rdm=True)
        return {"E_N": np.array([E, N]), "rdm": rdm}
    if kind == "spread":
        # a record of plain numbers; in single precision they carry H0 psi's own rounding
        return {"moments": [float(x) for x in eng.energy_spread(psi, state["ws"])], "h_psi": state["ws"]}
    ov, nphi, npsi = eng.overlap(state["phi"], psi)
    return {"overlap": np.array([ov.real, ov.imag, nphi, npsi])}


def work(case):
    """Bytes: each state read or written once; flops: 16 FMA an amplitude for a two-site
    gate or bond term (4 complex multiply-adds), 8 for a bond's density matrix."""
    L, n = case["L"], case["n"]
    amps, nb = float(1 << L), L - 1
    size = amps * (8 if case["dtype"] == "c64" else 16)
    kind = case["kind"]
    if kind == "evolve":
        return {"bytes": 2 * size, "flops": 32 * nb * amps * n}
    if kind == "step":
        return {"bytes": 2 * size, "flops": 32 * nb * amps * n + 16 * nb * amps}
    if kind == "energy":
        return {"bytes": size, "flops": 16 * nb * amps}
    if kind == "spread":
        return {"bytes": 2 * size, "flops": 32 * nb * amps + 16 * amps}
    if kind == "overlap":
        return {"bytes": size + amps * (8 if case["other"] == "c64" else 16), "flops": 16 * amps}
    # the forward writes a checkpoint every K periods and the backward reads them; it undoes each
    # gate on two states and sums the 28-FMA overlap of each quad
    seg = n // case["K"] if case["K"] else 1
    return {"bytes": (2 * seg + 2) * size, "flops": (3 * 32 + 28) * nb * amps * n}


# ------------------------------------- the same values in plain torch, 64 bits

def _order(L, dagger):
    odd, even = list(range(1, L - 1, 2)), list(range(0, L - 1, 2))
    return even + odd if dagger else odd + even


def _apply(v, L, b, G):
    """The 4x4 matrix G on sites (b, b+1)."""
    x = v.view(1 << b, 4, 1 << (L - 2 - b))
    G = torch.as_tensor(G, dtype=torch.complex128, device=v.device)
    out = G[None, :, 0, None] * x[:, 0:1]
    for j in range(1, 4):
        out.addcmul_(G[None, :, j, None], x[:, j:j + 1])
    return out.view(-1)


def _gates(h, T):
    return torch.linalg.matrix_exp(-0.5j * T * torch.as_tensor(h)).numpy()


def _evolve(v, L, G, n, dagger):
    for _ in range(n):
        for b in _order(L, dagger):
            v = _apply(v, L, b, np.conj(G[b].T) if dagger else G[b])
    return v


def _rdms(v, L):
    rho = np.zeros((L - 1, 4, 4), dtype=np.complex128)
    for b in range(L - 1):
        x = v.view(1 << b, 4, 1 << (L - 2 - b))
        for i in range(4):
            for j in range(i, 4):
                rho[b, i, j] = (x[:, i] * x[:, j].conj()).sum().item()
                rho[b, j, i] = np.conj(rho[b, i, j])
    return rho


def _energy(v, L, h):
    rho = _rdms(v, L)
    E = float(sum(np.sum(h[b] * rho[b].T).real for b in range(L - 1)))
    return E, float(v.abs().square().sum().item()), rho


def _gradient(case, d):
    """E_n / L and its gradient: the adjoint replay with dG from the block-triangular exponential."""
    L, n = case["L"], case["n"]
    theta = d["theta"].double().numpy()
    J, T = theta[:-1].reshape(L - 1, 3), float(theta[-1])
    h = _xyz(J, d["fields"])
    G = _gates(h, T)
    gens = [np.kron(s, s) for s in PAULI]
    dG = np.zeros((L - 1, 4, 4, 4), dtype=np.complex128)
    for b in range(L - 1):
        for a in range(3):
            M = np.zeros((8, 8), dtype=np.complex128)
            M[:4, :4] = M[4:, 4:] = -0.5j * T * h[b]
            M[:4, 4:] = -0.5j * T * gens[a]
            dG[b, a] = torch.linalg.matrix_exp(torch.as_tensor(M)).numpy()[:4, 4:]
        dG[b, 3] = -0.5j * h[b] @ G[b]
    psi = _evolve(_product(d["spinors"]).to(TORCH[case["dtype"]]).to(torch.complex128), L, G, n, False)
    E, _, rho = _energy(psi, L, h)
    grad = np.zeros((L - 1, 4))
    for b in range(L - 1):
        grad[b, :3] = [np.sum(g * rho[b].T).real for g in gens]
    lam = sum(_apply(psi, L, b, h[b]) for b in range(L - 1))
    for _ in range(n):
        for b in reversed(_order(L, False)):
            Gd = np.conj(G[b].T)
            psi = _apply(psi, L, b, Gd)
            x, y = psi.view(1 << b, 4, -1), lam.view(1 << b, 4, -1)
            M = torch.stack([(y[:, i:i + 1].conj() * x).sum(dim=(0, 2)) for i in range(4)]).cpu().numpy()
            grad[b] += 2.0 * np.real(np.einsum("aij,ij->a", dG[b], M))
            lam = _apply(lam, L, b, Gd)
    g = np.append(grad[:, :3].reshape(-1), grad[:, 3].sum())
    return {"loss": torch.tensor(E / L, dtype=torch.float64), "grad": torch.from_numpy(g / L)}


def exact(case, seed):
    L, n, kind = case["L"], case["n"], case["kind"]
    gates = {"evolve": n, "step": n + 2, "energy": 2, "spread": 2, "overlap": 0, "grad": 5 * n}[kind] * (L - 1)
    if gates * float(1 << L) > 2.5e11:
        return None     # tens of seconds in plain torch
    d = _inputs(case, seed)
    if kind == "grad":
        return _gradient(case, d)
    h = d["h"]
    v = d["psi"].to(torch.complex128)
    if kind in ("evolve", "step"):
        v = _evolve(v, L, _gates(h, d["T"]), n, case["dagger"])
        if kind == "evolve":
            return {"psi": v}
        E, N, _ = _energy(v, L, h)
        return {"psi": v, "e": torch.tensor(E / (L * N), dtype=torch.float64)}
    if kind == "energy":
        E, N, rho = _energy(v, L, h)
        out = np.array([E, N])
        if case["noalloc"]:
            return {"E_N": torch.from_numpy(out), "rdm": torch.from_numpy(rho.reshape(-1).view(np.float64).copy())}
        return {"E_N": out, "rdm": rho}
    if kind == "spread":
        w = sum(_apply(v, L, b, h[b]) for b in range(L - 1))
        N = v.abs().square().sum().item()
        E, E2 = (v.conj() * w).sum().real.item() / N, w.abs().square().sum().item() / N
        moments = (math.sqrt(max(E2 - E * E, 0.0)), E, E2)
        return {"moments": [torch.tensor(x, dtype=torch.float64) for x in moments], "h_psi": w}
    phi = d["phi"].to(torch.complex128)
    ov = (phi.conj() * v).sum().item()
    return {"overlap": np.array([ov.real, ov.imag, phi.abs().square().sum().item(), v.abs().square().sum().item()])}

"""What a user of this library has it do, as cases that a timing program can run.

listed() gives the cases, draw() more of the same ranges, prepare() what a
program holds before the call (handle, workspace, inputs), run() one pass
through the public entry points, work() what a pass cannot do without and
exact() the same result in plain 64-bit NumPy / torch where that is quick.

Kinds of case
  solve   one HOTRG solve on a kept handle: reset to new parameters, steps,
          ln Z read back (a temperature scan does this per point)
  qchain  the same for a quantum chain: steps along imaginary time, closed by
          the dominant eigenvalue of the column transfer matrix
  serve   a closed batch of solve requests through serve.Server
  chains  a batch of infinite chains evolved by iTEBD bond updates, with the
          energies and bond weights read back
  gemm    the index-mapped product by itself (binding.gemm_nt)

A solve's answer is ln Z per site (and the observables where they are
carried); the tensor behind it is defined only up to signs and rotations of
its bond bases, and so are a chain's site tensors, whose gauge-free part are
the bond weights.
"""
import math

import numpy as np
import torch

from paper_2602_05900_amd import binding, serve, workloads


def listed():
    return [
        # the smallest product: one launch, what a single call costs
        {"name": "gemm_small", "kind": "gemm", "m": 96, "n": 80, "k": 64, "precision": "fp64", "role": "generic",
         "panel": False},
        # the D^7 product on its own in the benchmark's precision, with the conversion of its operands
        {"name": "gemm_y_fp16x3", "kind": "gemm", "m": 48 ** 3, "n": 48 ** 2, "k": 48 ** 2, "precision": "fp16x3",
         "role": "y", "panel": True},
        # a quick look at a model: small D, every environment diagonalised in full
        {"name": "ising_d8", "kind": "solve", "model": "ising", "q": 2, "t": 2.27, "field": 0.0, "dmax": 8,
         "steps": 20, "precision": "fp64", "observables": False, "stepping": "whole"},
        # an odd bond dimension and a three-state model in a field, in split precision
        {"name": "potts_d21_bf16x6", "kind": "solve", "model": "potts", "q": 3, "t": 1.0, "field": 0.05, "dmax": 21,
         "steps": 30, "precision": "bf16x6", "observables": False, "stepping": "whole"},
        # one point of the D = 24 temperature scan, one solve at a time
        {"name": "ising_d24", "kind": "solve", "model": "ising", "q": 2, "t": 2.2, "field": 0.0, "dmax": 24,
         "steps": 30, "precision": "fp64", "observables": False, "stepping": "async"},
        # the same with two-sided truncation and both impurity tensors carried
        {"name": "observables_d24", "kind": "solve", "model": "ising", "q": 2, "t": 2.4, "field": 1e-3, "dmax": 24,
         "steps": 30, "precision": "fp64", "observables": True, "stepping": "async"},
        # the headline batch: D = 48 requests, four in flight
        {"name": "serve_d48_fp16x3", "kind": "serve", "t": 2.25, "dmax": 48, "steps": 30, "requests": 4, "slots": 4,
         "precision": "fp16x3"},
        # D = 48 in FP64, one solve alone
        {"name": "ising_d48_fp64", "kind": "solve", "model": "ising", "q": 2, "t": 2.3, "field": 0.0, "dmax": 48,
         "steps": 30, "precision": "fp64", "observables": False, "stepping": "async"},
        # the largest: D = 64 at criticality in the benchmark's precision
        {"name": "ising_d64_fp16x3", "kind": "solve", "model": "ising", "q": 2, "t": 2.269, "field": 0.0, "dmax": 64,
         "steps": 40, "precision": "fp16x3", "observables": False, "stepping": "async"},
        # the quantum chain at finite temperature
        {"name": "qchain_d32", "kind": "qchain", "g": 1.5, "temperature": 0.5, "dmax": 32, "steps": 10,
         "stepping": "async"},
        # the iTEBD benchmark: 512 chains, two per CU
        {"name": "chains_512x30", "kind": "chains", "chains": 512, "chi": 30, "updates": 128, "g": 1.5, "tau": 0.05},
        # a few chains of a middle size, where one chain's latency counts
        {"name": "chains_5x12", "kind": "chains", "chains": 5, "chi": 12, "updates": 24, "g": 1.5, "tau": 0.05},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "qchain", "serve", "chains", "chains", "gemm", "gemm"])
    if kind == "gemm":
        role = rng.choice(["generic", "x", "y", "tp"])
        n = {"generic": _log_int(rng, 8, 2400), "x": _log_int(rng, 64, 40000), "y": _log_int(rng, 64, 2400),
             "tp": _log_int(rng, 4, 64)}[role]
        return {"kind": "gemm", "m": _log_int(rng, 16, 30000), "n": n, "k": _log_int(rng, 4, 2400),
                "precision": rng.choice(["fp64", "fp64", "fp32", "bf16x3", "bf16x6"]), "role": role, "panel": False}
    if kind == "chains":
        return {"kind": "chains", "chains": _log_int(rng, 1, 512), "chi": rng.randint(2, 32),
                "updates": _log_int(rng, 8, 64), "g": round(rng.uniform(1.2, 2.0), 3), "tau": 0.05}
    if kind == "qchain":
        return {"kind": "qchain", "g": round(rng.uniform(1.2, 2.0), 3), "temperature": round(rng.uniform(0.4, 1.0), 3),
                "dmax": _log_int(rng, 4, 40), "steps": rng.randint(6, 10), "stepping": rng.choice(["whole", "async"])}
    if kind == "serve":
        precision = rng.choice(["fp16x3", "bf16x6", "fp64"])
        return {"kind": "serve", "t": round(rng.uniform(2.1, 2.5), 3),
                "dmax": rng.randint(9, 32 if precision == "fp64" else 44), "steps": rng.randint(20, 30),
                "requests": rng.randint(2, 6), "slots": rng.randint(2, 4), "precision": precision}
    model = rng.choice(["ising", "potts"])
    obs = rng.random() < 0.25
    precision = rng.choice(["fp64", "fp64", "fp32", "bf16x6"] + ([] if obs else ["fp16x3"]))
    t = rng.uniform(1.8, 2.8) if model == "ising" else rng.uniform(0.8, 1.25)
    return {"kind": "solve", "model": model, "q": 2 if model == "ising" else 3, "t": round(t, 3),
            "field": 0.0 if model == "ising" and not obs else 0.05, "dmax": _log_int(rng, 4, 32 if obs else 56 if precision == "fp16x3" else 44),
            "steps": rng.randint(10, 30), "precision": precision, "observables": obs,
            "stepping": rng.choice(["whole", "async"])}


# ---------------------------------------------------------------- inputs

def _jitter(case, seed, key):
    """The case's temperature or coupling moved by up to 1% from the seed: the points of a scan."""
    return float(case[key] * (1.0 + 0.01 * np.random.default_rng(seed).uniform(-1.0, 1.0)))


def _solve_params(case, seed):
    kw = dict(model=case["model"], q=case["q"], temperature=_jitter(case, seed, "t"), dmax=case["dmax"],
              precision=case["precision"], max_steps=case["steps"], field=case["field"])
    if case["observables"]:
        kw.update(two_sided=True, observables=("m", "e"))
    return kw


def _qchain_params(case, seed):
    tau = 1.0 / _jitter(case, seed, "temperature") / 2 ** case["steps"]
    return dict(model="qchain", bond_h=workloads.ising_transverse_bond(case["g"]), tau=tau, dmax=case["dmax"],
                max_steps=case["steps"])


def _requests(case, seed):
    rng = np.random.default_rng(seed)
    return [workloads.Request(i, 0.0, "ising", 2, float(case["t"] * (1.0 + 0.05 * rng.uniform(-1.0, 1.0))),
                              case["dmax"], case["steps"]) for i in range(case["requests"])]


def _chain_states(case, seed):
    return workloads.random_chain_states(case["chains"], case["chi"], seed=seed)


def _gemm_operands(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    kw = dict(dtype=torch.float64, device="cuda", generator=g)
    return torch.randn(case["m"], case["k"], **kw), torch.randn(case["n"], case["k"], **kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        a, b = _gemm_operands(case, seed)
        return {"case": case, "a": a, "b": b, "c": torch.empty(case["m"], case["n"], dtype=torch.float64, device="cuda")}
    if kind == "chains":
        h = workloads.ising_transverse_bond(case["g"])
        return {"case": case, "h": h, "states": _chain_states(case, seed)}
    if kind == "serve":
        return {"case": case, "requests": _requests(case, seed),
                "server": serve.Server(slots=case["slots"], budget=64 << 30, precision=case["precision"])}
    kw = _qchain_params(case, seed) if kind == "qchain" else _solve_params(case, seed)
    return {"case": case, "params": kw, "solve": binding.Solve(**kw)}


# ---------------------------------------------------------------- one pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        binding.gemm_nt(state["a"], state["b"], state["c"], m, n, k, k, k, (1, n, 0, n, 0, 1),
                        precision=case["precision"], role=case["role"], panel=case["panel"])
        return state["c"]
    if kind == "chains":
        c = binding.Chains(state["h"], state["states"], case["chi"])
        e = c.evolve(case["tau"], case["updates"]).energies()
        s = c.states()
        c.close()
        return {"energies": e, "weights": s[:, 4 * case["chi"] ** 2:]}
    if kind == "serve":
        return [c.lnz_per_site for c in state["server"].run(state["requests"], realtime=False)]
    s = state["solve"].reset(**state["params"])
    if case["stepping"] == "async":
        s.coarse_grain_async(case["steps"], exchange=kind != "qchain")
    else:
        s.coarse_grain(case["steps"], exchange=kind != "qchain")
    if kind == "qchain":
        return {"lnz": s.log_z_chain()}
    if case["observables"]:
        v = s.observables()
        return {"lnz": s.log_z(), "m": v["m"], "e": v["e"]}
    return {"lnz": s.log_z()}


# ---------------------------------------------------------------- the work

def _dims(case):
    """(Dx, Dy, D') entering each step."""
    dx = dy = 4 if case["kind"] == "qchain" else case.get("q", 2)
    out = []
    for _ in range(case["steps"]):
        dp = min(case["dmax"], dx * dx)
        out.append((dx, dy, dp))
        dx, dy = (dp, dy) if case["kind"] == "qchain" else (dy, dp)
    return out


def work(case):
    kind = case["kind"]
    if kind == "gemm":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": 8.0 * (m * k + n * k + m * n), "flops": 2.0 * m * n * k}
    if kind == "chains":
        # per update: contraction and gate, an SVD of the 2 chi x 2 chi pair with its right vectors
        # (4 n^3 + 8 n^3), the new left site
        chi, count = case["chi"], case["chains"] * case["updates"]
        n = 2 * chi
        flops = 2.0 * n * n * chi + 32.0 * chi * chi + 12.0 * n ** 3 + 4.0 * n * chi * chi
        return {"bytes": 16.0 * case["chains"] * (4 * chi * chi + 2 * chi), "flops": count * flops}
    # per step: the contractions of the O(D^7) order; T in and out
    obs = case.get("observables", False)
    flops = nbytes = 0.0
    for dx, dy, dp in _dims(case):
        env = 4.0 * dx ** 3 * dy ** 3 + 2.0 * dx ** 4 * dy ** 2
        x, y, tp = 2.0 * dp * dx ** 3 * dy ** 2, 2.0 * dp * dx ** 3 * dy ** 3, 2.0 * dp ** 2 * dx ** 2 * dy ** 2
        flops += env + x + y + tp
        tensors = 1
        if obs:
            flops += env + 2 * (x + 2.0 * y + tp)
            tensors = 3
        nbytes += 8.0 * tensors * (dx * dx * dy * dy + dp * dp * dy * dy)
    times = case.get("requests", 1)
    return {"bytes": times * nbytes, "flops": times * flops}


# ---------------------------------------------------------------- plain 64-bit results

def _initial(case, p):
    """T0[x,x',y,y'] = sum_s w(s) Q[s,x]Q[s,x']Q[s,y]Q[s,y'], and the impurity tensors of <m> and <e_b>."""
    q, beta = p["q"], 1.0 / p["temperature"]
    s = np.arange(q)
    ising = p["model"] == "ising"
    same = (s[:, None] == s[None, :]).astype(float)
    pair = 2.0 * same - 1.0 if ising else same
    f = np.where(s == 0, 1.0, -1.0 if ising else 0.0)
    m = np.where(s == 0, 1.0, -1.0 if ising else -1.0 / (q - 1.0))
    w = np.exp(beta * pair)
    lam, vec = np.linalg.eigh(w)
    root = (vec * np.sqrt(lam)) @ vec.T
    inv = (vec / np.sqrt(lam)) @ vec.T
    g = np.exp(beta * p["field"] * f)
    site = lambda c: np.einsum("k,ka,kb,kc,kd->abcd", c, root, root, root, root)  # noqa: E731
    t = site(g)
    return t, [site(m * g), np.einsum("ce,abed->abcd", inv @ (-pair * w) @ inv, t)]


def _chain_block(h, tau):
    """One tensor per two-site block and Trotter step of exp(-tau h_odd) exp(-tau h_even)."""
    lam, vec = np.linalg.eigh(np.asarray(h))
    gate = ((vec * np.exp(-tau * lam)) @ vec.T).reshape(2, 2, 2, 2)      # s1' s2' s1 s2
    u, sv, vt = np.linalg.svd(gate.transpose(0, 2, 1, 3).reshape(4, 4))
    a = (u * np.sqrt(sv)).T.reshape(4, 2, 2)                            # k s1' s1
    b = (np.sqrt(sv)[:, None] * vt).reshape(4, 2, 2)                    # k s2' s2
    t = np.einsum("lpx,rqy,xyst->lrstpq", b, a, gate)
    return t.reshape(4, 4, 4, 4)


def _environment(t):
    """E[(a1 a2), (b1 b2)] of the left legs of two tensors t[l, r, d, u] stacked along y."""
    dx, _, dy, _ = t.shape
    lo = t.permute(0, 3, 1, 2).reshape(dx * dy, dx * dy)
    up = t.permute(0, 2, 1, 3).reshape(dx * dy, dx * dy)
    a = (lo @ lo.T).reshape(dx, dy, dx, dy).permute(0, 2, 1, 3).reshape(dx * dx, dy * dy)
    b = (up @ up.T).reshape(dx, dy, dx, dy).permute(0, 2, 1, 3).reshape(dx * dx, dy * dy)
    e = (a @ b.T).reshape(dx, dx, dx, dx).permute(0, 2, 1, 3).reshape(dx * dx, dx * dx)
    return 0.5 * (e + e.T)


def _merge(lower, upper, u):
    """T'[l, r, d, u] of lower under upper, both fused x legs projected by u (n x D')."""
    dx, _, dy, _ = lower.shape
    dp = u.shape[1]
    iso = u.T.reshape(dp, dx, dx)                                       # l a1 a2
    x = torch.tensordot(iso, lower, dims=([1], [0]))                    # l a2 r1 d k
    y = torch.tensordot(x, upper, dims=([1, 4], [0, 2]))                # l r1 d r2 u
    return torch.tensordot(y, iso, dims=([1, 3], [1, 2])).permute(0, 3, 1, 2)


def _project(e, dp):
    lam, vec = torch.linalg.eigh(e)
    kept = lam[-dp:].sum()
    return vec[:, -dp:].flip(1), float((lam.sum() - kept) / lam.sum())


def _hotrg(t0, imps, dmax, steps, two_sided, exchange):
    t = torch.from_numpy(np.ascontiguousarray(t0))
    imps = [torch.from_numpy(np.ascontiguousarray(i)) for i in imps]
    c = float(t.abs().max())
    t, imps, acc = t / c, [i / c for i in imps], math.log(c)
    for n in range(1, steps + 1):
        dp = min(dmax, t.shape[0] ** 2)
        u, eps = _project(_environment(t), dp)
        if two_sided:
            ur, eps_r = _project(_environment(t.permute(1, 0, 2, 3)), dp)
            u = ur if eps_r < eps else u
        new = _merge(t, t, u)
        imps = [0.5 * (_merge(i, t, u) + _merge(t, i, u)) for i in imps]
        c = float(new.abs().max())
        turn = (2, 3, 0, 1) if exchange else (0, 1, 2, 3)
        t, imps = (new / c).permute(*turn), [(i / c).permute(*turn) for i in imps]
        acc += math.log(c) / 2 ** n
    return acc, t, imps


def _svd_update(b1, b2, l2, gate):
    """One bond update of the inverse-free iTEBD form; returns the new left and right sites and the weights."""
    chi = b1.shape[1]
    pair = np.einsum("oi,iab->oab", gate, np.einsum("sac,tcb->stab", b1, b2).reshape(4, chi, chi))
    pair = pair.reshape(2, 2, chi, chi).transpose(2, 0, 1, 3).reshape(2 * chi, 2 * chi)   # (a s), (t b)
    _, sv, vt = np.linalg.svd(np.repeat(l2, 2)[:, None] * pair)
    sv, vt = sv[:chi], vt[:chi]
    norm = math.sqrt(float((sv * sv).sum()))
    left = (pair @ vt.T / norm).reshape(chi, 2, chi).transpose(1, 0, 2)
    right = vt.reshape(chi, 2, chi).transpose(1, 0, 2)
    return right, left, sv / norm


def _chain(row, h, chi, tau, updates):
    nb = 2 * chi * chi
    b1, b2 = row[:nb].reshape(2, chi, chi), row[nb:2 * nb].reshape(2, chi, chi)
    l1, l2 = row[2 * nb:2 * nb + chi], row[2 * nb + chi:]
    lam, vec = np.linalg.eigh(np.asarray(h))
    gate = (vec * np.exp(-tau * lam)) @ vec.T
    for _ in range(updates):
        b1, b2, w = _svd_update(b1, b2, l2, gate)
        l1, l2 = l2, w
    energy = 0.0
    for x, y, w in ((b1, b2, l2), (b2, b1, l1)):
        th = (w[:, None, None, None] * np.einsum("sac,tcb->astb", x, y)).transpose(1, 2, 0, 3).reshape(4, -1)
        energy += 0.5 * float((th * (np.asarray(h) @ th)).sum() / (th * th).sum())
    return energy, np.concatenate([l1, l2])


def exact(case, seed):
    kind = case["kind"]
    if kind == "gemm":
        a, b = _gemm_operands(case, seed)
        return a @ b.T
    if kind == "chains":
        if case["chains"] * case["updates"] * (case["chi"] / 12.0) ** 2 > 2000:
            return None
        h = workloads.ising_transverse_bond(case["g"])
        got = [_chain(row, h, case["chi"], case["tau"], case["updates"]) for row in _chain_states(case, seed)]
        return {"energies": np.array([g[0] for g in got]), "weights": np.array([g[1] for g in got])}
    if case["dmax"] > 24 or kind == "serve":
        return None
    if kind == "qchain":
        p = _qchain_params(case, seed)
        acc, t, _ = _hotrg(_chain_block(p["bond_h"], p["tau"]), [], case["dmax"], case["steps"], False, False)
        lam = torch.linalg.eigvals(torch.einsum("lrss->lr", t)).abs().max()
        return {"lnz": acc + math.log(float(lam)) / 2 ** case["steps"]}
    p = _solve_params(case, seed)
    t0, imps = _initial(case, p)
    acc, t, imps = _hotrg(t0, imps if case["observables"] else [], case["dmax"], case["steps"], case["observables"],
                          True)
    tr = float(torch.einsum("xxyy->", t))
    out = {"lnz": acc + math.log(tr) / 2 ** case["steps"]}
    if case["observables"]:
        out.update({k: float(torch.einsum("xxyy->", i)) / tr for k, i in zip(("m", "e"), imps)})
    return out

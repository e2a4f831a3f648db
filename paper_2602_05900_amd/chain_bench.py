"""Stand-alone runs of the two chain workloads (for profiling and quick
measurements), one JSON line each:

    python -m paper_2602_05900_amd.chain_bench --what itebd  [--chains 512 --chi 30 --updates 2000]
    python -m paper_2602_05900_amd.chain_bench --what qchain [--dmax 32 --steps 12]

itebd: a batch of S = 1/2 antiferromagnetic Heisenberg chains from random
states, FP64 (include/itebd.h); qchain: the same chain's free energy at
beta = 1 by HOTRG along imaginary time (HOTRG_QCHAIN).
"""
from __future__ import annotations

import argparse
import json
import math
import time

import torch

from . import binding, workloads


def qr_flops(n: int) -> int:
    """Householder QR with column pivoting of an n x n matrix as the update
    kernel performs it: the first column norms (2 n^2), then per step k the
    reflector's norm over the r = n - k remaining rows (2 r) and, for each
    of the n - 1 - k trailing columns, its product with the reflector, the
    update and its new norm below row k (2 r + 2 r + 2 (r - 1))."""
    total = 2 * n * n
    for k in range(n - 1):
        r = n - k
        total += 2 * r + (n - 1 - k) * (6 * r - 2)
    return total


def itebd_flops(chi: int, updates: float, sweeps: float, rotations: float) -> float:
    """Algorithmic FLOPs of the device's work (see itebd_work): per update
    the contraction (2 n^2 chi), the gate (32 chi^2), the pivoted QR
    (qr_flops), the singular values (2 n^2) and B1' (4 n chi^2); per sweep
    the column norms and pair dot products (2 n^2 + n^2 (n - 1)); per rotation 6 n (two columns of
    R^T); n = 2 chi."""
    n = 2 * chi
    per_update = 2 * n * n * chi + 32 * chi * chi + qr_flops(n) + 2 * n * n + 4 * n * chi * chi
    return updates * per_update + sweeps * (2 * n * n + n * n * (n - 1)) + rotations * 6 * n


def run_itebd(chains: int, chi: int, updates: int, tau: float = 0.01) -> dict:
    h = workloads.heisenberg_bond()
    c = binding.Chains(h, workloads.random_chain_states(chains, chi, seed=2026), chi)
    c.evolve(0.1, 200)
    c.energies()
    sw0, rot0 = c.work()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    c.evolve(tau, updates)
    e = c.energies()
    dt = time.perf_counter() - t0
    sw1, rot1 = c.work()
    flops = itebd_flops(chi, chains * updates, sw1 - sw0, rot1 - rot0)
    c.close()
    return {"chains": chains, "chi": chi, "bond_updates_per_chain": updates, "seconds": dt,
            "updates_per_s": chains * updates / dt, "us_per_update_per_chain": dt / updates * 1e6,
            "mean_jacobi_sweeps": (sw1 - sw0) / (chains * updates), "achieved_tflops": flops / dt / 1e12,
            "energy_mean": float(e.mean()), "energy_minus_bethe_max": float(e.max() - (0.25 - math.log(2.0)))}


def run_qchain(dmax: int, steps: int, temperature: float = 1.0, stepping: str = "whole") -> dict:
    """stepping: "whole" (hotrg_coarse_grain_axis) or "engine" (host-polled
    steps driven by the library's progress thread, hotrg_coarse_grain_async)."""
    h = workloads.heisenberg_bond()
    tau = (1.0 / temperature) / 2 ** steps

    def advance(s):
        if stepping == "engine":
            s.coarse_grain_async(steps, exchange=False)
        else:
            s.coarse_grain(steps, exchange=False)

    s = binding.Solve(model="qchain", bond_h=h, tau=tau, dmax=dmax, max_steps=steps)
    advance(s)                                 # untimed warm-up solve
    s.log_z_chain()
    s.reset(model="qchain", bond_h=h, tau=tau, dmax=dmax, max_steps=steps)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    advance(s)
    f = -s.log_z_chain() / (2.0 * tau)
    dt = time.perf_counter() - t0
    s.close()
    return {"dmax": dmax, "steps": steps, "temperature": temperature, "stepping": stepping, "seconds": dt,
            "ms_per_step": dt / steps * 1e3, "free_energy": f}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--what", choices=("itebd", "qchain"), required=True)
    ap.add_argument("--chains", type=int, default=512)
    ap.add_argument("--chi", type=int, default=30)
    ap.add_argument("--updates", type=int, default=2000)
    ap.add_argument("--dmax", type=int, default=32)
    ap.add_argument("--steps", type=int, default=12)
    ap.add_argument("--stepping", choices=("whole", "engine"), default="whole",
                    help="quantum chain: whole steps or host-polled steps driven by the library's thread")
    a = ap.parse_args()
    out = (run_itebd(a.chains, a.chi, a.updates) if a.what == "itebd"
           else run_qchain(a.dmax, a.steps, stepping=a.stepping))
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()

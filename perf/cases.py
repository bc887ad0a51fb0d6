"""The work that a user of this framework has it do, as cases to be timed.

Every case goes through the public Python entry points. The mechanisms are the
named synthetic ones and the generic sizes of the padded-size tests; the cell
states are the seeded recipes of the workloads. Integrations make up most of
the list, since a run spends nearly all of its time there; the right-hand
side with its Jacobian and the batched LU are callable by themselves.
"""
import math
import os
import tempfile

import numpy as np
import torch

from paper_2112_05834_amd import chem, synth

DEV = "cuda:0"

# name: (species, reactions, third body, Troe, seed, activation energies by class,
#        pressure Pa, step s, recipe of its ordinary cells)
MECHS = {
    "tiny9": (9, 20, 4, 0, 9, False, synth.P_ATM, 1e-6, "uniform"),
    "mid25": (25, 90, 10, 3, 1025, True, 6.0e6, 1e-6, "bimodal"),
    "mid40": (40, 160, 20, 6, 1040, True, 6.0e6, 1e-6, "bimodal"),
    "spray54": (54, 269, 40, 12, 54, True, 6.0e6, 1e-6, "bimodal"),
    "mid100": (100, 450, 60, 15, 1100, True, 6.0e6, 1e-6, "bimodal"),
    "large160": (160, 800, 120, 40, 160, True, 4.0e6, 5e-7, "bimodal"),
}

# Mean attempted steps of one cell over one chemistry step, by recipe, and the
# factor of the looser tolerances; data-dependent, measured once and used for
# the flop count of work() only.
ATTEMPTS = {"uniform": 172.0, "bimodal": 55.0, "heavytail": 100.0, "heavytail_later": 12.0, "ambient": 22.0}
LOOSE = 0.32

_cache = {}


def _mechanism(name):
    """(synth mechanism, parsed handle), generated once per process."""
    if name not in _cache:
        ns, nr, n3, nt, seed, by_class = MECHS[name][:6]
        m = synth.generate_mechanism(ns, nr, n3, nt, seed, ea_by_class=by_class)
        d = tempfile.mkdtemp(prefix="cases_")
        path = synth.write_mech(m, os.path.join(d, name + ".mech"))
        _cache[name] = (m, chem.Mechanism(path))
    return _cache[name]


def _states(name, n, recipe, seed):
    m, _ = _mechanism(name)
    return synth.generate_states(m, n, MECHS[name][6], recipe, seed)


def _matrices(n, m, seed):
    """Diagonally shifted random matrices and right-hand sides: rows are
    interchanged, none is near singular."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    A = torch.randn((n, m, m), generator=g, device=DEV, dtype=torch.float64)
    A += 3.0 * torch.eye(m, device=DEV, dtype=torch.float64)
    return A, torch.randn((n, m), generator=g, device=DEV, dtype=torch.float64)


def _opts(case):
    kw = {"schedule": {"plain": chem.PLAIN, "persistent": chem.PERSISTENT,
                       "binned": chem.PERSISTENT_BINNED}[case.get("schedule", "plain")]}
    if case.get("loose"):
        kw.update(rtol=1e-5, atol=1e-8)
    if case.get("scheme") == "ros4":
        kw["scheme"] = chem.ROS4
    if case.get("jacobian") == "fd":
        kw["jacobian"] = chem.JAC_FD
    if case.get("state") == "no_bath":
        kw["state"] = chem.STATE_NO_BATH
    return chem.default_opts(**kw)


def listed():
    return [
        # the smallest mechanism, one step of 1024 cells with the default
        # options (several cells per wave): launch latency counts
        {"name": "tiny9_1024", "op": "integrate", "mech": "tiny9", "cells": 1024, "recipe": "uniform",
         "schedule": "plain"},
        # a small subdomain of the spray mechanism, fewer cells than the chip
        # has waves: the longest cell's own chain of steps
        {"name": "spray54_131", "op": "integrate", "mech": "spray54", "cells": 131, "recipe": "bimodal",
         "schedule": "persistent"},
        # an ordinary subdomain with the default options
        {"name": "spray54_16411_plain", "op": "integrate", "mech": "spray54", "cells": 16411, "recipe": "bimodal",
         "schedule": "plain"},
        # the headline workload: all of its cells, queue ordered by the
        # trained cost model
        {"name": "spray54_262144_binned", "op": "integrate", "mech": "spray54", "cells": 262144,
         "recipe": "bimodal", "schedule": "binned"},
        # the heavy-tailed workload: ten chained chemistry steps in one graph
        {"name": "spray54_heavytail_chain10", "op": "steps", "mech": "spray54", "cells": 8192,
         "recipe": "heavytail", "schedule": "persistent", "steps": 10},
        # the other scheme with the state without the bath gas
        {"name": "spray54_ros4_nobath_8192", "op": "integrate", "mech": "spray54", "cells": 8192,
         "recipe": "bimodal", "schedule": "persistent", "scheme": "ros4", "state": "no_bath"},
        # a mechanism between the compiled sizes at the shear-layer tolerances
        {"name": "mid40_loose_32768", "op": "integrate", "mech": "mid40", "cells": 32768, "recipe": "bimodal",
         "schedule": "persistent", "loose": True},
        # the large mechanism (one workgroup per cell)
        {"name": "large160_2048", "op": "integrate", "mech": "large160", "cells": 2048, "recipe": "bimodal",
         "schedule": "persistent"},
        # a mechanism between: one workgroup per cell, padded leading dimension
        {"name": "mid100_1500", "op": "integrate", "mech": "mid100", "cells": 1500, "recipe": "bimodal",
         "schedule": "persistent"},
        # ambient gas around the spray, mapped from one reference cell
        {"name": "spray54_zonal_65536", "op": "zonal", "mech": "spray54", "cells": 65536, "recipe": "ambient",
         "schedule": "persistent"},
        # right-hand side and Jacobian of every cell, as a coupled solver asks
        # for them
        {"name": "spray54_rhs_jac_8192", "op": "eval", "mech": "spray54", "cells": 8192, "recipe": "bimodal"},
        # batched LU with one solve
        {"name": "spray54_lu_16384", "op": "lu", "mech": "spray54", "cells": 16384},
    ]


# Cells up to which one drawn pass stays below the largest listed one.
_MOST = {"tiny9": 262144, "mid25": 131072, "mid40": 65536, "spray54": 131072, "mid100": 3072, "large160": 2048}


def draw(rng):
    def cells(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["integrate"] * 6 + ["steps", "zonal", "eval", "lu"])
    mech = rng.choice(list(MECHS))
    if op == "zonal" and mech == "tiny9":
        mech = "spray54"
    most = _MOST[mech]
    case = {"op": op, "mech": mech}
    if op in ("eval", "lu"):
        case["cells"] = cells(17, {"tiny9": 65536, "mid25": 32768, "mid100": 4096, "large160": 1024}.get(mech, 16384))
        if op == "eval":
            case["recipe"] = MECHS[mech][8]
        return case
    case["schedule"] = rng.choice(["plain", "persistent", "persistent", "binned"])
    recipe = MECHS[mech][8]
    if op == "zonal":
        case.update(recipe="ambient", schedule="persistent", cells=cells(100, most // 2))
        return case
    if recipe == "bimodal":
        recipe = rng.choice(["bimodal", "bimodal", "heavytail"])
    case["recipe"] = recipe
    if op == "steps":
        case.update(steps=rng.randint(2, 10), cells=cells(50, max(60, most // 16)),
                    schedule=rng.choice(["plain", "persistent"]))
        return case
    if recipe == "heavytail":
        most //= 4
    if rng.random() < 0.3:
        case["loose"] = True
    if rng.random() < 0.3:
        case["scheme"] = "ros4"
    if rng.random() < 0.2:
        case["state"] = "no_bath"
    if rng.random() < 0.12:
        case["jacobian"] = "fd"
        most //= 32
    case["cells"] = cells(20, most)
    return case


def prepare(case, seed):
    mech, handle = _mechanism(case["mech"])
    n, ns = case["cells"], mech.n_species
    s = {"op": case["op"], "dt": MECHS[case["mech"]][7], "steps": case.get("steps", 1)}
    s["solver"] = S = chem.Solver(handle, _opts(case), device=0)
    if case["op"] == "lu":
        s["A"], s["b"] = _matrices(n, ns + 1, seed)
        return s
    s["phi"] = torch.from_numpy(_states(case["mech"], n, case["recipe"], seed)).to(DEV)
    if case["op"] == "steps":
        s["h"] = torch.zeros(n, dtype=torch.float64, device=DEV)
        s["out"] = torch.empty_like(s["phi"])
    if case["op"] == "zonal":
        coupling, y_fuel, y_ox = synth.bilger_streams(mech)
        S.zone_config(coupling, y_fuel, y_ox, 1e-6, 1.0)
    if case.get("schedule") == "binned":
        # the cost model that such a program keeps: trained on the logged
        # substeps of other cells
        k = min(2048, max(64, n))
        sample = torch.from_numpy(_states(case["mech"], k, case["recipe"], seed + 1000003)).to(DEV)
        S.set_opts(schedule=chem.PERSISTENT)
        S.log_enable(k)
        S.integrate(sample, s["dt"], h_io=False)
        feats, target = S.log_fetch(k)
        S.log_enable(0)
        S.model_train(feats.contiguous(), target.contiguous())
        S.set_opts(schedule=chem.PERSISTENT_BINNED)
    return s


def _result(r):
    return {"phi": r.phi, "h": r.h, "n_acc": r.n_acc, "n_rej": r.n_rej, "status": r.status}


def run(state):
    S, op = state["solver"], state["op"]
    if op == "integrate":
        return _result(S.integrate(state["phi"], state["dt"]))
    if op == "steps":
        state["h"].zero_()
        return _result(S.integrate_steps(state["phi"], state["dt"], state["steps"], h_io=state["h"],
                                         out=state["out"]))
    if op == "zonal":
        r, mapped = S.integrate_zonal(state["phi"], state["dt"])
        return dict(_result(r), mapped=mapped)
    if op == "eval":
        f, J = S.eval_rhs_jac(state["phi"])
        return {"f": f, "J": J}
    A, piv, info, x = S.lu_batch(state["A"].clone(), state["b"].clone())
    return {"lu": A, "piv": piv, "info": info, "x": x}


def work(case):
    """Every input read and every output written once; flops of the method by
    the mechanism's structure (transcendentals count as one)."""
    _, handle = _mechanism(case["mech"])
    n, ns = case["cells"], handle.n_species
    m = ns + 1
    w = handle.work()
    f_rhs, f_jac = w["flops_rhs"] + w["trans_rhs"], w["flops_jac"] + w["trans_jac"]
    f_lu = m * (m - 1) / 2 + (m - 1) * m * (2 * m - 1) / 3
    f_solve = 2 * m * m - m
    row = 8.0 * (ns + 2)
    if case["op"] == "lu":
        return {"bytes": n * (16.0 * m * m + 16 * m + 4 * m + 4), "flops": n * (f_lu + f_solve)}
    if case["op"] == "eval":
        return {"bytes": n * (row + 8 * m + 8.0 * m * m), "flops": n * (f_rhs + f_jac)}
    att = ATTEMPTS[case["recipe"]] * (LOOSE if case.get("loose") else 1.0)
    if case["op"] == "steps" and case["recipe"] == "heavytail":
        att += ATTEMPTS["heavytail_later"] * (case["steps"] - 1)
    elif case["op"] == "steps":
        att *= case["steps"]
    jac = f_rhs * (m + 1) if case.get("jacobian") == "fd" else f_rhs + f_jac
    per = jac + 2 * f_rhs + m + 1 + f_lu + 4 * f_solve + 35 * m
    return {"bytes": n * (2 * row + 8 + 8 + 4 + 4 + 1), "flops": n * att * per}


# ---- results in 64 bits, from the rate laws themselves --------------------

_R, _PATM = 8.314462618, 101325.0


def _rates(mech, T, p, Y):
    """Rates of progress q [n, Nr], their derivatives by concentration
    [n, Nr, Ns] and by T, and the thermo pieces, in double precision."""
    n, ns, nr = len(T), mech.n_species, len(mech.reactions)
    a = np.where((T < synth.T_MID)[:, None, None], mech.nasa_lo[None], mech.nasa_hi[None])
    t = T[:, None]
    cp = a[..., 0] + t * (a[..., 1] + t * (a[..., 2] + t * (a[..., 3] + t * a[..., 4])))
    dcp = a[..., 1] + t * (2 * a[..., 2] + t * (3 * a[..., 3] + t * 4 * a[..., 4]))
    h = a[..., 0] + t * (a[..., 1] / 2 + t * (a[..., 2] / 3 + t * (a[..., 3] / 4 + t * a[..., 4] / 5))) + a[..., 5] / t
    s = a[..., 0] * np.log(t) + t * (a[..., 1] + t * (a[..., 2] / 2 + t * (a[..., 3] / 3 + t * a[..., 4] / 4))) + a[..., 6]
    g = h - s
    W = np.asarray(mech.W)
    rho = p / (_R * T * (Y / W).sum(axis=1))
    C = rho[:, None] * Y / W
    q = np.zeros((n, nr))
    qT = np.zeros((n, nr))
    qC = np.zeros((n, nr, ns))
    Ctot = C.sum(axis=1)
    for r, x in enumerate(mech.reactions):
        lnkf = math.log(x.A) + x.b * np.log(T) - x.Ea / (_R * T)
        dlnkf = (x.b + x.Ea / (_R * T)) / T
        kf = np.exp(lnkf)

        def product(side):
            P = np.ones(n)
            for sp, o in side:
                P = P * C[:, sp] ** o
            D = {}
            for sp, o in side:
                v = o * C[:, sp] ** (o - 1)
                for s2, o2 in side:
                    if s2 != sp:
                        v = v * C[:, s2] ** o2
                D[sp] = v
            return P, D

        Pf, Df = product(x.reac)
        Pr, Dr = product(x.prod)
        if x.reversible:
            dnu = sum(o for _, o in x.prod) - sum(o for _, o in x.reac)
            sg = sum(o * g[:, sp] for sp, o in x.prod) - sum(o * g[:, sp] for sp, o in x.reac)
            sh = sum(o * h[:, sp] for sp, o in x.prod) - sum(o * h[:, sp] for sp, o in x.reac)
            kr = np.exp(lnkf + sg + dnu * np.log(_R * T / _PATM))
            dlnkr = dlnkf - (sh - dnu) / T
        else:
            kr, dlnkr = np.zeros(n), np.zeros(n)
        q0 = kf * Pf - kr * Pr
        th, thM, thT = np.ones(n), np.zeros(n), np.zeros(n)
        alpha = np.ones(ns)
        if x.rtype != synth.ELEMENTARY:
            for sp, e in x.eff:
                alpha[sp] = e
            M = Ctot + sum((e - 1.0) * C[:, sp] for sp, e in x.eff)
            if x.rtype == synth.THIRD_BODY:
                th, thM = M, np.ones(n)
            else:
                A0, b0, E0, ta, T3, T1, T2, has = x.troe
                k0 = np.exp(math.log(A0) + b0 * np.log(T) - E0 / (_R * T))
                dlnk0 = (b0 + E0 / (_R * T)) / T
                pr = np.maximum(k0 * M / kf, 1e-300)
                e3, e1 = np.exp(-T / T3), np.exp(-T / T1)
                Fc = (1 - ta) * e3 + ta * e1
                dFc = -(1 - ta) / T3 * e3 - ta / T1 * e1
                if has:
                    e2 = np.exp(-T2 / T)
                    Fc, dFc = Fc + e2, dFc + T2 / T ** 2 * e2
                Fc = np.maximum(Fc, 1e-300)
                L, ln10 = np.log10(Fc), math.log(10.0)
                X = np.log10(pr) - 0.4 - 0.67 * L
                N = 0.75 - 1.27 * L
                den = N - 0.14 * X
                f1 = X / den
                F = 10.0 ** (L / (1 + f1 ** 2))
                # d log10 F by log10 Pr and by L
                dF_f1 = -L * 2 * f1 / (1 + f1 ** 2) ** 2
                dF_X = dF_f1 * N / den ** 2
                dF_L = 1 / (1 + f1 ** 2) + dF_f1 * (-0.67 * den - X * (-1.27 + 0.14 * 0.67)) / den ** 2
                lind = pr / (1 + pr)
                th = lind * F
                th_pr = F / (1 + pr) ** 2 + lind * F * dF_X / pr
                thM = th_pr * k0 / kf
                thT = th_pr * pr * (dlnk0 - dlnkf) + lind * F * dF_L * dFc / Fc
        q[:, r] = th * q0
        qT[:, r] = th * (kf * dlnkf * Pf - kr * dlnkr * Pr) + q0 * thT
        for sp, v in Df.items():
            qC[:, r, sp] += th * kf * v
        for sp, v in Dr.items():
            qC[:, r, sp] -= th * kr * v
        if x.rtype != synth.ELEMENTARY:
            qC[:, r] += (q0 * thM)[:, None] * alpha
    return q, qC, qT, C, rho, cp, dcp, h


def _eval_exact(mech, phi):
    n, ns = len(phi), mech.n_species
    W = np.asarray(mech.W)
    nu = np.zeros((ns, len(mech.reactions)))
    for r, x in enumerate(mech.reactions):
        for sp, o in x.reac:
            nu[sp, r] -= o
        for sp, o in x.prod:
            nu[sp, r] += o
    f, J = np.zeros((n, ns + 1)), np.zeros((n, ns + 1, ns + 1))
    step = max(1, 20_000_000 // (len(mech.reactions) * ns))
    for lo in range(0, n, step):
        T, p, Y = phi[lo:lo + step, 0], phi[lo:lo + step, 1], phi[lo:lo + step, 2:]
        q, qC, qT, C, rho, cp, dcp, h = _rates(mech, T, p, Y)
        om = q @ nu.T
        D = np.matmul(nu, qC)                       # d omega_i / d C_k at fixed T
        omT = qT @ nu.T
        Wbar = 1.0 / (Y / W).sum(axis=1)
        # C_k = rho Y_k / W_k with rho = p Wbar / (R T)
        sv = np.einsum("nik,nk->ni", D, C)
        domY = rho[:, None, None] * D / W - (Wbar[:, None] / W)[:, None, :] * sv[:, :, None]
        domT = omT - sv / T[:, None]
        drhoY = -rho[:, None] * Wbar[:, None] / W
        fY = W * om / rho[:, None]
        hm, cpm = h * _R * T[:, None], cp * _R / W  # molar enthalpy, cp per mass
        cpt = (Y * cpm).sum(axis=1)
        Q = (hm * om).sum(axis=1)
        fT = -Q / (rho * cpt)
        sl = slice(lo, lo + len(T))
        f[sl, 0], f[sl, 1:] = fT, fY
        J[sl, 1:, 1:] = (W / rho[:, None])[:, :, None] * domY - (fY / rho[:, None])[:, :, None] * drhoY[:, None, :]
        J[sl, 1:, 0] = W / rho[:, None] * domT + fY / T[:, None]
        rc = rho * cpt
        dQY = np.einsum("ni,nik->nk", hm, domY)
        drc = drhoY * cpt[:, None] + rho[:, None] * cpm
        J[sl, 0, 1:] = -(dQY + fT[:, None] * drc) / rc[:, None]
        dQT = (cp * _R * om + hm * domT).sum(axis=1)
        drcT = -rc / T + rho * (Y * dcp * _R / W).sum(axis=1)
        J[sl, 0, 0] = -(dQT + fT * drcT) / rc
    return {"f": f, "J": J}


def exact(case, seed):
    """Right-hand side, Jacobian and LU in plain double precision. The
    integrations take up to hundreds of adaptive steps a cell and have no such
    value within the time."""
    mech, _ = _mechanism(case["mech"])
    n, m = case["cells"], mech.n_species + 1
    if case["op"] == "eval" and n * len(mech.reactions) * m * m < 8e9:
        return _eval_exact(mech, _states(case["mech"], n, case["recipe"], seed))
    if case["op"] == "lu" and n * m ** 3 < 2e10:
        A, b = (t.cpu() for t in _matrices(n, m, seed))
        lu, piv = torch.linalg.lu_factor(A)
        x = torch.linalg.lu_solve(lu, piv, b.unsqueeze(-1)).squeeze(-1)
        return {"lu": lu, "piv": None, "info": None, "x": x}
    return None

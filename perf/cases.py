"""Measured cases: the work a user has this library do, through the public
entry points of the Python binding.

Four kinds of call:

* loops     tsm_loops, the whole estimate of Eq. 4 (the production call);
* solve     tsm_solve_batch on a block of Z4 sources: the low-precision (LP)
            and high-precision (HP) solves with each solver;
* dslash    tm_dslash on fields held as torch tensors;
* contract  tsm_contract of given solutions, for each loop estimator and for
            the projection onto every momentum.

Every case uses kappa, a*mu and link spread of the repository's workloads
(kappa 0.1632, a*mu 0.003 or 0.004, eps 0.25; the 4^4 lattice kappa 0.160,
a*mu 0.03125, eps 0.3).  Training of the learned preconditioner is set-up
work, done once per ensemble, and is not timed here.

The links, sources and solutions of a case come from its seed alone.  The
exact values (`exact`) are plain torch in complex128: the operator with full
3x3 links and the four gammas, CG without any storage rounding, direct phase
sums.  Results of 16-bit and FP32 solves are taken in the storage precision
the caller chose (out_prec), and the estimate from LP solves stored in 16 or
32 bits is recorded in single precision: its statistical error is per cents.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_1211_0126_amd as tq

PRECS = {"f64": tq.PREC_F64, "f32": tq.PREC_F32, "f16": tq.PREC_F16, "bf16": tq.PREC_BF16}
SOLVERS = {"cg": tq.SOLVER_CG, "eo": tq.SOLVER_CG_EO, "fcg": tq.SOLVER_FCG_LEARNED}
ESTIMATORS = {"standard": tq.LOOP_STANDARD, "isovector": tq.LOOP_ONEEND_ISOVECTOR,
              "generalized": tq.LOOP_ONEEND_GENERALIZED, "derivative": tq.LOOP_DERIVATIVE}
OPS = {"m": tq.OP_M, "mdag": tq.OP_MDAG, "mdagm": tq.OP_MDAGM, "hop": tq.OP_HOP}
T_BC = -1  # antiperiodic time, as in every workload


def listed():
    return [
        # the smallest estimate (the 4^4 workload as it stands): launches and
        # host round trips, FP64 throughout
        {"name": "loops_f64_4x4x4x4", "kind": "loops", "lx": 4, "ly": 4, "lz": 4, "lt": 4, "mu": 0.03125,
         "prec": "f64", "solver": "cg", "n_hp": 4, "n_lp": 32, "block": 4, "hp_tol": 1e-12, "momenta": 1},
        # the production call on the largest workload's lattice, with fewer
        # sources: FP16 LP solves in blocks of 16, HP solves stored in FP16
        # with FP64 reliable updates, 27 momenta
        {"name": "loops_f16_32x32x32x64", "kind": "loops", "lx": 32, "ly": 32, "lz": 32, "lt": 64, "mu": 0.003,
         "prec": "f16", "solver": "eo", "n_hp": 8, "n_lp": 40, "block": 16, "hp_tol": 1e-10, "momenta": 27},
        # LP solves whose solutions the caller keeps, two blocks of sources,
        # on an extent that is no power of two
        {"name": "solve_eo_f16_24x24x24x48", "kind": "solve", "lx": 24, "ly": 24, "lz": 24, "lt": 48, "mu": 0.004,
         "prec": "f16", "solver": "eo", "n": 32, "block": 16, "tol": 1e-2},
        # HP solves of one block: FP16 storage, FP64 reliable updates
        {"name": "solve_hp_f16_24x24x24x48", "kind": "solve", "lx": 24, "ly": 24, "lz": 24, "lt": 48, "mu": 0.004,
         "prec": "f16", "solver": "eo", "n": 16, "block": 16, "tol": 1e-10, "hp": True},
        # odd extents, where the even-odd solver does not apply: CG on the
        # whole lattice in FP32, a ragged number of sources
        {"name": "solve_cg_f32_9x11x7x13", "kind": "solve", "lx": 9, "ly": 11, "lz": 7, "lt": 13, "mu": 0.004,
         "prec": "f32", "solver": "cg", "n": 7, "block": 4, "tol": 1e-2},
        # CG on the whole lattice with FP16 storage (the solver of the paper),
        # the traversal that the tuner picks set as a program keeps it
        {"name": "solve_cg_f16_24x24x24x48", "kind": "solve", "lx": 24, "ly": 24, "lz": 24, "lt": 48, "mu": 0.004,
         "prec": "f16", "solver": "cg", "n": 16, "block": 16, "tol": 1e-2, "nr": 2, "march": 8},
        # flexible CG with the Neumann-series network
        {"name": "solve_fcg_f16_16x16x16x32", "kind": "solve", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "mu": 0.004,
         "prec": "f16", "solver": "fcg", "n": 16, "block": 16, "tol": 1e-2, "nr": 2, "march": 8},
        # one application of M to one field: the call a user's own solver makes
        {"name": "dslash_m_f32_16x16x16x32", "kind": "dslash", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "mu": 0.004,
         "prec": "f32", "op": "m", "n": 1},
        # M^dag M in FP64 on a few fields (residual checks, eigensolvers)
        {"name": "dslash_mdagm_f64_24x24x24x48", "kind": "dslash", "lx": 24, "ly": 24, "lz": 24, "lt": 48,
         "mu": 0.004, "prec": "f64", "op": "mdagm", "n": 4},
        # loops of stored solutions, 16 Gamma and 27 momenta
        {"name": "contract_standard_32x32x32x64", "kind": "contract", "lx": 32, "ly": 32, "lz": 32, "lt": 64,
         "mu": 0.003, "estimator": "standard", "n": 4, "momenta": 27},
        # the one-derivative loops in all four directions
        {"name": "contract_derivative_24x24x24x48", "kind": "contract", "lx": 24, "ly": 24, "lz": 24, "lt": 48,
         "mu": 0.004, "estimator": "derivative", "n": 4, "momenta": 27},
        # the Fourier transform to every momentum
        {"name": "contract_allmom_16x16x16x32", "kind": "contract", "lx": 16, "ly": 16, "lz": 16, "lt": 32,
         "mu": 0.004, "estimator": "standard", "n": 4, "momenta": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same kinds: lattices of 4^4 to about 24^3 x 48
    sites, extents that need not be powers of two (nor even, where the solver
    allows it), 1 to 32 sources, each storage, solver and estimator."""
    kind = rng.choice(["loops", "solve", "solve", "dslash", "contract"])
    solver = rng.choice(["eo", "eo", "cg", "fcg"])
    odd = kind in ("dslash", "contract") or (kind == "solve" and solver != "eo")

    def extent(lo, hi):
        e = _log_int(rng, lo, hi)
        return e if odd and rng.random() < 0.5 else e + e % 2

    top = 16 if kind == "loops" else 24
    d = [extent(4, top) for _ in range(3)] + [extent(4, 2 * top)]
    case = {"kind": kind, "lx": d[0], "ly": d[1], "lz": d[2], "lt": d[3], "mu": rng.choice([0.003, 0.004])}
    if kind == "loops":
        prec = rng.choice(["f64", "f32"])
        case.update(prec=prec, solver=rng.choice(["eo", "cg"]), n_hp=rng.choice([1, 2, 4]), n_lp=_log_int(rng, 4, 32),
                    block=rng.choice([4, 8, 16]), hp_tol=1e-10, momenta=rng.choice([1, 27]))
    elif kind == "solve":
        case.update(prec=rng.choice(["f32", "f16", "f16", "bf16"]), solver=solver, n=_log_int(rng, 1, 32),
                    block=rng.choice([4, 8, 16]), tol=1e-2)
        if solver == "eo" and rng.random() < 0.3:
            case.update(prec=rng.choice(["f32", "f16"]), hp=True, tol=1e-10)
    elif kind == "dslash":
        case.update(prec=rng.choice(["f64", "f32", "f16", "bf16"]), op=rng.choice(["m", "mdag", "mdagm", "hop"]),
                    n=_log_int(rng, 1, 16))
    else:
        case.update(estimator=rng.choice(list(ESTIMATORS)), n=_log_int(rng, 1, 8), momenta=rng.choice([1, 27]))
        if case["estimator"] == "standard" and rng.random() < 0.3:
            # (the loops of one source are then as large as 16 fields)
            case["momenta"] = 0
            case["n"] = min(case["n"], max(1, 500000 // _volume(case)))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def _volume(case):
    return case["lx"] * case["ly"] * case["lz"] * case["lt"]


def _physics(case):
    small = case["mu"] == 0.03125  # the 4^4 workload
    return (0.160 if small else 0.1632), case["mu"], (0.3 if small else 0.25)


def _momenta(n):
    if n == 1:
        return np.zeros((1, 3), dtype=np.int32)
    return np.array([(i % 3 - 1, (i // 3) % 3 - 1, i // 9 - 1) for i in range(27)], dtype=np.int32)


def _device_of(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _links(case, seed):
    """Near-identity SU(3) links, complex128 [V][4][3][3] on the GPU: 1 + eps
    times a complex Gaussian matrix, rows orthonormalised, determinant phase
    removed (the recipe of the workloads)."""
    eps = _physics(case)[2]
    n = 4 * _volume(case)
    w = torch.randn((n, 3, 3), dtype=torch.complex128, device="cuda", generator=_device_of(seed)) * eps
    w += torch.eye(3, dtype=torch.complex128, device="cuda")
    rows = []
    for i in range(3):
        u = w[:, i]
        for v in rows:
            u = u - (v.conj() * w[:, i]).sum(-1, keepdim=True) * v
        rows.append(u / torch.linalg.vector_norm(u, dim=-1, keepdim=True))
    a, b, c = rows
    det = (a * torch.linalg.cross(b, c)).sum(-1, keepdim=True)
    ph = torch.polar(torch.ones_like(det.real), -torch.angle(det) / 3)
    return torch.stack([a * ph, b * ph, c * ph], 1).reshape(n // 4, 4, 3, 3)


def _mix(z):
    """The output mix of splitmix64 on int64 (two's complement) tensors."""
    def srl(v, k):
        return (v >> k) & ((1 << (64 - k)) - 1)

    z = (z ^ srl(z, 30)) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ srl(z, 27)) * (0x94D049BB133111EB - (1 << 64))
    return z ^ srl(z, 31)


def _noise(case, seed, j):
    """The Z4 source of id j as complex128 [4][3][T][Z][Y][X]."""
    lx, ly, lz, lt = _dims(case)
    V = _volume(case)
    start = _mix(torch.tensor([int(seed)], dtype=torch.int64, device="cuda"))
    count = 1 + j * V + torch.arange(V, dtype=torch.int64, device="cuda")
    h = _mix(start + count * (0x9E3779B97F4A7C15 - (1 << 64)))
    units = torch.tensor([1, 1j, -1, -1j], dtype=torch.complex128, device="cuda")
    k = torch.stack([(h >> (2 * c)) & 3 for c in range(12)])
    return units[k].reshape(4, 3, lt, lz, ly, lx)


def _canonical(fields):
    """[n] of [4][3][T][Z][Y][X] as [n][V][4][3]."""
    return torch.stack([f.reshape(12, -1).T.reshape(-1, 4, 3) for f in fields])


def _given_solutions(case, seed, op):
    """What a solve leaves behind, to a few per cent: three terms of the
    hopping expansion of M^-1 eta."""
    out = []
    for j in range(case["n"]):
        eta = _noise(case, seed, j)
        s = eta
        for _ in range(2):
            s = eta + op.kappa * op.hop(s) - 1j * op.tw * op.g5(s)
        out.append(s)
    return out


def _caps(case):
    kind = case["kind"]
    if kind == "loops":
        lp, hp = _loop_params(case)
        return tq.caps([lp, hp], max_sources=case["n_hp"] + case["n_lp"], max_mom=case["momenta"])
    if kind == "solve":
        return tq.caps([_solve_params(case)], max_sources=case["n"])
    if kind == "dslash":
        return tq.caps([], max_sources=1, field_rhs=case["n"])
    return tq.caps([], max_sources=case["n"], max_mom=max(case["momenta"], 1), estimators=(ESTIMATORS[case["estimator"]],),
                   all_mom_sources=0 if case["momenta"] else case["n"])


def _solve_params(case):
    prec = PRECS[case["prec"]]
    if case.get("hp"):
        # handed on in FP32: what is left after that is the solve's own 1e-10
        return tq.solve_params(prec=prec, tol=case["tol"], reliable=1, delta=3e-3, rhs_block=case["block"],
                               true_resid=1, stop=tq.STOP_TRUE, solver=SOLVERS[case["solver"]], out_prec=tq.PREC_F32)
    return tq.solve_params(prec=prec, tol=case["tol"], rhs_block=case["block"], true_resid=0,
                           solver=SOLVERS[case["solver"]], out_prec=prec)


def _loop_params(case):
    prec, solver = PRECS[case["prec"]], SOLVERS[case["solver"]]
    lp = tq.solve_params(prec=prec, tol=1e-2, rhs_block=case["block"], true_resid=0, solver=solver)
    if case["prec"] == "f64":
        hp = tq.solve_params(prec=prec, tol=case["hp_tol"], rhs_block=case["block"], solver=solver)
    else:
        hp = tq.solve_params(prec=prec, tol=case["hp_tol"], reliable=1, delta=3e-3, rhs_block=min(case["block"], 8),
                             true_resid=1, stop=tq.STOP_TRUE, solver=solver)
    return lp, hp


def prepare(case, seed):
    kappa, mu, _ = _physics(case)
    links = _links(case, seed)
    state = {"case": case, "seed": seed}
    # solves and estimates run on a stream of their own (iterations are then
    # replayed as graphs); operator calls on the program's current stream
    stream = torch.cuda.Stream() if case["kind"] in ("loops", "solve") else torch.cuda.current_stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ctx = tq.tm_create(_dims(case), kappa, mu, T_BC, stream=stream, caps=_caps(case))
        tq.tm_gauge_load(ctx, links.cpu().numpy())
    state.update(ctx=ctx, stream=stream)
    kind = case["kind"]
    if kind in ("loops", "solve"):
        prec = PRECS[case["prec"]]
        if "nr" in case or kind == "loops" and case["prec"] == "f16":
            tq.tm_set_lane_rhs(ctx, prec, case.get("nr", 2))
        if "march" in case:
            tq.tm_set_march(ctx, prec, case["march"])
        if case["solver"] == "fcg":
            tq.tm_precond_train(ctx, seed, 0, 0, 0, 1, init_mode=1, init_scale=0.0)  # the Neumann-series network
    if kind == "loops":
        state.update(params=_loop_params(case), mom=_momenta(case["momenta"]))
    elif kind == "solve":
        state.update(params=_solve_params(case), ids=list(range(case["n"])))
    elif kind == "dslash":
        x = _field(case, seed)
        state.update(x=x, out=torch.empty_like(x))
    else:
        op = _Operator(case, links)
        state.update(sol=_canonical(_given_solutions(case, seed, op)).contiguous(), ids=list(range(case["n"])),
                     mom=_momenta(case["momenta"]) if case["momenta"] else None)
    torch.cuda.synchronize()
    return state


def _field(case, seed):
    """Gaussian fields in the storage type of the operator call."""
    x = torch.randn((case["n"], _volume(case), 4, 3), dtype=torch.complex128, device="cuda",
                    generator=_device_of(seed + 7))
    if case["prec"] == "f64":
        return x
    if case["prec"] == "f32":
        return x.to(torch.complex64)
    return torch.view_as_real(x).to(torch.float16 if case["prec"] == "f16" else torch.bfloat16).contiguous()


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    with torch.cuda.stream(state["stream"]):
        if kind == "loops":
            lp, hp = state["params"]
            full = case["prec"] == "f64"
            r = tq.tsm_loops(ctx, state["seed"], case["n_hp"], case["n_lp"], lp, hp, state["mom"], per_source=full)
            if full:
                return {"loops": r["loops"], "err": r["err"], "per_source": r["per_source"]}
            return {"loops": r["loops"].astype(np.complex64)}
        if kind == "solve":
            return tq.tsm_solve_batch(ctx, state["params"], state["seed"], state["ids"])[0]
        if kind == "dslash":
            return tq.tm_dslash(ctx, OPS[case["op"]], PRECS[case["prec"]], state["x"], out=state["out"])
        return tq.tsm_contract(ctx, state["seed"], state["ids"], state["sol"], state["mom"],
                               estimator=ESTIMATORS[case["estimator"]])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
_BYTES = {"f64": 16, "f32": 8, "f16": 4, "bf16": 4}  # per complex number
_M_FLOPS = 1368 + 48  # one application of M to one site
# CG iterations these links need (two M per iteration on a whole lattice; the
# Schur complement counts one M per Mhat)
_ITERS = {"cg": 16, "eo": 6, "fcg": 4}


def _solve_flops(case, solver, n, hp):
    its = (120 if solver == "cg" else 38) if hp else _ITERS[solver]
    ops = 2 + (6 if solver == "fcg" else 0)
    return float(_volume(case)) * n * its * (ops * _M_FLOPS + 12 * 10)


def work(case):
    """Links, inputs and outputs once; the arithmetic of the operator
    applications and of the projections."""
    V, kind = float(_volume(case)), case["kind"]
    L = float(case["lt"])
    if kind == "loops":
        n = case["n_hp"] + case["n_lp"]
        links = V * 4 * 9 * _BYTES[case["prec"]]
        out = ((n * 2 + 6) * 16 if case["prec"] == "f64" else 3 * 16) * case["momenta"] * L * 16
        fl = _solve_flops(case, case["solver"], n, False) + _solve_flops(case, case["solver"], case["n_hp"], True)
        return {"bytes": links + out, "flops": fl + (n + case["n_hp"]) * V * 500}
    if kind == "solve":
        out = V * 12 * case["n"] * (8 if case.get("hp") else _BYTES[case["prec"]])
        return {"bytes": V * 36 * _BYTES[case["prec"]] + out,
                "flops": _solve_flops(case, case["solver"], case["n"], bool(case.get("hp")))}
    if kind == "dslash":
        b = _BYTES[case["prec"]]
        return {"bytes": V * (24 * case["n"] + 36) * b, "flops": V * case["n"] * _M_FLOPS * (2 if case["op"] == "mdagm" else 1)}
    sets = 4 if case["estimator"] == "derivative" else 1
    nm = case["momenta"] or case["lx"] * case["ly"] * case["lz"]
    links = V * 36 * 16 if case["estimator"] in ("generalized", "derivative") else 0.0
    fl = V * case["n"] * {"standard": 500, "isovector": 900, "generalized": 900 + _M_FLOPS, "derivative": 4 * 1200}[case["estimator"]]
    if not case["momenta"]:
        fl += V * case["n"] * 16 * 5 * math.log2(nm)
    return {"bytes": V * 12 * 16 * case["n"] + links + case["n"] * sets * 16 * nm * L * 16, "flops": fl}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
class _Operator:
    """M = 1 - kappa H + i tw g5, tw = 2 kappa mu, on complex128 fields
    [4][3][T][Z][Y][X]; upper and lower spins u, d, with g_mu = [[0, B],
    [B^dag, 0]] in the Euclidean chiral basis."""

    def __init__(self, case, links):
        lx, ly, lz, lt = _dims(case)
        self.kappa = _physics(case)[0]
        self.tw = 2 * self.kappa * case["mu"]
        self.U = links.reshape(lt, lz, ly, lx, 4, 3, 3).permute(4, 5, 6, 0, 1, 2, 3).contiguous()
        par = sum(torch.meshgrid(*[torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)], indexing="ij")) % 2
        self.even = (par == 0)

    @staticmethod
    def _b(mu, d, dag):
        """B d (B^dag d if dag) for the two lower (upper) spins d[2][3]."""
        s = 1j if dag else -1j
        if mu == 0:
            return torch.stack([s * d[1], s * d[0]])
        if mu == 1:
            return torch.stack([d[1], -d[0]]) if dag else torch.stack([-d[1], d[0]])
        if mu == 2:
            return torch.stack([s * d[0], -s * d[1]])
        return d

    @staticmethod
    def shift(f, mu, step):
        """f(x + step mu) over the last four axes, with the time sign."""
        ax = f.dim() - 1 - mu
        g = torch.roll(f, -step, ax)
        if mu == 3:
            g.select(ax, g.shape[ax] - 1 if step > 0 else 0).mul_(T_BC)
        return g

    def transport(self, mu, h, dag):
        """U_mu(x) h(x + mu), or U_mu(x - mu)^dag h(x - mu); h [..][3][site]."""
        U = self.U[mu]
        if not dag:
            h = self.shift(h, mu, 1)
            return torch.stack([U[i, 0] * h[:, 0] + U[i, 1] * h[:, 1] + U[i, 2] * h[:, 2] for i in range(3)], 1)
        C = U.conj()
        g = torch.stack([C[0, i] * h[:, 0] + C[1, i] * h[:, 1] + C[2, i] * h[:, 2] for i in range(3)], 1)
        return self.shift(g, mu, -1)

    def hop(self, p):
        out = torch.zeros_like(p)
        for mu in range(4):
            bd = self._b(mu, p[2:], False)
            for sg, dag in ((1, False), (-1, True)):
                g = self.transport(mu, p[:2] - sg * bd, dag)
                out[:2] += g
                out[2:] -= sg * self._b(mu, g, True)
        return out

    @staticmethod
    def g5(p):
        return torch.cat([p[:2], -p[2:]])

    def apply(self, name, p):
        if name == "hop":
            return self.hop(p)
        if name == "m":
            return p - self.kappa * self.hop(p) + 1j * self.tw * self.g5(p)
        if name == "mdag":
            return p - self.kappa * self.g5(self.hop(self.g5(p))) - 1j * self.tw * self.g5(p)
        return self.apply("mdag", self.apply("m", p))

    def d(self, p, sg=1):
        return p + 1j * sg * self.tw * self.g5(p)

    def dinv(self, p, sg=1):
        return (p - 1j * sg * self.tw * self.g5(p)) / (1 + self.tw ** 2)

    def schur(self, p, dag=False):
        """Mhat p = D p - kappa^2 H_oe D^-1 H_eo p for p on the odd sites."""
        if not dag:
            return self.d(p) - self.kappa ** 2 * self.hop(self.dinv(self.hop(p)))
        q = self.hop(self.dinv(self.hop(self.g5(p)), -1))
        return self.d(p, -1) - self.kappa ** 2 * self.g5(q)

    def neumann(self, p, dag=False):
        """1 + A + A^2 + A^3 with A = 1 - M (the network of the flexible CG)."""
        s = p
        for _ in range(3):
            s = p + s - self.apply("mdag" if dag else "m", s)
        return s


def _cg(mul, b, tol, prec=None):
    """(Preconditioned) CG from zero until |r| <= tol |b|."""
    def dot(a, c):
        return torch.vdot(a.reshape(-1), c.reshape(-1)).real

    x, r = torch.zeros_like(b), b.clone()
    z = r if prec is None else prec(r)
    p, rz, bb = z.clone(), dot(r, z), float(dot(b, b))
    for _ in range(2000):
        q = mul(p)
        a = rz / dot(p, q)
        x += a * p
        r -= a * q
        if float(dot(r, r)) <= tol * tol * bb:
            break
        z = r if prec is None else prec(r)
        new = dot(r, z)
        p = z + (new / rz) * p
        rz = new
    return x


def _exact_solve(op, solver, eta, tol):
    if solver == "cg":
        return _cg(lambda p: op.apply("mdagm", p), op.apply("mdag", eta), tol)
    if solver == "fcg":
        return _cg(lambda p: op.apply("mdagm", p), op.apply("mdag", eta), tol,
                   lambda r: op.neumann(op.neumann(r, dag=True)))
    e = eta * op.even
    src = (eta - e) + op.kappa * op.hop(op.dinv(e))
    xo = _cg(lambda p: op.schur(op.schur(p), dag=True), op.schur(src, dag=True), tol)
    return xo + op.dinv(e + op.kappa * op.hop(xo))


def _gammas():
    g = np.zeros((5, 4, 4), dtype=np.complex128)
    sig = [np.array(s, dtype=np.complex128) for s in ([[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]])]
    for k in range(3):
        g[k, :2, 2:], g[k, 2:, :2] = -1j * sig[k], 1j * sig[k]
    g[3, :2, 2:] = g[3, 2:, :2] = np.eye(2)
    g[4] = np.diag([1, 1, -1, -1])
    basis = []
    for n in range(16):
        m = np.eye(4, dtype=np.complex128)
        for b in range(4):
            if (n >> b) & 1:
                m = m @ g[b]
        basis.append(m)
    return np.array(basis), g[4]


def _traces(u, v, gam):
    """sum over spin and colour of conj(v)_ac Gamma_n[a][b] u_bc at every site."""
    out = torch.zeros((16,) + u.shape[2:], dtype=torch.complex128, device=u.device)
    S = [[(u[b] * v[a].conj()).sum(0) for b in range(4)] for a in range(4)]
    for n in range(16):
        for a in range(4):
            for b in range(4):
                if gam[n, a, b] != 0:
                    out[n] += complex(gam[n, a, b]) * S[a][b]
    return out


def _project(tr, momenta):
    """[16][n_mom][Lt] sums over space with exp(-i p.x)."""
    n, lt, lz, ly, lx = tr.shape
    if momenta == 0:
        f = torch.fft.fftn(tr, dim=(2, 3, 4))
        return f.reshape(n, lt, -1).transpose(1, 2).contiguous()
    out = []
    for k in _momenta(momenta).tolist():
        f = tr
        for m, size in zip(k, (lx, ly, lz)):
            f = (f * torch.exp(-2j * math.pi * m / size * torch.arange(size, dtype=torch.float64, device=tr.device))).sum(-1)
        out.append(f)
    return torch.stack(out, 1)


def _loops(op, est, eta, s, momenta, basis, g5):
    """The loops of one source, [16][n_mom][Lt] (derivative: four of them)."""
    if est == "standard":
        return _project(_traces(s, eta, basis), momenta)
    if est == "isovector":
        return -2j * op.tw * _project(_traces(s, s, g5 @ basis), momenta)
    if est == "generalized":
        ds = s - op.kappa * op.hop(s)
        return 2 * _project(_traces(ds, s, g5 @ basis @ g5), momenta)
    out = []
    for mu in range(4):
        f = op.transport(mu, s, False) - op.transport(mu, s, True)
        g = op.transport(mu, eta, False) - op.transport(mu, eta, True)
        out.append(0.25 * _project(_traces(f, eta, basis) - _traces(s, g, basis), momenta))
    return torch.stack(out)


def exact(case, seed):
    links = _links(case, seed)
    kind = case["kind"]
    op = _Operator(case, links)
    lx, ly, lz, lt = _dims(case)
    if kind == "dslash":
        x = _field(case, seed)
        x = x.to(torch.complex128) if x.is_complex() else torch.view_as_complex(x.double())
        y = _canonical([op.apply(case["op"], f.reshape(-1, 12).T.reshape(4, 3, lt, lz, ly, lx)) for f in x])
        return y if case["prec"] in ("f64", "f32") else torch.view_as_real(y.contiguous())
    basis, g5 = _gammas()
    if kind == "contract":
        sols = _given_solutions(case, seed, op)
        return torch.stack([_loops(op, case["estimator"], _noise(case, seed, j), s, case["momenta"], basis, g5)
                            for j, s in enumerate(sols)])
    if kind == "solve":
        tol = 1e-13 if case.get("hp") else case["tol"]
        y = _canonical([_exact_solve(op, case["solver"], _noise(case, seed, j), tol) for j in range(case["n"])])
        return y if case.get("hp") or case["prec"] == "f32" else torch.view_as_real(y.contiguous())
    n_hp, n_lp = case["n_hp"], case["n_lp"]
    ps = torch.zeros((n_hp + n_lp, 2, 16, case["momenta"], lt), dtype=torch.complex128, device="cuda")
    for j in range(n_hp + n_lp):
        eta = _noise(case, seed, j)
        for slot, tol in ((0, 1e-2), (1, 1e-13)):
            if slot == 0 or j < n_hp:
                s = _exact_solve(op, case["solver"], eta, tol)
                ps[j, slot] = _loops(op, "standard", eta, s, case["momenta"], basis, g5)
    diff, low = ps[:n_hp, 1] - ps[:n_hp, 0], ps[n_hp:, 0]
    loops = torch.stack([diff.mean(0), low.mean(0), diff.mean(0) + low.mean(0)])
    if case["prec"] != "f64":
        return {"loops": loops}

    def spread(v):
        r = torch.view_as_real(v)
        if len(r) < 2:
            return torch.zeros_like(r[0])
        return ((r - r.mean(0)) ** 2).sum(0) / (len(r) - 1) / len(r)

    vc, vb = spread(diff), spread(low)
    return {"loops": loops, "err": torch.view_as_complex(torch.stack([vc, vb, vc + vb]).sqrt()), "per_source": ps}

"""Performance cases of the domain-wall operator, its solver and its serving pool.

A case names an entry point ("op"), a lattice "L" (x, y, z, t as text
"16x16x16x32"), the fifth-dimension extent, the action, the storage precision
and the number of right-hand sides. Inputs are drawn on the GPU from the seed:
Haar-random links for the operators, smoothed links exp(0.3 i H) for the
solves, Gaussian spinors.

`exact` evaluates the same operator in complex128 with plain torch in the
canonical layout, from the inputs as rounded to the storage type, and lays the
result out as the library documents it (sites of a parity in traversal order,
interleaved complex blocked over the slices of a site).
"""
import math
import random

import numpy as np
import torch

from paper_2112_01852_amd import qdwf as q

DEV = "cuda"
PREC = {"f64": q.QDWF_F64, "f32": q.QDWF_F32, "f16": q.QDWF_F16, "bf16": q.QDWF_BF16}
SIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
MOBIUS = {"M5": 1.8, "mf": 0.01, "b": 1.5, "c": 0.5}
SHAMIR = {"M5": 1.8, "mf": 0.01, "b": 1.0, "c": 0.0}
BC = (1, 1, 1, -1)
HOP_FLOPS = 1320          # per 5D site and hop application
DW_MASS = 0.1
SERVED_VOLUMES = (8, 12, 16)
SERVED_LS = (8, 12, 16)


def listed():
    return [
        # one application on the smallest lattice in use: call overhead and launch latency
        {"name": "d_f64_4x4x4x4_ls8", "op": "D", "L": "4x4x4x4", "Ls": 8, "action": "shamir",
         "prec": "f64", "dagger": 0, "nrhs": 1},
        # the Dslash headline: the full operator on 32^4 x 16 in single precision
        {"name": "d_f32_32x32x32x32_ls16", "op": "D", "L": "32x32x32x32", "Ls": 16,
         "action": "mobius", "prec": "f32", "dagger": 0, "nrhs": 1},
        # a volume of the domain-wall table, double precision, the short fifth dimension
        {"name": "d_f64_16x16x16x32_ls8", "op": "D", "L": "16x16x16x32", "Ls": 8,
         "action": "shamir", "prec": "f64", "dagger": 0, "nrhs": 1},
        # the adjoint on a lattice that fits no power of two, Ls of the served requests
        {"name": "ddag_f32_12x12x12x24_ls12", "op": "D", "L": "12x12x12x24", "Ls": 12,
         "action": "mobius", "prec": "f32", "dagger": 1, "nrhs": 1},
        # the operator of a plain double-precision solve, and of every reliable update
        {"name": "normal_f64_24x24x24x24_ls16", "op": "MdagM", "L": "24x24x24x24", "Ls": 16,
         "action": "mobius", "prec": "f64", "nrhs": 1},
        # the inner operator of the mixed-precision solve at the same volume
        {"name": "normal_f16_24x24x24x24_ls16", "op": "MdagM", "L": "24x24x24x24", "Ls": 16,
         "action": "mobius", "prec": "f16", "nrhs": 1},
        # one hop of the batched solve of 12 sources (one per spin and colour)
        {"name": "deo_f32_16x16x16x16_ls16_rhs12", "op": "Deo", "L": "16x16x16x16", "Ls": 16,
         "action": "mobius", "prec": "f32", "dagger": 0, "nrhs": 12},
        # the 5D-local inverse of the even-odd scheme, a launch of its own where Ls is not 16
        {"name": "meeinv_f32_16x16x16x32_ls12", "op": "Mee", "L": "16x16x16x32", "Ls": 12,
         "action": "mobius", "prec": "f32", "dagger": 0, "inverse": 1, "nrhs": 1},
        # the Wilson kernel (4D fields) at the largest volume of its table
        {"name": "wilson_f32_32x32x32x64", "op": "Dh", "L": "32x32x32x64", "Ls": 1,
         "action": "shamir", "prec": "f32", "dagger": 0, "nrhs": 1},
        # a new configuration: load its links, pack a source, apply D, unpack the result
        {"name": "config_f64_16x16x16x32_ls16", "op": "config", "L": "16x16x16x32", "Ls": 16,
         "action": "mobius", "prec": "f64", "dagger": 0, "nrhs": 1},
        # a whole mixed-precision solve of the normal equations
        {"name": "solve_f16_16x16x16x16_ls16", "op": "solve", "L": "16x16x16x16", "Ls": 16,
         "action": "mobius", "prec": "f16", "mf": 0.05, "nrhs": 1},
        # a served batch: requests of mixed volume, Ls and mass through the pool until all are done
        {"name": "serve_f16_6_requests", "op": "serve", "prec": "f16", "requests": 6,
         "largest": 12, "mix": 7},
    ]


def _extent(rng, lo, hi):
    """An even extent, log-uniform in [lo, hi]."""
    return max(lo, min(hi, 2 * round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / 2)))


def draw(rng):
    op = rng.choice(["D", "D", "D", "MdagM", "MdagM", "Deo", "Mee", "Dh", "Dw", "config", "solve",
                     "serve"])
    if op == "serve":
        return {"op": op, "prec": rng.choice(["f16", "f16", "f32"]), "requests": rng.randint(2, 7),
                "largest": rng.choice([8, 12]), "mix": rng.randrange(1 << 20)}
    four_d = op in ("Dh", "Dw")
    prec = rng.choice(["f64", "f32", "f32", "f16", "bf16"])
    while True:
        top = 48 if four_d else 16 if op == "solve" else 32
        if rng.random() < 0.5:      # a cubic space and its own time extent
            l = _extent(rng, 8 if four_d else 4, top)
            L = (l, l, l, _extent(rng, 4, 64))
        else:
            L = tuple(_extent(rng, 4, top) for _ in range(4))
        Ls = 1 if four_d else rng.choice([8, 12, 16, 16, 16, 20, 10])
        V = L[0] * L[1] * L[2] * L[3]
        nrhs = rng.choice([1, 1, 1, 2, 3, 4, 12]) if op in ("Deo", "MdagM") else 1
        if four_d and (V // 2) % 16:
            continue
        if op == "solve" and not 2 ** 12 <= V <= 16 ** 4:
            continue
        if V * Ls * nrhs * SIZE[prec] <= (2 if op == "config" else 3) * 2 ** 24 and V >= 256:
            break
    case = {"op": op, "L": "x".join(map(str, L)), "Ls": Ls,
            "action": rng.choice(["mobius", "mobius", "shamir"]), "prec": prec, "nrhs": nrhs}
    if op in ("D", "Deo", "Dh", "Dw", "Mee", "config"):
        case["dagger"] = rng.randint(0, 1)
    if op == "Mee":
        case["inverse"] = rng.randint(0, 1)
    if op == "solve":
        case["action"] = "mobius"
        case["mf"] = round(rng.uniform(0.03, 0.1), 4)
    return case


# ---- inputs ---------------------------------------------------------------------
def _extents(case):
    return tuple(int(v) for v in case["L"].split("x"))


def _action(case):
    a = dict(MOBIUS if case["action"] == "mobius" else SHAMIR)
    if "mf" in case:
        a["mf"] = case["mf"]
    return a


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _gaussian(shape, seed, real=torch.float64):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=_gen(seed), device=DEV,
                                             dtype=real))


def _haar(L, seed, real=torch.float64):
    """Haar SU(3) links [4][t][z][y][x][3][3]: Gram-Schmidt of Gaussian rows."""
    n = 4 * L[0] * L[1] * L[2] * L[3]
    m = _gaussian((n, 2, 3), seed)
    r1, r2 = m[:, 0], m[:, 1]
    r1 = r1 / r1.abs().square().sum(1, keepdim=True).sqrt()
    r2 = r2 - (r1.conj() * r2).sum(1, keepdim=True) * r1
    r2 = r2 / r2.abs().square().sum(1, keepdim=True).sqrt()
    r3 = torch.stack([r1[:, 1] * r2[:, 2] - r1[:, 2] * r2[:, 1],
                      r1[:, 2] * r2[:, 0] - r1[:, 0] * r2[:, 2],
                      r1[:, 0] * r2[:, 1] - r1[:, 1] * r2[:, 0]], 1).conj()
    U = torch.stack([r1, r2, r3], 1).reshape(4, L[3], L[2], L[1], L[0], 3, 3)
    return (U if real == torch.float64 else U.to(torch.complex64)).contiguous()


def _mul3(A, B):
    """3x3 complex products, element by element."""
    return sum(A[..., :, b, None] * B[..., None, b, :] for b in range(3))


def _smooth(L, seed, eps=0.3):
    """exp(i eps H), H = sum_a h_a lambda_a / 2, h_a ~ N(0, 1), by its power series."""
    n = 4 * L[0] * L[1] * L[2] * L[3]
    h = torch.randn((n, 8), generator=_gen(seed), device=DEV, dtype=torch.float64) * 0.5
    z = torch.zeros(n, device=DEV, dtype=torch.float64)
    d8 = h[:, 7] / math.sqrt(3.0)
    rows = [[torch.complex(h[:, 2] + d8, z), torch.complex(h[:, 0], -h[:, 1]),
             torch.complex(h[:, 3], -h[:, 4])],
            [torch.complex(h[:, 0], h[:, 1]), torch.complex(d8 - h[:, 2], z),
             torch.complex(h[:, 5], -h[:, 6])],
            [torch.complex(h[:, 3], h[:, 4]), torch.complex(h[:, 5], h[:, 6]),
             torch.complex(-2 * d8, z)]]
    X = 1j * eps * torch.stack([torch.stack(r, 1) for r in rows], 1)
    U = torch.eye(3, device=DEV, dtype=torch.complex128).expand(n, 3, 3).clone()
    term = U.clone()
    for k in range(1, 26):
        term = _mul3(term, X) / k
        U = U + term
    return U.reshape(4, L[3], L[2], L[1], L[0], 3, 3).contiguous()


def _real(case):
    """Real type of the canonical inputs: complex128 for FP64 storage and whole calls."""
    whole = case["op"] in ("config", "solve")
    return torch.float64 if case["prec"] == "f64" or whole else torch.float32


def _links(case, seed):
    L = _extents(case)
    return _smooth(L, 2 * seed + 1) if case["op"] == "solve" else _haar(L, 2 * seed + 1, _real(case))


def _spinor(case, seed):
    """[rhs][s][t][z][y][x][4][3]; 4D fields have one slice."""
    L = _extents(case)
    return _gaussian((case["nrhs"], case["Ls"], L[3], L[2], L[1], L[0], 4, 3), 2 * seed + 2,
                     _real(case))


def _subset(case):
    """(subset of the input, subset of the output) of an operator."""
    if case["op"] in ("MdagM", "solve"):
        return q.QDWF_ODD, q.QDWF_ODD
    if case["op"] == "Deo":
        return q.QDWF_ODD, q.QDWF_EVEN
    return q.QDWF_FULL, q.QDWF_FULL


def _requests(case, seed):
    """The served mix: (extent, Ls, mf, link seed, source seed) of each request."""
    r = random.Random(case["mix"])
    vols = [v for v in SERVED_VOLUMES if v <= case["largest"]]
    out = []
    for i in range(case["requests"]):
        l = case["largest"] if i == 0 else r.choice(vols)
        out.append((l, r.choice(SERVED_LS), 10 ** r.uniform(-1.5, -1.0), 1000 * seed + 2 * i + 1,
                    1000 * seed + 2 * i + 2))
    return out


def prepare(case, seed):
    if case["op"] == "serve":
        prm = q.solve_params(inner_prec=PREC[case["prec"]], tol=1e-12, check_every=8)
        reqs, need = [], q.qdwf_pool_overhead_bytes(16)
        for l, Ls, mf, us, bs in _requests(case, seed):
            L = (l, l, l, l)
            act = q.make_action(L, Ls, M5=1.8, b=1.5, c=0.5, mf=mf, bc=BC)
            b = _gaussian((Ls, l, l, l, l, 4, 3), bs)
            reqs.append((act, _smooth(L, us), b, torch.zeros_like(b)))
            need += q.qdwf_request_bytes(act, prm) + 4096
        arena = torch.empty(need, dtype=torch.uint8, device=DEV)
        return _Served(q.qdwf_pool_create(0, arena, 16, prm), arena, prm, reqs)

    op, prec, nrhs = case["op"], PREC[case["prec"]], case["nrhs"]
    D = q.Dirac(_extents(case), case["Ls"], bc=BC, **_action(case))
    U = _links(case, seed)
    psi = _spinor(case, seed)
    state = {"case": case, "D": D, "prec": prec}
    sin, sout = _subset(case)
    if op == "config":
        state.update(U=U, psi=psi, f=D.field(prec), g=D.field(prec), back=torch.empty_like(psi))
        return state
    D.set_gauge(U)
    if op == "solve":
        state["b"] = D.pack(psi, q.QDWF_F64, q.QDWF_RIRI, sin, nrhs)
        state["x"] = D.field(q.QDWF_F64, sout, nrhs)
        state["ws"] = D.workspace(q.QDWF_OP_SOLVE, prec, nrhs)
        state["prm"] = q.solve_params(inner_prec=prec, tol=1e-12, check_every=8, use_graph=1)
        return state
    state["f"] = D.pack(psi, prec, q.QDWF_RIRI, sin, nrhs)
    state["g"] = D.field(prec, sout, nrhs)
    if op == "MdagM":
        state["ws"] = D.workspace(q.QDWF_OP_MDAGM, prec, nrhs)
    return state


class _Served:
    """A pool, its arena and the requests a program submits to it."""

    def __init__(self, pool, arena, prm, reqs):
        self.pool, self.arena, self.prm, self.reqs = pool, arena, prm, reqs

    def __del__(self):
        q.qdwf_pool_destroy(self.pool)


def run(state):
    if isinstance(state, _Served):
        ids = [q.qdwf_pool_submit(state.pool, act, U, b, x, state.prm) for act, U, b, x in state.reqs]
        while ids:
            q.qdwf_pool_step(state.pool)
            ids = [i for i in ids if not q.qdwf_pool_poll(state.pool, i)[0]]
        return [x for _, _, _, x in state.reqs]
    case, ctx, prec = state["case"], state["D"].ctx, state["prec"]
    op, lay, nrhs = case["op"], q.QDWF_RIRI, case["nrhs"]
    if op == "config":
        q.qdwf_set_gauge(ctx, state["U"])
        q.qdwf_pack_spinor(ctx, state["f"], prec, lay, state["psi"], q.QDWF_FULL, nrhs)
        q.qdwf_apply_D(ctx, state["g"], state["f"], case["dagger"], prec, lay, nrhs)
        q.qdwf_unpack_spinor(ctx, state["back"], state["g"], prec, lay, q.QDWF_FULL, nrhs)
        return state["back"]
    if op == "solve":
        q.qdwf_solve(ctx, state["x"], state["b"], nrhs, state["prm"], state["ws"])
        return state["x"]
    f, g = state["f"], state["g"]
    if op == "D":
        q.qdwf_apply_D(ctx, g, f, case["dagger"], prec, lay, nrhs)
    elif op == "Deo":
        q.qdwf_apply_Deo(ctx, g, f, q.QDWF_EVEN, case["dagger"], prec, lay, nrhs)
    elif op == "MdagM":
        q.qdwf_apply_MdagM(ctx, g, f, prec, lay, nrhs, state["ws"])
    elif op == "Mee":
        which = q.QDWF_MEE_INV if case["inverse"] else q.QDWF_MEE_FWD
        q.qdwf_apply_Mee(ctx, g, f, q.QDWF_FULL, case["dagger"], which, prec, lay, nrhs)
    elif op == "Dh":
        q.qdwf_apply_Dh(ctx, g, f, q.QDWF_FULL, case["dagger"], prec, lay, nrhs)
    else:
        q.qdwf_apply_Dw(ctx, g, f, DW_MASS, case["dagger"], prec, lay, nrhs)
    return g


# ---- bytes and operations a pass cannot do without ----------------------------------
def work(case):
    if case["op"] == "serve":
        # links, source and solution once per request; each iteration at least reads and
        # writes x, r and p of the inner solve and the links once
        by = fl = 0.0
        s = SIZE[case["prec"]]
        for l, Ls, _, _, _ in _requests(case, 0):
            V = l ** 4
            half = V / 2 * Ls * 24
            by += V * 72 * 16 / 2 + 2 * half * 8 + 150 * (3 * half * s + V * 72 * s)
            fl += 150 * 4 * HOP_FLOPS * V / 2 * Ls
        return {"bytes": by, "flops": fl}
    L, Ls, nrhs, s = _extents(case), case["Ls"], case["nrhs"], SIZE[case["prec"]]
    V = L[0] * L[1] * L[2] * L[3]
    full, links = V * Ls * 24 * nrhs, V * 72
    n5 = V * Ls * nrhs
    op = case["op"]
    if op == "MdagM":
        return {"bytes": (full + links) * s, "flops": 2 * HOP_FLOPS * n5}
    if op == "Deo":
        return {"bytes": (full + links) * s, "flops": HOP_FLOPS * n5 / 2}
    if op == "Mee":
        return {"bytes": 2 * full * s, "flops": 4 * 24 * n5}
    if op == "config":
        return {"bytes": links * 8 + 2 * full * 8, "flops": HOP_FLOPS * n5}
    if op == "solve":
        its = 150
        return {"bytes": full * 8 + its * (3 * full / 2 + links) * s,
                "flops": its * 2 * HOP_FLOPS * n5}
    return {"bytes": (2 * full + links) * s, "flops": HOP_FLOPS * n5}


# ---- the same in 64 bits ---------------------------------------------------------------
# gamma_mu psi = factor * psi[source], rows 0..3 (DeGrand-Rossi basis)
_GAMMA = [((3, 2, 1, 0), (1j, 1j, -1j, -1j)), ((3, 2, 1, 0), (-1, 1, 1, -1)),
          ((2, 3, 0, 1), (1j, -1j, -1j, 1j)), ((2, 3, 0, 1), (1, 1, 1, 1))]


def _gamma(mu, v):
    src, fac = _GAMMA[mu]
    f = torch.tensor(fac, device=DEV, dtype=torch.complex128)
    return v[..., list(src), :] * f[:, None]


def _colour(U, v):
    """U v at every site and slice, spin by spin."""
    return sum(U[..., None, :, b] * v[..., :, b, None] for b in range(3))


class _Exact:
    """The domain-wall operator on [s][t][z][y][x][4][3] in complex128."""

    def __init__(self, L, Ls, U, M5, mf, b, c):
        self.L, self.Ls, self.mf, self.b, self.c = L, Ls, mf, b, c
        self.alpha, self.beta = b * (4 - M5) + 1, c * (4 - M5) - 1
        U = U.to(torch.complex128).clone()
        for mu in range(4):     # the boundary factor sits on the last link of each direction
            U[mu].select(3 - mu, L[mu] - 1).mul_(BC[mu])
        self.U = U
        x = torch.arange(L[0], device=DEV).view(1, 1, 1, -1) + torch.arange(L[1], device=DEV).view(1, 1, -1, 1)
        x = x + torch.arange(L[2], device=DEV).view(1, -1, 1, 1) + torch.arange(L[3], device=DEV).view(-1, 1, 1, 1)
        self.odd = (x % 2).view(1, L[3], L[2], L[1], L[0], 1, 1)
        Sd = torch.zeros(Ls, Ls, dtype=torch.float64)
        for s in range(Ls):
            Sd[s, (s - 1) % Ls] = 1.0 if s else -mf
        self.Sd = Sd.to(DEV)

    def hop(self, v, dag):
        out = torch.zeros_like(v)
        sg = -1 if dag else 1
        for mu in range(4):
            dim, U = 4 - mu, self.U[mu]
            out += _colour(U, torch.roll(v - sg * _gamma(mu, v), -1, dim))
            out += torch.roll(_colour(U.transpose(-1, -2).conj(), v + sg * _gamma(mu, v)), 1, dim)
        return out

    def chiral(self, K, v, dag=False):
        """K on the upper spins and its reflection in s on the lower ones (S_u for S_d)."""
        K = K.to(torch.complex128)
        P = torch.flip(K, (0, 1))
        if dag:
            K, P = K.T.contiguous(), P.T.contiguous()
        up, lo = v[..., :2, :].contiguous(), v[..., 2:, :].contiguous()
        up = (K @ up.reshape(self.Ls, -1)).reshape(up.shape)
        lo = (P @ lo.reshape(self.Ls, -1)).reshape(lo.shape)
        return torch.cat([up, lo], -2)

    def A(self, v, dag):
        return self.b * v + self.c * self.chiral(self.Sd, v, dag) if self.c else self.b * v

    def local(self, v, dag=False, inverse=False):
        M = self.alpha * torch.eye(self.Ls, device=DEV, dtype=torch.float64) + self.beta * self.Sd
        return self.chiral(torch.linalg.inv(M.cpu()).to(DEV) if inverse else M, v, dag)

    def off(self, v, dag):
        """-1/2 D_h A, or its adjoint: the part that changes the parity."""
        return -0.5 * (self.A(self.hop(v, True), True) if dag else self.hop(self.A(v, False), False))

    def D(self, v, dag):
        return self.off(v, dag) + self.local(v, dag)

    def Mpc(self, v, dag):
        """On odd sites (v is zero on the even ones; so is the result)."""
        return self.local(v, dag) - self.off(self.local(self.off(v, dag), dag, True), dag)

    def MdagM(self, v):
        return self.Mpc(self.Mpc(v, False), True)

    def solve(self, b, tol=3e-15, most=1500):
        x, r = torch.zeros_like(b), b.clone()
        p, rr = r.clone(), float(torch.linalg.vector_norm(r)) ** 2
        stop = tol * tol * rr
        for _ in range(most):
            Ap = self.MdagM(p)
            a = rr / float((p.conj() * Ap).real.sum())
            x += a * p
            r -= a * Ap
            new = float(torch.linalg.vector_norm(r)) ** 2
            if new <= stop:
                break
            p = r + (new / rr) * p
            rr = new
        return x


def _site_order(L):
    """Lex index of the sites of each parity in the documented traversal order:
    8 slabs along z, (x, y, z) tiles of 32 x 4 x Lz/8 in each, swept along t."""
    lex = np.arange(L[0] * L[1] * L[2] * L[3])
    x = [lex % L[0], lex // L[0] % L[1], lex // (L[0] * L[1]) % L[2], lex // (L[0] * L[1] * L[2])]
    tile = (min(L[0], 32), min(L[1], 4), max(1, L[2] // 8))
    keys = [x[0] % tile[0], x[1] % tile[1], x[2] % tile[2], x[3], x[0] // tile[0], x[1] // tile[1],
            x[2] // tile[2], x[2] * 8 // L[2]]
    order = np.lexsort(keys)
    par = (x[0] + x[1] + x[2] + x[3]) % 2
    return [torch.from_numpy(order[par[order] == p]).to(DEV) for p in (0, 1)]


def _internal(v, L, Ls, subset):
    """Canonical [rhs][s][t][z][y][x][4][3] -> the interleaved internal field."""
    v = torch.view_as_real(v.reshape(v.shape[0], Ls, -1, 12)).reshape(v.shape[0], Ls, -1, 24)
    order, parts = _site_order(L), []
    for p in ((0, 1) if subset == q.QDWF_FULL else (subset,)):
        h = v[:, :, order[p]]
        if Ls == 1:      # 16 consecutive sites play the role of the slices
            h = h.reshape(h.shape[0], -1, 16, 6, 4).transpose(2, 3)
        else:
            h = h.reshape(h.shape[0], Ls, -1, 6, 4).permute(0, 2, 3, 1, 4)
        parts.append(h.reshape(h.shape[0], -1))
    return torch.cat(parts, 1).reshape(-1)


def _stored(z, prec):
    """Complex values as rounded to the storage type, in complex128."""
    r = torch.view_as_real(z).to(q.TORCH_DTYPE[PREC[prec]]).to(torch.float64)
    return torch.view_as_complex(r.contiguous())


def exact(case, seed):
    if case["op"] == "serve":
        out = []
        for l, Ls, mf, us, bs in _requests(case, seed):
            L = (l, l, l, l)
            E = _Exact(L, Ls, _smooth(L, us), 1.8, mf, 1.5, 0.5)
            out.append(E.solve(_gaussian((Ls, l, l, l, l, 4, 3), bs) * E.odd))
        return out
    L, Ls, op = _extents(case), case["Ls"], case["op"]
    store = "f64" if op == "solve" else case["prec"]
    E = _Exact(L, Ls, _stored(_links(case, seed), store), **_action(case))
    psi = _stored(_spinor(case, seed), store)
    sout = _subset(case)[1]
    res = []
    for v in psi:
        if op in ("D", "config"):
            w = E.D(v, case["dagger"])
        elif op == "Deo":
            w = E.off(v * E.odd, case["dagger"])
        elif op == "MdagM":
            w = E.MdagM(v * E.odd)
        elif op == "Mee":
            w = E.local(v, case["dagger"], case["inverse"])
        elif op == "solve":
            w = E.solve(v * E.odd)
        else:
            w = E.hop(v, case["dagger"])
            if op == "Dw":
                w = (4 + DW_MASS) * v - 0.5 * w
        res.append(w)
    w = torch.stack(res)
    return w if op == "config" else _internal(w, L, Ls, sout)

"""Workloads of the twisted-mass clover library, for timing one build against another.

A case is one call (or the few calls that belong together) a lattice program
makes through the Python binding: operator applications on the caller's own
internal fields, solves, forces, a new gauge configuration, the learned
preconditioner and its training gradient.  Lattices run from 4^4 to 32^3x64,
extents even as the library asks, many of them no powers of two.

``exact`` evaluates the same quantities in 64-bit torch arithmetic on full
lattices (spinors [t][z][y][x][flavour][spin][colour]) straight from the
definitions of include/tmx.h.
"""
import math

import numpy as np
import torch

import paper_2212_06635_amd.tmx as tmx

# physics parameters of the repository's benchmark
KAPPA, CSW, MU, MUBAR, EPSBAR, T_BC, RHO = 0.1394, 1.69, 0.00072, 0.1246, 0.1315, -1, 0.02
C128 = torch.complex128
OPS = {"plus": tmx.TMX_OP_PLUS, "minus": tmx.TMX_OP_MINUS, "nd": tmx.TMX_OP_ND,
       "wplus": tmx.TMX_OP_WPLUS, "wminus": tmx.TMX_OP_WMINUS}
KINDS = {"cg": tmx.TMX_SOLVER_CG, "mpcg_f32": tmx.TMX_SOLVER_MPCG_F32, "mpcg_f16": tmx.TMX_SOLVER_MPCG_F16}


def _case(what, dims, **more):
    return {"what": what, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], **more}


def listed():
    big, mid, std, small = (32, 32, 32, 64), (24, 24, 24, 48), (16, 16, 16, 32), (8, 8, 8, 8)
    return [
        # N = Mhat^dagger Mhat on the smallest lattice of the tests and the smoke
        # check: launches and latency
        {"name": "n_f64_8x8x8x8", **_case("n", small, op="plus", prec="f64")},
        # the Schur operator at the benchmark's size: the headline, and what the
        # reliable updates and true residuals of every solve are made of
        {"name": "mhat_f64_32x32x32x64", **_case("mhat", big, op="plus", prec="f64", dagger=0)},
        # the heavy sector's operator (two flavours, adjoint) in the precision of
        # its inner iterations
        {"name": "mhat_nd_f32_24x24x24x48", **_case("mhat", mid, op="nd", prec="f32", dagger=1)},
        # the inner iteration of the FP16 mixed-precision CG, on a lattice whose
        # extents fit no tile
        {"name": "n_f16_20x12x28x36", **_case("n", (20, 12, 28, 36), op="minus", prec="f16")},
        # a whole FP64 CG where every kernel is short
        {"name": "cg_f64_8x8x8x8", **_case("solve", small, op="plus", kind="cg", nrhs=1)},
        # the fastest light-sector solve, at the benchmark's size
        {"name": "mpcg_f16_32x32x32x64", **_case("solve", big, op="plus", kind="mpcg_f16", nrhs=1)},
        # twelve sources (the spin-colour components of a propagator) in the heavy sector
        {"name": "mpcg_nd_r12_16x16x16x32", **_case("solve", std, op="nd", kind="mpcg_f32", nrhs=12)},
        # the twelve poles of the heavy sector's rational approximation
        {"name": "multishift_nd_12_24x24x24x48", **_case("multishift", mid, op="nd", nshift=12, inner="f32")},
        # one shift's force (hopping and clover terms) of a momentum update
        {"name": "force_32x32x32x64", **_case("force", big, op="plus")},
        # a new gauge configuration: upload, clover term, site inverses, and the
        # first application on a canonical field (pack and unpack)
        {"name": "new_gauge_16x16x16x32", **_case("gauge", std, op="plus")},
        # the learned preconditioner's production form P_1, once per iteration
        {"name": "pc_p1_24x24x24x48", **_case("pc", mid, mode=3)},
        # forward and backward through the network: the gradient of one training batch
        {"name": "pc_grad_16x16x16x32", **_case("grad", std, npairs=4)},
    ]


def _draw_dims(rng, vmax):
    """Even extents, time the longest, volume spread over its logarithm up to vmax."""
    while True:
        v = math.exp(rng.uniform(math.log(256), math.log(vmax)))
        s = (v / 2) ** 0.25
        d = [max(4, 2 * round(s * math.exp(rng.uniform(-0.3, 0.3)) / 2)) for _ in range(3)]
        d.append(max(4, 2 * round(v / (d[0] * d[1] * d[2]) / 2)))
        if d[0] * d[1] * d[2] * d[3] <= vmax and d[3] <= 96:
            return tuple(d)


def draw(rng):
    what = rng.choice(["n", "mhat", "mhat", "solve", "solve", "multishift", "force", "force", "gauge", "pc", "grad"])
    big, mid, std = 32 ** 3 * 64, 24 ** 3 * 48, 16 ** 3 * 32
    if what == "n":
        return _case(what, _draw_dims(rng, big), op=rng.choice(["plus", "minus", "nd", "wplus"]),
                     prec=rng.choice(["f64", "f32", "f16"]))
    if what == "mhat":
        return _case(what, _draw_dims(rng, big), op=rng.choice(["plus", "minus", "nd", "wminus"]),
                     prec=rng.choice(["f64", "f32", "f16"]), dagger=rng.choice([0, 1]))
    if what == "solve":
        op, nrhs = rng.choice(["plus", "minus", "nd", "wplus"]), rng.choice([1, 1, 1, 2, 3, 12])
        vmax = mid if op != "nd" and nrhs == 1 else std
        return _case(what, _draw_dims(rng, vmax), op=op, kind=rng.choice(["cg", "mpcg_f32", "mpcg_f16"]), nrhs=nrhs)
    if what == "multishift":
        return _case(what, _draw_dims(rng, mid), op=rng.choice(["plus", "nd", "nd"]),
                     nshift=rng.choice([3, 6, 8, 10, 12]), inner=rng.choice(["f32", "f32", "f16", "f64"]))
    if what == "force":
        return _case(what, _draw_dims(rng, big), op=rng.choice(["plus", "minus", "nd"]))
    if what == "gauge":
        return _case(what, _draw_dims(rng, mid), op=rng.choice(["plus", "minus", "nd"]))
    if what == "pc":
        return _case(what, _draw_dims(rng, mid), mode=rng.choice([0, 1, 2, 3]))
    return _case(what, _draw_dims(rng, std), npairs=rng.choice([1, 2, 4]))


# ---------------------------------------------------------------------------
# inputs (torch on the GPU, from the seed alone)
# ---------------------------------------------------------------------------
def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def _nf(case):
    return 2 if case.get("op") == "nd" else 1


def _gen(seed, k):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * int(seed) + k)
    return g


def _mm(a, b):
    """3x3 products, entry by entry."""
    return torch.stack([torch.stack([sum(a[..., i, k] * b[..., k, j] for k in range(3)) for j in range(3)], -1)
                        for i in range(3)], -2)


def _dag(a):
    return a.conj().transpose(-1, -2).resolve_conj()


def _links(dims, seed, eps=0.25):
    """SU(3) links exp(i eps H), H = sum_a w_a lambda_a / 2 with Gaussian w; [t][z][y][x][mu][3][3]."""
    lx, ly, lz, lt = dims
    out = torch.empty((lt, lz, ly, lx, 4, 3, 3), dtype=C128, device="cuda")
    for mu in range(4):
        w = torch.randn((8, lt, lz, ly, lx), dtype=torch.float64, device="cuda", generator=_gen(seed, mu)) * (eps / 2)
        h = torch.zeros((lt, lz, ly, lx, 3, 3), dtype=C128, device="cuda")
        for n, (i, j) in enumerate(((0, 1), (0, 2), (1, 2))):
            h[..., i, j] = torch.complex(w[2 * n], -w[2 * n + 1])
            h[..., j, i] = torch.complex(w[2 * n], w[2 * n + 1])
        h[..., 0, 0] = w[6] + w[7] / math.sqrt(3)
        h[..., 1, 1] = -w[6] + w[7] / math.sqrt(3)
        h[..., 2, 2] = -2 * w[7] / math.sqrt(3)
        u = torch.eye(3, dtype=C128, device="cuda") + 1j * h / 12
        for k in range(11, 0, -1):  # the exponential's series, innermost factor first
            u = torch.eye(3, dtype=C128, device="cuda") + (1j / k) * _mm(h, u)
        r0 = u[..., 0, :] / torch.linalg.vector_norm(u[..., 0, :], dim=-1, keepdim=True)
        r1 = u[..., 1, :] - (r0.conj() * u[..., 1, :]).sum(-1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
        out[..., mu, 0, :], out[..., mu, 1, :] = r0, r1
        for c in range(3):
            a, b = (c + 1) % 3, (c + 2) % 3
            out[..., mu, 2, c] = (r0[..., a] * r1[..., b] - r0[..., b] * r1[..., a]).conj()
    return out


def _gauss(dims, nf, n, seed, k):
    """n Gaussian odd fields, canonical order."""
    vh = dims[0] * dims[1] * dims[2] * dims[3] // 2
    re, im = (torch.randn(n * vh * nf * 12, dtype=torch.float64, device="cuda", generator=_gen(seed, k + j)) for j in (0, 1))
    return torch.complex(re, im)


def _weights(seed):
    """Network weights near the identity, as training starts from: C_0 = 1, Gamma_0 = 1, the rest N(0, 1e-2)."""
    rng, parts = np.random.default_rng([int(seed), 9]), []
    for ci, co in ((1, 8), (8, 8), (8, 8), (8, 1)):
        for d in range(9):
            for a, b in ((co, ci), (4, 4)):
                m = np.eye(a, b) + 0j if d == 0 else 1e-2 * (rng.standard_normal((a, b)) + 1j * rng.standard_normal((a, b)))
                parts.append(np.stack([m.real.reshape(-1), m.imag.reshape(-1)], 1).reshape(-1))
    return np.concatenate(parts).astype(np.float32)


def _shifts(n):
    """Poles of an approximation of N^(-1/2) over five decades, closely geometric."""
    return np.geomspace(1.6e-6, 5.8, n)


def _context(dims, U):
    ctx = tmx.Context(dims)
    ctx.set_params(tmx.Params(KAPPA, CSW, MU, MUBAR, EPSBAR, T_BC, RHO))
    ctx.load_gauge(U, 1.0)
    ctx.load_clover()
    return ctx


def _training_pairs(dims, U, n, seed):
    """b_i = Mhat x_i for Gaussian x_i."""
    x = _gauss(dims, 1, n, seed, 30)
    f = _Fields(dims, U)
    b = torch.cat([f.cb(f.mhat(f.full(v, 1), 1)) for v in x.view(n, -1)])
    return b, x


def prepare(case, seed):
    dims, nf = _dims(case), _nf(case)
    s = dict(case)
    links = _links(dims, seed)
    U = links.cpu().numpy()
    s["ctx"] = ctx = _context(dims, U)
    vh = ctx.Vh
    if case["what"] in ("n", "mhat"):
        kind, prec = (tmx.TMX_FIELD_ODD_ND if nf == 2 else tmx.TMX_FIELD_ODD), tmx.PREC[case["prec"]]
        s["in"] = ctx.pack(_gauss(dims, nf, 1, seed, 10), kind, prec)
        s["out"] = ctx.empty(kind, prec)
    elif case["what"] == "solve":
        s["b"] = _gauss(dims, nf, case["nrhs"], seed, 10)
        s["x"] = torch.zeros_like(s["b"])
    elif case["what"] == "multishift":
        s["b"] = _gauss(dims, nf, 1, seed, 10)
        s["x"] = torch.zeros(case["nshift"] * vh * nf * 12, dtype=C128, device="cuda")
    elif case["what"] == "force":
        s["X"], s["Y"] = _gauss(dims, nf, 1, seed, 10), _gauss(dims, nf, 1, seed, 20)
        s["F"] = torch.zeros(ctx.V * 36, dtype=C128, device="cuda")
    elif case["what"] == "gauge":
        s["U"], s["id"], s["phi"] = U, 1.0, _gauss(dims, nf, 1, seed, 10)
    elif case["what"] == "pc":
        ctx.pc_set_weights(_weights(seed))
        s["b"] = _gauss(dims, 1, 1, seed, 10)
        s["x"] = torch.empty_like(s["b"])
    else:
        ctx.pc_set_weights(_weights(seed))
        s["b"], s["x"] = _training_pairs(dims, links, case["npairs"], seed)
    return s


def _field_values(buf, prec, n):
    """A field buffer in its own number type: FP64, FP32, or FP16 values and their FP32 scales (n reals)."""
    if prec == "f16":
        return [buf[:2 * n].view(torch.float16), buf[2 * n:].view(torch.float32)]
    return buf.view(torch.float64 if prec == "f64" else torch.float32)


def run(state):
    s = state
    ctx, what = s["ctx"], s["what"]
    nf, op = _nf(s), OPS.get(s.get("op"))
    if what == "n":
        ctx.apply_mdagm(s["out"], s["in"], op, tmx.PREC[s["prec"]])
        return _field_values(s["out"], s["prec"], ctx.Vh * nf * 24)
    if what == "mhat":
        ctx.apply_mhat(s["out"], s["in"], op, tmx.PREC[s["prec"]], dagger=s["dagger"])
        return _field_values(s["out"], s["prec"], ctx.Vh * nf * 24)
    if what == "solve":
        ctx.solve(s["x"], s["b"], s["nrhs"], kind=KINDS[s["kind"]], op=op, tol=1e-11)
        return s["x"]
    if what == "multishift":
        ctx.multishift_solve(s["x"], s["b"], _shifts(s["nshift"]), op=op, tol=1e-11, inner_prec=tmx.PREC[s["inner"]])
        return s["x"]
    if what == "force":
        ctx.hop_force(s["F"], s["X"], s["Y"], op=op)
        ctx.clover_force(s["F"], s["X"], s["Y"], op=op, accumulate=1)
        return s["F"]
    if what == "gauge":
        s["id"] += 1.0  # the next configuration of the trajectory
        ctx.load_gauge(s["U"], s["id"])
        ctx.load_clover()
        kind = tmx.TMX_FIELD_ODD_ND if nf == 2 else tmx.TMX_FIELD_ODD
        v = ctx.pack(s["phi"], kind, tmx.TMX_F64)
        out = ctx.empty(kind, tmx.TMX_F64)
        ctx.apply_mhat(out, v, op, tmx.TMX_F64)
        return ctx.unpack(out, kind, tmx.TMX_F64)
    if what == "pc":
        ctx.pc_apply(s["x"], s["b"], dagger=s["mode"])
        return s["x"]
    loss, grad = ctx.pc_loss_grad(s["b"], s["x"], s["npairs"])
    return {"loss": loss, "grad": grad}


# ---------------------------------------------------------------------------
# what a pass cannot do without: inputs read once, outputs written once, and
# for a solve every iteration's operator and the vectors it advances
# ---------------------------------------------------------------------------
def work(case):
    dims, nf, what = _dims(case), _nf(case), case["what"]
    vh = dims[0] * dims[1] * dims[2] * dims[3] // 2
    hop = 1320 * nf  # flops of one hopping term per site
    real = {"f64": 8, "f32": 4, "f16": 2}

    def mhat(b):  # two-row links of both parities, site blocks of both parities, field in and out
        return vh * b * (96 + 144 + 48 * nf), vh * (2 * hop + 1104 * nf)

    if what in ("n", "mhat"):
        by, fl = mhat(real[case["prec"]])
        return {"bytes": by, "flops": (2 if what == "n" else 1) * fl}
    if what in ("solve", "multishift"):
        inner = case.get("inner") or {"cg": "f64", "mpcg_f32": "f32", "mpcg_f16": "f16"}[case["kind"]]
        n, its = case.get("nrhs", 1), 80 if nf == 1 else 115
        by, fl = mhat(real[inner])
        per = by + (n - 1) * vh * real[inner] * 48 * nf
        vec = 4 * n + 4 * case.get("nshift", 0) // 2
        return {"bytes": its * (2 * per + vec * vh * 24 * nf * real[inner]), "flops": its * 2 * n * fl}
    if what == "force":  # links, clover terms, the two fields, and every link's force
        return {"bytes": 2 * vh * (48 + 72) * 8 + vh * 48 * nf * 8 + 2 * vh * 576, "flops": 2 * vh * (8000 + 4000 * nf)}
    if what == "gauge":  # the links over the host link and through memory, the derived fields, one application
        by, fl = mhat(8)
        return {"bytes": 2 * vh * 576 + 2 * vh * 72 * 8 + vh * 48 * nf * 8 + by, "flops": fl + 2 * vh * 30000}
    layer = 2 * vh * 2 * 9 * (8 * 12 * 8 + 8 * 36)
    if what == "pc":  # links (BF16) and the field in and out
        return {"bytes": 2 * vh * 4 * 36 + vh * 384, "flops": layer * (2 if case["mode"] < 3 else 0.2)}
    return {"bytes": case["npairs"] * (2 * vh * 4 * 36 * 8 + 2 * vh * 8 * 48 * 8), "flops": case["npairs"] * 6 * layer}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
# gamma_mu psi: component s of the result is phase[s] psi[perm[s]]
GAMMA = [((3, 2, 1, 0), (-1j, -1j, 1j, 1j)), ((3, 2, 1, 0), (-1, 1, 1, -1)),
         ((2, 3, 0, 1), (-1j, 1j, 1j, -1j)), ((2, 3, 0, 1), (1, 1, 1, 1))]


def _gamma_matrix(mu):
    m = torch.zeros((4, 4), dtype=C128)
    for s in range(4):
        m[s, GAMMA[mu][0][s]] = GAMMA[mu][1][s]
    return m


class _Fields:
    """Operators on full-lattice fields [t][z][y][x][nf][4][3]."""

    def __init__(self, dims, U, clover=True):
        self.dims, self.U = dims, U
        lx, ly, lz, lt = dims
        t, z, y, x = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)), indexing="ij")
        self.odd = ((x + y + z + t) % 2 == 1)
        self.coord = (x, y, z, t)
        self.g5 = torch.tensor([1, 1, -1, -1], device="cuda", dtype=torch.float64)[:, None]
        self.A = self.clover() if clover else None
        self.inverse = {}

    def full(self, v, nf):
        f = torch.zeros(self.odd.shape + (nf, 4, 3), dtype=C128, device="cuda")
        f[self.odd] = v.view(-1, nf, 4, 3)
        return f

    def cb(self, f):
        return f[self.odd].reshape(-1)

    def shift(self, f, mu, d):
        return torch.roll(f, -d, 3 - mu)

    def clover(self):
        """A = 1 + T as [..][chirality][6][6]."""
        U = self.U
        T = torch.zeros(self.odd.shape + (4, 3, 4, 3), dtype=C128, device="cuda")
        for mu in range(4):
            for nu in range(mu + 1, 4):
                um, un = U[..., mu, :, :], U[..., nu, :, :]
                # the four leaves at x, each beginning and ending there
                m_m, n_m = self.shift(um, mu, -1), self.shift(un, mu, -1)  # links at x - mu
                m_n, n_n = self.shift(um, nu, -1), self.shift(un, nu, -1)  # at x - nu
                m_mn, n_mn = self.shift(m_n, mu, -1), self.shift(n_n, mu, -1)  # at x - mu - nu
                Q = (_mm(_mm(um, self.shift(un, mu, 1)), _mm(_dag(self.shift(um, nu, 1)), _dag(un)))
                     + _mm(_mm(un, _dag(self.shift(m_m, nu, 1))), _mm(_dag(n_m), m_m))
                     + _mm(_mm(_dag(m_m), _dag(n_mn)), _mm(m_mn, n_n))
                     + _mm(_mm(_dag(n_n), m_n), _mm(self.shift(n_n, mu, 1), _dag(um))))
                F = (Q - _dag(Q)) / 8
                gm, gn = _gamma_matrix(mu), _gamma_matrix(nu)
                sig = 0.5j * (gm @ gn - gn @ gm)
                for a in range(4):
                    for c in range(4):
                        if sig[a, c] != 0:
                            T[..., a, :, c, :] += (1j * KAPPA * CSW * complex(sig[a, c])) * F
        T = T.reshape(self.odd.shape + (12, 12))
        A = torch.stack([T[..., :6, :6], T[..., 6:, 6:]], -3)
        return A + torch.eye(6, dtype=C128, device="cuda")

    def site(self, f, sgn, nf, nu):
        """(A + twist) f"""
        v = f.reshape(f.shape[:4] + (nf, 2, 6))
        w = (self.A[:, :, :, :, None] * v[..., None, :]).sum(-1)
        ch = torch.tensor([1, -1], device="cuda", dtype=torch.float64)[:, None]
        tau = torch.tensor([1, -1][:nf], device="cuda", dtype=torch.float64)[:, None, None]
        w = w + 1j * sgn * nu * ch * tau * v
        if nf == 2:
            w = w - 2 * KAPPA * EPSBAR * v.flip(4)
        return w.reshape(f.shape)

    def blocks_inverse(self, sgn, nf):
        """(A + twist)^-1 on each chirality: 6x6, or 12x12 over the flavours, by elimination."""
        if (sgn, nf) in self.inverse:
            return self.inverse[sgn, nf]
        n = 6 * nf
        M = torch.zeros(self.odd.shape + (2, n, n), dtype=C128, device="cuda")
        eye = torch.eye(6, dtype=C128, device="cuda")
        for c in range(2):
            for f in range(nf):
                nu = 2 * KAPPA * (MU if nf == 1 else MUBAR) * sgn * (1 - 2 * c) * (1 - 2 * f)
                M[..., c, 6 * f:6 * f + 6, 6 * f:6 * f + 6] = self.A[..., c, :, :] + 1j * nu * eye
            if nf == 2:
                M[..., c, :6, 6:] = M[..., c, 6:, :6] = -2 * KAPPA * EPSBAR * eye
        inv = torch.eye(n, dtype=C128, device="cuda").expand(M.shape).clone()
        for k in range(n):
            p = 1 / M[..., k, k][..., None]
            rm, ri = M[..., k, :] * p, inv[..., k, :] * p
            col = M[..., :, k].clone()
            col[..., k] = 0
            M = M - col[..., None] * rm[..., None, :]
            inv = inv - col[..., None] * ri[..., None, :]
            M[..., k, :], inv[..., k, :] = rm, ri
        self.inverse[sgn, nf] = inv
        return inv

    def site_inverse(self, f, sgn):
        nf = f.shape[4]
        inv = self.blocks_inverse(sgn, nf)
        v = f.reshape(f.shape[:4] + (nf, 2, 6)).transpose(4, 5).reshape(f.shape[:4] + (2, 6 * nf))
        w = sum(inv[..., k] * v[..., k, None] for k in range(6 * nf))
        return w.reshape(f.shape[:4] + (2, nf, 6)).transpose(4, 5).reshape(f.shape)

    def transport(self, f, mu, d):
        """U_mu(x) f(x + mu), or U_mu(x - mu)^dagger f(x - mu), with the time boundary's factor."""
        g = self.shift(f, mu, d)
        u = self.U[..., mu, :, :]
        u = u if d > 0 else _dag(self.shift(u, mu, -1))
        if mu == 3:
            edge = self.coord[3] == (self.dims[3] - 1 if d > 0 else 0)
            g = g * torch.where(edge, float(T_BC), 1.0).view(edge.shape + (1,) * (g.dim() - 4))
        u = u.view(u.shape[:4] + (1,) * (g.dim() - 5) + (3, 3))
        return u[..., 0] * g[..., 0:1] + u[..., 1] * g[..., 1:2] + u[..., 2] * g[..., 2:3]

    def gamma(self, f, mu):
        perm, ph = GAMMA[mu]
        return f[..., list(perm), :] * torch.tensor(ph, dtype=C128, device="cuda")[:, None]

    def hop(self, f, parity):
        out = torch.zeros_like(f)
        for mu in range(4):
            a, b = self.transport(f, mu, 1), self.transport(f, mu, -1)
            out = out + a + b - self.gamma(a - b, mu)
        return out * (self.odd if parity else ~self.odd)[..., None, None, None]

    def mhat(self, f, sgn):
        nf = f.shape[4]
        u = self.site_inverse(self.hop(f, 0), sgn)
        nu = 2 * KAPPA * (MU if nf == 1 else MUBAR)
        return self.site(f, sgn, nf, nu) * self.odd[..., None, None, None] - KAPPA ** 2 * self.hop(u, 1)

    def mhat_dag(self, f, sgn):
        return self.g5 * self.mhat(self.g5 * f, -sgn)

    def what(self, f, sgn):
        return self.g5 * self.mhat(f, sgn) + 1j * sgn * 2 * KAPPA * RHO * f

    def apply(self, f, op, dagger):
        sgn = -1 if op in ("minus", "wminus") else 1
        if op[0] == "w":
            return self.what(f, -sgn if dagger else sgn)
        return self.mhat_dag(f, sgn) if dagger else self.mhat(f, sgn)

    def normal(self, f, op):
        return self.apply(self.apply(f, op, 0), op, 1)


def _internal(case, f, F):
    """A full-lattice field's odd sites in the order and number format of the internal fields:
    vectors of 2 (FP64), 4 (FP32) or 8 (FP16) reals, sites fastest; x/2 and y run fastest over
    the sites, then the (z, t) planes in tiles of 2 x 8 (the largest power of two that divides)."""
    lx, ly, lz, lt = _dims(case)
    zb, tb = 2, next(k for k in (8, 4, 2) if lt % k == 0)
    x, y, z, t = (c[F.odd] for c in F.coord)
    plane = ((t // tb) * (lz // zb) + z // zb) * (zb * tb) + (t % tb) * zb + z % zb
    order = torch.argsort((plane * ly + y) * (lx // 2) + x // 2)
    v = torch.view_as_real(f[F.odd][order].reshape(order.numel(), -1, 12)).reshape(order.numel(), -1, 24)
    scale = v.abs().amax(-1)
    w = {"f64": 2, "f32": 4, "f16": 8}[case["prec"]]
    if case["prec"] == "f16":
        v = v / scale[..., None]
    out = v.reshape(v.shape[0], v.shape[1], 24 // w, w).permute(1, 2, 0, 3).reshape(-1)
    return [out, scale.t().reshape(-1)] if case["prec"] == "f16" else out


def _dot(a, b):
    return float((a.real * b.real + a.imag * b.imag).sum())


def _solve(F, b, op, shifts, tol=1e-13, maxiter=400):
    """(N + s)^-1 b for every shift s (ascending), one Krylov space for all (Jegerlehner's recurrences)."""
    n = len(shifts)
    xs, ps = [torch.zeros_like(b) for _ in range(n)], [b.clone() for _ in range(n)]
    r, bb = b.clone(), _dot(b, b)
    rr, zeta, zold, aold, bold = bb, [1.0] * n, [1.0] * n, 1.0, 0.0
    for _ in range(maxiter):
        q = F.normal(ps[0], op) + shifts[0] * ps[0]
        a = rr / _dot(ps[0], q)
        r = r - a * q
        new = _dot(r, r)
        beta = new / rr
        for k in range(n):
            if zeta[k] ** 2 * rr <= (tol * 1e-2) ** 2 * bb:
                continue
            zn = zeta[k] * zold[k] * aold / (a * bold * (zold[k] - zeta[k]) + zold[k] * aold * (1 + (shifts[k] - shifts[0]) * a))
            xs[k] += (a * zn / zeta[k]) * ps[k]
            ps[k] = zn * r + (beta * (zn / zeta[k]) ** 2) * ps[k]
            zold[k], zeta[k] = zeta[k], zn
        rr, aold, bold = new, a, beta
        if rr <= tol * tol * bb:
            break
    return xs


def _force(F, X, Y, op, nf):
    """The link derivative of Re<Y, Mhat X>: with u = A_ee^-1 H_eo X and w = A_ee^-dagger H_oe^dagger Y
    held, its variation is that of Re<Y, A X> - kappa^2 (Re<Y, H u> + Re<w, H X> - Re<w, A u>)."""
    sgn = -1 if op == "minus" else 1
    with torch.no_grad():
        u = F.site_inverse(F.hop(X, 0), sgn)
        w = F.site_inverse(F.g5 * F.hop(F.g5 * Y, 0), -sgn)
    U = F.U.clone().requires_grad_(True)
    V = _Fields(F.dims, U)
    s = _re(Y, V.site(X, sgn, nf, 0.0)) - KAPPA ** 2 * (
        _re(Y, V.hop(u, 1)) + _re(w, V.hop(X, 0)) - _re(w, V.site(u, sgn, nf, 0.0)))
    (G,) = torch.autograd.grad(s, U)
    Q = _mm(F.U, _dag(G))
    A = 0.5 * (Q - _dag(Q))
    tr = A.diagonal(dim1=-2, dim2=-1).sum(-1) / 3
    return (A - tr[..., None, None] * torch.eye(3, dtype=C128, device="cuda")).reshape(-1)


def _re(a, b):
    return (a.real * b.real + a.imag * b.imag).sum()


def _network(F, w, f, mode):
    """K (0), K^dagger (1), P = L1+ L2+ L2 L1 (2) or P_1 = L1+ L1 (3) of channels [..][c][4][3]."""
    layers, k = [], 0
    for ci, co in ((1, 8), (8, 8), (8, 8), (8, 1)):
        paths = []
        for d in range(9):
            C = torch.view_as_complex(w[k:k + 2 * co * ci].view(co, ci, 2))
            k += 2 * co * ci
            G = torch.view_as_complex(w[k:k + 32].view(4, 4, 2))
            k += 32
            paths.append((C, G))
        layers.append(paths)

    def mix(C, G, v):
        v = sum(G[:, t, None] * v[..., t:t + 1, :] for t in range(4))
        return sum(C[:, i, None, None] * v[..., i:i + 1, :, :] for i in range(C.shape[1]))

    def move(v, d):
        return v if d == 0 else F.transport(v, (d - 1) // 2, 1 if d % 2 else -1)

    def forward(paths, v):
        return sum(mix(C, G, move(v, d)) for d, (C, G) in enumerate(paths))

    def adjoint(paths, v):
        back = [0, 2, 1, 4, 3, 6, 5, 8, 7]
        return sum(move(mix(_dag(C), _dag(G), v), back[d]) for d, (C, G) in enumerate(paths))

    L1, L2, L3, L4 = layers
    if mode == 0:
        f = forward(L4, forward(L3, forward(L2, forward(L1, f))))
    elif mode == 1:
        f = adjoint(L1, adjoint(L2, adjoint(L3, adjoint(L4, f))))
    elif mode == 2:
        f = adjoint(L1, adjoint(L2, forward(L2, forward(L1, f))))
    else:
        f = adjoint(L1, forward(L1, f))
    return f * F.odd[..., None, None, None]


def exact(case, seed):
    dims, nf, what = _dims(case), _nf(case), case["what"]
    U = _links(dims, seed)
    F = _Fields(dims, U, clover=what != "pc")
    if what in ("n", "mhat"):
        f = F.full(_gauss(dims, nf, 1, seed, 10), nf)
        return _internal(case, F.normal(f, case["op"]) if what == "n" else F.apply(f, case["op"], case["dagger"]), F)
    if what in ("solve", "multishift"):
        if 2 * F.odd.sum() * nf * case.get("nrhs", 1) > 14e5:
            return None  # over twenty seconds of iterations
        b = _gauss(dims, nf, case.get("nrhs", 1), seed, 10)
        shifts = [float(v) for v in _shifts(case["nshift"])] if what == "multishift" else [0.0]
        return torch.cat([F.cb(x) for v in b.view(case.get("nrhs", 1), -1) for x in _solve(F, F.full(v, nf), case["op"], shifts)])
    if what == "force":
        X, Y = (F.full(_gauss(dims, nf, 1, seed, k), nf) for k in (10, 20))
        return _force(F, X, Y, case["op"], nf)
    if what == "gauge":
        return F.cb(F.apply(F.full(_gauss(dims, nf, 1, seed, 10), nf), case["op"], 0))
    w = torch.from_numpy(_weights(seed).astype(np.float64)).cuda()
    if what == "pc":
        return F.cb(_network(F, w, F.full(_gauss(dims, 1, 1, seed, 10), 1), case["mode"]))
    n = case["npairs"]
    b, x = _training_pairs(dims, U, n, seed)
    loss, grad = 0.0, torch.zeros_like(w)
    for bi, xi in zip(b.view(n, -1), x.view(n, -1)):
        wi = w.clone().requires_grad_(True)
        out = _network(F, wi, F.full(bi, 1), 0)
        e = out.detach() - F.full(xi, 1)
        q, bb = F.mhat(e, 1), _dot(bi, bi)
        loss += _dot(q, q) / bb / n
        delta = (2 / bb / n) * F.mhat_dag(q, 1)  # of the real and imaginary parts of K b
        (g,) = torch.autograd.grad(_re(delta, out), wi)
        grad += g
    return {"loss": torch.tensor(loss, dtype=torch.float64), "grad": grad}

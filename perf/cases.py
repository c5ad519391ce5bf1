"""Cases of the work that a program has this library do, each through the
public entry points: stencil applies (one field, blocks of fields, the even/odd
hopping block), sign and D_N applies with exact low modes, a whole mixed
precision solve, a differentiated action, and the Gram matrix of a block.

A case names an operation (``op``), a lattice ``n0 x n1 x n2 x n3``, the storage
(``sp`` spinors, ``lp`` links, ``recon`` reals per link) and what the operation
needs besides.  The Wilson mass, the link width and the approximant's interval
are those of the solve workload of bench.py.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1010_5636_amd as ndq

M = -1.4          # Wilson mass
MQ = 0.05         # quark mass of D_N^m
LAM = 6.6         # bound on |Q|
WIDTH = 0.3       # width of the random links
EPS = 0.00894     # lower end of the approximant's interval on (Q/LAM)^2
SPINOR_BYTES = {"f64": 192, "f32": 96, "f16": 52}
REAL_BYTES = {"f64": 8, "f32": 4, "f16": 2}
PREC = {"f64": ndq.F64, "f32": ndq.F32, "f16": ndq.F16}
DEV = "cuda"


def _case(name, op, dims, sp, lp, recon, nrhs=1, **more):
    c = {"name": name, "op": op, "n0": dims[0], "n1": dims[1], "n2": dims[2], "n3": dims[3],
         "sp": sp, "lp": lp, "recon": recon, "nrhs": nrhs}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: Q on a test lattice, where only the call itself costs
        _case("q_4c4_f64", "q", (4, 4, 4, 4), "f64", "f64", 18),
        # the even/odd hopping block on the dslash benchmark lattice
        _case("dslash_16c32_f32", "dslash", (32, 16, 16, 16), "f32", "f32", 12),
        # one field of the mixed solve: every Clenshaw step of its inner operator
        _case("q_24c48_f32", "q", (48, 24, 24, 24), "f32", "f32", 12),
        # the FP64 operator of its outer residuals and of the plain solve
        _case("q_24c48_f64", "q", (48, 24, 24, 24), "f64", "f64", 12),
        # the 12 spin-colour point sources in one apply, on the largest lattice
        _case("q12_32c64_f32", "q", (64, 32, 32, 32), "f32", "f32", 18, 12),
        # the same block on half precision storage, as the F16 inner solver has it
        _case("q12_24c48_f16", "q", (48, 24, 24, 24), "f16", "f16", 12, 12),
        # the block of the low-mode filter: 20 wanted and 40 extra vectors, FP64
        _case("q60_24c48_f64", "q", (48, 24, 24, 24), "f64", "f64", 12, 60),
        # one sign apply of the inner solver: polynomial and projection on 20 modes
        _case("sign_24c48_f32", "sign", (48, 24, 24, 24), "f32", "f32", 12, 1, nev=20, degree=67, sandwich=True),
        # one D_N apply of the batched solve of the 12 point sources
        _case("dn12_24c48_f32", "dn", (48, 24, 24, 24), "f32", "f32", 12, 12, nev=20, degree=67, sandwich=True),
        # a whole mixed solve on a small lattice, where launches and round trips count
        _case("solve_8c16", "solve", (16, 8, 8, 8), "f64", "f64", 12, 1, degree=67),
        # forward and backward of the action psi^H Q^2 psi through autograd
        _case("grad_16c32_f64", "grad", (32, 16, 16, 16), "f64", "f64", 18),
        # the Rayleigh-Ritz matrix of the low-mode block
        _case("gram60_24c48", "gram", (48, 24, 24, 24), "f64", "f64", 18, 60),
    ]


def _extent(rng, hi):
    """An even extent in [4, hi], spread over the logarithm."""
    return 2 * int(round(math.exp(rng.uniform(math.log(2.0), math.log(hi / 2.0)))))


def _dims(rng, vmin, vmax):
    while True:
        d = (_extent(rng, 64), _extent(rng, 32), _extent(rng, 32), _extent(rng, 32))
        if vmin <= d[0] * d[1] * d[2] * d[3] <= vmax:
            return d


def draw(rng):
    op = rng.choice(("q", "q", "q1", "q1", "dslash", "sign", "dn", "solve", "grad", "gram"))
    sp = rng.choice(("f64", "f32", "f32", "f16"))
    lp = sp
    recon = rng.choice((18, 12) if sp == "f16" else (18, 12, 12, 8))
    vmax = 64 * 32 ** 3
    if op in ("q", "q1", "dslash"):
        d = _dims(rng, 4 ** 4, vmax)
        nrhs = 1 if op == "q1" else int(round(math.exp(rng.uniform(math.log(2.0), math.log(60.0)))))
        if op == "dslash":
            nrhs = rng.choice((1, 1, nrhs))
        nrhs = max(1, min(nrhs, 60 * 48 * 24 ** 3 // (d[0] * d[1] * d[2] * d[3])))
        return _case("", "dslash" if op == "dslash" else "q", d, sp, lp, recon, nrhs)
    if op in ("sign", "dn"):
        d = _dims(rng, 4 ** 4, 48 * 24 ** 3)
        nrhs = 1 if op == "sign" else rng.randint(2, 12)
        return _case("", op, d, sp, lp, 12, nrhs, nev=rng.randint(1, 20), degree=rng.randint(20, 67),
                     sandwich=rng.random() < 0.7)
    if op == "solve":
        d = _dims(rng, 4 ** 4, 16 * 8 ** 3)
        return _case("", "solve", d, "f64", "f64", 12, rng.randint(1, 4), degree=rng.randint(50, 67))
    if op == "grad":
        return _case("", "grad", _dims(rng, 4 ** 4, 48 * 24 ** 3), "f64", "f64", 18)
    return _case("", "gram", _dims(rng, 4 ** 4, 48 * 24 ** 3), "f64", "f64", 18, rng.randint(2, 60))


# ---- inputs (canonical complex128, lexicographic sites) ------------------------

def _volume(c):
    return c["n0"] * c["n1"] * c["n2"] * c["n3"]


def _dims_of(c):
    return (c["n0"], c["n1"], c["n2"], c["n3"])


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1) + what)
    return g


def _mm(a, b):
    """Products of 3 x 3 matrices, without a batched library call."""
    out = a[..., :, 0, None] * b[..., 0, None, :]
    out += a[..., :, 1, None] * b[..., 1, None, :]
    out += a[..., :, 2, None] * b[..., 2, None, :]
    return out


def _links(v, seed):
    """Random SU(3) links exp(i H), H = sum_a omega_a lambda_a / 2, omega_a ~ N(0, WIDTH^2); [v, 4, 3, 3]."""
    w = torch.randn((v * 4, 8), generator=_gen(seed, 1), dtype=torch.float64, device=DEV) * (0.5 * WIDTH)
    h = torch.zeros((v * 4, 3, 3), dtype=torch.complex128, device=DEV)
    s3 = 1.0 / math.sqrt(3.0)
    h[:, 0, 0] = w[:, 2] + s3 * w[:, 7]
    h[:, 1, 1] = -w[:, 2] + s3 * w[:, 7]
    h[:, 2, 2] = -2.0 * s3 * w[:, 7]
    for (r, k, a, b) in ((0, 1, 0, 1), (0, 2, 3, 4), (1, 2, 5, 6)):
        h[:, r, k] = torch.complex(w[:, a], -w[:, b])
        h[:, k, r] = torch.complex(w[:, a], w[:, b])
    del w
    h *= 1j
    one = torch.eye(3, dtype=torch.complex128, device=DEV)
    u = h / 12.0 + one
    for k in range(11, 0, -1):      # Taylor polynomial of the exponential, Horner form
        u = _mm(h, u) / k
        u += one
    # onto SU(3): orthonormal columns a, b and c = conj(a x b)
    a = u[..., 0]
    a = a / torch.linalg.vector_norm(a, dim=-1, keepdim=True)
    b = u[..., 1]
    b = b - (a.conj() * b).sum(-1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=-1, keepdim=True)
    return torch.stack([a, b, torch.linalg.cross(a, b).conj()], dim=-1).reshape(v, 4, 3, 3)


def _field(n, seed, what, dtype=torch.complex128):
    """Complex Gaussian spinors of n sites, Re and Im ~ N(0, 1/2); [n, 4, 3]."""
    return torch.randn((n, 4, 3), generator=_gen(seed, what), dtype=dtype, device=DEV)


def _modes(v, nev, seed):
    """nev orthonormal fields [nev, v, 4, 3] (Cholesky QR of Gaussian ones) and signs of their eigenvalues."""
    a = torch.stack([_field(v, seed, 500 + k).reshape(-1) for k in range(nev)])
    low = torch.linalg.cholesky((a.conj() @ a.t()).conj())
    a = torch.linalg.solve_triangular(low, a, upper=False)
    sg = np.where(np.random.RandomState(seed % (1 << 31)).rand(nev) < 0.5, -1.0, 1.0)
    return a.reshape(nev, v, 4, 3), sg


def _coeffs(eps, degree):
    """Chebyshev coefficients of 1/sqrt(y) on [eps, 1] (the Clenshaw form of the sign)."""
    n = 4 * (degree + 1)
    th = (np.arange(n) + 0.5) * np.pi / n
    f = 1.0 / np.sqrt(0.5 * ((1.0 - eps) * np.cos(th) + 1.0 + eps))
    c = np.array([2.0 / n * np.sum(f * np.cos(k * th)) for k in range(degree + 1)])
    c[0] *= 0.5
    return c


def _pack(g, c, seed, nrhs, parity, what=2):
    """A packed block of nrhs random fields, packed one field at a time."""
    prec = PREC[c["sp"]]
    out = ndq.SpinorField(g, prec, parity, nrhs)
    per = out.buf.numel() // nrhs
    for r in range(nrhs):
        one = ndq.SpinorField.pack(g, _field(out.nsites, seed, what + r), prec, parity)
        out.buf[r * per:(r + 1) * per].copy_(one.buf)
    return out


# ---- what a program has in hand -------------------------------------------------

def prepare(case, seed):
    c = case
    v = _volume(c)
    g = ndq.Geometry(_dims_of(c))
    op = c["op"]
    s = {"op": op, "g": g, "sp": c["sp"]}
    if op == "gram":
        s["a"] = _pack(g, c, seed, c["nrhs"], ndq.FULL, 2)
        s["b"] = _pack(g, c, seed, c["nrhs"], ndq.FULL, 200)
        return s
    links = _links(v, seed)
    if op == "grad":
        s["psi"] = _field(v, seed, 2).requires_grad_(True)
        s["links"] = links.requires_grad_(True)
        return s
    s["U"] = ndq.GaugeField.pack(g, links, PREC[c["lp"]], c["recon"])
    if op == "solve":
        s["Ulo"] = ndq.GaugeField.pack(g, links, ndq.F32, 12)
        s["x"] = _pack(g, c, seed, c["nrhs"], ndq.FULL)
        s["y"] = s["x"].like()
        s["ov"] = ndq.Overlap(g, M, ndq.Approx.from_coeffs(ndq.MINMAX_POLY, _coeffs(EPS, 143), lo=EPS), LAM, mq=MQ)
        s["ovlo"] = ndq.Overlap(g, M, ndq.Approx.from_coeffs(ndq.MINMAX_POLY, _coeffs(EPS, c["degree"]), lo=EPS), LAM,
                                mq=MQ)
        return s
    del links
    s["x"] = _pack(g, c, seed, c["nrhs"], ndq.ODD if op == "dslash" else ndq.FULL)
    s["y"] = s["x"].like(ndq.EVEN if op == "dslash" else ndq.FULL)
    if op in ("sign", "dn"):
        modes, sg = _modes(v, c["nev"], seed)
        s["modes"] = ndq.SpinorField.pack(g, modes, ndq.F64, ndq.FULL)
        s["ov"] = ndq.Overlap(g, M, ndq.Approx.from_coeffs(ndq.MINMAX_POLY, _coeffs(EPS, c["degree"]), lo=EPS), LAM,
                              modes=s["modes"], nu=0.6 * sg, mq=MQ,
                              form=ndq.SANDWICH if c["sandwich"] else ndq.LITERAL)
        s["ov"].workspace(PREC[c["sp"]], ndq.ndq.OP_SIGN if op == "sign" else ndq.ndq.OP_DN, c["nrhs"])
    return s


def _numbers(f, sp):
    """The numbers a packed block holds, field 0 apart from the rest, in the type of its storage."""
    rows = f.buf.view(f.nrhs, -1)
    if sp == "f16":     # three planes of scaled halves and the scales
        cut = 48 * f.nsites
        parts = [rows[:, :cut].view(torch.float16), rows[:, cut:].view(torch.float32)]
    else:
        parts = [rows.view(torch.float64 if sp == "f64" else torch.float32)]
    return [p[a:b] for p in parts for a, b in ((0, 1), (1, f.nrhs)) if b > a]


def run(state):
    s = state
    op, g = s["op"], s["g"]
    if op == "q":
        ndq.apply_Q(g, s["U"], M, s["x"], s["y"])
    elif op == "dslash":
        ndq.apply_dslash(g, s["U"], s["x"], s["y"])
    elif op == "sign":
        ndq.apply_sign(g, s["U"], s["ov"], s["x"], s["y"])
    elif op == "dn":
        ndq.apply_DN(g, s["U"], s["ov"], s["x"], s["y"])
    elif op == "solve":
        s["y"].buf.zero_()
        ndq.solve_DN(g, s["U"], s["ov"], s["x"], s["y"], tol=1e-11, U_lo=s["Ulo"], ov_lo=s["ovlo"], inner_prec=ndq.F32)
    elif op == "grad":
        s["psi"].grad = s["links"].grad = None
        y = ndq.QFunction.apply(s["psi"], s["links"], g, M)
        torch.view_as_real(y).square().sum().backward()
        return [y.detach(), s["psi"].grad, s["links"].grad]
    else:
        return ndq.spinor_gram(g, s["a"], s["b"])
    return _numbers(s["y"], s["sp"])


# ---- what a pass cannot do without -------------------------------------------------

def work(case):
    c = case
    v, r = _volume(c), c["nrhs"]
    sb, lb = SPINOR_BYTES[c["sp"]], c["recon"] * REAL_BYTES[c["lp"]]
    op = c["op"]
    if op == "dslash":
        return {"bytes": v // 2 * (8 * lb + 2 * r * sb), "flops": 1320 * (v // 2) * r}
    q = 1368 * v * r    # Q: the hopping term, the site term and the sum
    if op == "q":
        return {"bytes": v * (4 * lb + 2 * r * sb), "flops": q}
    if op in ("sign", "dn"):
        # fields, links and modes once, the operations of 2 n + 1 applies and of the projection
        n, e = c["degree"], c["nev"]
        return {"bytes": v * (4 * lb + 2 * r * sb + 192 * e), "flops": (2 * n + 1) * q + 4 * 96 * v * e * r}
    if op == "solve":
        # one residual of the FP64 operator per right-hand side is the least there is; the
        # iteration count follows from the data
        return {"bytes": v * (4 * lb + 2 * r * sb), "flops": 2 * 287 * q}
    if op == "grad":
        # read psi and the links, write y and the two gradients, canonical complex128
        return {"bytes": v * (2 * 576 + 3 * 192), "flops": 2 * q + 4 * 2200 * v}
    return {"bytes": 2 * v * 192 * r + 16 * r * r, "flops": 96 * v * r * r}


# ---- the same in 64 bits with plain torch ---------------------------------------------

def _spin(mu):
    """The 2 x 2 block A_mu of gamma_mu = [[0, A], [A^H, 0]]: A_0 = -1, A_k = -i sigma_k."""
    m = [[[-1, 0], [0, -1]], [[0, -1j], [-1j, 0]], [[0, -1], [1, 0]], [[-1j, 0], [0, 1j]]][mu]
    return m


def _spin_mul(m, x):
    """(m x)_s = sum_t m[s][t] x_t on the spin axis (-2) of a two-spinor."""
    return torch.stack([sum(m[s][t] * x[..., t, :] for t in (0, 1) if m[s][t] != 0) for s in (0, 1)], dim=-2)


def _dag(m):
    return [[complex(m[t][s]).conjugate() for t in (0, 1)] for s in (0, 1)]


def _neg(m):
    return [[-m[s][t] for t in (0, 1)] for s in (0, 1)]


def _col(u, h):
    """u[v, 3, 3] on the colour axis of h[..., v, 2, 3]."""
    out = u[..., None, :, 0] * h[..., 0, None]
    out += u[..., None, :, 1] * h[..., 1, None]
    out += u[..., None, :, 2] * h[..., 2, None]
    return out


def _shift(x, dims, mu, sign):
    """x at the neighbour x + sign * mu; site axis first or second from the left of a spinor block."""
    lead = x.shape[:-3]
    y = x.reshape(lead + tuple(dims) + x.shape[-2:])
    return torch.roll(y, -sign, dims=len(lead) + mu).reshape(x.shape)


def _hop(u, psi, dims):
    """H psi = sum_mu U (1 - gamma_mu) psi(x + mu) + U^H(x - mu) (1 + gamma_mu) psi(x - mu); psi [..., v, 4, 3]."""
    out = torch.zeros_like(psi)
    for mu in range(4):
        a = _spin(mu)
        um = u[:, mu]
        p = _shift(psi, dims, mu, 1)
        h = _col(um, p[..., :2, :] - _spin_mul(a, p[..., 2:, :]))
        out[..., :2, :] += h
        out[..., 2:, :] += _spin_mul(_neg(_dag(a)), h)
        h = _col(um.conj().transpose(-1, -2), psi[..., :2, :] + _spin_mul(a, psi[..., 2:, :]))
        h = _shift(h, dims, mu, -1)
        out[..., :2, :] += h
        out[..., 2:, :] += _spin_mul(_dag(a), h)
    return out


def _q64(u, psi, dims):
    d = (4.0 + M) * psi - 0.5 * _hop(u, psi, dims)
    d[..., 2:, :] *= -1.0
    return d


def _sign64(u, x, c, dims, modes, sg):
    """Eq. 11 with the polynomial of _coeffs: the forward Chebyshev recurrence on Z = (2 X^2 - 1 - e) / (1 - e)."""
    def z(f):
        q2 = _q64(u, _q64(u, f, dims), dims)
        return (2.0 / (LAM * LAM) * q2 - (1.0 + EPS) * f) / (1.0 - EPS)

    def proj(f, w):
        d = modes.reshape(len(sg), -1).conj() @ f.reshape(-1)
        return ((d * w) @ modes.reshape(len(sg), -1)).reshape(f.shape)

    sgt = torch.as_tensor(sg, device=DEV, dtype=torch.complex128)
    one = torch.ones_like(sgt)
    src = x - proj(x, one) if c["sandwich"] else x
    co = _coeffs(EPS, c["degree"])
    t0, t1 = src, z(src)
    acc = co[0] * t0 + co[1] * t1
    for k in range(2, len(co)):
        t0, t1 = t1, 2.0 * z(t1) - t0
        acc += co[k] * t1
    t = _q64(u, acc, dims) / LAM
    return t - proj(t, one) + proj(x, sgt)


def _packed(x, dims, sp, parity):
    """A canonical field [v, 4, 3] in the order of the packed storage, as _numbers gives it (one field)."""
    n = x.shape[0]
    if parity == ndq.FULL:
        i = torch.arange(n, device=DEV)
        p = (i + i // dims[3] + i // (dims[3] * dims[2]) + i // (dims[3] * dims[2] * dims[1])) % 2
        x = torch.cat([x[p == 0], x[p == 1]])
    r = torch.view_as_real(x.reshape(n, 12)).reshape(n, 24)
    words = {"f64": 2, "f32": 4, "f16": 8}[sp]
    out = []
    if sp == "f16":
        big = r.abs().amax(1, keepdim=True)
        r = r / big
        out = [big.reshape(1, -1)]
    return [r.reshape(n, 24 // words, words).permute(1, 0, 2).reshape(1, -1)] + out


def _inputs64(c, seed, r=0, parity=ndq.FULL):
    """Field r as the packed storage holds it (rounded to it), canonical complex128."""
    n = _volume(c) // (1 if parity == ndq.FULL else 2)
    x = _field(n, seed, 2 + r)
    if c["sp"] == "f32":
        x = x.to(torch.complex64).to(torch.complex128)
    elif c["sp"] == "f16":
        f = torch.view_as_real(x).to(torch.float32)
        big = f.abs().amax((1, 2, 3), keepdim=True)
        f = (f * (1.0 / big)).to(torch.float16).to(torch.float64) * big
        x = torch.view_as_complex(f.contiguous())
    return x


def _links64(c, seed):
    """The links as the packed storage holds them."""
    u = _links(_volume(c), seed)
    if c["recon"] == 8:
        return u
    t = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16}[c["lp"]]
    u = torch.view_as_complex(torch.view_as_real(u).to(t).to(torch.float64).contiguous())
    if c["recon"] == 12:
        u[..., 2] = torch.linalg.cross(u[..., 0].contiguous(), u[..., 1].contiguous()).conj()
    return u


def exact(case, seed):
    c = case
    dims, op = _dims_of(c), c["op"]
    v = _volume(c)
    if op == "solve":
        return None
    if op == "gram":
        a = torch.stack([_field(v, seed, 2 + k).reshape(-1) for k in range(c["nrhs"])])
        b = torch.stack([_field(v, seed, 200 + k).reshape(-1) for k in range(c["nrhs"])])
        return a.conj() @ b.t()
    if op == "grad":
        u = _links(v, seed)
        psi = _field(v, seed, 2)
        y = _q64(u, psi, dims)
        gy = 2.0 * y
        chi = gy.clone()
        chi[..., 2:, :] *= -1.0
        gu = torch.empty_like(u)
        for mu in range(4):
            a = _spin(mu)
            sf, cf = _shift(psi, dims, mu, 1), _shift(chi, dims, mu, 1)
            h = sf[..., :2, :] - _spin_mul(a, sf[..., 2:, :])
            h = torch.cat([h, _spin_mul(_neg(_dag(a)), h)], dim=-2)          # (1 - gamma) psi(x + mu)
            k = psi[..., :2, :] + _spin_mul(a, psi[..., 2:, :])
            k = torch.cat([k, _spin_mul(_dag(a), k)], dim=-2)                # (1 + gamma) psi(x)
            hm = (h[..., :, :, None] * chi[..., :, None, :].conj()).sum(-3)
            km = (k[..., :, :, None] * cf[..., :, None, :].conj()).sum(-3)
            um = u[:, mu]
            gm = _mm(um, hm) - _mm(km, um.conj().transpose(-1, -2))
            # F^a = 1/2 Im tr(T_a G); 2 sum_a F^a T_a is half the traceless part of (G - G^H) / 2i
            an = (gm - gm.conj().transpose(-1, -2)) / 2j
            tr = (an[..., 0, 0] + an[..., 1, 1] + an[..., 2, 2]) / 3.0
            an = an - tr[..., None, None] * torch.eye(3, dtype=torch.complex128, device=DEV)
            gu[:, mu] = _mm(0.5j * an, um)
        return [y, _q64(u, gy, dims), gu]
    u = _links64(c, seed)
    parity = ndq.FULL
    if op == "dslash":
        # the odd field on its sites of the whole lattice, zero on the even ones
        parity = ndq.EVEN
        i = torch.arange(v, device=DEV)
        p = (i + i // dims[3] + i // (dims[3] * dims[2]) + i // (dims[3] * dims[2] * dims[1])) % 2
        full = torch.zeros((v, 4, 3), dtype=torch.complex128, device=DEV)
        full[p == 1] = _inputs64(c, seed, 0, ndq.ODD)
        y = _hop(u, full, dims)[p == 0]
    elif op == "q":
        y = _q64(u, _inputs64(c, seed), dims)
    else:
        modes, sg = _modes(v, c["nev"], seed)
        x = _inputs64(c, seed)
        y = _sign64(u, x, c, dims, modes, sg)
        if op == "dn":
            y[..., 2:, :] *= -1.0
            y = (-M - 0.5 * MQ) * (x + y) + MQ * x
    out = _packed(y, dims, c["sp"], parity)
    # field 0 alone; the other fields of a block hold the same operation
    return [w for o in out for w in ((o, None) if c["nrhs"] > 1 else (o,))]

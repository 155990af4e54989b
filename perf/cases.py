"""The work that users of lq have it do, as cases that can be timed.

Two calls carry the library: `lq_solve` (a propagator: D x = b for a batch of
sources, the reason the library exists) and `lq_apply` (one operator on a batch
of columns, for programs with their own outer loop).  The listed cases take both
over the lattices, column counts, precisions and actions of this repository's
benchmark, serving mix and tests; `draw` gives others of the same ranges.

A case is a dict of plain values:
  call    "apply" or "solve"
  action  "wilson", "tm" (twisted clover), "hisq" or "overlap"
  lx, ly, lz, lt   even extents
  cols    right-hand sides in one call
  apply:  op ("d", "ddag", "hop", "schur", "normal_even", "hw", "sign"), prec
          (storage 64, 32 or 16), order (Chebyshev order of "sign")
  solve:  sloppy (storage of the inner iterations), tol, masses (HISQ), mg
          (multigrid GCR), full (HISQ: all sites of the solution)

Every run takes device tensors and returns what the call computed, whole.  Calls
at FP32 and FP16 storage hand their result back in that storage (complex64, or
pairs of float16), as a program does that keeps its vectors at the precision at
which it had them computed.
"""
import math

import torch

from paper_2201_09004_amd import lq

DEV = "cuda:0"
# Parameters of the benchmark workloads: twisted clover (24^3 x 64), HISQ
# (32^3 x 96, masses 0.002 ... 0.05), overlap (rho 1.5), Wilson (kappa 0.12).
TM = {"m": -0.0695, "mu": 0.01, "c_sw": 1.0509}
WILSON_M = 1.0 / (2 * 0.12) - 4.0
RHO, OVERLAP_M = 1.5, 0.015
# Interval that holds the spectrum of H_W^2 on links exp(0.2 i H): |H_W| <= 8 - rho
# always, and the lower edge stays above 0.25 on such fields.
CHEB_A, CHEB_B = 0.2, 42.5
HISQ_M0, HISQ_M1 = 0.002, 0.05
NVEC, NU_POST, GCR_KMAX = 30, 4, 8

_CTX = []


def ctx():
    if not _CTX:
        _CTX.append(lq.lq_init(0))
    return _CTX[0]


def _case(name, call, action, L, cols, **kw):
    c = {"call": call, "action": action, "lx": L[0], "ly": L[1], "lz": L[2], "lt": L[3], "cols": cols, **kw}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one column, one operator, where latency is all (the smallest lattice of the tests
        # that is also a benchmark workload)
        _case("tm_d_8x8x8x8", "apply", "tm", (8, 8, 8, 8), 1, op="d", prec=64),
        # a program's own Krylov loop on an odd-shaped lattice: D^dag for a batch that no register block divides
        _case("wilson_ddag_ragged", "apply", "wilson", (6, 10, 14, 18), 5, op="ddag", prec=64),
        # the operator of the twisted-clover benchmark at its full size, in its inner precision
        _case("tm_schur_24x24x24x64", "apply", "tm", (24, 24, 24, 64), 12, op="schur", prec=32),
        # staggered: one time slice's colours for several times on a ragged lattice in half storage ...
        _case("hisq_d_ragged", "apply", "hisq", (12, 20, 14, 36), 7, op="d", prec=16),
        # ... and the even normal operator of the HISQ benchmark at its full size
        _case("hisq_normal_32x32x32x96", "apply", "hisq", (32, 32, 32, 96), 12, op="normal_even", prec=32),
        # the sign function, all of an overlap propagator's cost: order 200 in half storage on the benchmark lattice
        _case("overlap_sign_24x24x24x64", "apply", "overlap", (24, 24, 24, 64), 12, op="sign", prec=16, order=200),
        # the smallest solve: CG on the normal equations, one column (the Wilson workload of the benchmark)
        _case("wilson_cgne_8x8x8x8", "solve", "wilson", (8, 8, 8, 8), 1, sloppy=64, tol=1e-12),
        # a staggered propagator of the serving mix: three colour columns, one mass
        _case("hisq_16x16x16x32", "solve", "hisq", (16, 16, 16, 32), 3, sloppy=16, tol=1e-11, masses=1, full=0),
        # a twisted-clover propagator of the serving mix: twelve spin-colour columns, BiCGStab
        _case("tm_bicgstab_16x16x16x32", "solve", "tm", (16, 16, 16, 32), 12, sloppy=32, tol=1e-12, mg=0),
        # the benchmark propagator on a gauge field with a multigrid setup
        _case("tm_mg_24x24x24x64", "solve", "tm", (24, 24, 24, 64), 12, sloppy=32, tol=1e-12, mg=1),
        # the HISQ workload of the benchmark, eight masses at once, on its smaller serving lattice
        _case("hisq_8masses_24x24x24x64", "solve", "hisq", (24, 24, 24, 64), 12, sloppy=16, tol=1e-11, masses=8,
              full=0),
    ]


def draw(rng):
    def extents(sites, lo=4, hi=32):
        """Four even extents with about that many sites."""
        side = sites ** 0.25
        L = []
        for _ in range(3):
            v = 2 * round(side * math.exp(rng.uniform(-0.4, 0.4)) / 2)
            L.append(min(hi, max(lo, v)))
        v = 2 * round(sites / (L[0] * L[1] * L[2]) / 2)
        return L + [min(96, max(lo, v))]

    def log_uniform(a, b):
        return math.exp(rng.uniform(math.log(a), math.log(b)))

    kind = rng.choice(["apply", "apply", "apply", "apply", "sign", "wilson", "tm", "mg", "hisq", "hisq"])
    if kind == "apply":
        action, op = rng.choice([("wilson", "d"), ("wilson", "ddag"), ("wilson", "hop"), ("tm", "d"), ("tm", "ddag"),
                                 ("tm", "schur"), ("hisq", "d"), ("hisq", "hop"), ("hisq", "normal_even"),
                                 ("overlap", "hw")])
        prec = rng.choice([64, 32] if action == "tm" else [64, 32, 16])
        cols = rng.randint(1, 13)
        return _case(None, "apply", action, extents(log_uniform(3000, 7e5)), cols, op=op, prec=prec)
    if kind == "sign":
        return _case(None, "apply", "overlap", extents(log_uniform(4000, 2e5)), rng.randint(1, 12), op="sign",
                     prec=rng.choice([64, 32, 16]), order=rng.randint(20, 120))
    if kind == "wilson":
        return _case(None, "solve", "wilson", extents(log_uniform(1500, 1e5)), rng.randint(1, 6),
                     sloppy=rng.choice([64, 32, 16]), tol=1e-12)
    if kind == "tm":
        return _case(None, "solve", "tm", extents(log_uniform(4000, 1.6e5)), rng.randint(1, 12),
                     sloppy=rng.choice([64, 32, 32]), tol=1e-12, mg=0)
    if kind == "mg":
        L = [rng.choice([8, 16, 24]) for _ in range(3)] + [rng.choice([16, 24, 32])]
        return _case(None, "solve", "tm", L, rng.randint(1, 12), sloppy=32, tol=1e-12, mg=1)
    return _case(None, "solve", "hisq", extents(log_uniform(6000, 3e5)), rng.randint(1, 9),
                 sloppy=rng.choice([64, 32, 16, 16]), tol=1e-11, masses=rng.choice([1, 1, 2, 3, 5, 8]),
                 full=rng.choice([0, 1]))


# ------------------------------------------------------------------ inputs
def _extents(c):
    return (c["lx"], c["ly"], c["lz"], c["lt"])


def _volume(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _nc(c):
    return 3 if c["action"] == "hisq" else 12


def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + salt)


def _links(V, eps, g, with_trace=False):
    """V x 4 links exp(i eps H), H = sum_a h_a lambda_a / 2 (plus h_0 / sqrt 6 for U(3)), h ~ N(0, 1).  They are
    drawn from 32768 such matrices, which keeps the preparation short."""
    n = 32768
    h = torch.randn(n, 9, dtype=torch.float64, device=DEV, generator=g)
    H = torch.zeros(n, 3, 3, dtype=torch.complex128, device=DEV)
    for k, (i, j) in enumerate([(0, 1), (0, 2), (1, 2)]):
        z = torch.complex(h[:, 2 * k], -h[:, 2 * k + 1]) / 2
        H[:, i, j], H[:, j, i] = z, z.conj()
    d3, d8 = h[:, 6] / 2, h[:, 7] / (2 * math.sqrt(3.0))
    tr = h[:, 8] / math.sqrt(6.0) if with_trace else torch.zeros_like(d3)
    for i, v in enumerate((d3 + d8, d8 - d3, -2 * d8)):
        H[:, i, i] = torch.complex(v + tr, torch.zeros_like(v))
    w, Q = torch.linalg.eigh(H.cpu())
    pool = ((Q * torch.exp(1j * eps * w)[:, None, :]) @ Q.mH).to(DEV)
    at = torch.randint(n, (V * 4,), device=DEV, generator=g)
    return pool[at].reshape(V, 4, 3, 3)


class Field:
    """A resident gauge field, freed with its last user."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        lq.lq_field_free(self.handle)


def _gauge(c, seed):
    """The links of a case: (U,) or, for HISQ, (fat, long)."""
    V = _volume(c)
    if c["action"] == "hisq":
        return (_links(V, 0.1, _gen(seed, 1)), _links(V, 0.2, _gen(seed, 2), True) * (-1.0 / 24.0))
    return (_links(V, 0.3 if c["action"] == "wilson" else 0.2, _gen(seed, 1)),)


def _columns(c, seed):
    """Gaussian columns for an operator; point sources at a random site for a solve (Gaussian ones for the Wilson
    workload), on even sites for HISQ, whose solver works there."""
    V, nc = _volume(c), _nc(c)
    shape = (c["cols"], V, 3) if nc == 3 else (c["cols"], V, 4, 3)
    g = _gen(seed, 3)
    if c["call"] == "apply" or c["action"] == "wilson":
        return torch.randn(shape, dtype=torch.complex128, device=DEV, generator=g)
    b = torch.zeros((c["cols"], V, nc), dtype=torch.complex128, device=DEV)
    for k in range(c["cols"]):
        x, y, z, t = (int(torch.randint(n, (1,), device=DEV, generator=g)) for n in _extents(c))
        x = (x // 2) * 2 + (y + z + t) % 2
        s = x + c["lx"] * (y + c["ly"] * (z + c["lz"] * t))
        b[k, s, k % nc] = 1.0
    return b.reshape(shape)


def _masses(c):
    n = c["masses"]
    return [HISQ_M0 * (HISQ_M1 / HISQ_M0) ** (k / (n - 1)) for k in range(n)] if n > 1 else [0.01]


def _action(c):
    if c["action"] == "wilson":
        return lq.action(lq.LQ_WILSON, m=WILSON_M)
    if c["action"] == "tm":
        return lq.action(lq.LQ_TM_CLOVER, **TM)
    if c["action"] == "hisq":
        return lq.action(lq.LQ_HISQ, m=_masses(c)[0] if c["call"] == "solve" else 0.01)
    return lq.action(lq.LQ_OVERLAP, m=OVERLAP_M, rho=RHO, cheb_N=c.get("order", 1), cheb_a=CHEB_A, cheb_b=CHEB_B)


OPS = {"d": lq.LQ_OP_D, "ddag": lq.LQ_OP_DDAG, "hop": lq.LQ_OP_HOP, "schur": lq.LQ_OP_SCHUR,
       "normal_even": lq.LQ_OP_NORMAL_EVEN, "hw": lq.LQ_OP_HW, "sign": lq.LQ_OP_SIGN}


def prepare(case, seed):
    """A resident gauge field with what belongs to it (multigrid setup, measured spectrum of H_W) and the sources."""
    c, L = case, _extents(case)
    links = _gauge(c, seed)
    load = lq.lq_hisq_load if c["action"] == "hisq" else lq.lq_gauge_load
    field = Field(load(ctx(), L, *links))
    act = _action(c)
    if c.get("mg"):
        lq.lq_mg_setup(ctx(), act, field.handle, lq.mg_params(n_vec=NVEC, nu_post=NU_POST, gcr_kmax=GCR_KMAX, seed=seed + 1))
    if c.get("op") == "sign":
        # the library measures the spectrum of H_W once per field
        one = lq.action(lq.LQ_OVERLAP, m=OVERLAP_M, rho=RHO, cheb_N=1, cheb_a=CHEB_A, cheb_b=CHEB_B)
        lq.lq_apply(ctx(), one, field.handle, lq.LQ_OP_SIGN, 64,
                    torch.ones((1, _volume(c), 4, 3), dtype=torch.complex128, device=DEV))
    return {"case": c, "field": field, "action": act, "b": _columns(c, seed)}


def run(state):
    c = state["case"]
    if c["call"] == "apply":
        out = lq.lq_apply(ctx(), state["action"], state["field"].handle, OPS[c["op"]], c["prec"], state["b"])
        if c["prec"] == 64:
            return out
        return out.to(torch.complex64) if c["prec"] == 32 else torch.view_as_real(out).to(torch.float16)
    masses = _masses(c) if c["action"] == "hisq" and c["masses"] > 1 else None
    prm = lq.params(tol=c["tol"], sloppy_bits=c["sloppy"], masses=masses, reconstruct_full=c.get("full", 0),
                    solver=3 if c.get("mg") else 0)
    x, st = lq.lq_solve(ctx(), state["action"], state["field"].handle, prm, state["b"])
    if st["status"] != 0:
        raise RuntimeError(f"the solve ended with status {st['status']}")
    return x


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Bytes and flops of one pass.

    An operator reads its links, site matrices and input columns once and writes its output once, in the caller's
    FP64 layout on the outside (the input and output tensors) and without any intermediate.  A solve counts, per
    iteration, each link and site matrix and the columns that every matrix product must read and write in the inner
    precision, plus the least vector traffic of its recurrence, times a typical number of iterations of these
    ensembles (counted once on the listed sizes)."""
    c = case
    V, n, nc = _volume(c), c["cols"], _nc(c)
    dof = 2 * nc
    site_flops = 1146.0 if nc == 3 else 1320.0
    if c["call"] == "apply":
        rb = c["prec"] / 8
        links = V * 4 * 18 * rb * (2 if nc == 3 else 1)
        clov = V * 72 * rb if c["action"] == "tm" else 0
        half = 0.5 if c["op"] in ("schur", "normal_even") else 1.0
        io = V * n * dof * 8 * (1 + half)  # the whole output is written, zeros among it
        if c["op"] == "sign":
            per = V * (4 * 18 + 4 * n * dof) * rb
            return {"bytes": io + c["order"] * 2 * per, "flops": (2 * c["order"] + 1) * V * n * site_flops}
        flops = V * n * site_flops + (V * n * 576 if c["op"] == "schur" else 0)
        return {"bytes": links + (2 if c["op"] == "schur" else 1) * clov + io, "flops": flops}
    rb = c["sloppy"] / 8
    if c["action"] == "wilson":
        its, mats, vecs = 150, 2 * V * 8 * 18 / 2 * rb, 2 * 2 + 8
        flops = its * 2 * V * n * site_flops
    elif c["action"] == "tm":
        # multigrid: fine-level products of its steps only
        its = 20 * 6 if c["mg"] else 480
        mats, vecs = 2 * V * (8 * 18 + 144) / 2 * rb, (2 * 2 + (4 if c["mg"] else 13)) / 2
        flops = its * 2 * V * n * (site_flops + 576) / 2 * 2
    else:
        its, mats = 450, 2 * V * 16 * 18 / 2 * rb
        vecs = (2 + 2 + 8) / 2 * (c["masses"] if c["masses"] > 1 else 1)
        flops = its * V * n * site_flops
    return {"bytes": its * (mats + V * n * dof * rb * vecs), "flops": flops}


# ------------------------------------------------------------------ the same in plain torch, FP64
AXIS = {0: 3, 1: 2, 2: 1, 3: 0}


def _grid(c, f):
    """[V, ...] as [t, z, y, x, ...]."""
    return f.reshape((c["lt"], c["lz"], c["ly"], c["lx"]) + tuple(f.shape[1:]))


def _shift(f, mu, k):
    """f(x + k mu), periodic."""
    return torch.roll(f, -k, dims=AXIS[mu])


def _mul(U, v):
    """Colour matrix on the last index of v [..., spin, colour]."""
    return torch.stack([sum(U[..., a, b, None] * v[..., b] for b in range(3)) for a in range(3)], dim=-1)


def _mul_dag(U, v):
    return torch.stack([sum(U[..., b, a, None].conj() * v[..., b] for b in range(3)) for a in range(3)], dim=-1)


def _gammas():
    s = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=torch.complex128)
    g = torch.zeros(4, 4, 4, dtype=torch.complex128)
    for k in range(3):
        g[k, :2, 2:], g[k, 2:, :2] = -1j * s[k], 1j * s[k]
    g[3, :2, 2:] = g[3, 2:, :2] = torch.eye(2)
    return g


def _spin(G, v):
    """Spin matrix with few entries on v [..., spin, colour]."""
    rows = []
    for i in range(4):
        r = 0
        for j in range(4):
            if G[i, j] != 0:
                r = r + complex(G[i, j]) * v[..., j, :]
        rows.append(r if not isinstance(r, int) else torch.zeros_like(v[..., 0, :]))
    return torch.stack(rows, dim=-2)


def _fermion_links(c, U):
    """The links of every direction with the antiperiodic sign on the last time slice."""
    W = [U[..., mu, :, :].clone() for mu in range(4)]
    W[3][-1] *= -1
    return W


def _wilson_hop(W, v):
    """sum_mu (1 - g_mu) U_mu(x) v(x + mu) + (1 + g_mu) U_mu^dag(x - mu) v(x - mu)."""
    out = torch.zeros_like(v)
    for mu, G in enumerate(_gammas()):
        f, b = _mul(W[mu], _shift(v, mu, 1)), _shift(_mul_dag(W[mu], v), mu, -1)
        out += f + b + _spin(G, b - f)
    return out


def _g5(v):
    return torch.cat([v[..., :2, :], -v[..., 2:, :]], dim=-2)


def _site_matrix(U):
    """(4 + m) + C + i mu g5 as 12 x 12 matrices, C = -(c_sw / 2) sum_{mu<nu} g_mu g_nu F_mu_nu."""
    g = _gammas().to(U.device)
    A = torch.zeros(U.shape[:4] + (4, 3, 4, 3), dtype=torch.complex128, device=U.device)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            am, bm = _shift(a, mu, -1), _shift(b, nu, -1)
            q = a @ _shift(b, mu, 1) @ _shift(a, nu, 1).mH.contiguous() @ b.mH.contiguous()
            q = q + b @ _shift(am, nu, 1).mH.contiguous() @ _shift(b, mu, -1).mH.contiguous() @ am
            q = q + am.mH.contiguous() @ _shift(bm, mu, -1).mH.contiguous() @ _shift(am, nu, -1) @ bm
            q = q + bm.mH.contiguous() @ _shift(a, nu, -1) @ _shift(bm, mu, 1) @ a.mH.contiguous()
            F = (q - q.mH) / 8
            F = F - torch.diagonal(F, dim1=-2, dim2=-1).sum(-1)[..., None, None] / 3 * torch.eye(3, device=U.device)
            S = g[mu] @ g[nu]
            for i in range(4):
                for j in range(4):
                    if S[i, j] != 0:
                        A[..., i, :, j, :] += -0.5 * TM["c_sw"] * S[i, j] * F
    A = A.reshape(U.shape[:4] + (12, 12))
    diag = torch.full((12,), 4 + TM["m"], dtype=torch.complex128, device=U.device)
    diag[:6] += 1j * TM["mu"]
    diag[6:] -= 1j * TM["mu"]
    return A + torch.diag(diag)


def _apply_site(A, v):
    return (A @ v.reshape(v.shape[:-2] + (12, 1))).reshape(v.shape)


def _parity(c):
    ax = [torch.arange(n, device=DEV) for n in (c["lt"], c["lz"], c["ly"], c["lx"])]
    t, z, y, x = torch.meshgrid(*ax, indexing="ij")
    return (x + y + z + t) % 2, (x, y, z, t)


def _stag_hop(c, fat, lng, v):
    _, (x, y, z, t) = _parity(c)
    eta = [1 - 2 * (n % 2) for n in (t, t + x, t + x + y, torch.zeros_like(t))]
    out = torch.zeros_like(v)
    for mu in range(4):
        for links, k in ((fat, 1), (lng, 3)):
            W = links[..., mu, :, :].clone()
            if mu == 3:
                W[-k:] *= -1
            f = _mul(W, _shift(v, mu, k))
            b = _shift(_mul_dag(W, v), mu, -k)
            out += 0.5 * eta[mu][..., None, None] * (f - b)
    return out


def exact(case, seed):
    """The operator in torch's FP64, column by column.  None for the long recursions on large lattices and for the
    solves, except the Wilson workload's, which plain CG reaches to rounding."""
    c = case
    V = _volume(c)
    if c["call"] == "solve" and (c["action"] != "wilson" or V * c["cols"] > 20000):
        return None
    if c.get("op") == "sign" and V * c["cols"] * c["order"] > 2.5e7:
        return None
    links = [_grid(c, u) for u in _gauge(c, seed)]
    b = _columns(c, seed)
    par, _ = _parity(c)
    even = (par == 0)[..., None, None]
    W = _fermion_links(c, links[0]) if c["action"] != "hisq" else None
    A = _site_matrix(links[0]) if c["action"] == "tm" else None

    def hw(v):
        return _g5((4 - RHO) * v - 0.5 * _wilson_hop(W, v))

    def wilson(v):
        return (4 + WILSON_M) * v - 0.5 * _wilson_hop(W, v)

    if c["call"] == "solve":
        def normal(v):
            return _g5(wilson(_g5(wilson(v))))
    elif c["op"] == "schur":
        A = torch.linalg.inv(A.reshape(V, 12, 12).cpu() if V < 5000 else A.reshape(V, 12, 12)).to(DEV).reshape(A.shape)

    def column(v):
        if c["call"] == "solve":
            rhs = _g5(wilson(_g5(v)))
            x, r = torch.zeros_like(v), rhs.clone()
            p, rr = r.clone(), float((r.abs() ** 2).sum())
            stop = rr * 1e-30
            for _ in range(2000):
                q = normal(p)
                a = rr / float((p.conj() * q).sum().real)
                x, r = x + a * p, r - a * q
                rn = float((r.abs() ** 2).sum())
                if rn < stop:
                    break
                p, rr = r + (rn / rr) * p, rn
            return x
        op = c["op"]
        if c["action"] == "hisq":
            h = lambda u: _stag_hop(c, links[0], links[1], u)  # noqa: E731
            if op == "normal_even":
                v = v * even
                return (1e-4 * v - h(h(v))) * even
            return h(v) if op == "hop" else 0.01 * v + h(v)
        if op == "hop":
            return -0.5 * _wilson_hop(W, v)
        if op == "hw":
            return hw(v)
        if op == "sign":
            N, a, e = c["order"], CHEB_A, CHEB_B
            th = [math.pi * (j + 0.5) / (N + 1) for j in range(N + 1)]
            f = [1 / math.sqrt(0.5 * (e - a) * math.cos(t) + 0.5 * (e + a)) for t in th]
            k = [2 / (N + 1) * math.fsum(math.cos(i * t) * y for t, y in zip(th, f)) for i in range(N + 1)]
            b1, b2 = torch.zeros_like(v), torch.zeros_like(v)
            for i in range(N, 0, -1):
                z = (2 * hw(hw(b1)) - (a + e) * b1) / (e - a)
                b1, b2 = k[i] * v + 2 * z - b2, b1
            y = 0.5 * k[0] * v + (2 * hw(hw(b1)) - (a + e) * b1) / (e - a) - b2
            return hw(y)
        if op == "schur":
            v = v * even
            t = _apply_site(A, -0.5 * _wilson_hop(W, v)) * ~even
            return v - _apply_site(A, -0.5 * _wilson_hop(W, t)) * even
        dag = op == "ddag"
        if c["action"] == "wilson":
            return _g5(wilson(_g5(v))) if dag else wilson(v)
        B = A.mH.contiguous() if dag else A
        hop = _g5(_wilson_hop(W, _g5(v))) if dag else _wilson_hop(W, v)
        return _apply_site(B, v) - 0.5 * hop

    out = torch.empty_like(b)
    for k in range(c["cols"]):
        v = _grid(c, b[k])
        if c["action"] == "hisq":
            v = v[..., None, :]
        out[k] = column(v).reshape(b[k].shape)
    if c["call"] == "apply" and c["prec"] != 64:
        return torch.view_as_real(out).contiguous() if c["prec"] == 16 else out
    return out

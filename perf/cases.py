"""Timed workloads of the twisted-mass loop library, through its Python binding.

Every case is one call (or the one call chain) that a program measuring
disconnected loops makes on a resident gauge field:

  dslash    tm_dslash_ex: one operator on a batch of right-hand sides
  update    tm_cg_update: the CG direction update on a batch of fields
  contract  tm_contract: spin matrices of given solutions with their Z4 noise
  solve     tm_cg_solve: even-odd CG for a batch of sources
  loops     tm_loops_tsm: the truncated-solver estimate of the 90 loop operators

Lattices are those of the benchmark and the tests (4^4 to 32^3 x 64) and
ragged ones with even extents that are not powers of two.  ``exact`` computes
the same quantities in 64 bits with plain torch.

Solves and loops end in double precision, but a low-precision solve carries
only the rounding of 16-bit storage; the case of such a solve keeps its
solutions in half precision, as a program does that stores many of them.
"""
import math

import torch

from paper_1401_6749_amd import tm

EPS = 0.4          # disorder of the synthetic links, as in the benchmark's inputs
KAPPA, TWO_KAPPA_MU = 0.1636, 0.0033
LINK_BYTES = {"f64": 96, "f32": 48, "f16": 24, "bf16": 24}   # two rows of a link
SPIN_BYTES = {"f64": 192, "f32": 96, "f16": 52, "bf16": 52}  # a spinor (halves: with its scale)
HOP_FLOPS = 1320   # eight projected SU(3) products and their sum, per output site
HALF_FAMILY = ("mhat", "mhat_dag", "mhat_dag_mhat")          # act on the even sites


def _case(kind, dims, prec, nrhs, **more):
    c = {"kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3], "prec": prec, "nrhs": nrhs,
         "kappa": KAPPA, "mu": TWO_KAPPA_MU, "t_bc": -1}
    c.update(more)
    return c


def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def listed():
    named = [
        # the hop of every low-precision CG iteration at the benchmark's lattice and batch
        ("hop_f16_32c64_x12", _case("dslash", (32, 32, 32, 64), "f16", 12, op="hop")),
        # bfloat16 storage, a lattice with no power-of-two extent and a partly filled batch
        ("mdag_bf16_ragged_x5", _case("dslash", (12, 10, 14, 18), "bf16", 5, op="mdag")),
        # the operator that the FP32 part of a mixed high-precision solve iterates
        ("mdagm_f32_24c48_x12", _case("dslash", (24, 24, 24, 48), "f32", 12, op="mhat_dag_mhat")),
        # one FP64 application for one source: residual checks, a program's own solver
        ("m_f64_16c32_x1", _case("dslash", (16, 16, 16, 32), "f64", 1, op="m")),
        # the smallest lattice of the tests: launches and latency only
        ("mhat_f64_4c4_x1", _case("dslash", (4, 4, 4, 4), "f64", 1, op="mhat")),
        # the vector update that ends every low-precision CG iteration
        ("update_f16_32c64_x12", _case("update", (32, 32, 32, 64), "f16", 12)),
        # contraction of a batch of low-precision solutions (widened to FP32)
        ("contract_f32_24c48_x12", _case("contract", (24, 24, 24, 48), "f32", 12)),
        # contraction of a few FP64 solutions
        ("contract_f64_16c32_x3", _case("contract", (16, 16, 16, 32), "f64", 3)),
        # plain FP64 solve of one source on a small lattice: latency of an iteration and of the call
        ("solve_f64_8c16_x1", _case("solve", (8, 8, 8, 16), "f64", 1, kappa=0.12, mu=0.01, tol=1e-10, iters=0)),
        # high-precision solves of a full batch: FP32 CG with FP64 reliable updates
        ("solve_mixed_16c32_x12", _case("solve", (16, 16, 16, 32), "mixed", 12, tol=1e-12, iters=0)),
        # low-precision solves truncated after a few iterations, kept in half precision
        ("solve_lp_24c48_x12", _case("solve", (24, 24, 24, 48), "lp", 12, tol=1e-2, iters=7)),
        # the whole estimator: mixed correction set, truncated FP64 bulk set
        ("tsm_16c32", _case("loops", (16, 16, 16, 32), "f64", 12, n_hp=4, n_lp=32, tol=1e-2)),
    ]
    return [dict(c, name=n) for n, c in named]


def _lattice(rng, most):
    """Even extents with at most `most` sites, the volume spread over its logarithm."""
    while True:
        if rng.random() < 0.5:
            l = rng.choice((4, 6, 8, 10, 12, 16, 20, 24, 28, 32))
            dims = (l, l, l, l * rng.choice((1, 2)))
        else:
            v = math.exp(rng.uniform(math.log(256), math.log(most)))
            l = v ** 0.25
            dims = tuple(max(2, 2 * round(l * math.exp(rng.uniform(-0.6, 0.6)) / 2)) for _ in range(4))
        if 256 <= dims[0] * dims[1] * dims[2] * dims[3] <= most:
            return dims


def draw(rng):
    kind = rng.choice(("dslash", "dslash", "dslash", "update", "contract", "contract", "solve", "solve", "loops"))
    more = {"kappa": round(rng.uniform(0.11, KAPPA), 4), "mu": round(10 ** rng.uniform(-2.5, -1.0), 5),
            "t_bc": rng.choice((-1, -1, 1))}
    if kind in ("dslash", "update"):
        prec = rng.choice(("f64", "f32", "f16", "bf16"))
        if kind == "dslash":
            ops = ("hop", "m", "mdag", "bh") if prec in ("f16", "bf16") else ("hop", "m", "mdag", "bh") + HALF_FAMILY
            more["op"] = rng.choice(ops)
        return _case(kind, _lattice(rng, 1 << 20), prec, rng.choice((1, 1, 2, 3, 5, 8, 12, 12, 16)), **more)
    if kind == "contract":
        return _case(kind, _lattice(rng, 1 << 19), rng.choice(("f64", "f32")), rng.choice((1, 2, 3, 6, 12, 12, 16)), **more)
    if kind == "solve":
        prec = rng.choice(("f64", "mixed", "lp"))
        more["tol"], more["iters"] = {"f64": (1e-10, 0), "mixed": (1e-12, 0), "lp": (1e-2, rng.choice((5, 7)))}[prec]
        return _case(kind, _lattice(rng, 1 << 17), prec, rng.choice((1, 1, 2, 4, 7, 12)), **more)
    return _case(kind, _lattice(rng, 1 << 16), "f64", rng.choice((1, 4, 12)), n_hp=rng.choice((2, 3, 4)),
                 n_lp=rng.randint(6, 24), tol=1e-2, **more)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _rng(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _links(dims, gen):
    """Random SU(3) links near one, [V][4][3][3] complex128 on the GPU."""
    v = dims[0] * dims[1] * dims[2] * dims[3]
    u = EPS * torch.randn(v, 4, 2, 3, dtype=torch.complex128, device="cuda", generator=gen)
    u[:, :, 0, 0] += 1
    u[:, :, 1, 1] += 1
    a = u[:, :, 0] / u[:, :, 0].norm(dim=-1, keepdim=True)
    b = u[:, :, 1] - a * (a.conj() * u[:, :, 1]).sum(-1, keepdim=True)
    b = b / b.norm(dim=-1, keepdim=True)
    return torch.stack((a, b, torch.linalg.cross(a, b).conj()), dim=2)


def _spinors(n, dims, gen):
    """n canonical spinor fields, [n][V][4][3][2] float64."""
    v = dims[0] * dims[1] * dims[2] * dims[3]
    return torch.randn(n, v, 4, 3, 2, dtype=torch.float64, device="cuda", generator=gen)


class Lattice:
    """A resident gauge field; all of a program's fields share one context."""

    ctx = None

    def __init__(self, case, links):
        if Lattice.ctx is None:
            Lattice.ctx = tm.tm_create(0)
        self.dims = _dims(case)
        prec = {"mixed": ("f32",), "lp": ("f32", "f16")}.get(case["prec"], (case["prec"],))
        if case["kind"] == "loops":
            prec = ("f32",)
        self.gauge = tm.tm_load_gauge(self.ctx, self.dims, links.cpu().numpy(), case["t_bc"], precs=prec)

    def __del__(self):
        if getattr(self, "gauge", None) and tm is not None:
            tm.tm_free_gauge(self.ctx, self.gauge)


def _fields(lat, prec, n, full):
    """Device buffer of n fields, one pitch apart (the field and 17 x 256 bytes)."""
    size = tm.tm_field_bytes(lat.gauge, prec, full)
    pitch = (size + 255) // 256 * 256 + 17 * 256
    return torch.zeros(n * pitch, dtype=torch.uint8, device="cuda"), pitch


def _load(lat, prec, spinors, buf, pitch, full):
    """Canonical spinors into a buffer of fields (their even halves for half fields)."""
    size = tm.tm_field_bytes(lat.gauge, prec, True)
    part = size if full else size // 2
    tmp = torch.empty(size, dtype=torch.uint8, device="cuda")
    for i in range(spinors.shape[0]):
        tm.tm_field_import(lat.ctx, lat.gauge, prec, 1, spinors[i], tmp)
        buf[i * pitch:i * pitch + part].copy_(tmp[:part])


def _view(buf, pitch, n, dims, prec, full):
    """The numbers of n fields: [n][parity][..] in their own type, halves with their per-site scales."""
    half_v = dims[0] * dims[1] * dims[2] * dims[3] // 2
    par, site = (2 if full else 1), SPIN_BYTES[prec]
    if prec in ("f64", "f32"):
        t, b = (torch.float64, 8) if prec == "f64" else (torch.float32, 4)
        return buf.view(t).as_strided((n, par, 24 * half_v), (pitch // b, 24 * half_v, 1))
    t = torch.float16 if prec == "f16" else torch.bfloat16
    values = buf.view(t).as_strided((n, par, 24 * half_v), (pitch // 2, site * half_v // 2, 1))
    scale = buf.view(torch.float32).as_strided((n, par, half_v), (pitch // 4, site * half_v // 4, 1), 12 * half_v)
    return {"values": values, "scale": scale}


def _coefs(case, gen):
    """alpha and beta per right-hand side; beta below one, as in a converging solve."""
    return torch.rand(2, case["nrhs"], dtype=torch.float64, device="cuda", generator=gen).mul_(0.8).add_(0.1).tolist()


def prepare(case, seed):
    gen, dims, n, kind = _rng(seed), _dims(case), case["nrhs"], case["kind"]
    lat = Lattice(case, _links(dims, gen))
    st = {"case": case, "lat": lat, "ctx": lat.ctx, "gauge": lat.gauge}
    if kind == "loops":
        st["params"] = tm.tsm_params(case["kappa"], case["mu"], 1000 + seed, case["n_hp"], case["n_lp"],
                                     hp=tm.solver_params("mixed", tol=1e-12),
                                     lp=tm.solver_params("f64", tol=case["tol"]), batch=n)
    elif kind == "solve":
        st["b"] = _spinors(n, dims, gen)
        st["x"] = torch.empty_like(st["b"])
        st["params"] = tm.solver_params(case["prec"], tol=case["tol"], fixed_iters=case["iters"])
    elif kind == "contract":
        st["s"], st["pitch"] = _fields(lat, case["prec"], n, True)
        _load(lat, case["prec"], _spinors(n, dims, gen), st["s"], st["pitch"], True)
        st["seed"], st["ids"] = 1000 + seed, list(range(n))
        st["raw"] = torch.empty(n, 9, dims[3], 4, 4, 2, dtype=torch.float64, device="cuda")
    elif kind == "update":
        for k in ("p", "r", "x"):
            st[k], st["pitch"] = _fields(lat, case["prec"], n, False)
            _load(lat, case["prec"], _spinors(n, dims, gen), st[k], st["pitch"], False)
        st["alpha"], st["beta"] = _coefs(case, gen)
        st["out"] = {k: _view(st[k], st["pitch"], n, dims, case["prec"], False) for k in ("p", "x")}
    else:
        full = case["op"] not in HALF_FAMILY
        for k in ("in", "res"):
            st[k], st["pitch"] = _fields(lat, case["prec"], n, full)
        _load(lat, case["prec"], _spinors(n, dims, gen), st["in"], st["pitch"], full)
        st["out"] = _view(st["res"], st["pitch"], n, dims, case["prec"], full)
    return st


def run(st):
    case, ctx, gauge = st["case"], st["ctx"], st["gauge"]
    n, kappa, mu, kind = case["nrhs"], case["kappa"], case["mu"], case["kind"]
    if kind == "dslash":
        tm.tm_dslash_ex(ctx, gauge, case["op"], kappa, mu, case["prec"], n, st["in"], st["pitch"], st["res"], st["pitch"])
        return st["out"]
    if kind == "update":
        tm.tm_cg_update(ctx, gauge, case["prec"], n, st["p"], st["r"], st["x"], st["pitch"], st["alpha"], st["beta"])
        return st["out"]
    if kind == "contract":
        tm.tm_contract(ctx, gauge, case["prec"], n, st["s"], st["pitch"], st["seed"], st["ids"], st["raw"])
        return st["raw"]
    if kind == "solve":
        tm.tm_cg_solve(ctx, gauge, kappa, mu, st["params"], n, st["b"], st["x"])
        return st["x"].half() if case["prec"] == "lp" else st["x"]
    res = tm.tm_loops_tsm(ctx, gauge, st["params"], case["lt"])
    return {k: res[k] for k in ("est", "var_re", "var_im")}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    v = case["lx"] * case["ly"] * case["lz"] * case["lt"]
    kind, n = case["kind"], case["nrhs"]
    if kind == "loops":
        hp, lp = case["n_hp"], case["n_hp"] + case["n_lp"]
        flops = _solve_flops(v, hp, 255) + _solve_flops(v, lp, 10) + 5568 * v * (hp + lp)
        return {"bytes": _solve_bytes(v, hp, 255, "f32", n) + _solve_bytes(v, lp, 10, "f64", n) + (hp + lp) * 576 * v, "flops": flops}
    if kind == "solve":
        prec = {"mixed": "f32", "lp": "f16"}.get(case["prec"], "f64")
        iters = case["iters"] or (255 if case["kappa"] > 0.15 else 60)
        return {"bytes": 2 * 192 * v * n + _solve_bytes(v, n, iters, prec, n), "flops": _solve_flops(v, n, iters)}
    s, l = SPIN_BYTES[case["prec"]], LINK_BYTES[case["prec"]]
    if kind == "update":
        return {"bytes": 5 * s * v // 2 * n, "flops": 48 * 2 * v // 2 * n}
    if kind == "contract":
        return {"bytes": (n * s + 4 * l) * v, "flops": 5568 * v * n}
    if case["op"] in HALF_FAMILY:
        hops = 2 if case["op"] == "mhat_dag_mhat" else 1   # in applications to the whole lattice
        return {"bytes": 4 * l * v + 2 * s * v // 2 * n, "flops": HOP_FLOPS * v * n * hops}
    return {"bytes": 4 * l * v + 2 * s * v * n, "flops": HOP_FLOPS * v * n}


def _solve_flops(v, n, iters):
    return (iters + 2) * n * v * 2 * HOP_FLOPS


def _solve_bytes(v, n, iters, prec, batch):
    """Per iteration: the links once per batch of right-hand sides and the five CG
    vector passes (four half-lattice hops, the updates of x, r and p) of each."""
    return iters * v * (math.ceil(n / batch) * 4 * LINK_BYTES[prec] + n * 17 * SPIN_BYTES[prec] // 2)


# ---------------------------------------------------------------------------
# the same in 64 bits (torch, complex128, fields [n][t][z][y][x][4][3])
# ---------------------------------------------------------------------------
def _gammas():
    g = torch.zeros(5, 4, 4, dtype=torch.complex128)
    g[0, 0, 3] = g[0, 1, 2] = -1j
    g[0, 2, 1] = g[0, 3, 0] = 1j
    g[1, 0, 3] = g[1, 3, 0] = -1
    g[1, 1, 2] = g[1, 2, 1] = 1
    g[2, 0, 2] = g[2, 3, 1] = -1j
    g[2, 1, 3] = g[2, 2, 0] = 1j
    g[3, 0, 2] = g[3, 1, 3] = g[3, 2, 0] = g[3, 3, 1] = 1
    g[4] = g[0] @ g[1] @ g[2] @ g[3]
    return g.cuda()


class Exact:
    def __init__(self, case, links):
        self.case, self.dims = case, _dims(case)
        lx, ly, lz, lt = self.dims
        self.shape = (lt, lz, ly, lx)
        self.u = links.reshape(self.shape + (4, 3, 3))
        self.g = _gammas()
        self.ch = torch.tensor([1.0, 1.0, -1.0, -1.0], dtype=torch.float64, device="cuda")[:, None]  # gamma5
        t, z, y, x = torch.meshgrid(*(torch.arange(k, device="cuda") for k in self.shape), indexing="ij")
        self.even = ((x + y + z + t) % 2 == 0)[..., None, None]
        flat = self.even.reshape(-1)
        self.order = [torch.nonzero(flat).reshape(-1), torch.nonzero(~flat).reshape(-1)]

    def field(self, spinor):
        return torch.view_as_complex(spinor.contiguous()).reshape(self.shape + (4, 3))

    def shift(self, f, mu, sign):
        """f(x + sign mu), with the boundary sign in time."""
        f = torch.roll(f, -sign, 3 - mu)
        if mu == 3 and self.case["t_bc"] < 0:
            f[-1 if sign > 0 else 0] *= -1
        return f

    def transport(self, f, mu, sign):
        """U_mu(x) f(x + mu), or U_mu(x - mu)^dagger f(x - mu)."""
        if sign > 0:
            u, h = self.u[..., mu, :, :], self.shift(f, mu, 1)
            return sum(u[..., None, :, c] * h[..., :, None, c] for c in range(3))
        u = self.u[..., mu, :, :]
        return self.shift(sum(u[..., None, c, :].conj() * f[..., :, None, c] for c in range(3)), mu, -1)

    def spin(self, m, f):
        return torch.stack([sum(m[a, b] * f[..., b, :] for b in range(4) if m[a, b] != 0) for a in range(4)], dim=-2)

    def hop(self, f):
        out = torch.zeros_like(f)
        for mu in range(4):
            w = self.transport(f, mu, 1)
            out += w
            d = w
            w = self.transport(f, mu, -1)
            out += w
            out -= self.spin(self.g[mu], d - w)
        return out

    def m(self, f, dag=False):
        k, a = self.case["kappa"], self.case["mu"]
        if dag:
            return f - 1j * a * self.ch * f - k * self.ch * self.hop(self.ch * f)
        return f + 1j * a * self.ch * f - k * self.hop(f)

    def ainv(self, f, dag=False):
        a = self.case["mu"]
        return (1 + (1j if dag else -1j) * a * self.ch) * f / (1 + a * a)

    def mhat(self, f, dag=False):
        """On even fields (zero on odd sites)."""
        k, a = self.case["kappa"], self.case["mu"]
        hop = (lambda v: self.ch * self.hop(self.ch * v)) if dag else self.hop
        return f + (-1j if dag else 1j) * a * self.ch * f - k * k * hop(self.ainv(hop(f), dag))

    def op(self, name, f):
        if name == "hop":
            return self.hop(f)
        if name in ("m", "mdag"):
            return self.m(f, name == "mdag")
        if name == "bh":
            return -self.case["kappa"] * self.ainv(self.hop(f))
        f = f * self.even
        if name == "mhat_dag_mhat":
            return self.mhat(self.mhat(f), True)
        return self.mhat(f, name == "mhat_dag")

    def solve(self, eta, tol, iters=0):
        """M s = eta by even-odd CG on the normal equations from zero."""
        k = self.case["kappa"]
        b = (eta + k * self.hop(self.ainv(eta * ~self.even))) * self.even
        r = self.mhat(b, True)
        x, p = torch.zeros_like(r), r
        rr = rr0 = r.abs().square().sum()
        done = 0
        while (done < iters) if iters else (rr > tol * tol * rr0 and done < 2000):
            u = self.mhat(p)
            alpha = rr / u.abs().square().sum()
            x = x + alpha * p
            r = r - alpha * self.mhat(u, True)
            new = r.abs().square().sum()
            p = r + (new / rr) * p
            rr = new
            done += 1
        return x + self.ainv(eta + k * self.hop(x)) * ~self.even

    def noise(self, seed, src):
        """Z4 noise from word 0 of Philox4x64-10 (Salmon et al., SC'11)."""
        def signed(v):
            v &= (1 << 64) - 1
            return v - (1 << 64) if v >> 63 else v

        def mulhi(m, c):
            lo, hi = c & 0xFFFFFFFF, (c >> 32) & 0xFFFFFFFF
            ml, mh = m & 0xFFFFFFFF, m >> 32
            def parts(v):   # the two halves of an unsigned 64-bit product
                return v & 0xFFFFFFFF, (v >> 32) & 0xFFFFFFFF
            (_, a1), (b0, b1), (c0, c1), d = parts(lo * ml), parts(lo * mh), parts(hi * ml), hi * mh
            return d + b1 + c1 + ((a1 + b0 + c0) >> 32)

        n = self.u.numel() // 36
        z = torch.zeros(n, dtype=torch.int64, device="cuda")
        c, key = [torch.arange(n, device="cuda"), z + src, z, z], [seed, 0]
        for _ in range(10):
            h0, l0 = mulhi(0xD2E7470EE14C6C93, c[0]), c[0] * signed(0xD2E7470EE14C6C93)
            h1, l1 = mulhi(0xCA5A826395121157, c[2]), c[2] * signed(0xCA5A826395121157)
            c = [h1 ^ c[1] ^ signed(key[0]), l1, h0 ^ c[3] ^ signed(key[1]), l0]
            key = [key[0] + 0x9E3779B97F4A7C15, key[1] + 0xBB67AE8584CAA73B]
        bits = (c[0][:, None] >> torch.arange(24, device="cuda")) & 1
        v = (1 - 2 * bits).to(torch.float64).reshape(-1, 12, 2) / math.sqrt(2)
        return torch.view_as_complex(v).reshape(self.shape + (4, 3))

    def contract(self, eta, s):
        """Spin matrices [9][t][4][4] of the local, forward and backward kinds."""
        def dot(l, w):
            l, w = l.reshape(self.shape[0], -1, 4, 3), w.reshape(self.shape[0], -1, 4, 3)
            return torch.stack([torch.stack([(l[:, :, a].conj() * w[:, :, b]).sum((1, 2)) for b in range(4)], -1)
                                for a in range(4)], -2)
        return torch.stack([dot(eta, s)] + [dot(eta, self.transport(s, nu, 1)) for nu in range(4)]
                           + [dot(self.transport(eta, nu, 1), s) for nu in range(4)])

    def project(self, raw):
        """The 90 operators [90][t] of spin matrices [9][t][4][4]."""
        g = self.g
        ins = [torch.eye(4, dtype=torch.complex128, device="cuda"), *g, *(g[m] @ g[4] for m in range(4))]
        ins += [0.5j * (g[m] @ g[n] - g[n] @ g[m]) for m in range(4) for n in range(m + 1, 4)]
        tr = torch.einsum("gab,ktab->gkt", torch.stack(ins), raw)
        der = torch.empty(16, 4, self.shape[0], dtype=torch.complex128, device="cuda")
        for nu in range(4):
            d = tr[:, 1 + nu] - tr[:, 5 + nu]
            der[:, nu] = 0.25 * (d + (torch.roll(d, 1, -1) if nu == 3 else d))
        sym = [0.5 * (der[1 + m, n] + der[1 + n, m]) for m in range(4) for n in range(m, 4)]
        return torch.cat((tr[:, 0], der.reshape(64, -1), torch.stack(sym)))

    def pack(self, fields, prec, full):
        """Fields in the library's layout of prec: what _view shows of them."""
        out, scale = [], []
        for f in fields:
            f = f.reshape(-1, 12)
            for par in range(2 if full else 1):
                h = f[self.order[par]]
                if prec in ("f16", "bf16"):
                    mx = torch.view_as_real(h).abs().amax((1, 2))
                    scale.append(mx)
                    h = h / mx[:, None]
                g = {"f64": 1, "f32": 2}.get(prec, 4)   # components side by side
                out.append(torch.view_as_real(h.reshape(-1, 12 // g, g).transpose(0, 1).contiguous()).reshape(-1))
        n = len(fields)
        out = torch.stack(out).reshape(n, -1, out[0].numel())
        return {"values": out, "scale": torch.stack(scale).reshape(n, -1, scale[0].numel())} if scale else out


def _stored(ex, spinors, prec, full):
    """The fields as the storage of prec holds them: the inputs that an operator sees."""
    res = []
    for s in spinors:
        f = ex.field(s)
        if prec == "f32":
            f = f.to(torch.complex64).to(torch.complex128)
        elif prec in ("f16", "bf16"):
            r = torch.view_as_real(f)
            mx = r.float().abs().amax((-1, -2, -3), keepdim=True)
            q = (r.float() * (1 / mx)).to(torch.float16 if prec == "f16" else torch.bfloat16)
            f = torch.view_as_complex(q.double() * mx.double())
        res.append(f if full else f * ex.even)
    return res


def exact(case, seed):
    gen, dims, n, kind, prec = _rng(seed), _dims(case), case["nrhs"], case["kind"], case["prec"]
    ex = Exact(case, _links(dims, gen))
    if kind == "loops":
        hp, lp = [], []
        for i in range(case["n_hp"] + case["n_lp"]):
            eta = ex.noise(1000 + seed, i)
            if i < case["n_hp"]:
                hp.append(ex.project(ex.contract(eta, ex.solve(eta, 1e-14))))
            lp.append(ex.project(ex.contract(eta, ex.solve(eta, case["tol"]))))
        corr, bulk = torch.stack(hp) - torch.stack(lp[:len(hp)]), torch.stack(lp[len(hp):])
        var = [sum(part(v).var(0) / v.shape[0] for v in (corr, bulk)) for part in (torch.real, torch.imag)]
        return {"est": (corr.mean(0) + bulk.mean(0)).cpu().numpy(), "var_re": var[0].cpu().numpy(), "var_im": var[1].cpu().numpy()}
    if kind == "solve":
        b = _spinors(n, dims, gen)
        tol = case["tol"] if prec == "lp" else 1e-14
        return torch.stack([torch.view_as_real(ex.solve(ex.field(v), tol, case["iters"])).reshape(v.shape) for v in b])
    if kind == "contract":
        s = _stored(ex, _spinors(n, dims, gen), prec, True)
        return torch.stack([torch.view_as_real(ex.contract(ex.noise(1000 + seed, i), s[i])) for i in range(n)])
    if kind == "update":
        p, r, x = (_stored(ex, _spinors(n, dims, gen), prec, False) for _ in range(3))
        alpha, beta = _coefs(case, gen)
        x = [x[i] + alpha[i] * p[i] for i in range(n)]
        p = [r[i] + beta[i] * p[i] for i in range(n)]
        return {"p": ex.pack(p, prec, False), "x": ex.pack(x, prec, False)}
    full = case["op"] not in HALF_FAMILY
    return ex.pack([ex.op(case["op"], f) for f in _stored(ex, _spinors(n, dims, gen), prec, full)], prec, full)

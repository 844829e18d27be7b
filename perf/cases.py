"""Performance cases: the library's work as a user's program gives it, through the public entry points.

  listed()           the cases
  draw(rng)          one more case from the ranges that the listed ones stand for
  prepare(case, s)   inputs made from the seed alone, and the buffers and handles a program keeps
  run(state)         one pass
  work(case)         bytes and flops that a pass cannot do without
  exact(case, s)     the pass's result in 64 bits by plain torch (no code of the library)

Lattices are (T, Z, Y, X).  The parameters (kappa 0.1373, c_sw 1.5, links exp(i 0.6 H), FGMRES(8) defect
correction with 4 SAP cycles of 4 MR steps) are those of bench.py's workloads.  Sources of
solves are point sources (a propagator's columns), taken to 1e-11, a digit below the benchmark's, so that
solutions agree to well under 1e-9; operator and smoother get Gaussian fields.

FP32 and BF16 paths are measured on internal buffers, which a program keeps resident between calls,
and return those buffers as they are: [nsys][6 units][V tiled][4 reals].
"""
import itertools

import torch

import paper_1610_02370_amd as tm

KAPPA, CSW, EPS = 0.1373, 1.5, 0.6
TOL = 1e-11
CYCLES, MR = 4, 4
_tags = itertools.count(1)  # a program numbers its gauge configurations

AXIS = (0, 3, 2, 1)  # array axis of direction mu = t, x, y, z


# ------------------------------------------------------------------------------------- cases

def _case(name, kind, dims, nsys, storage="f64", mu=0.0009, **more):
    c = {"kind": kind, "T": dims[0], "Z": dims[1], "Y": dims[2], "X": dims[3], "nsys": nsys, "storage": storage,
         "mu": mu}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one application on the smallest lattice, both flavours: launches and host work count
        _case("apply_f64_4^4", "apply", (4, 4, 4, 4), 2, mu=0.01),
        # odd and ragged extents (small tiles), antiperiodic in time, twisted in space, shifted masses
        _case("apply_f64_6x10x7x9", "apply", (6, 10, 7, 9), 3, mu=0.2, twisted=True),
        # a new gauge configuration: links taken in and checked, clover term built, one application
        _case("new_links_f64_32^3x64", "apply", (64, 32, 32, 32), 1, mu=0.001, new_links=True),
        # the solver's FP32 operator on the largest lattice of the benchmark's full propagator
        _case("apply_f32_48^3x96", "apply", (96, 48, 48, 48), 12, storage="f32"),
        # FP64 smoother on one system (plain FP64 solves), canonical buffers
        _case("smooth_f64_32^3x64", "smooth", (64, 32, 32, 32), 1, mu=0.001),
        # FP32 smoother over a whole propagator: the largest case
        _case("smooth_f32_48^3x96", "smooth", (96, 48, 48, 48), 12, storage="f32"),
        # 16-bit storage, 12 sources of both flavours in one batch
        _case("smooth_bf16_32^3x64", "smooth", (64, 32, 32, 32), 24, storage="bf16", mu=0.001),
        # the paper's smoother: even-odd preconditioned block solves
        _case("smooth_eo_f32_32^3x64", "smooth", (64, 32, 32, 32), 2, storage="f32", mu=0.001, eo=True),
        # a propagator on a small lattice: few blocks, many launches
        _case("solve_dc_f32_16^4", "solve", (16, 16, 16, 16), 12, storage="f32", form="defect_correction",
              restart=8),
        # both flavours, FP64 FGMRES(20) preconditioned by the FP32 smoother
        _case("solve_flex_f32_32^3x64", "solve", (64, 32, 32, 32), 2, storage="f32", mu=0.001, form="flexible",
              restart=20),
        # the FP64 CG baseline on the even-odd normal equations
        _case("cg_f64_16^3x32", "cg", (32, 16, 16, 16), 1),
        # a new configuration with the two-level method: setup, then a spin's three columns solved with it
        _case("two_level_16^4", "two_level", (16, 16, 16, 16), 3, storage="f32", form="defect_correction",
              restart=8, n_vec=20, setup_iters=3),
    ]


def _spread(rng, lo, hi):
    """An integer from lo..hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def _dims(rng, step, lo, hi, sites):
    """Four extents, multiples of `step` in lo..hi, of at most `sites` sites together."""
    while True:
        d = [step * _spread(rng, max(1, lo // step), hi // step) for _ in range(4)]
        if d[0] * d[1] * d[2] * d[3] <= sites:
            return d


def draw(rng):
    """One more case.  Solves stay on lattices of multiples of 8 (4^4 blocks, two per direction)."""
    kind = rng.choice(("apply", "apply", "new_links", "smooth", "smooth", "smooth_blocks", "smooth_eo", "solve",
                       "solve", "cg", "two_level"))
    mu = rng.choice((0.0009, 0.001, 0.003, 0.01))
    if kind == "apply":
        if rng.random() < 0.5:  # any extents, FP64, canonical buffers
            return _case(None, "apply", _dims(rng, 1, 3, 24, 200000), rng.randint(1, 6), mu=mu,
                         twisted=rng.random() < 0.5)
        # an extent of at least 8 keeps every internal buffer free of padding
        return _case(None, "apply", _dims(rng, 4, 4, 48, 1 << 21), rng.randint(1, 12),
                     storage=rng.choice(("f32", "bf16")), mu=mu, twisted=rng.random() < 0.5)
    if kind == "new_links":
        return _case(None, "apply", _dims(rng, 2, 4, 40, 1 << 20), rng.randint(1, 4), mu=mu, new_links=True)
    if kind == "smooth":
        return _case(None, "smooth", _dims(rng, 8, 8, 48, 1 << 20), rng.randint(1, 12),
                     storage=rng.choice(("f64", "f32", "f32", "bf16")), mu=mu, twisted=rng.random() < 0.3)
    if kind == "smooth_blocks":  # other Schwarz blocks than 4^4
        b = rng.choice(((2, 2, 2, 2), (4, 4, 4, 2), (6, 4, 4, 4), (4, 6, 2, 4), (3, 3, 3, 4), (8, 4, 4, 4)))
        n = [2 * rng.randint(1, 3) for _ in range(4)]
        return _case(None, "smooth", [x * y for x, y in zip(b, n)], rng.randint(1, 6),
                     storage=rng.choice(("f64", "f32")), mu=mu, bT=b[0], bZ=b[1], bY=b[2], bX=b[3])
    if kind == "smooth_eo":
        return _case(None, "smooth", _dims(rng, 8, 8, 32, 1 << 19), rng.randint(1, 6),
                     storage=rng.choice(("f64", "f32", "f32")), mu=mu, eo=True)
    if kind == "solve":
        form = rng.choice(("defect_correction", "flexible"))
        storage = "f32" if form == "defect_correction" else rng.choice(("f64", "f32"))
        return _case(None, "solve", _dims(rng, 8, 8, 24, 1 << 17), rng.randint(1, 8), storage=storage, mu=mu,
                     form=form, restart=8 if form == "defect_correction" else 20)
    if kind == "cg":
        return _case(None, "cg", _dims(rng, 2, 8, 32, 1 << 17), rng.randint(1, 2), mu=mu)
    return _case(None, "two_level", _dims(rng, 8, 8, 24, 1 << 16), rng.randint(1, 6), storage="f32", mu=mu,
                 form="defect_correction", restart=8, n_vec=rng.randint(4, 24), setup_iters=rng.randint(1, 3))


# ------------------------------------------------------------------------------------ inputs

def _dims_of(c):
    return (c["T"], c["Z"], c["Y"], c["X"])


def _volume(c):
    return c["T"] * c["Z"] * c["Y"] * c["X"]


def _block(c):
    return (c.get("bT", 4), c.get("bZ", 4), c.get("bY", 4), c.get("bX", 4))


def _mus(c):
    """Both flavours by turns."""
    return [c["mu"] if k % 2 == 0 else -c["mu"] for k in range(c["nsys"])]


def _boundary(c):
    if not c.get("twisted"):
        return {}
    return {"antiperiodic_t": True, "theta": (0.0, 0.3, -0.9, 0.5), "mu_shift": (0.003, -0.002)}


def _generator(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) % (1 << 62))
    return g


def _mm(a, b):
    """Products of 3x3 matrices [..., 3, 3]."""
    return a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :]


def _links(c, seed):
    """SU(3) links [V, 4, 3, 3] complex128 near exp(i eps H), H Gaussian in the Gell-Mann basis."""
    n = 4 * _volume(c)
    gen = _generator(seed, 1)
    out = torch.empty((n, 3, 3), dtype=torch.complex128, device="cuda")
    for a in range(0, n, 1 << 21):
        m = min(1 << 21, n - a)
        h = torch.randn((m, 8), dtype=torch.float64, device="cuda", generator=gen) * (0.5 * EPS)
        x = torch.zeros((m, 3, 3), dtype=torch.complex128, device="cuda")  # i eps H
        for (i, j, k) in ((0, 1, 0), (0, 2, 3), (1, 2, 5)):
            x[:, i, j] = torch.complex(h[:, k + 1], h[:, k])
            x[:, j, i] = torch.complex(-h[:, k + 1], h[:, k])
        d = h[:, 7] / 3 ** 0.5
        for i, v in enumerate((h[:, 2] + d, d - h[:, 2], -2 * d)):
            x[:, i, i] = torch.complex(torch.zeros_like(v), v)
        u = x.clone()
        for k in range(6, 1, -1):  # 1 + x (1 + x/2 (1 + x/3 ...)), made exactly special unitary below
            u = _mm(x, u / k) + x
        for i in range(3):
            u[:, i, i] += 1
        r0 = u[:, 0] / u[:, 0].abs().square().sum(-1, keepdim=True).sqrt()
        r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(-1, keepdim=True) * r0
        r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
        out[a:a + m, 0], out[a:a + m, 1] = r0, r1
        out[a:a + m, 2] = torch.linalg.cross(r0, r1).conj()
    return out.reshape(-1, 4, 3, 3)


def _gaussian(c, seed, k):
    """System k's Gaussian field [1, V, 4, 3]."""
    g = _generator(seed, 100 + k)
    return torch.randn((1, _volume(c), 4, 3), dtype=torch.complex128, device="cuda", generator=g)


def _points(c, seed):
    """Point sources [nsys, V, 4, 3]: the columns of a propagator from one random site, flavours by turns."""
    g = torch.Generator()
    g.manual_seed(int(seed))
    site = int(torch.randint(_volume(c), (1,), generator=g))
    b = torch.zeros((c["nsys"], _volume(c), 4, 3), dtype=torch.complex128, device="cuda")
    for k in range(c["nsys"]):
        b[k, site, (k // 3) % 4, k % 3] = 1.0
    return b


def _internal(c):
    return c["storage"] in ("f32", "bf16") and c["kind"] in ("apply", "smooth")


def _layout(c):
    """The tile of internal buffers: the Schwarz block, or the library's default for an application."""
    return _block(c) if c["kind"] == "smooth" else None


def _buffer(c):
    kind = {"f32": torch.float32, "bf16": torch.bfloat16}[c["storage"]]
    n = tm.tm_spinor_bytes(_dims_of(c), c["nsys"], c["storage"], layout_block=_layout(c))
    return torch.zeros(n // (4 if kind is torch.float32 else 2), dtype=kind, device="cuda")


def prepare(case, seed):
    c, dims = case, _dims_of(case)
    st = {"case": c, "U": _links(c, seed), "tag": 0 if c.get("new_links") else next(_tags)}
    if c["kind"] in ("solve", "cg", "two_level"):
        st["b"] = _points(c, seed)
        st["x"] = torch.zeros_like(st["b"])
        if c["kind"] == "two_level":
            g = _generator(seed, 2)
            st["v0"] = torch.randn((c["n_vec"], _volume(c), 4, 3), dtype=torch.complex128, device="cuda", generator=g)
    elif _internal(c):
        st["b"] = _buffer(c)
        for k in range(c["nsys"]):
            tm.tm_spinor_import_range(dims, _gaussian(c, seed, k), st["b"], c["nsys"], k, storage=c["storage"],
                                      layout_block=_layout(c))
        st["x"] = _buffer(c)
    else:
        st["b"] = torch.cat([_gaussian(c, seed, k) for k in range(c["nsys"])])
        st["x"] = torch.zeros_like(st["b"])
    return st


# --------------------------------------------------------------------------------------- run

def run(st):
    c = st["case"]
    dims, mus, io = _dims_of(c), _mus(c), "internal" if _internal(c) else "canonical"
    if c["kind"] == "apply":
        return tm.tm_dirac_apply(dims, st["U"], st["b"], KAPPA, mus, CSW, out=st["x"], storage=c["storage"], io=io,
                                 gauge_tag=st["tag"], **_boundary(c))
    if c["kind"] == "smooth":
        st["x"].zero_()
        return tm.tm_sap_smooth(dims, st["U"], st["b"], st["x"], KAPPA, mus, CSW, _block(c), CYCLES, MR,
                                storage=c["storage"], io=io, gauge_tag=st["tag"], eo=bool(c.get("eo")),
                                **_boundary(c))
    if c["kind"] == "cg":
        st["x"].zero_()
        tm.tm_cg_solve(dims, st["U"], st["b"], st["x"], KAPPA, mus, CSW, TOL, gauge_tag=st["tag"])
        return st["x"]
    mg = None
    if c["kind"] == "two_level":
        mg = tm.MG(dims, st["U"], KAPPA, c["mu"], CSW, st["v0"], gauge_tag=st["tag"], n_vec=c["n_vec"],
                   setup_iters=c["setup_iters"])
    tm.tm_fgmres_solve(dims, st["U"], st["b"], st["x"], KAPPA, mus, CSW, TOL, storage=c["storage"], form=c["form"],
                       restart=c["restart"], n_cycles=CYCLES, mr_iters=MR, block_dims=(4, 4, 4, 4), x_in=False,
                       gauge_tag=st["tag"], mg=mg)
    if mg is not None:
        mg.close()
    return st["x"]


# -------------------------------------------------------------------------------------- work

# Flops per site and system: an application (8 hops of 168, clover with twist 552, 48 more); an MR step
# on 4^4 blocks (6 in-block hops on average, clover, dot products and updates).
APPLY, MR_STEP = 8 * 168 + 552 + 48, 6 * 168 + 552 + 24 + 336


def work(case):
    c = case
    V, n, s = _volume(c), c["nsys"], c["storage"]
    real = {"f64": 8, "f32": 4, "bf16": 2}[s]
    link, clover = 48 * real, 72 * max(real, 4)
    smooth = CYCLES * (APPLY + MR * MR_STEP) - APPLY // 2
    if c["kind"] == "apply":
        if c.get("new_links"):  # canonical links in; 24 plaquettes of three products, 6 spin structures
            return {"bytes": V * (576.0 + n * 384), "flops": V * (24.0 * 3 * 198 + n * APPLY)}
        return {"bytes": V * (link + clover + n * (48.0 * real if _internal(c) else 384)), "flops": V * n * float(APPLY)}
    if c["kind"] == "smooth":
        return {"bytes": V * (link + clover + n * (48.0 * real if _internal(c) else 384)), "flops": V * n * float(smooth)}
    # solves: canonical links, b and x; flops of the steps that these systems take (about 14 FGMRES
    # steps, 140 CG steps of two reduced operators; setup: vectors times smoother and applications)
    bytes_ = V * (576.0 + n * 384)
    if c["kind"] == "cg":
        return {"bytes": bytes_, "flops": V * n * 140.0 * 2 * APPLY}
    flops = V * n * 14.0 * (smooth + APPLY)
    if c["kind"] == "two_level":
        flops += V * c["n_vec"] * (c["setup_iters"] * float(smooth) + 9 * 552)
    return {"bytes": bytes_, "flops": flops}


# ------------------------------------------------------------------------- 64-bit reference

_I = 1j
# B_mu on a pair (p0, p1): (source, factor) of each component; B_mu^+ likewise
_B = (((0, -1), (1, -1)), ((1, -_I), (0, -_I)), ((1, -1), (0, 1)), ((0, -_I), (1, _I)))
_BD = (((0, -1), (1, -1)), ((1, _I), (0, _I)), ((1, 1), (0, -1)), ((0, _I), (1, -_I)))


def _pair(table, p):
    """Spin matrix of `table` on pairs [..., 2, 3]."""
    return torch.stack([f * p[..., s, :] for s, f in table], dim=-2)


def _mul(U, h):
    """U h for links [sites..., 3, 3] and pairs [..., sites, 2, 3]."""
    return sum(U[..., None, :, k] * h[..., k:k + 1] for k in range(3))


class _Lattice:
    """The operator of section 2.1 on [n, T, Z, Y, X, 4, 3] fields, complex128, and its restriction to blocks."""

    def __init__(self, c, seed):
        self.c, self.dims = c, _dims_of(c)
        b = _boundary(c)
        self.theta = list(b.get("theta", (0.0,) * 4))
        if b.get("antiperiodic_t"):
            self.theta[0] += torch.pi
        self.shift = b.get("mu_shift", (0.0, 0.0))
        U = _links(c, seed).reshape(*self.dims, 4, 3, 3)
        self.U = [U[..., mu, :, :].contiguous() for mu in range(4)]
        del U
        self.A = self._clover()
        at = [torch.arange(n, device="cuda").reshape([-1 if a == k else 1 for k in range(4)])
              for a, n in enumerate(self.dims)]
        self.at = at
        self.parity = (at[0] + at[1] + at[2] + at[3]) % 2

    def _clover(self):
        """m + 4 - c_sw/16 sum_{mu<nu} gamma_mu gamma_nu (Q - Q^+): two 6x6 blocks [sites..., 2, 6, 6]."""
        A = torch.zeros((*self.dims, 2, 6, 6), dtype=torch.complex128, device="cuda")
        for i in range(6):
            A[..., i, i] += 1 / (2 * KAPPA)
        up = lambda f, mu: torch.roll(f, -1, AXIS[mu])  # noqa: E731  f(x + mu)
        dn = lambda f, mu: torch.roll(f, 1, AXIS[mu])  # noqa: E731
        dag = lambda m: m.transpose(-1, -2).conj()  # noqa: E731
        for mu in range(4):
            for nu in range(mu + 1, 4):
                u, v = self.U[mu], self.U[nu]
                a, b = _mm(u, up(v, mu)), _mm(v, up(u, nu))  # the two ways to x + mu + nu
                # the four leaves at x: the plaquette above it, and those to the left, below and both
                Q = _mm(a, dag(b))
                Q = Q + dn(_mm(_mm(up(v, mu), dag(b)), u), mu)
                Q = Q + dn(dn(_mm(dag(b), a), mu), nu)
                Q = Q + dn(_mm(dag(v), _mm(a, dag(up(u, nu)))), nu)
                F = Q - dag(Q)
                for blk, (t1, t2) in enumerate(((_B[mu], _BD[nu]), (_BD[mu], _B[nu]))):
                    for s, (k, f) in enumerate(t1):  # row s of the product of two monomial spin matrices
                        j, g = t2[k]
                        A[..., blk, 3 * s:3 * s + 3, 3 * j:3 * j + 3] -= CSW / 16 * f * g * F
        return A

    def mass(self, mu):
        return mu + torch.tensor(self.shift, dtype=torch.float64, device="cuda")[self.parity]

    def diagonal(self, psi, mu, A=None):
        A = self.A if A is None else A
        v = psi.reshape(*psi.shape[:-2], 2, 6)
        out = sum(A[..., k] * v[..., k:k + 1] for k in range(6))
        if mu is not None:
            tw = (1j * self.mass(mu))[..., None]
            out[..., 0, :] += tw * v[..., 0, :]
            out[..., 1, :] -= tw * v[..., 1, :]
        return out.reshape(psi.shape)

    def hops(self, psi, blocks=None):
        """-1/2 sum of the eight hops; with `blocks`, those inside a block only."""
        acc = torch.zeros_like(psi)
        ax0 = psi.dim() - 6
        for mu in range(4):
            ax, n = AXIS[mu], self.dims[AXIS[mu]]
            at = self.at[ax]
            ph = torch.exp(1j * torch.tensor(self.theta[mu], dtype=torch.float64, device="cuda"))
            one = torch.ones_like(at, dtype=torch.complex128)
            f, b = torch.where(at == n - 1, ph, one), torch.where(at == 0, ph.conj(), one)
            if blocks:
                f = torch.where(at % blocks[ax] == blocks[ax] - 1, 0 * one, one)
                b = torch.where(at % blocks[ax] == 0, 0 * one, one)
            for sign, w in ((-1, f), (1, b)):
                if sign < 0:
                    h = psi[..., :2, :] - _pair(_B[mu], psi[..., 2:, :])
                    g = _mul(self.U[mu], torch.roll(h, -1, ax0 + ax) * w[..., None, None])
                else:
                    h = psi[..., :2, :] + _pair(_B[mu], psi[..., 2:, :])
                    g = torch.roll(_mul(self.U[mu].transpose(-1, -2).conj(), h), 1, ax0 + ax) * w[..., None, None]
                acc[..., :2, :] += g
                acc[..., 2:, :] += sign * _pair(_BD[mu], g)
        return acc.mul_(-0.5)

    def apply(self, psi, mu, blocks=None):
        return self.hops(psi, blocks).add_(self.diagonal(psi, mu))

    # ---- the smoother (section 2.4)

    def block_sum(self, f, blocks):
        """Sums over blocks of [T, Z, Y, X], spread back over the sites."""
        s = f.reshape([w for n, b in zip(self.dims, blocks) for w in (n // b, b)]).sum((1, 3, 5, 7), keepdim=True)
        return s.expand([w for n, b in zip(self.dims, blocks) for w in (n // b, b)]).reshape(self.dims)

    def mr(self, op, r, blocks, steps):
        e, rho = torch.zeros_like(r), r
        for _ in range(steps):
            q = op(rho)
            qq = self.block_sum(q.abs().square().sum((-1, -2)), blocks)
            qr = self.block_sum((q.conj() * rho).sum((-1, -2)), blocks)
            al = torch.where(qq > 0, qr / torch.where(qq > 0, qq, torch.ones_like(qq)), 0 * qr)[..., None, None]
            e, rho = e + al * rho, rho - al * q
        return e

    def inverse(self, mu):
        """(A + i mu Gamma5)^-1 by elimination (the diagonal dominates: no pivoting)."""
        M = self.A.clone()
        tw = 1j * self.mass(mu)
        for i in range(6):
            M[..., 0, i, i] += tw
            M[..., 1, i, i] -= tw
        X = torch.zeros_like(M)
        for i in range(6):
            X[..., i, i] = 1
        for k in range(6):
            d = 1 / M[..., k:k + 1, k:k + 1]
            M[..., k:k + 1, :], X[..., k:k + 1, :] = M[..., k:k + 1, :] * d, X[..., k:k + 1, :] * d
            f = M[..., :, k:k + 1].clone()
            f[..., k, :] = 0
            M, X = M - f * M[..., k:k + 1, :], X - f * X[..., k:k + 1, :]
        return X

    def smooth(self, b, mu):
        blocks = _block(self.c)
        col = sum(a // w for a, w in zip(self.at, blocks)) % 2
        x = torch.zeros_like(b)
        odd = (self.parity == 1)[..., None, None]
        inv = self.inverse(mu) if self.c.get("eo") else None
        hop = lambda v: self.hops(v, blocks)  # noqa: E731
        zero = torch.zeros((), dtype=b.dtype, device="cuda")
        for _ in range(CYCLES):
            for colour in (0, 1):
                here = (col == colour)[..., None, None]
                r = torch.where(here, b - self.apply(x, mu), zero)
                if inv is None:
                    e = self.mr(lambda v: self.apply(v, mu, blocks), r, blocks, MR)
                else:
                    ee = lambda v: torch.where(odd, zero, self.diagonal(v, None, inv))  # noqa: E731
                    rhat = torch.where(odd, r - hop(ee(r)), zero)
                    e = self.mr(lambda v: torch.where(odd, self.diagonal(v, mu) - hop(ee(hop(v))), zero), rhat,
                                blocks, MR)
                    e = e + ee(r - hop(e))
                x = torch.where(here, x + e, x)
        return x

    def solve(self, b, mu):
        """D^-1 b: BiCGStab, started again from the true residual until that is at rounding."""
        x, dot = torch.zeros_like(b), lambda u, v: (u.conj() * v).sum()  # noqa: E731
        norm = b.norm()
        for _ in range(8):
            r = b - self.apply(x, mu)
            if r.norm() <= 2e-15 * norm:
                break
            goal, r0, p, rho = max(2e-15 * float(norm), 1e-10 * float(r.norm())), r, r, dot(r, r)
            for _ in range(400):
                v = self.apply(p, mu)
                al = rho / dot(r0, v)
                s = r - al * v
                t = self.apply(s, mu)
                om = dot(t, s) / dot(t, t)
                x = x + al * p + om * s
                r = s - om * t
                if float(r.norm()) <= goal:
                    break
                new = dot(r0, r)
                p = r + (new / rho) * (al / om) * (p - om * v)
                rho = new
        return x


def _tiled(c, v):
    """[V, 4, 3] complex -> an internal buffer's system [6, V, 4] reals."""
    d = _dims_of(c)
    tile = _layout(c) or [4 if n % 4 == 0 else 2 if n % 2 == 0 else 1 for n in d]
    w = torch.view_as_real(v).reshape([k for n, b in zip(d, tile) for k in (n // b, b)] + [6, 4])
    return w.permute(8, 0, 2, 4, 6, 1, 3, 5, 7, 9).reshape(-1)


def exact(case, seed):
    c, V = case, _volume(case)
    if c["kind"] == "smooth" and V * c["nsys"] > 1 << 26:
        return None  # minutes
    L = _Lattice(c, seed)
    out = torch.empty((c["nsys"], 24 * V), dtype=torch.float64, device="cuda")
    points = _points(c, seed) if c["kind"] in ("solve", "cg", "two_level") else None
    for k, mu in enumerate(_mus(c)):
        b = (points[k:k + 1] if points is not None else _gaussian(c, seed, k))
        if c["storage"] == "bf16":  # what the buffer holds
            b = torch.view_as_complex(torch.view_as_real(b).to(torch.bfloat16).double())
        elif c["storage"] == "f32":
            b = b.to(torch.complex64).to(torch.complex128)
        b = b.reshape(1, *_dims_of(c), 4, 3)
        if c["kind"] == "apply":
            x = L.apply(b, mu)
        elif c["kind"] == "smooth":
            x = L.smooth(b, mu)
        else:
            x = L.solve(b, mu)
        out[k] = _tiled(c, x.reshape(V, 4, 3)) if _internal(c) else torch.view_as_real(x.reshape(V, 4, 3)).reshape(-1)
    if _internal(c):
        return out.reshape(-1)
    return torch.view_as_complex(out.reshape(c["nsys"], V, 4, 3, 2))

"""The work a plane-wave program has this library do, as measurable cases.

Every case is one call (or the few calls of one SCF iteration) through the
public binding, over the sizes the library takes: a few bands of a small cell up
to the 115313-plane-wave, 2048-band block; cubic and slab-shaped cells; FFT edges
with and without compile-time passes; complex128 and the mixed complex64 form;
forward, adjoint and batched filters; S = I and PAW-like overlaps.

Inputs are seeded synthetic systems: Gaussian wells of depth 4 Ha on random
atoms (at least 3 bohr apart), four Gaussian s + p projectors per atom, a random
Hermitian D per atom, and N(0,1) blocks, which is what a solver starts from.
The filter's interval is fixed per case (a wanted part that ends a little above
the lowest bands' energies, an upper bound just above the cut-off), as a solver
has it from its second cycle on.

Results of the mixed form that the library hands out in 64 bits although they
carry 32-bit (or split-BF16) rounding - Ritz values of the intermediate cycles,
their density, the gradients of the mixed adjoint - are taken in 32 bits, the
precision of the block.  Ritz vectors have an arbitrary phase each, so the cases
that compute them return what a program forms from them: the density.
"""
import math

import numpy as np
import torch

from paper_2604_11139_amd import binding as B

WELL, SIGMA, RC = -4.0, 0.8, 1.0


# ---- the cases ---------------------------------------------------------------------
def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, a1=10.0, a2=10.0, a3=10.0, n1=32, n2=32, n3=32, ecut=10.0,
             kx=0.0, ky=0.0, kz=0.0, natom=2, nband=32, degree=8, mixed=False)
    c.update(kw)
    return c


def _cube(a, n):
    return dict(a1=a, a2=a, a3=a, n1=n, n2=n, n3=n)


def listed():
    return [
        # One H application on a few bands of a small cell at a k-point: the inner call of a
        # program with its own iteration (latency and launches).
        _case("apply_small_mixed", "apply", **_cube(9.3, 30), ecut=12.0, kx=0.13, ky=0.31, kz=0.22,
              natom=3, nband=17, mixed=True),
        # The smallest whole filter: 1503 plane waves, 32 bands, complex128.
        _case("filter_small_fp64", "filter", **_cube(10.0, 32), ecut=10.0, natom=2, nband=32,
              degree=8),
        # The ordinary mixed filter: 64 atoms, 22119 plane waves, 512 bands.
        _case("filter_medium_mixed", "filter", **_cube(20.0, 36), ecut=15.0, natom=64, nband=512,
              degree=10, mixed=True),
        # A slab: a long cell, a box that is not a cube, an odd number of bands.
        _case("filter_slab_mixed", "filter", a1=16.0, a2=16.0, a3=40.0, n1=36, n2=36, n3=80,
              ecut=15.0, natom=72, nband=347, degree=10, mixed=True),
        # complex128 at a k-point in a box whose edge (54) is none of the tuned ones.
        _case("filter_kpt_fp64", "filter", **_cube(24.5, 54), ecut=14.0, kx=0.25, ky=0.1, kz=0.4,
              natom=96, nband=411, degree=8),
        # The headline workload: 216 atoms, 115313 plane waves, 2048 bands, degree 12, mixed.
        _case("filter_large_mixed", "filter", **_cube(30.0, 64), ecut=20.0, natom=216, nband=2048,
              degree=12, mixed=True),
        # The same block in complex128, one H application (the Rayleigh-Ritz step's).
        _case("apply_large_fp64", "apply", **_cube(30.0, 64), ecut=20.0, natom=216, nband=2048),
        # PAW / ultrasoft: the filter of S^-1 H with the Woodbury inverse.
        _case("paw_filter_mixed", "paw", **_cube(20.0, 36), ecut=15.0, natom=64, nband=512,
              degree=10, mixed=True),
        # Backward of the mixed filter: gradients for V_loc, D and the block.
        _case("adjoint_medium_mixed", "adjoint", **_cube(20.0, 36), ecut=15.0, natom=64, nband=512,
              degree=10, mixed=True),
        # Sixteen small cells (8-16 bohr, 1-8 atoms, 32-256 bands) filtered in one call.
        dict(name="batch16_mixed", kind="batch", nsys=16, mix=4, ecut=12.0, degree=8, mixed=True),
        # One SCF iteration: two cycles of the eigensolver, occupations, density, potential.
        _case("scf_medium_fp64", "scf", **_cube(20.0, 36), ecut=15.0, natom=64, nband=512,
              degree=10),
        # Rayleigh-Ritz of an intermediate mixed cycle at the headline size, and the density.
        _case("rr_large_mixed", "rr", **_cube(30.0, 64), ecut=20.0, natom=216, nband=2048,
              degree=12, mixed=True),
    ]


def _smooth(m):
    while True:
        r = m
        for p in (2, 3, 5):
            while r % p == 0:
                r //= p
        if r == 1:
            return m
        m += 1


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _npw(c):
    return c["a1"] * c["a2"] * c["a3"] * (2.0 * c["ecut"]) ** 1.5 / (6.0 * math.pi ** 2)


def draw(rng):
    kind = rng.choice(["apply", "filter", "filter", "filter", "paw", "adjoint", "batch", "scf", "rr"])
    if kind == "batch":
        return dict(kind="batch", nsys=rng.randint(4, 16), mix=rng.randint(0, 10 ** 6),
                    ecut=rng.uniform(9.0, 12.0), degree=rng.randint(6, 10),
                    mixed=rng.random() < 0.75)
    mixed = True if kind == "rr" else False if kind == "scf" else rng.random() < 0.6
    while True:
        ecut = rng.uniform(8.0, 20.0)
        gmax = math.sqrt(2.0 * ecut)
        a = math.exp(rng.uniform(math.log(9.0), math.log(30.0)))
        slab = rng.random() < 0.35
        cell = [a, a, a * rng.uniform(1.3, 2.6)] if slab else [a, a, a]
        room = rng.uniform(1.0, 1.5)
        grid = [_smooth(int(math.ceil(room * (2 * math.floor(gmax * x / (2 * math.pi) + 0.5) + 2))))
                for x in cell]
        if max(grid) > 96:
            continue
        c = dict(kind=kind, a1=cell[0], a2=cell[1], a3=cell[2], n1=grid[0], n2=grid[1], n3=grid[2],
                 ecut=ecut, kx=rng.uniform(0.0, 0.5), ky=rng.uniform(0.0, 0.5),
                 kz=rng.uniform(0.0, 0.5),
                 natom=max(1, min(216, int(cell[0] * cell[1] * cell[2] / rng.uniform(120, 500)))),
                 degree=rng.randint(6, 12), mixed=mixed)
        npw = _npw(c)
        top = dict(apply=2048, filter=1024, paw=768, adjoint=640, scf=640, rr=1500)[kind]
        top = int(min(top, npw / 12))
        # as much work as the largest listed filter at the most; complex128 products and
        # several products a step (adjoint, SCF) count for what they take
        weight = dict(apply=1, filter=c["degree"], paw=1.3 * c["degree"], adjoint=3 * c["degree"],
                      scf=6 * c["degree"], rr=4)[kind] * (1.0 if mixed else 5.0)
        per_band = 16.0 * npw * 4 * c["natom"] + 400.0 * grid[0] * grid[1] * grid[2]
        top = int(min(top, 0.8 * 12 * 2048 * (16.0 * 115313 * 864 + 400.0 * 64 ** 3)
                      / (weight * per_band)))
        if top < 16:
            continue
        c["nband"] = _log_int(rng, 8 if kind in ("apply", "filter") else 16, top)
        return c


# ---- inputs ------------------------------------------------------------------------
class _System:
    """What the binding reads of one Hamiltonian."""


def _hermitian(rng, natom):
    d = rng.uniform(-1, 1, (natom, 4, 4)) + 1j * rng.uniform(-1, 1, (natom, 4, 4))
    d = np.triu(d, 1)
    return d + np.conj(np.swapaxes(d, 1, 2)) + np.eye(4) * rng.uniform(-1, 1, (natom, 1, 4))


def _system(c, seed):
    rng = np.random.default_rng([2604, 11139, int(seed)])
    cell = np.array([c["a1"], c["a2"], c["a3"]])
    tau = np.zeros((c["natom"], 3))
    k = 0
    while k < c["natom"]:
        t = rng.uniform(0.0, 1.0, 3) * cell
        d = tau[:k] - t
        d -= cell * np.round(d / cell)
        if k == 0 or (d * d).sum(1).min() >= 9.0:
            tau[k] = t
            k += 1
    s = _System()
    s.lattice, s.kpt_red = np.diag(cell), np.array([c["kx"], c["ky"], c["kz"]])
    s.ecut, s.ngrid = c["ecut"], (c["n1"], c["n2"], c["n3"])
    s.tau, s.rc = tau, RC
    g = []
    for x, n, col in zip(cell, s.ngrid, tau.T):
        d = (np.arange(n) * (x / n))[None, :, None] - col[:, None, None] - np.arange(-2, 3) * x
        g.append(np.exp(-(d * d) / (2 * SIGMA * SIGMA)).sum(2))
    xy = g[1][:, :, None] * g[0][:, None, :]
    s.vloc = WELL * (g[2].T @ xy.reshape(c["natom"], -1)).reshape(-1)
    s.dij = _hermitian(rng, c["natom"])
    s.qij = 10.0 * (_hermitian(rng, c["natom"]) + 1.5 * np.eye(4)) if c["kind"] == "paw" else None
    return s


def _block(nband, npw, mixed, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) * 7919 + 17)
    x = torch.randn((nband, npw, 2), generator=g, device="cuda", dtype=torch.float64)
    x = torch.view_as_complex(x)
    return x.to(torch.complex64) if mixed else x


def _bounds(c):
    b = 1.05 * c["ecut"] + 1.0 if c["kind"] == "paw" else c["ecut"] + 0.5
    return 1.5, b, -1.0


def _cells(c):
    """The cells of a batch: their sizes are the case's own, not the seed's."""
    rng = np.random.default_rng([4, c["mix"]])
    out = []
    for _ in range(c["nsys"]):
        a = float(rng.integers(8, 17))
        k = rng.uniform(0.0, 0.5, 3)
        n = _smooth(int(3 * a))
        out.append(dict(kind="filter", **_cube(a, n), ecut=c["ecut"], kx=k[0], ky=k[1], kz=k[2],
                        natom=int(rng.integers(1, 9)), nband=int(rng.choice([32, 64, 128, 256])),
                        degree=c["degree"], mixed=c["mixed"]))
    return out


def _sphere(c):
    """(miller (npw, 3), box index, k+G, G) of {G : 0.5|k+G|^2 < ecut}, ascending box index."""
    n = (c["n1"], c["n2"], c["n3"])
    m = [np.rint(np.fft.fftfreq(v) * v) for v in n]
    b = [2 * np.pi / c[x] for x in ("a1", "a2", "a3")]
    g = np.stack([x.reshape(-1) for x in
                  np.meshgrid(m[2] * b[2], m[1] * b[1], m[0] * b[0], indexing="ij")][::-1], 1)
    q = g + np.array([c["kx"] * b[0], c["ky"] * b[1], c["kz"] * b[2]])
    at = np.flatnonzero(0.5 * (q * q).sum(1) < c["ecut"])
    return at, q[at], g[at]


def _filtered(c, kin, seed):
    """A block as a filter leaves it: N(0,1) columns times the filter's polynomial of the
    kinetic energy."""
    a, b, a0 = _bounds(c)
    x = (kin - (a + b) / 2) / ((b - a) / 2)
    x0 = (a0 - (a + b) / 2) / ((b - a) / 2)
    t0, t1, u0, u1 = torch.ones_like(x), x, 1.0, x0
    for _ in range(c["degree"] - 1):
        t0, t1 = t1, 2 * x * t1 - t0
        u0, u1 = u1, 2 * x0 * u1 - u0
    return (_block(c["nband"], kin.numel(), False, seed) * (t1 / u1)).to(torch.complex64)


def _weights(nband, device="cuda"):
    """Fixed smooth occupations of the lowest half of the bands."""
    i = torch.arange(nband, dtype=torch.float64, device=device)
    return 2.0 / (1.0 + torch.exp((i - 0.5 * nband) / (0.05 * nband)))


def prepare(case, seed):
    c = case
    prec = B.ABI_PREC_MIXED if c["mixed"] else B.ABI_PREC_FP64
    if c["kind"] == "batch":
        cells = _cells(c)
        h = B.Batch([_system(x, seed * 64 + i) for i, x in enumerate(cells)], prec)
        return dict(kind="batch", h=h, degree=c["degree"], bounds=[_bounds(x) for x in cells],
                    X=[_block(x["nband"], h.systems[i].npw, c["mixed"], seed * 64 + i)
                       for i, x in enumerate(cells)])
    s = _system(c, seed)
    h = B.System(s, prec)
    st = dict(kind=c["kind"], h=h, degree=c["degree"], bounds=_bounds(c), nband=c["nband"])
    if c["kind"] == "rr":
        _, q, _ = _sphere(c)
        kin = torch.from_numpy(0.5 * (q * q).sum(1)).cuda()
        st.update(X=_filtered(c, kin, seed), w=_weights(c["nband"]))
        return st
    st["X"] = _block(c["nband"], h.npw, c["mixed"], seed)
    if c["kind"] == "adjoint":
        st["W"] = _block(c["nband"], h.npw, c["mixed"], seed + 500000)
    if c["kind"] == "scf":
        st.update(v0=_block(1, h.npw, False, seed + 500000)[0], vion=torch.from_numpy(s.vloc).cuda(),
                  nelec=float(c["nband"]), kT=0.05)
    return st


# ---- one pass ----------------------------------------------------------------------
def run(state):
    kind, h, X = state["kind"], state["h"], state["X"]
    if kind == "apply":
        return h.apply_H(X)
    if kind in ("filter", "paw"):
        return h.cheb_filter(X, state["degree"], *state["bounds"])
    if kind == "batch":
        return h.cheb_filter(X, state["degree"], state["bounds"])
    if kind == "adjoint":
        dV, dD, dX = h.filter_backward(X, state["W"], state["degree"], *state["bounds"])
        if X.dtype == torch.complex64:  # gradients in the block's precision
            dV, dD = dV.float(), dD.to(torch.complex64)
        return dict(dV=dV, dD=dD, dX=dX)
    if kind == "rr":
        Y = X.clone()  # the call overwrites its block
        ev, _, _ = h.rayleigh_ritz(Y, lowprec=True)
        return dict(eval=ev.astype(np.float32), rho=h.density(Y, state["w"]).float())
    Y = X.clone()
    ev, res, _ = h.solve(Y, state["v0"], state["degree"], 2, state["nband"], 1e-9)
    f, _ = B.occupations(ev, state["nelec"], state["kT"])
    rho = h.density(Y, f)
    return dict(eval=ev, res=res, rho=rho, vout=h.scf_potential(rho, state["vion"]))


# ---- what a pass cannot do without ---------------------------------------------------
def _work(c):
    """(bytes of the tables, bytes of a block, flops of one H application of the block)."""
    npw, box, nproj = _npw(c), c["n1"] * c["n2"] * c["n3"], 4 * c["natom"]
    e = 8 if c["mixed"] else 16
    fft = 2 * 5.0 * box * math.log2(box)
    return (e * npw * nproj + e / 2 * box, e * npw * c["nband"],
            c["nband"] * (fft + 2 * 8.0 * npw * nproj + 8.0 * npw + 6.0 * box))


def work(case):
    c = case
    if c["kind"] == "batch":
        w = [_work(x) for x in _cells(c)]
        return dict(bytes=sum(t + 2 * b for t, b, _ in w), flops=c["degree"] * sum(f for _, _, f in w))
    t, b, f = _work(c)
    m, npw = c["nband"], _npw(c)
    if c["kind"] == "apply":
        return dict(bytes=t + 2 * b, flops=f)
    if c["kind"] in ("filter", "paw"):
        more = 3 * 8.0 * (4 * c["natom"]) ** 2 * m if c["kind"] == "paw" else 0.0
        return dict(bytes=t + 2 * b, flops=c["degree"] * (f + more))
    if c["kind"] == "adjoint":
        return dict(bytes=t + 3 * b, flops=2 * c["degree"] * f)
    # Rayleigh-Ritz: two Hermitian products, H Y, the rotation, the dense steps
    rr = 8.0 * m * m * npw + 8.0 * m * m * npw + f + (4 / 3 + 16 / 3 + 8 + 12) * m ** 3
    if c["kind"] == "rr":
        return dict(bytes=t + 2 * b, flops=rr)
    return dict(bytes=t + 2 * b, flops=2 * (c["degree"] * f + rr))


# ---- the same in 64 bits, with torch alone ---------------------------------------------
class _Exact:
    """H (and S^-1) of one system on (nband, npw) complex128 blocks."""

    def __init__(self, c, seed):
        s = _system(c, seed)
        at, q, g = _sphere(c)
        self.grid = (c["n3"], c["n2"], c["n1"])
        self.box = c["n1"] * c["n2"] * c["n3"]
        self.omega = c["a1"] * c["a2"] * c["a3"]
        self.at = torch.from_numpy(at).cuda()
        self.kin = torch.from_numpy(0.5 * (q * q).sum(1)).cuda()
        self.V = torch.from_numpy(s.vloc).cuda()
        self.D = torch.from_numpy(s.dij).cuda()
        self.natom = c["natom"]
        qc, gc, tau = (torch.from_numpy(v).cuda() for v in (q, g, s.tau))
        ph = tau @ gc.T
        gauss = torch.exp(-self.kin * RC * RC) / math.sqrt(self.omega)
        e = torch.complex(torch.cos(ph), -torch.sin(ph)) * gauss
        w = torch.cat([torch.ones_like(qc[:, :1]), RC * qc], 1).T
        self.P = (e[:, None, :] * w[None]).reshape(4 * self.natom, -1)
        self.PH = self.P.conj().T.resolve_conj().contiguous()
        self.K = None
        if s.qij is not None:
            Q = torch.block_diag(*torch.from_numpy(s.qij).cuda())
            I = torch.eye(4 * self.natom, dtype=torch.complex128, device="cuda")
            self.K = torch.linalg.solve(I + Q @ (self.P.conj() @ self.P.T), Q)

    def real(self, X):
        """Unnormalised inverse transforms of some sphere vectors."""
        b = torch.zeros((X.shape[0], self.box), dtype=torch.complex128, device="cuda")
        b[:, self.at] = X
        return torch.fft.ifftn(b.view(-1, *self.grid), dim=(1, 2, 3), norm="forward").view(-1, self.box)

    def parts(self, X):
        n = max(1, (1 << 24) // self.box)
        return [slice(i, min(i + n, X.shape[0])) for i in range(0, X.shape[0], n)]

    def blockwise(self, C, D):
        return (C.view(-1, self.natom, 1, 4) * D).sum(-1).reshape(C.shape)

    def H(self, X):
        out = self.blockwise(X @ self.PH, self.D) @ self.P
        out += self.kin * X
        for p in self.parts(X):
            r = (self.real(X[p]) * self.V).view(-1, *self.grid)
            out[p] += torch.fft.fftn(r, dim=(1, 2, 3), norm="forward").view(-1, self.box)[:, self.at]
        return out

    def A(self, X):
        h = self.H(X)
        return h if self.K is None else h - ((h @ self.PH) @ self.K.T) @ self.P

    def density(self, X, w):
        rho = torch.zeros(self.box, dtype=torch.float64, device="cuda")
        for p in self.parts(X):
            r = torch.view_as_real(self.real(X[p])).square().sum(-1)
            rho += (w[p, None] * r).sum(0)
        return rho / self.box


def _coefs(degree, a, b, a0):
    e, c = (b - a) / 2, (b + a) / 2
    s1 = e / (a0 - c)
    s, gamma, delta = s1, [s1 / e], [0.0]
    for _ in range(degree - 1):
        t = 1 / (2 / s1 - s)
        gamma.append(2 * t / e)
        delta.append(s * t)
        s = t
    return c, gamma, delta


def _exact_filter(h, X, degree, bounds, keep=False):
    c, gamma, delta = _coefs(degree, *bounds)
    ys, y0, y1 = [X], None, X
    for g, d in zip(gamma, delta):
        y2 = g * (h.A(y1) - c * y1)
        if y0 is not None:
            y2 -= d * y0
        y0, y1 = y1, y2
        if keep:
            ys.append(y1)
    return ys if keep else y1


def _exact_adjoint(h, X, W, degree, bounds):
    c, gamma, delta = _coefs(degree, *bounds)
    ys = _exact_filter(h, X, degree, bounds, keep=True)
    dV = torch.zeros(h.box, dtype=torch.float64, device="cuda")
    dD = torch.zeros((h.natom, 4, 4), dtype=torch.complex128, device="cuda")
    a2, a1 = None, W
    for k in range(degree - 1, -1, -1):
        for p in h.parts(X):
            dV += gamma[k] / h.box * (h.real(a1[p]).conj() * h.real(ys[k][p])).real.sum(0)
        ca, cy = ((v @ h.PH).view(-1, h.natom, 4) for v in (a1, ys[k]))
        for i in range(4):
            for j in range(4):
                dD[:, i, j] += gamma[k] * (ca[:, :, i] * cy[:, :, j].conj()).sum(0)
        a0 = gamma[k] * (h.H(a1) - c * a1)
        if a2 is not None:
            a0 -= delta[k + 1] * a2
        a2, a1 = a1, a0
    return dict(dV=dV, dD=dD, dX=a1)


def _exact_ritz(X, HX):
    """(values, vectors, H times the vectors) of Rayleigh-Ritz on the rows of X."""
    G = X.conj() @ X.T
    L = torch.linalg.cholesky((G + G.conj().T) / 2)
    M = X.conj() @ HX.T
    M = torch.linalg.solve_triangular(L, (M + M.conj().T) / 2, upper=False)
    M = torch.linalg.solve_triangular(L, M.conj().T.contiguous(), upper=False)
    w, Z = torch.linalg.eigh((M + M.conj().T) / 2)
    T = torch.linalg.solve_triangular(L.conj().T.contiguous(), Z, upper=True).T.contiguous()
    return w, T @ X, T @ HX


def _exact_top(h, v0, steps=10):
    """The filter's upper bound: Lanczos with full reorthogonalisation."""
    v = v0[None] / v0.norm()
    vs, al, be = [v], [], []
    for _ in range(steps):
        w = h.H(vs[-1])
        al.append(float((vs[-1].conj() * w).sum().real))
        for _ in range(2):
            for u in vs:
                w = w - (u.conj() * w).sum() * u
        be.append(float(w.norm()))
        vs.append(w / be[-1])
    return float(np.linalg.eigvalsh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))[-1]) + be[-1]


def _exact_scf(h, c, seed):
    X = _block(c["nband"], h.kin.numel(), False, seed)
    HX = h.H(X)
    rq = (X.conj() * HX).sum(1).real / (X.conj() * X).sum(1).real
    a, a0 = float(rq.max()), float(rq.min())
    b = _exact_top(h, _block(1, h.kin.numel(), False, seed + 500000)[0])
    for _ in range(2):
        X = _exact_filter(h, X, c["degree"], (a, b, a0))
        ev, X, HX = _exact_ritz(X, h.H(X))
        a, a0 = float(ev[-1]), float(ev[0])
    res = torch.linalg.vector_norm(HX - ev[:, None] * X, dim=1)
    lo, hi = float(ev[0]) - 10.0, float(ev[-1]) + 10.0
    for _ in range(200):
        mu = (lo + hi) / 2
        f = 2.0 / (1.0 + torch.exp((ev - mu) / 0.05))
        lo, hi = (mu, hi) if float(f.sum()) < c["nband"] else (lo, mu)
    rho = h.density(X, f)
    n = rho * (h.box / h.omega)
    gs = [torch.fft.fftfreq(k, 1.0 / k, dtype=torch.float64, device="cuda") * (2 * math.pi / c[x])
          for k, x in zip(h.grid, ("a3", "a2", "a1"))]
    g2 = gs[0][:, None, None] ** 2 + gs[1][:, None] ** 2 + gs[2] ** 2
    nG = torch.fft.fftn(n.view(h.grid), norm="forward")
    vH = torch.where(g2 > 0, 4 * math.pi * nG / torch.where(g2 > 0, g2, 1.0), 0.0)
    vH = torch.fft.ifftn(vH, norm="forward").real.reshape(-1)
    vx = -(3.0 * n.clamp(min=0.0) / math.pi) ** (1.0 / 3.0)
    return dict(eval=ev, res=res, rho=rho, vout=h.V + vH + vx)


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        out = []
        for i, x in enumerate(_cells(c)):
            h = _Exact(x, seed * 64 + i)
            X = _block(x["nband"], h.kin.numel(), c["mixed"], seed * 64 + i).to(torch.complex128)
            out.append(_exact_filter(h, X, c["degree"], _bounds(x)))
        return out
    h = _Exact(c, seed)
    if c["kind"] == "scf":
        return _exact_scf(h, c, seed)
    if c["kind"] == "rr":
        X = _filtered(c, h.kin, seed).to(torch.complex128)
        ev, X, _ = _exact_ritz(X, h.H(X))
        return dict(eval=ev, rho=h.density(X, _weights(c["nband"])))
    X = _block(c["nband"], h.kin.numel(), c["mixed"], seed).to(torch.complex128)
    if c["kind"] == "apply":
        return h.H(X)
    if c["kind"] == "adjoint":
        W = _block(c["nband"], h.kin.numel(), c["mixed"], seed + 500000).to(torch.complex128)
        return _exact_adjoint(h, X, W, c["degree"], _bounds(c))
    return _exact_filter(h, X, c["degree"], _bounds(c))

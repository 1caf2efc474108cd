"""Performance cases of the constant-potential electrostatics library.

A case is one call that a program makes in earnest on a capacitor cell of the
shape the workloads have (graphene electrodes, coarse-grained ionic liquid):

    solve      charges, forces and energies of one configuration
    grad       the adjoint loss gradient, forward and backward
    batch      many frames times a sweep of potential differences
    md         a stretch of the constant-potential MD loop
    profile    density and potential profile averaged over a trajectory
    elastance  the elastance matrix of an electrode geometry, its projected
               inverse, and the first solve with it

listed() holds the cases that stand for these uses, draw() gives others of the
same ranges: cells of 256 to 1760 atoms per sheet, finite field, doubled cell
and slab, one or three charged sheets, FP64 and mixed precision, PPPM and (for
the small cell) explicit Ewald, 1 to 4096 frames and 1 to 32 potentials.

prepare() makes the inputs and the context that a program keeps, run() is one
call, exact() the same results in plain 64-bit torch arithmetic.
"""

import functools
import math

import numpy as np
import torch

from paper_2201_12963_amd import Context, MDLoop
from paper_2201_12963_amd.autograd import cpm_loss
from workloads import Workload, md_setup
from workloads.cells import MIN_SEP, electrode, molecule_sizes, random_electrolyte

KE = 1.43996454784           # Coulomb constant, eV nm / e^2
EV_KJ = 96.48533212          # kJ/mol per eV
KB = 0.0083144626            # kJ/mol/K
SPACING = 0.1973             # nm, mesh spacing of the paper-shaped cells (1e-5 force accuracy)
PAIR_DENSITY = 320 / (3.4 * 3.4 * 9.4)   # ion pairs per nm^3 between the electrodes
HONEYCOMB = (3.4 / 11, 0.34)             # rectangular graphene cell of the paper-shaped sheets, nm


def _case(kind, nx=11, ny=10, gap=10.0, pairs=320, geometry="ff", layers=1, kspace="pppm", mixed=False, **more):
    return dict(kind=kind, nx=nx, ny=ny, gap=gap, pairs=pairs, geometry=geometry, layers=layers, kspace=kspace,
                mixed=mixed, **more)


def listed():
    return [
        # the smallest call: the 72-atom test cell with explicit Ewald sums, where launches count
        dict(_case("solve", 6, 3, 4.34, 50, kspace="ewald"), name="solve_small_ewald"),
        # a step of the paper's cell in the finite field (N_e = 880, N_l = 1280), as an MD code calls it
        dict(_case("solve"), name="solve_ff"),
        # and in the doubled cell (N_e = 1760, N_l = 2560), the benchmark's headline
        dict(_case("solve", geometry="dc"), name="solve_dc"),
        # a snapshot re-solved with three sheets charged, slab geometry, a cell of odd sizes
        dict(_case("solve", 9, 9, 7.7, 173, "slab", 3), name="solve_slab_three_sheets"),
        # a step of the four times larger cell in mixed precision (N_e = 3520, N_l = 5120)
        dict(_case("solve", 22, 20, pairs=1280, mixed=True), name="solve_large_mixed"),
        # a training step: loss and gradient of the larger cell
        dict(_case("grad", 22, 20, pairs=1280), name="grad_large"),
        # a stretch of production MD, charges every fifth step
        dict(_case("md", steps=25), name="md_ff"),
        # a few frames at a few potentials: an odd cell, too few frames to fill the chip
        dict(_case("batch", 13, 9, 8.3, 259, frames=37, n_dv=3), name="batch_few_frames"),
        # the largest call: a trajectory's frames times a sweep of potentials
        dict(_case("batch", frames=4096, n_dv=32), name="batch_sweep"),
        # a trajectory of the doubled cell at one potential, mixed precision
        dict(_case("batch", geometry="dc", mixed=True, frames=777, n_dv=1), name="batch_dc_mixed"),
        # the potential profile of a trajectory
        dict(_case("profile", frames=3000, bins=800), name="profile"),
        # a new electrode geometry: elastance, inverse, first solve
        dict(_case("elastance", geometry="dc"), name="elastance_dc"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "grad", "batch", "batch", "batch", "md", "profile", "elastance"])
    if kind in ("solve", "grad") and rng.random() < 0.2:
        # the small cell: narrower than two cutoffs, explicit Ewald sums
        return _case(kind, rng.randint(6, 8), rng.randint(3, 5), round(rng.uniform(3.5, 5.5), 2),
                     rng.randint(31, 60), rng.choice(["ff", "dc"]), kspace="ewald")
    geometry = rng.choice(["ff", "ff", "dc", "slab"])
    layers = rng.choice([1, 1, 3]) if kind in ("solve", "batch", "grad") else 1
    most = (80 if geometry == "dc" else 150) if layers == 3 else 200 if geometry == "dc" else 440
    if kind == "elastance":
        most = {"ff": 200, "dc": 105, "slab": 105}[geometry]
    area = math.exp(rng.uniform(math.log(64), math.log(most)))
    if kind == "md":
        area = max(110.0, min(area, 240.0))       # the Lennard-Jones cutoff needs 3.2 nm across
    nx = max(8, min(22, int(round(math.sqrt(area) * rng.uniform(0.92, 1.08)))))
    ny = max(8, min(20, int(round(area / nx))))
    if kind == "md":
        nx, ny = max(nx, 11), max(ny, 10)
    gap = round(rng.uniform(5.0, 10.0), 2)
    volume = nx * HONEYCOMB[0] * ny * HONEYCOMB[1] * (gap - 2 * MIN_SEP)
    pairs = int(volume * PAIR_DENSITY * rng.uniform(0.75, 1.0))
    more = {}
    if kind == "batch":
        cost = pairs / 320 * (2 if geometry == "dc" else 1) * (1.5 if layers == 3 else 1)
        more["frames"] = max(1, min(4096, int(_log_int(rng, 1, 4096) / (1.3 * cost))))
        more["n_dv"] = min(_log_int(rng, 1, 32), max(1, int(24 * 4096 / (cost * more["frames"]))))
    elif kind == "md":
        more["steps"] = rng.randint(5, 40)
    elif kind == "profile":
        more["frames"] = _log_int(rng, 1, 4096)
        more["bins"] = rng.randint(100, 2048)
    mixed = kind in ("solve", "batch") and rng.random() < 0.25
    return _case(kind, nx, ny, gap, pairs, geometry, layers, mixed=mixed, **more)


# ------------------------------------------------------------------- inputs

def _smooth(n):
    """The smallest product of 2, 3 and 5 that is at least n."""
    while True:
        m = n
        for p in (2, 3, 5):
            while m % p == 0:
                m //= p
        if m == 1:
            return n
        n += 1


@functools.lru_cache(maxsize=None)
def _cell(nx, ny, gap, pairs, geometry, layers, kspace):
    """The cell of a case: electrodes, ions placed at random, and the numerical parameters."""
    if kspace == "ewald":
        lx, ly, lz, z_lo, sites = nx * 0.246, ny * 0.42608, gap + 1.66, 0.0, 1
        par = dict(alpha=2.97, rcut=1.2, kcut=24.0, alpha_exact=2.97, rcut_exact=2.0, kcut_exact=33.0)
    else:
        lx, ly, lz, z_lo, sites = nx * HONEYCOMB[0], ny * HONEYCOMB[1], gap + 2.625, 1.3125, 3
        par = dict(alpha=2.21, rcut=1.2, kcut=0.0, alpha_exact=2.21, rcut_exact=2.7, kcut_exact=24.5)
        if lx * ly > 30.0:
            par.update(alpha_exact=1.6, rcut_exact=3.7, kcut_exact=17.5)
    z_hi = z_lo + gap
    mesh = [_smooth(int(math.ceil(L / SPACING))) for L in (lx, ly, lz)]
    lo, lo_l = electrode(nx, ny, lx, ly, z_lo, -1, 3)
    hi, hi_l = electrode(nx, ny, lx, ly, z_hi, +1, 3)
    lj = np.concatenate([lo, hi], axis=1)
    lo, lo_l, hi, hi_l = lo[:, lo_l < layers], lo_l[lo_l < layers], hi[:, hi_l < layers], hi_l[hi_l < layers]
    x, q = random_electrolyte(np.random.default_rng(nx * ny + pairs), pairs, lx, ly, z_lo + MIN_SEP, z_hi - MIN_SEP,
                              sites)
    e, n = np.concatenate([lo, hi], axis=1), lo.shape[1]
    side, lay = np.repeat(np.array([-1, 1], np.int8), n), np.concatenate([lo_l, hi_l])
    sub, mol = None, molecule_sizes(q)
    zmin, zmax = np.full(q.shape, z_lo + MIN_SEP), np.full(q.shape, z_hi - MIN_SEP)
    box = np.array([lx, ly, lz])
    if geometry == "dc":      # a second cell on top: electrodes shifted, polarity swapped, electrolyte mirrored
        up = np.array([[0.0], [0.0], [lz]])
        x2 = x.copy()
        x2[2] = lz + z_lo + z_hi - x[2]
        sub = np.repeat(np.array([1, 0], np.uint8), 2 * n)
        e, side, lay = np.concatenate([e, e + up], axis=1), np.concatenate([side, -side]), np.tile(lay, 2)
        lj, x, q, mol = np.concatenate([lj, lj + up], axis=1), np.concatenate([x, x2], axis=1), np.tile(q, 2), np.tile(mol, 2)
        zmin, zmax = np.concatenate([zmin, zmin + lz]), np.concatenate([zmax, zmax + lz])
        box[2], mesh[2] = 2 * lz, 2 * mesh[2]
    elif geometry == "slab":  # the cell in the middle of a period three times as long
        up = np.array([[0.0], [0.0], [lz]])
        e, lj, x, zmin, zmax = e + up, lj + up, x + up, zmin + lz, zmax + lz
        box[2], mesh[2] = 3 * lz, _smooth(3 * mesh[2])
    return Workload(name="cell", geometry=geometry, box=box, eta=19.79, kspace=kspace, mesh=tuple(mesh), order=5,
                    elec_xyz=np.ascontiguousarray(e), elec_side=side, elec_sub=sub, elec_layer=lay,
                    site_xyz=np.ascontiguousarray(x), site_q=q, site_zmin=zmin, site_zmax=zmax, mol_size=mol,
                    lj_elec_xyz=lj, **par)


def _workload(case):
    return _cell(case["nx"], case["ny"], case["gap"], case["pairs"], case["geometry"], case["layers"], case["kspace"])


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _inputs(case, seed):
    """The case's tensors, from the seed alone."""
    w, dev = _workload(case), _device()
    g = torch.Generator(device=dev).manual_seed(seed)
    box = torch.tensor(w.box, device=dev)
    base = torch.tensor(w.site_xyz, device=dev)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float64)

    if case["kind"] == "md":
        # whole molecules moved a little (the cations stay rigid), velocities at 400 K
        s = md_setup(w)
        mol = torch.tensor(np.repeat(np.arange(w.mol_size.size), w.mol_size), device=dev)
        x = base + 0.01 * normal(3, w.mol_size.size)[:, mol]
        v = normal(3, w.n_site) * torch.tensor(np.sqrt(KB * s.temperature / s.site_mass), device=dev)
        return dict(x=x.contiguous(), v=v.contiguous(), dv=2.0)
    frames = case.get("frames", 1)
    x = base[None] + 0.05 * normal(frames, 3, w.n_site)
    x -= box[None, :, None] * torch.floor(x / box[None, :, None])
    if case["kind"] == "batch":
        return dict(x=x, dvs=np.linspace(0.0, 4.0, case["n_dv"]) if case["n_dv"] > 1 else np.array([2.0]))
    if case["kind"] == "profile":
        # charges of the size a 2 V solve gives: polarised per electrode, each frame neutral
        side = torch.tensor(w.elec_side.astype(np.float64), device=dev)
        q = 0.01 * normal(frames, w.n_elec) + 0.005 * side
        return dict(x=x, q=q - q.mean(1, keepdim=True), dv=2.0, bulk=(w.box[2] * 0.4, w.box[2] * 0.6))
    return dict(x=x[0].contiguous(), dv=2.0, target=0.01 * normal(w.n_elec))


_STREAM = []


def _stream():
    """The program's one stream: every state's calls go through it."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def prepare(case, seed):
    w, s = _workload(case), _stream()
    st = dict(kind=case["kind"], **_inputs(case, seed))
    torch.cuda.current_stream().synchronize()
    with torch.cuda.stream(s):
        ctx = Context.from_workload(w, precision=1 if case["mixed"] else 0, stream=s)
        if case["kind"] != "elastance":
            ctx.build_elastance()
        st["ctx"] = ctx
        if case["kind"] == "md":
            st["md"], st["steps"] = MDLoop(ctx, md_setup(w)), case["steps"]
        if case["kind"] == "grad":
            st["x"].requires_grad_(True)
            st["dv"] = torch.tensor(st["dv"], dtype=torch.float64, requires_grad=True)
        if case["kind"] == "profile":
            st["bins"] = case["bins"]
    return st


def run(st):
    kind, ctx = st["kind"], st["ctx"]
    with torch.cuda.stream(_stream()):
        if kind == "solve":
            return ctx.solve(st["x"], st["dv"])
        if kind == "grad":
            loss, q = cpm_loss(ctx, st["x"], st["dv"], st["target"])
            dx, ddv = torch.autograd.grad(loss, (st["x"], st["dv"]))
            return loss.detach(), dx, ddv, q
        if kind == "batch":
            return ctx.solve_batch(st["x"], st["dvs"])
        if kind == "md":
            q, thermo = st["md"].run(st["x"], st["v"], st["dv"], st["steps"])
            return st["x"], st["v"], q, thermo
        if kind == "profile":
            return ctx.profile(st["x"], st["q"], st["dv"], st["bins"], st["bulk"])
        ctx.build_elastance()
        return ctx.solve(st["x"], st["dv"])


def work(case):
    """Inputs read once and outputs written once; S counts as an input of every call that solves.
    Operations: 2 per element of S and frame, 50 per site pair and 130 per electrode pair within the cutoff (b and
    force), the mesh transforms (5 N log2 N each, 1 + 1 + 1 + 3) and 5^3 stencil points per particle, both ways."""
    w = _workload(case)
    ne, ns, frames, n_dv = w.n_elec, w.n_site, case.get("frames", 1), case.get("n_dv", 1)
    if case["kind"] == "profile":
        return dict(bytes=8.0 * frames * (ns + ne) + 16.0 * case["bins"], flops=4.0 * frames * (ns + ne))
    vol = float(w.box[0] * w.box[1]) * (case["gap"] - 2 * MIN_SEP) * (2 if case["geometry"] == "dc" else 1)
    near = 2 * math.pi / 3 * w.rcut ** 3 * ns / vol              # partners per site, each pair once
    face = math.pi * w.rcut ** 3 * 0.2 * ns / vol                # sites within reach of an electrode atom
    M = float(np.prod(w.mesh))
    fft = 6 * 5 * M * math.log2(M) + 2 * 2 * 125 * (ns + ne) if w.kspace == "pppm" else 0.0
    per_frame = 50 * near * ns + 130 * face * ne + fft + 2.0 * ne * ne
    inputs, s = 8.0 * 3 * ns, 8.0 * ne * ne
    outputs = 8.0 * (ne + 3 * ns + 2)
    if case["kind"] == "md":
        steps = case["steps"]
        return dict(bytes=2 * 2 * inputs + 8.0 * ne + 32.0 * steps + s * (steps // 5), flops=steps * per_frame)
    if case["kind"] == "grad":
        return dict(bytes=inputs + 2 * s + outputs + 8.0 * ne, flops=per_frame + 2.0 * ne * ne)
    if case["kind"] == "elastance":
        kvecs = 0.5 * 4 / 3 * math.pi * w.kcut_exact ** 3 / (2 * math.pi) ** 3 * float(np.prod(w.box))
        return dict(bytes=24.0 * ne + 2 * s + inputs + outputs, flops=2.0 * kvecs * ne * ne + 2.0 * ne ** 3 + per_frame)
    return dict(bytes=frames * (inputs + n_dv * outputs) + s, flops=frames * per_frame)


# ------------------------------------------- the same results in plain torch

def _t(a, dev=None):
    return torch.as_tensor(np.asarray(a, dtype=np.float64), device=dev or _device())


def _images(box, rcut):
    m = [int(math.floor(rcut / L + 0.5)) for L in box]
    return [(a, b, c) for a in range(-m[0], m[0] + 1) for b in range(-m[1], m[1] + 1) for c in range(-m[2], m[2] + 1)]


def _pairs(xa, xb, box, rcut, same, body):
    """body(d, r, inside) for every chunk and periodic image: d the three components of xa - xb + n L.
    xa [.., 3, na], xb [.., 3, nb]."""
    L = [float(v) for v in box]
    for n in _images(box, rcut):
        d = []
        for k in range(3):
            t = xa[..., k, :, None] - xb[..., k, None, :]
            d.append(t - L[k] * torch.round(t / L[k]) + n[k] * L[k])
        r = torch.sqrt(d[0] ** 2 + d[1] ** 2 + d[2] ** 2)
        inside = r < rcut
        if same and n == (0, 0, 0):
            inside = inside & ~torch.eye(r.shape[-1], dtype=torch.bool, device=r.device)
        body(d, torch.where(inside, r, torch.ones_like(r)), inside)


def _erfc_r(a, r):
    return torch.special.erfc(a * r) / r


def _slope(a, r):
    """-d/dr of erfc(a r)/r."""
    return torch.special.erfc(a * r) / r ** 2 + 2 * a / math.sqrt(math.pi) * torch.exp(-(a * r) ** 2) / r


class _Exact:
    """The cell's electrostatics in 64 bits: PPPM (or Ewald) sums over frames [F, 3, n]."""

    def __init__(self, w):
        self.w, self.box = w, [float(v) for v in w.box]
        self.vol = float(np.prod(w.box))
        self.e, self.q = _t(w.elec_xyz), _t(w.site_q)
        self.ze = self.e[2] - self.box[2] * torch.floor(self.e[2] / self.box[2])
        self.d = 0.5 * _t(w.elec_side)
        self.c = self.d - self.ze / self.box[2] if w.geometry == "ff" else self.d
        self.kappa = KE * 4 * math.pi / self.vol if w.geometry == "slab" else 0.0
        self.A, self.S = self._matrices()
        if w.kspace == "pppm":
            self.G, self.D = self._influence()
        else:
            self.k = self._kvectors(w.kcut)
            self.wk = self._weight(self.k, w.alpha)

    def _kvectors(self, kcut):
        m = [int(math.floor(kcut * L / (2 * math.pi))) for L in self.box]
        n = np.stack(np.meshgrid(*[np.arange(-v, v + 1) for v in m], indexing="ij"), -1).reshape(-1, 3)
        k = 2 * math.pi * n / np.array(self.box)
        k2 = (k * k).sum(1)
        half = (n[:, 0] > 0) | ((n[:, 0] == 0) & ((n[:, 1] > 0) | ((n[:, 1] == 0) & (n[:, 2] > 0))))
        return _t(k[half & (k2 <= kcut * kcut)])

    def _weight(self, k, alpha):
        k2 = (k * k).sum(1)
        return 2 * 4 * math.pi / self.vol * torch.exp(-k2 / (4 * alpha * alpha)) / k2      # both k and -k

    def _matrices(self):
        w, n = self.w, self.w.n_elec
        a, g = w.alpha_exact, w.eta / math.sqrt(2.0)
        A = torch.zeros((n, n), dtype=torch.float64, device=self.e.device)
        for i in range(0, n, 256):
            def add(d, r, inside):
                v = torch.where(inside, _erfc_r(a, r) - _erfc_r(g, r), torch.zeros_like(r))
                A[i:i + 256] += v
            # (an atom's own image at n = 0 sits on the shifted diagonal of this block)
            def off_diagonal(d, r, inside):
                add(d, r, inside & (d[0] ** 2 + d[1] ** 2 + d[2] ** 2 > 1e-20))
            _pairs(self.e[:, i:i + 256], self.e, w.box, w.rcut_exact, False, off_diagonal)
        k = self._kvectors(w.kcut_exact)
        wt = torch.sqrt(self._weight(k, a))
        for i in range(0, k.shape[0], 8192):
            ph = k[i:i + 8192] @ self.e
            for f in (torch.cos(ph), torch.sin(ph)):
                f = f * wt[i:i + 8192, None]
                A += f.T @ f
        A += torch.eye(n, dtype=torch.float64, device=A.device) * (math.sqrt(2.0) * w.eta - 2 * a) / math.sqrt(math.pi)
        A = KE * A + self.kappa * torch.outer(self.ze, self.ze)
        S = torch.linalg.inv(A.cpu()).to(A.device)
        S = 0.5 * (S + S.T)
        for v in [torch.ones(n, dtype=torch.float64, device=A.device)] + (
                [_t(w.elec_sub)] if w.geometry == "dc" else []):
            u = S @ v
            S = S - torch.outer(u, u) / (v @ u)
        return A, S

    def _influence(self):
        w, P = self.w, self.w.order
        ns = [np.rint(np.fft.fftfreq(K, 1.0 / K)).astype(int) for K in w.mesh]
        k = [2 * math.pi * n / L for n, L in zip(ns, self.box)]
        num, den = 0.0, 0.0
        alias = []
        for n, K, L in zip(ns, w.mesh, self.box):
            rows = []
            for m in range(-3, 4):
                nm = n + m * K
                x = math.pi * nm / K
                u2 = np.where(x == 0, 1.0, np.sin(x) / np.where(x == 0, 1.0, x)) ** (2 * P)
                rows.append((_t(2 * math.pi * nm / L), _t(np.where(np.abs(nm) <= 2.5 * K, u2, 0.0))))
            alias.append(rows)
        kx, ky, kz = _t(k[0])[:, None, None], _t(k[1])[None, :, None], _t(k[2])[None, None, :]
        k2 = kx ** 2 + ky ** 2 + kz ** 2
        for ax, ux in alias[0]:
            for ay, uy in alias[1]:
                for az, uz in alias[2]:
                    u2 = ux[:, None, None] * uy[None, :, None] * uz[None, None, :]
                    q2 = ax[:, None, None] ** 2 + ay[None, :, None] ** 2 + az[None, None, :] ** 2
                    safe = torch.where(q2 == 0, torch.ones_like(q2), q2)
                    R = torch.where(q2 == 0, torch.zeros_like(q2), 4 * math.pi * torch.exp(-safe / (4 * w.alpha ** 2)) / safe)
                    num = num + u2 * R * (kx * ax[:, None, None] + ky * ay[None, :, None] + kz * az[None, None, :])
                    den = den + u2
        G = torch.where(k2 > 0, num / (torch.where(k2 > 0, k2, torch.ones_like(k2)) * den ** 2), torch.zeros_like(k2))
        D = [_t(np.where((K % 2 == 0) & (n == -(K // 2)), 0.0, kk)) for n, K, kk in zip(ns, w.mesh, k)]
        return G, [D[0][:, None, None], D[1][None, :, None], D[2][None, None, :]]

    def _stencil(self, x):
        """Mesh index and weight of the P^3 points of every particle: x [F, 3, n] -> [F, n, P^3] each."""
        w, P = self.w, self.w.order

        def spline(order, t):
            if order == 1:
                return ((t >= 0) & (t < 1)).to(t.dtype)
            return (t * spline(order - 1, t) + (order - t) * spline(order - 1, t - 1)) / (order - 1)

        idx, wt = [], []
        for k in range(3):
            K, L = w.mesh[k], self.box[k]
            u = (x[:, k] - L * torch.floor(x[:, k] / L)) / (L / K)
            first = torch.floor(u - P / 2.0).to(torch.int64) + 1
            m = first[..., None] + torch.arange(P, device=x.device)
            idx.append(torch.remainder(m, K))
            wt.append(spline(P, u[..., None] - m + P / 2.0))
        shape = x.shape[0], x.shape[2], P ** 3
        index = (idx[0][..., :, None, None] * w.mesh[1] + idx[1][..., None, :, None]) * w.mesh[2] + idx[2][..., None, None, :]
        weight = wt[0][..., :, None, None] * wt[1][..., None, :, None] * wt[2][..., None, None, :]
        return index.reshape(shape), weight.reshape(shape)

    def _spread(self, st, q):
        """Charge mesh [F, Kx, Ky, Kz]; q [F or 1, n]."""
        idx, wt = st
        F, M = idx.shape[0], int(np.prod(self.w.mesh))
        mesh = torch.zeros(F * M, dtype=torch.float64, device=wt.device)
        at = idx + torch.arange(F, device=idx.device)[:, None, None] * M
        mesh.index_add_(0, at.reshape(-1), (wt * q[..., None]).reshape(-1))
        return mesh.reshape(F, *self.w.mesh)

    def _gather(self, st, mesh):
        idx, wt = st
        flat = mesh.reshape(mesh.shape[0], -1)
        return (torch.gather(flat, 1, idx.reshape(idx.shape[0], -1)).reshape(idx.shape) * wt).sum(-1)

    def _field(self, rho_hat, st, scale):
        return torch.stack([scale * self._gather(st, torch.fft.ifftn(-1j * D * self.G * rho_hat, dim=(1, 2, 3)).real)
                            for D in self.D], 1)

    def frames(self, x):
        """Everything about frames x [F, 3, n] that does not need electrode charges: b, U_elyt, and a function
        of charges q [F, n_elec] giving the Coulomb forces [F, 3, n] (linear part and constant part apart)."""
        w, F = self.w, x.shape[0]
        phi = torch.zeros((F, w.n_elec), dtype=torch.float64, device=x.device)
        u_pair = torch.zeros(F, dtype=torch.float64, device=x.device)
        f_pair = torch.zeros((F, 3, w.n_site), dtype=torch.float64, device=x.device)
        near = []

        def elec(d, r, inside):
            z = torch.zeros_like(r)
            phi.add_(torch.where(inside, _erfc_r(w.alpha, r) - _erfc_r(w.eta, r), z).transpose(1, 2) @ self.q)
            s = torch.where(inside, (_slope(w.alpha, r) - _slope(w.eta, r)) / r, z)
            near.append([s * t for t in d])

        def site(d, r, inside):
            z = torch.zeros_like(r)
            u_pair.add_(0.5 * ((torch.where(inside, _erfc_r(w.alpha, r), z) @ self.q) * self.q).sum(-1))
            s = torch.where(inside, _slope(w.alpha, r) / r, z)
            for k in range(3):
                f_pair[:, k] += (s * d[k]) @ self.q

        _pairs(x, self.e, w.box, w.rcut, False, elec)
        _pairs(x, x, w.box, w.rcut, True, site)
        self_e = w.alpha / math.sqrt(math.pi) * (self.q ** 2).sum()
        if w.kspace == "pppm":
            M = float(np.prod(w.mesh))
            st, se = self._stencil(x), self._stencil(self.e[None])
            rho = self._spread(st, self.q[None])
            hat = torch.fft.fftn(rho, dim=(1, 2, 3))
            pot = torch.fft.ifftn(self.G * hat, dim=(1, 2, 3)).real * (M / self.vol)
            many = tuple(t.expand(F, -1, -1) for t in se)
            phi_k = self._gather(many, pot)
            u_k = 0.5 * (rho * pot).sum((1, 2, 3))
            site_field = self._field(hat, st, M / self.vol)

            def elec_field(q):
                h = torch.fft.fftn(self._spread(many, q), dim=(1, 2, 3))
                return self._field(h, st, M / self.vol)
        else:
            cs, sn = torch.cos(self.k @ x[0]), torch.sin(self.k @ x[0])
            ce, se = torch.cos(self.k @ self.e), torch.sin(self.k @ self.e)
            re, im = cs @ self.q, sn @ self.q
            phi_k = ((self.wk * re) @ ce + (self.wk * im) @ se)[None]
            u_k = 0.5 * (self.wk * (re ** 2 + im ** 2)).sum()[None]

            def of(re, im):
                return (-(self.k * self.wk[:, None]).T @ (cs * im[:, None] - sn * re[:, None]))[None]

            site_field = of(re, im)

            def elec_field(q):
                return of(ce @ q[0], se @ q[0])
        zs = x[:, 2] - self.box[2] * torch.floor(x[:, 2] / self.box[2])
        dip = zs @ self.q
        b = -KE * (phi + phi_k) - self.kappa * dip[:, None] * self.ze
        u = KE * (u_pair + u_k - self_e) + 0.5 * self.kappa * dip ** 2
        fixed = KE * self.q * (f_pair + site_field)
        fixed[:, 2] -= self.kappa * self.q * dip[:, None]

        def force_of(q):
            f = elec_field(q)
            for parts in near:
                for k in range(3):
                    f[:, k] += (parts[k] @ q[..., None])[..., 0]
            f = KE * self.q * f
            f[:, 2] -= self.kappa * self.q * (q @ self.ze)[:, None]
            return f

        return b, u, dip, fixed, force_of

    def energies(self, q, b, u, dip, dv):
        coul = u - (q * b).sum(-1) + 0.5 * ((q @ self.A) * q).sum(-1)
        cp = coul - dv * (q @ self.d)
        if self.w.geometry == "ff":
            cp = cp + dv / self.box[2] * (q @ self.ze + dip)
        return coul, cp

    def solve(self, x, dvs):
        """q [F, V, n_elec], f [F, V, 3, n], e [F, V, 2]."""
        b, u, dip, fixed, force_of = self.frames(x)
        q0, qc = b @ self.S.T, self.S @ self.c
        f0, f1 = fixed + force_of(q0), force_of(qc.expand(x.shape[0], -1).contiguous())
        if self.w.geometry == "ff":
            f1[:, 2] -= self.q / self.box[2]
        q = torch.stack([q0 + v * qc for v in dvs], 1)
        e = torch.stack([torch.stack(self.energies(q[:, i], b, u, dip, v), -1) for i, v in enumerate(dvs)], 1)
        return q, torch.stack([f0 + v * f1 for v in dvs], 1), e


@functools.lru_cache(maxsize=2)
def _exact_of(*key):
    return _Exact(_cell(*key))


def exact(case, seed):
    w, p = _workload(case), _inputs(case, seed)
    if case["kind"] == "profile":
        return _exact_profile(w, p, case["bins"])
    ex = _exact_of(case["nx"], case["ny"], case["gap"], case["pairs"], case["geometry"], case["layers"], case["kspace"])
    if case["kind"] == "batch":
        q = torch.empty((case["frames"], case["n_dv"], w.n_elec), dtype=torch.float64, device=_device())
        f = torch.empty((case["frames"], case["n_dv"], 3, w.n_site), dtype=torch.float64, device=_device())
        e = torch.empty((case["frames"], case["n_dv"], 2), dtype=torch.float64, device=_device())
        step = max(1, int(1.5e8 / (w.n_site * max(w.n_site, w.n_elec))))
        for i in range(0, case["frames"], step):
            q[i:i + step], f[i:i + step], e[i:i + step] = ex.solve(p["x"][i:i + step], [float(v) for v in p["dvs"]])
        return q, f, e
    if case["kind"] == "md":
        return _exact_md(w, ex, p, case["steps"])
    if case["kind"] == "grad":
        b, u, dip, fixed, force_of = ex.frames(p["x"][None])
        q = b[0] @ ex.S.T + p["dv"] * (ex.S @ ex.c)
        coul, _ = ex.energies(q[None], b, u, dip, p["dv"])
        lam = ex.S @ (2 * (q - p["target"]) + p["dv"] * ex.c)
        dx = -(fixed + force_of((q - lam)[None]))[0]
        return ((q - p["target"]) ** 2).sum() + coul[0], dx, lam @ ex.c, q
    q, f, e = ex.solve(p["x"][None], [p["dv"]])
    return q[0, 0], f[0, 0], e[0, 0]


def _exact_profile(w, p, n):
    lz, area = float(w.box[2]), float(w.box[0] * w.box[1])
    h = lz / n
    z = p["x"][:, 2] - lz * torch.floor(p["x"][:, 2] / lz)
    k = torch.clamp((z / h).to(torch.int64), max=n - 1)
    charge = torch.zeros(n, dtype=torch.float64, device=z.device)
    for i in range(0, z.shape[0], 256):
        charge.index_add_(0, k[i:i + 256].reshape(-1), _t(w.site_q).expand(k[i:i + 256].shape).reshape(-1))
    e = _t(w.elec_xyz)[2]
    e = e - lz * torch.floor(e / lz)
    edges = torch.arange(n + 1, device=z.device, dtype=torch.float64) * h
    qsum = p["q"].sum(0)
    for m in (-1, 0, 1):
        cdf = 0.5 * torch.special.erf(w.eta * (edges[None] - (e + m * lz)[:, None]))
        charge += qsum @ (cdf[:, 1:] - cdf[:, :-1])
    rho = charge / z.shape[0] / (area * h)
    # psi'' = -rho/eps0 by second differences, with the ends of the geometry
    r = (-rho * (4 * math.pi * KE)).cpu().numpy()
    A = np.zeros((n + 1, n + 1))
    i = np.arange(n)
    A[i, i] = -2.0
    A[i[1:], i[:-1]] = A[i[:-1], i[1:]] = 1.0
    if w.geometry == "slab":
        A[0, 0] = A[n - 1, n - 1] = -1.0
    else:
        A[0, n - 1] += 1.0
        A[n - 1, 0] += 1.0
    rhs = np.concatenate([r * h * h, [0.0]])
    if w.geometry == "ff":
        rhs[0] += p["dv"]
        rhs[n - 1] -= p["dv"]
    A[:n, n] = A[n, :n] = 1.0
    psi = np.linalg.solve(A, rhs)[:n]
    zc = (i + 0.5) * h
    return rho, _t(psi - psi[(zc >= p["bulk"][0]) & (zc < p["bulk"][1])].mean())


def _exact_md(w, ex, p, steps):
    s, box = md_setup(w), _t(w.box)[:, None]
    dev = box.device
    m, dt, kt = _t(s.site_mass), s.dt, KB * s.temperature
    size = torch.tensor(s.mol_size, device=dev)
    mol = torch.repeat_interleave(torch.arange(size.numel(), device=dev), size)
    group = torch.tensor(s.mol_group, device=dev).to(torch.int64)[mol]
    first = (torch.cumsum(size, 0) - size)[size == 3]
    tri = [(first, first + 1, s.bond), (first, first + 2, s.bond), (first + 1, first + 2, s.bond * math.sqrt(3.0))]
    nf = torch.stack([3.0 * (group == g).sum() - 3.0 * (group[first] == g).sum() for g in range(s.n_groups)])
    Q = nf * kt * s.tau ** 2
    image = lambda d: d - box * torch.round(d / box)  # noqa: E731
    sides = lambda x: [image(x[:, i] - x[:, j]) for i, j, _ in tri]  # noqa: E731

    def pulls(dirs, lam):
        """Displacement of every site by the three multipliers along `dirs`, times 1/m."""
        out = torch.zeros((3, w.n_site), dtype=torch.float64, device=dev)
        for (i, j, _), d, l in zip(tri, dirs, lam):
            out.index_add_(1, i, l * d)
            out.index_add_(1, j, -l * d)
        return out / m

    def system(rows, dirs):
        """Jacobian [mol, 3, 3] of the three sides' projections on `rows` under the pulls along `dirs`."""
        J = torch.zeros((first.numel(), 3, 3), dtype=torch.float64, device=dev)
        for b, (i, j, _) in enumerate(tri):
            for a, (k, l, _) in enumerate(tri):
                t = ((k == i).double() / m[k] - (k == j).double() / m[k] - (l == i).double() / m[l] + (l == j).double() / m[l])
                J[:, a, b] = t * (rows[a] * dirs[b]).sum(0)
        return J

    def shake(x, x_old):
        old = sides(x_old)
        for _ in range(12):
            r = sides(x)
            gap = torch.stack([0.5 * (d * d - (v * v).sum(0)) for (_, _, d), v in zip(tri, r)], 1)
            x = x + pulls(old, torch.linalg.solve(system(r, old).cpu(), gap.cpu()).to(dev).T)
        return x

    def rattle(v, x):
        r = sides(x)
        rel = torch.stack([((v[:, i] - v[:, j]) * d).sum(0) for (i, j, _), d in zip(tri, r)], 1)
        return v - pulls(r, torch.linalg.solve(system(r, r).cpu(), rel.cpu()).to(dev).T)

    carbon = _t(s.lj_elec_xyz)
    sig, eps = _t(s.site_sigma), _t(s.site_eps)

    def lj_part(x, y, sg, ep, keep):
        d = [x[k][:, None] - y[k][None] for k in range(3)]
        d = [t - float(w.box[k]) * torch.round(t / float(w.box[k])) for k, t in enumerate(d)]
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2
        ok = keep & (r2 < s.lj_cut ** 2) & (r2 > 0)
        r2 = torch.where(ok, r2, torch.ones_like(r2))
        a, c = (sg * sg / r2) ** 3, (sg * sg / s.lj_cut ** 2) ** 3
        u = torch.where(ok, 4 * ep * (a * a - a - c * c + c), torch.zeros_like(r2))
        f = torch.where(ok, 24 * ep * (2 * a * a - a) / r2, torch.zeros_like(r2))
        return torch.stack([(f * t).sum(1) for t in d]), u.sum()

    def lj(x):
        f, u = lj_part(x, x, 0.5 * (sig[:, None] + sig), torch.sqrt(eps[:, None] * eps), mol[:, None] != mol)
        g, t = lj_part(x, carbon, 0.5 * (sig[:, None] + s.carbon_sigma),
                       torch.sqrt(eps[:, None] * s.carbon_eps).expand(-1, carbon.shape[1]), True)
        return f + g, 0.5 * u + t

    def forces(x, q):
        b, u, dip, fixed, force_of = ex.frames(x[None])
        e = None
        if q is None:
            q = b[0] @ ex.S.T + p["dv"] * (ex.S @ ex.c)
            e = ex.energies(q[None], b, u, dip, p["dv"])[1][0]
        f = (fixed + force_of(q[None]))[0]
        if w.geometry == "ff":
            f[2] -= ex.q * p["dv"] / w.box[2]
        g, u_lj = lj(x)
        return g + EV_KJ * f, q, u_lj, e

    xi = torch.zeros(s.n_groups, dtype=torch.float64, device=dev)
    eta = torch.zeros_like(xi)

    def k2(v):
        return torch.zeros_like(xi).index_add_(0, group, m * (v * v).sum(0))

    def half(v):
        k = k2(v)
        xi.add_(0.25 * dt * (k - nf * kt) / Q)
        eta.add_(0.5 * dt * xi)
        scale = torch.exp(-0.5 * dt * xi)
        xi.add_(0.25 * dt * (k * scale * scale - nf * kt) / Q)
        return v * scale[group]

    x, v = p["x"], rattle(p["v"], p["x"])
    f, q, _, e_cp = forces(x, None)
    rows = []
    for n in range(1, steps + 1):
        v = half(v) + 0.5 * dt * f / m
        new = shake(x + dt * v, x)
        v, x = (new - x) / dt, new
        update = n % s.charge_every == 0
        f, q, u_lj, e = forces(x, None if update else q)
        e_cp = e if update else e_cp
        v = half(rattle(v + 0.5 * dt * f / m, x))
        rows.append(torch.stack([0.5 * k2(v).sum(), u_lj, EV_KJ * e_cp, (0.5 * Q * xi ** 2 + nf * kt * eta).sum()]))
    return x, v, q, torch.stack(rows)

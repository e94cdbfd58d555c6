"""Performance cases of the ChFSI library: what a user's program has it do.

Each case is one call (or the few calls that belong together) through the
Python binding, at sizes of the named workloads (`synth/workloads.py`), of the
GPU tests and of the density network's training.  Clusters are hydrogen-
passivated Si spheres on the h = 0.7 bohr grid; `d` is the cluster's diameter
in nm, `m` the number of vectors.

`exact` gives the same results in 64 bits from the definitions alone: the
spherical grid on a cubic box, the 37-point star as shifted rows, the
projectors as (point, atom) pairs, the network as sums of shifted matrix
products.  Only the rows' order (blocks of 8^3 points along a Hilbert curve)
and the weights' layout follow the library's documented formats.
"""
from __future__ import annotations

import math
import os

import numpy as np
import torch

from paper_2303_00790_amd import binding as B
from paper_2303_00790_amd import scf as S
from synth.cluster import make_cluster, n_states
from synth.workloads import MODEL_PP as PP

H = 0.7
HALF = 6
BOHR = 0.529177210903            # angstrom, only for size estimates
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WEIGHTS = os.path.join(ROOT, "results", "dnet_c32.npy")
DT = {"f32": torch.float32, "f64": torch.float64}


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: H times two FP64 vectors (a residual check, one
        # Lanczos step) on the SCF-parity cluster Si35H36
        {"name": "apply-1.1nm-f64-2", "kind": "apply", "d": 1.1, "dtype": "f64", "m": 2},
        # a ChFSI filter of the SCF-parity workload: 128 FP64 states, degree 10
        {"name": "filter-1.1nm-f64-128", "kind": "filter", "d": 1.1, "dtype": "f64", "m": 128, "w": 128, "degree": 10},
        # a ragged block: an odd number of FP64 vectors with no padding
        {"name": "filter-2nm-f64-97", "kind": "filter", "d": 2.0, "dtype": "f64", "m": 97, "w": 97, "degree": 10},
        # the FP64 filter workload (3 nm, one 128-vector block, degree 12)
        {"name": "filter-3nm-f64-128", "kind": "filter", "d": 3.0, "dtype": "f64", "m": 128, "w": 128, "degree": 12},
        # the filter inside a mixed-precision SCF step: all 1024 states of the
        # 2.5 nm cluster through a 256-column work block (four column blocks)
        {"name": "filter-2.5nm-f32-1024", "kind": "filter", "d": 2.5, "dtype": "f32", "m": 1024, "w": 256, "degree": 12},
        # the mixed-precision workload at scale (5 nm, 256 FP32 vectors)
        {"name": "filter-5nm-f32-256", "kind": "filter", "d": 5.0, "dtype": "f32", "m": 256, "w": 256, "degree": 12},
        # the spectrum's upper bound, taken in every SCF step
        {"name": "lanczos-3nm", "kind": "lanczos", "d": 3.0, "k": 10},
        # a Hartree potential from zero, as in the first SCF step
        {"name": "hartree-2.5nm", "kind": "hartree", "d": 2.5},
        # Cholesky-QR of a filtered block: all FP32 states of the 2.5 nm cluster
        {"name": "ortho-2.5nm-f32-1024", "kind": "ortho", "d": 2.5, "dtype": "f32", "m": 1024},
        # the first SCF step (four ChFSI iterations) of the parity workload
        {"name": "scf-1.1nm-f64", "kind": "scf", "d": 1.1, "degree": 10},
        # the learned start density of a 2.5 nm cluster: network and high-pass
        # on its 96^3 box
        {"name": "net-predict-96", "kind": "predict", "edge": 96, "sigma": 8.0},
        # one training step on a 64^3 patch, the edge the network is trained on
        {"name": "net-train-64", "kind": "train", "edge": 64, "batch": 1},
    ]


def _points(d):
    """About the number of grid points of a cluster of diameter d."""
    return 4.0 / 3.0 * math.pi * ((5.0 * d / BOHR + 7.5) / H) ** 3


def draw(rng):
    def spread(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    kind = rng.choice(["filter", "filter", "filter", "apply", "lanczos", "hartree", "ortho", "scf", "predict", "train"])
    if kind in ("filter", "apply"):
        dtype = rng.choice(["f32", "f64"])
        d = round(spread(1.0, 4.5), 2)
        degree = rng.randint(8, 16) if kind == "filter" else 1
        # no more values than the 5 nm case moves; an odd FP32 width takes the
        # neighbour-table kernel, which is several times slower
        most = 2.0e6 * 256 * 12 * 4 / (_points(d) * degree * (4 if dtype == "f32" else 8))
        m = int(spread(1, min(1024, max(2.0, 0.5 * most))))
        if dtype == "f32" and m % 2 and m > most / 8:
            m += 1
        if kind == "apply":
            return {"kind": kind, "d": d, "dtype": dtype, "m": m}
        w = m if m <= 256 else rng.choice([192, 256])
        return {"kind": kind, "d": d, "dtype": dtype, "m": m, "w": w, "degree": degree}
    if kind == "lanczos":
        return {"kind": kind, "d": round(spread(1.0, 4.5), 2), "k": rng.randint(6, 16)}
    if kind == "hartree":
        return {"kind": kind, "d": round(spread(1.0, 3.0), 2)}
    if kind == "ortho":
        return {"kind": kind, "d": round(spread(1.0, 2.5), 2), "dtype": rng.choice(["f32", "f64"]), "m": int(spread(16, 600))}
    if kind == "scf":
        return {"kind": kind, "d": round(rng.uniform(1.0, 1.5), 2), "degree": rng.randint(8, 12)}
    if kind == "predict":
        return {"kind": kind, "edge": 8 * rng.randint(4, 12), "sigma": round(rng.uniform(4.0, 10.0), 1)}
    edge = 8 * rng.randint(2, 8)
    return {"kind": kind, "edge": edge, "batch": rng.randint(1, max(1, min(8, 64 ** 3 // edge ** 3)))}


def _cluster(case):
    """The cluster; its geometry belongs to the case (one seed per diameter)."""
    return make_cluster(5.0 * case["d"], 1000 + round(100 * case["d"]))


# ---------------------------------------------------------------------------
# inputs (shared by prepare and exact), from the seed alone
# ---------------------------------------------------------------------------
def _rows_block(rows, n_rows, m, dtype, seed):
    """N(0, 1) on the rows that hold points, zero on the padding rows."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    X = torch.zeros((n_rows, m), dtype=dtype, device="cuda")
    X[rows] = torch.randn((rows.numel(), m), generator=gen, dtype=dtype, device="cuda")
    return X


def _filtered_block(rows, n_rows, m, dtype, seed):
    """A block as the filter leaves it: columns that overlap, condition ~30."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 1)
    Q = torch.linalg.qr(torch.randn((m, m), generator=gen, dtype=torch.float64, device="cuda"))[0]
    s = torch.logspace(0, -1.5, m, dtype=torch.float64, device="cuda")
    return _rows_block(rows, n_rows, m, dtype, seed) @ (s[:, None] * Q.T).to(dtype)


def _rho(rows, n_rows, xyz2, radius, n_electrons, seed):
    """A smooth positive density that falls off towards the sphere's edge,
    with point-to-point structure from the seed."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    f = torch.exp(-8.0 * xyz2 / radius ** 2) * (1.0 + 0.5 * torch.rand(rows.numel(), generator=gen, dtype=torch.float64, device="cuda"))
    rho = torch.zeros(n_rows, dtype=torch.float64, device="cuda")
    rho[rows] = f * (n_electrons / (H ** 3 * f.sum()))
    return rho


def _patch(edge, seed):
    """A scaled density box: Gaussian atoms at the crystal's density inside a
    sphere, and a correction of its short wavelengths to learn."""
    rng = np.random.default_rng(seed)
    g = np.arange(edge) - (edge - 1) / 2
    inside = (g[:, None, None] ** 2 + g[None, :, None] ** 2 + g[None, None, :] ** 2) < (0.4 * edge) ** 2
    atoms = (rng.random((edge,) * 3) < 0.00254) & inside

    def blur(a, sigma):
        k = np.fft.fftfreq(edge)
        kz = np.fft.rfftfreq(edge)
        t = np.exp(-2 * (math.pi * sigma) ** 2 * (k[:, None, None] ** 2 + k[None, :, None] ** 2 + kz[None, None, :] ** 2))
        return np.fft.irfftn(np.fft.rfftn(a) * t, s=a.shape, axes=(0, 1, 2))

    x = np.maximum(blur(30.0 * 4.0 / H ** 3 * atoms, 3.7), 0.0)
    t = 0.2 * (x - blur(x, 4.0))
    return torch.from_numpy(x.astype(np.float32).ravel()).cuda(), torch.from_numpy(t.astype(np.float32).ravel()).cuda()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("predict", "train"):
        net = B.DensityNet(32, seed=1)
        net.set_params(np.load(WEIGHTS))
        patches = [_patch(case["edge"], seed + 1000 * k) for k in range(case.get("batch", 1))]
        x = patches[0][0]
        return {"case": case, "net": net, "patches": patches, "y": torch.zeros_like(x), "dy": torch.zeros_like(x),
                "hp": torch.zeros_like(x), "work": torch.zeros(2 * x.numel(), dtype=torch.float32, device="cuda"), "step": 0}
    c = _cluster(case)
    if kind == "scf":
        st = S.setup(c, PP, H, dtype="f64", degree=case["degree"], x_seed=seed, lanczos_seed=seed + 1)
        rho0 = st["H"].sad_density(c.pos, c.species, c.n_electrons)
        return {"case": case, "scf": st, "rho0": rho0, "rho": torch.zeros_like(rho0), "vh": torch.zeros_like(rho0)}
    dtype = case.get("dtype", "f64")
    odd32 = dtype == "f32" and case["m"] % 2 == 1
    ham = B.Hamiltonian(c.pos, c.species, PP, H, c.domain_radius(), B.ORDER_HILBERT, keep_nbr=odd32, dtypes=3)
    ijk, rows_np, _ = ham.export_ordering()
    rows = torch.from_numpy(rows_np).cuda()
    ctx = B.Context(0)
    st = {"case": case, "ham": ham, "ctx": ctx}
    if kind in ("lanczos", "filter"):
        st["v0"] = _rows_block(rows, ham.n_rows, 1, torch.float64, seed + 1)[:, 0].contiguous()
    if kind in ("apply", "filter"):
        st["X"] = _rows_block(rows, ham.n_rows, case["m"], DT[dtype], seed)
        st["W"] = torch.zeros((ham.n_rows, case.get("w", case["m"])), dtype=DT[dtype], device="cuda")
        if kind == "filter":
            b, tmin, _ = ham.lanczos_bound(ctx, st["v0"], 10)
            st["bounds"] = (tmin + 0.1 * (b - tmin), b, tmin)
    elif kind == "ortho":
        st["X"] = _filtered_block(rows, ham.n_rows, case["m"], DT[dtype], seed)
    elif kind == "hartree":
        xyz = torch.from_numpy(ijk).cuda().double() * H
        st["rho"] = _rho(rows, ham.n_rows, (xyz * xyz).sum(1), c.domain_radius(), c.n_electrons, seed)
        st["vh"] = torch.zeros_like(st["rho"])
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "apply":
        st["ham"].apply(st["X"], st["W"])
        return st["W"]
    if kind == "filter":
        a, b, a0 = st["bounds"]
        st["ham"].filter(st["X"], st["W"], case["degree"], a, b, a0)
        return st["X"]
    if kind == "lanczos":
        return st["ham"].lanczos_bound(st["ctx"], st["v0"], case["k"])
    if kind == "hartree":
        st["vh"].zero_()                      # the solve starts from the vector's contents
        st["ham"].hartree(st["ctx"], st["rho"], st["vh"])
        return st["vh"]
    if kind == "ortho":
        B.orthonormalize(st["ctx"], st["X"])
        return st["X"]
    if kind == "scf":
        # a new SCF from the given density; a second pass starts from the
        # block the first one left, as a restarted run does.  The block itself
        # is not returned: its columns are fixed only up to their sign.
        res = S.run(st["scf"], st["rho0"], max_steps=1)
        st["scf"]["scf"].fields(st["rho"], st["vh"])
        return {"energy": res.energy, "eig": res.eig, "rho": st["rho"], "vh": st["vh"]}
    net = st["net"]
    if kind == "predict":
        net.forward(st["patches"][0][0], st["y"])
        B.highpass(st["y"], case["edge"], case["sigma"], st["hp"], st["work"])
        return {"y": st["y"], "highpass": st["hp"]}
    loss = 0.0
    for x, t in st["patches"]:                # the gradients of a batch accumulate
        net.forward(x, st["y"])
        loss += net.mse(st["y"], t, st["dy"])
        net.backward(st["dy"])
    grads = net.get_grads()
    st["step"] += 1
    net.adam(1e-5, st["step"])                # a fine-tuning step; it clears the gradients
    return {"y": st["y"], "loss": loss, "grads": grads}


# ---------------------------------------------------------------------------
# bytes and operations no evaluation can do without
# ---------------------------------------------------------------------------
def _sphere(case):
    """(points, projector pairs, cluster) of a case, counted."""
    c = _cluster(case)
    r = c.domain_radius()
    n_r, thr = math.floor(r / H), math.floor((r / H) ** 2 + 1e-9)
    g = np.arange(-n_r, n_r + 1) ** 2
    n = int(((g[:, None, None] + g[None, :, None] + g[None, None, :]) <= thr).sum())
    return n, c.n_si * 4.0 / 3.0 * math.pi * (PP.r_cut / H) ** 3, c


# the 37-point star: per distance five additions and a multiply-add; then the
# diagonal and the three-term update.  A projector pair: four channels in and out.
STAR, PAIR = 6 * 7 + 6, 16


def work(case):
    kind = case["kind"]
    if kind in ("predict", "train"):
        n = case["edge"] ** 3
        w = np.load(WEIGHTS, mmap_mode="r").size
        # multiply-adds per cell of the finest level: 27 taps x (1 + 32 + 32 + 64 + 32) x 32 there, the
        # coarser levels' share, and the 1^3 output layer
        conv = 27 * 32 * 32
        per = 27 * 32 + conv * (1 + 1 + 2 + 1) + 32 + conv * ((3 + 4) / 8 + (3 + 4) / 64 + 3 / 512)
        if kind == "predict":
            taps = 2 * math.ceil(3 * case["sigma"]) + 1
            return {"bytes": 12.0 * n + 4.0 * w, "flops": n * (2.0 * per + 6 * taps)}
        return {"bytes": 12.0 * n * case["batch"] + 4.0 * w * 8, "flops": 6.0 * per * n * case["batch"]}
    n, pairs, c = _sphere(case)
    if kind in ("apply", "filter"):
        es = 4 if case["dtype"] == "f32" else 8
        return {"bytes": float(n) * es * (2 * case["m"] + 1),
                "flops": float(case.get("degree", 1)) * case["m"] * (STAR * n + PAIR * pairs)}
    if kind == "lanczos":
        return {"bytes": 16.0 * n, "flops": float(case["k"]) * ((STAR + 10) * n + PAIR * pairs)}
    if kind == "hartree":                     # at least one iteration per point of the radius
        return {"bytes": 16.0 * n, "flops": (STAR + 10.0) * n * c.domain_radius() / H}
    if kind == "ortho":
        es, passes = (4, 2) if case["dtype"] == "f32" else (8, 1)
        return {"bytes": 2.0 * es * n * case["m"], "flops": passes * 2.0 * n * case["m"] ** 2}
    m = n_states(c.n_electrons)               # four ChFSI iterations: filter, Cholesky-QR, H X, two products, rotation
    per = (case["degree"] + 1) * m * (STAR * n + PAIR * pairs) + (2 + 1 + 2) * float(n) * m * m
    return {"bytes": 8.0 * n * (2 * m + 4), "flops": 4.0 * per}


# ---------------------------------------------------------------------------
# the same results in 64 bits, from the definitions
# ---------------------------------------------------------------------------
def _hilbert(x, y, z, bits):
    """Index along the 3-D Hilbert curve (Skilling's transpose form, x first)."""
    v = [x.copy(), y.copy(), z.copy()]
    for lev in reversed(range(1, bits)):
        q, low = 1 << lev, (1 << lev) - 1
        for i in range(3):
            on = (v[i] & q) != 0
            t = np.where(on, 0, (v[0] ^ v[i]) & low)
            v[0] = np.where(on, v[0] ^ low, v[0] ^ t)
            v[i] = v[i] ^ t
    v[1] ^= v[0]
    v[2] ^= v[1]
    f = np.zeros_like(x)
    for lev in range(1, bits):
        f ^= np.where((v[2] >> lev) & 1, (1 << lev) - 1, 0)
    key = np.zeros_like(x)
    for lev in reversed(range(bits)):
        for a in range(3):
            key = (key << 1) | (((v[a] ^ f) >> lev) & 1)
    return key


class _Exact:
    """The Hamiltonian of a case on the points of its sphere, FP64."""

    def __init__(self, case):
        c = self.c = _cluster(case)
        self.radius = c.domain_radius()
        n_r, thr = math.floor(self.radius / H), math.floor((self.radius / H) ** 2 + 1e-9)
        g = np.arange(-n_r, n_r + 1)
        p = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
        p = p[(p * p).sum(1) <= thr]
        blk, loc = np.divmod(p + n_r, 8)
        key = _hilbert(blk[:, 0], blk[:, 1], blk[:, 2], max(1, (2 * n_r // 8).bit_length()))
        slots, at = np.unique(key, return_inverse=True)
        row = at.reshape(-1) * 512 + loc @ np.array([1, 8, 64])
        p = p[np.argsort(row)]                # points in the order of their rows
        self.n_rows, self.rows = len(slots) * 512, torch.from_numpy(np.sort(row)).cuda()
        edge = 2 * n_r + 1 + 2 * HALF
        self.stride = (1, edge, edge * edge)
        self.at = torch.from_numpy((p + n_r + HALF) @ np.array(self.stride)).cuda()
        self.cells = edge ** 3
        self.ijk = torch.from_numpy(p).cuda()
        self.xyz = self.ijk.double() * H
        # second derivative, 12th order: c_k = 2 (-1)^(k+1) (6!)^2 / (k^2 (6-k)! (6+k)!)
        f = math.factorial
        self.ck = [0.0] + [2.0 * (-1) ** (k + 1) * f(6) ** 2 / (k * k * f(6 - k) * f(6 + k)) / H ** 2 for k in range(1, 7)]
        self.ck[0] = -2.0 * sum(self.ck)

    def lap(self, X):
        u = torch.zeros((self.cells, X.shape[1]), dtype=torch.float64, device="cuda")
        u[self.at] = X
        Y = 3.0 * self.ck[0] * X
        for s in self.stride:
            for k in range(1, 7):
                Y.add_(u[self.at + k * s].add_(u[self.at - k * s]), alpha=self.ck[k])
        return Y

    def potential(self):
        v = torch.zeros(len(self.xyz), dtype=torch.float64, device="cuda")
        for pos, sp in zip(torch.from_numpy(self.c.pos).cuda(), self.c.species):
            z, w = (PP.z_si, PP.r_loc) if sp == 0 else (PP.z_h, PP.r_loc_h)
            d = ((self.xyz - pos) ** 2).sum(1).sqrt()
            near = torch.full_like(d, 2.0 * z / (math.sqrt(math.pi) * w))
            v -= torch.where(d < 1e-8, near, z * torch.erf(d / w) / d.clamp_min(1e-300))
        return v

    def set_up(self, veff=None):
        """V_eff and the (point, atom) pairs; only the s channel has an energy
        in the model pseudopotential (h_p = 0)."""
        assert PP.h_p == 0.0
        self.veff = (self.potential() if veff is None else veff)[:, None]
        point = torch.full((self.cells,), -1, dtype=torch.int64, device="cuda")
        point[self.at] = torch.arange(len(self.at), device="cuda")
        r = math.ceil(PP.r_cut / H) + 1
        g = torch.arange(-r, r + 1, device="cuda")
        off = torch.stack(torch.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
        pos = torch.from_numpy(self.c.pos[self.c.species == 0]).cuda()
        n_r = math.floor(self.radius / H)
        cell = torch.round(pos / H).long()[:, None, :] + off
        ok = (cell.abs() <= n_r).all(-1)
        lin = ((cell + n_r + HALF) * torch.tensor(self.stride, device="cuda")).sum(-1)
        pt = torch.where(ok, point[lin.clamp(0, self.cells - 1)], -1)
        d2 = ((cell.double() * H - pos[:, None, :]) ** 2).sum(-1)
        self.atom, slot = torch.nonzero((pt >= 0) & (d2 <= PP.r_cut ** 2), as_tuple=True)
        self.pt, d2 = pt[self.atom, slot], d2[self.atom, slot]
        norm = math.sqrt(4.0 / (math.sqrt(math.pi) * PP.r_c ** 3)) / math.sqrt(4.0 * math.pi)
        self.beta = (norm * torch.exp(-d2 / (2.0 * PP.r_c ** 2)))[:, None]
        self.n_si = len(pos)
        return self

    def ham(self, X):
        Y = self.lap(X).mul_(-0.5)
        Y += self.veff * X
        C = torch.zeros((self.n_si, X.shape[1]), dtype=torch.float64, device="cuda")
        C.index_add_(0, self.atom, X[self.pt].mul_(self.beta))
        return Y.index_add_(0, self.pt, C[self.atom].mul_(self.beta), alpha=PP.h_s * H ** 3)

    def lanczos(self, v0, k):
        v, last, beta, a, b = v0 / v0.norm(), None, 0.0, [], []
        for j in range(k):
            f = self.ham(v)
            if j:
                f -= beta * last
            a.append(float((v * f).sum()))
            f -= a[-1] * v
            beta = float(f.norm())
            b.append(beta)
            last, v = v, f / beta
        th = np.linalg.eigvalsh(np.diag(a) + np.diag(b[:-1], 1) + np.diag(b[:-1], -1))
        return float(th[-1] + b[-1]), float(th[0]), float(th[-1])

    def filter(self, X, degree, a, b, a0):
        e, c = (b - a) / 2, (b + a) / 2
        s1 = s = e / (a0 - c)
        last, X = X, (self.ham(X) - c * X) * (s1 / e)
        for _ in range(2, degree + 1):
            t = 1.0 / (2.0 / s1 - s)
            last, X = X, (self.ham(X) - c * X).mul_(2.0 * t / e) - (s * t) * last
            s = t
        return X

    def hartree(self, rho, v, rtol=1e-14):
        """-L v = 4 pi rho; outside the sphere the multipole expansion, l <= 4."""
        mono = [torch.ones((len(rho), 1), dtype=torch.float64, device="cuda")]
        for _ in range(4):
            mono.append((mono[-1][:, :, None] * self.xyz[:, None, :]).reshape(len(rho), -1))
        M = [H ** 3 * (rho @ t) for t in mono]            # sum q x^(l), 3^l entries
        rhs = 4.0 * math.pi * rho
        for axis in range(3):
            for k in (*range(-6, 0), *range(1, 7)):
                q = self.ijk.clone()
                q[:, axis] += k
                thr = math.floor((self.radius / H) ** 2 + 1e-9)
                out = torch.nonzero((q * q).sum(1) > thr)[:, 0]
                r = q[out].double() * H
                r2 = (r * r).sum(1)
                w = [torch.ones((len(out), 1), dtype=torch.float64, device="cuda")]
                for _ in range(4):
                    w.append((w[-1][:, :, None] * r[:, None, :]).reshape(len(out), -1))
                eye = torch.eye(3, dtype=torch.float64, device="cuda").reshape(-1)
                T = [w[i] @ M[i] for i in range(5)]
                S0 = M[2] @ eye
                S1 = w[1] @ (M[3].reshape(3, 9) @ eye)
                M4 = M[4].reshape(9, 9) @ eye
                S2, Q0 = w[2] @ M4, M4 @ eye
                d = r2.sqrt()
                pot = (T[0] / d + T[1] / d ** 3 + (3 * T[2] - r2 * S0) / (2 * d ** 5) + (5 * T[3] - 3 * r2 * S1) / (2 * d ** 7)
                       + (35 * T[4] - 30 * r2 * S2 + 3 * r2 * r2 * Q0) / (8 * d ** 9))
                rhs[out] += self.ck[abs(k)] * pot
        v = v.clone()
        r = rhs + self.lap(v[:, None])[:, 0]
        p, rr, stop = r.clone(), float(r @ r), rtol * float(rhs.norm())
        for _ in range(4000):
            if math.sqrt(rr) <= stop:
                break
            ap = -self.lap(p[:, None])[:, 0]
            al = rr / float(p @ ap)
            v += al * p
            r -= al * ap
            rn = float(r @ r)
            p = r + (rn / rr) * p
            rr = rn
        return v

    def to_rows(self, X):
        out = torch.zeros((self.n_rows, *X.shape[1:]), dtype=torch.float64, device="cuda")
        out[self.rows] = X
        return out


def _lda(rho):
    """(eps_xc, v_xc), Perdew-Zunger, zero below 1e-14."""
    ok = rho >= 1e-14
    rs = (3.0 / (4.0 * math.pi * torch.where(ok, rho, torch.ones_like(rho)))) ** (1.0 / 3.0)
    cx = 0.75 * (9.0 / (4.0 * math.pi ** 2)) ** (1.0 / 3.0)
    sq, ln = rs.sqrt(), rs.log()
    den = 1.0 + 1.0529 * sq + 0.3334 * rs
    lo = rs >= 1.0
    ec = torch.where(lo, -0.1423 / den, 0.0311 * ln - 0.048 + 0.0020 * rs * ln - 0.0116 * rs)
    dec = torch.where(lo, 0.1423 * (0.5 * 1.0529 / sq + 0.3334) / den ** 2, 0.0311 / rs + 0.0020 * (ln + 1.0) - 0.0116)
    e = ec - cx / rs
    v = e - rs / 3.0 * (dec + cx / rs ** 2)
    return torch.where(ok, e, torch.zeros_like(e)), torch.where(ok, v, torch.zeros_like(v))


def _cholesky_qr(X):
    """X R^-1 with X^T X = R^T R; twice, which leaves rounding errors only."""
    for _ in range(2):
        L = torch.linalg.cholesky(X.T @ X)
        eye = torch.eye(len(L), dtype=torch.float64, device="cuda")
        X = X @ torch.linalg.solve_triangular(L, eye, upper=False).T.contiguous()
    return X


def _exact_scf(case, seed):
    E = _Exact(case)
    c, ne = E.c, E.c.n_electrons
    m, occ, h3 = n_states(ne), ne // 2, H ** 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    step = max(1, (1 << 27) // m)
    X = torch.cat([torch.randn((min(step, len(E.xyz) - r), m), generator=gen, dtype=torch.float64, device="cuda")
                   for r in range(0, len(E.xyz), step)])
    v0 = torch.from_numpy(np.random.default_rng(seed + 1).standard_normal(len(E.xyz))).cuda()
    rho = torch.zeros(len(E.xyz), dtype=torch.float64, device="cuda")
    for pos, sp in zip(torch.from_numpy(c.pos).cuda(), c.species):
        al, z = (0.074, 4.0) if sp == 0 else (0.21, 1.0)
        rho += z * (al / math.pi) ** 1.5 * torch.exp(-al * ((E.xyz - pos) ** 2).sum(1))
    rho *= ne / (h3 * rho.sum())
    vh = E.hartree(rho, torch.zeros_like(rho))
    exc, vxc = _lda(rho)
    E.set_up(E.potential() + vh + vxc)
    b, tmin, _ = E.lanczos(v0[:, None], 10)
    a0, a = tmin, tmin + 0.1 * (b - tmin)
    for _ in range(4):
        X = E.filter(X, case["degree"], a, b, a0)
        X = _cholesky_qr(X)
        Hs = X.T @ E.ham(X)
        eig, Q = torch.linalg.eigh(0.5 * (Hs + Hs.T))
        X = X @ Q
        a0, a = float(eig[0]), float(eig[-1])
    out = (X[:, :occ] ** 2).sum(1)
    out *= ne / (h3 * out.sum())
    pos, z = c.pos, np.where(c.species == 0, PP.z_si, PP.z_h)
    d = np.sqrt(((pos[:, None] - pos[None]) ** 2).sum(-1)) + np.eye(len(z))
    e_ion = 0.5 * (np.outer(z, z) / d)[~np.eye(len(z), dtype=bool)].sum()
    energy = 2.0 * float(eig[:occ].sum()) - h3 * float(rho @ (0.5 * vh + vxc - exc)) + e_ion
    return {"energy": energy, "eig": eig, "rho": E.to_rows(rho + 0.1 * (out - rho)), "vh": E.to_rows(vh)}


def _exact_net(x):
    """The network on x [S, S, S], FP64: (output, {offset: weight or bias})."""
    flat = np.load(WEIGHTS).astype(np.float64)
    par, at = [], 0
    for i in range(21):
        cin, cout, k = 1 if i == 0 else 64 if i in (12, 15, 18) else 32, 1 if i == 20 else 32, 1 if i == 20 else 3
        cp, op, t = 4 * -(-cin // 4), 16 * -(-cout // 16), k ** 3
        w = torch.from_numpy(flat[at:at + op * t * cp].reshape(op, t, cp)[:cout, :, :cin].copy()).cuda().requires_grad_()
        bias = torch.from_numpy(flat[at + op * t * cp:at + op * t * cp + cout].copy()).cuda().requires_grad_()
        par.append((at, op, t, cp, w, bias))
        at += op * t * cp + op

    def conv(i, u, stride=1, act=True):
        w, bias = par[i][4:]
        D, cin = u.shape[0], u.shape[-1]
        k = round(w.shape[1] ** (1 / 3))
        up = torch.nn.functional.pad(u, (0, 0) + (k // 2,) * 6)
        z = bias
        for t in range(k ** 3):
            a, b, c = t // (k * k), t // k % k, t % k
            part = up[a:a + D:stride, b:b + D:stride, c:c + D:stride].reshape(-1, cin)
            z = z + part @ w[:, t].T
        D = D // stride
        return (z * torch.sigmoid(z) if act else z).reshape(D, D, D, -1)

    def grow(u):
        return u.repeat_interleave(2, 0).repeat_interleave(2, 1).repeat_interleave(2, 2)

    e1 = conv(1, conv(0, x[..., None]))
    e2 = conv(4, conv(3, conv(2, e1, 2)))
    e3 = conv(7, conv(6, conv(5, e2, 2)))
    g = conv(10, conv(9, conv(8, e3, 2)))
    for i, e in ((11, e3), (14, e2), (17, e1)):
        g = conv(i + 2, conv(i + 1, torch.cat([conv(i, grow(g)), e], -1)))
    return conv(20, g, act=False)[..., 0], par, at


def exact(case, seed):
    kind = case["kind"]
    if kind == "predict":
        n, s = case["edge"], case["sigma"]
        with torch.no_grad():
            y, _, _ = _exact_net(_patch(n, seed)[0].double().reshape(n, n, n))
        k = np.arange(n)
        g = np.arange(-math.ceil(3 * s), math.ceil(3 * s) + 1)
        t = np.exp(-(k[:, None] - k[None, :]) ** 2 / (2 * s * s)) * (abs(k[:, None] - k[None, :]) <= math.ceil(3 * s))
        t = torch.from_numpy(t / np.exp(-g * g / (2 * s * s)).sum()).cuda()
        z = y
        for _ in range(3):
            z = (t @ z.reshape(n, n * n)).reshape(n, n, n).permute(1, 2, 0).contiguous()
        return {"y": y.reshape(-1), "highpass": (y - z).reshape(-1)}
    if kind == "train":
        n, total, flat = case["edge"], 0.0, 0.0
        for k in range(case["batch"]):
            x, t = (v.double().reshape(n, n, n) for v in _patch(n, seed + 1000 * k))
            y, par, size = _exact_net(x)
            loss = ((y - t) ** 2).mean()
            loss.backward()
            total += float(loss.detach())
            one = torch.zeros(size, dtype=torch.float64, device="cuda")
            for at, op, taps, cp, w, bias in par:
                v = one[at:at + op * taps * cp].reshape(op, taps, cp)
                v[:w.shape[0], :, :w.shape[2]] = w.grad
                one[at + op * taps * cp:at + op * taps * cp + len(bias)] = bias.grad
            flat = flat + one
        return {"y": y.detach().reshape(-1), "loss": total, "grads": flat}
    if kind == "scf":
        return _exact_scf(case, seed)
    E = _Exact(case)
    if kind == "hartree":
        rho = _rho(E.rows, E.n_rows, (E.xyz * E.xyz).sum(1), E.radius, E.c.n_electrons, seed)[E.rows]
        return E.to_rows(E.hartree(rho, torch.zeros_like(rho)))
    if kind == "ortho":
        X = _filtered_block(E.rows, E.n_rows, case["m"], DT[case["dtype"]], seed).double()
        return _cholesky_qr(X)
    E.set_up()
    if kind == "apply":
        X = _rows_block(E.rows, E.n_rows, case["m"], DT[case["dtype"]], seed)[E.rows].double()
        return E.to_rows(E.ham(X))
    v0 = _rows_block(E.rows, E.n_rows, 1, torch.float64, seed + 1)[E.rows]
    if kind == "lanczos":
        return E.lanczos(v0, case["k"])
    b, tmin, _ = E.lanczos(v0, 10)
    X = _rows_block(E.rows, E.n_rows, case["m"], DT[case["dtype"]], seed)[E.rows].double()
    return E.to_rows(E.filter(X, case["degree"], tmin + 0.1 * (b - tmin), b, tmin))

"""Workloads of the Kohn-Sham library, for timing and for comparing outputs.

Each case is one call sequence that a program of this library makes, on seeded
synthetic inputs of the shapes that the package's own generator draws
(Gaussian local potential and Kleinman-Bylander spheres, E_cut = 10 Ha, random
plane-wave coefficients):

* ``hpsi``     H psi of orbitals on the box (``System.ham_apply``): a caller
               with its own eigensolver or propagator;
* ``step``     resident Taylor-4 propagation with the density and the norms
               after every step, then the orbitals (``State.propagate``,
               ``State.download``): the library's main path;
* ``batch``    ragged batched steps of several resident systems of one grid
               (``Batch.propagate``): the serving loop's inner call;
* ``etrs``     density-dependent propagation with Hartree and local-density
               xc (``State.propagate_etrs``);
* ``ground``   steepest-descent iterations from orthonormal orbitals
               (``State.eigensolve``), forward products, subspace
               diagonalisation and orthonormalisation included;
* ``observe``  density, norms and band energy, Hartree and xc potentials and
               the dipole of orbitals on the box (analysis of a snapshot).

Fields: ``kind``; ``n0`` and ``n1`` (grid n0 x n1 x n1); ``h`` (grid spacing in
bohr, L_a = h n_a); ``norb``; ``natoms``; ``mixed`` (complex64 transforms);
``proj`` (1: the split-BF16 projection product); ``steps``; ``tune`` (True:
the program runs the launch-schedule autotuner at set-up); ``x_shape`` (a
stored launch shape, -1: the default).
"""
import math

import numpy as np
import torch

from paper_2106_03872_amd import ks

ECUT = 10.0
R_CUT = 2.0
SIGMA = 0.8
DT = 0.05
OCC = 2.0
MEMBERS = 8   # systems of a batch, drawn from the seeds MEMBERS * seed + i


def _case(name, kind, n0, n1, h, norb, natoms, mixed=False, proj=0, steps=1, tune=False, x_shape=-1):
    return {"name": name, "kind": kind, "n0": n0, "n1": n1, "h": h, "norb": norb, "natoms": natoms, "mixed": mixed,
            "proj": proj, "steps": steps, "tune": tune, "x_shape": x_shape}


def listed():
    return [
        # the smallest system of the package's configurations: a latency-bound call
        _case("hpsi_16_8_fp64", "hpsi", 16, 16, 0.625, 8, 2),
        # a small resident system propagated on its own, as a small serving request is
        _case("step_24_10_mixed", "step", 24, 24, 0.33, 10, 3, mixed=True, steps=5),
        # an odd orbital count on a non-cubic cell, through the box interface
        _case("hpsi_48x40_33_fp64", "hpsi", 48, 40, 0.3125, 33, 6),
        # a serving request of the larger grids, stepped on its own
        _case("step_60_96_mixed", "step", 60, 60, 0.33, 96, 20, mixed=True, steps=2),
        # ragged requests of one grid stepped together, as the serving loop does
        _case("batch_32_8x_mixed", "batch", 32, 32, 0.33, 131, 17, mixed=True, steps=4),
        # the 64-point workload: an ordinary molecule or cluster
        _case("step_64_128_fp64", "step", 64, 64, 0.3125, 128, 32, steps=2),
        # density-dependent dynamics at the same size
        _case("etrs_64_96_fp64", "etrs", 64, 64, 0.3125, 96, 24),
        # two ground-state iterations at the same size
        _case("ground_64_128_fp64", "ground", 64, 64, 0.3125, 128, 32, steps=2),
        # analysis of a snapshot on a non-cubic cell, odd orbital count
        _case("observe_72x80_75_fp64", "observe", 72, 80, 0.3125, 75, 40),
        # the headline workload: 96^3, 512 orbitals, 128 atoms, double precision, autotuned
        _case("step_96_512_fp64", "step", 96, 96, 0.3125, 512, 128, steps=2, tune=True),
        # the same size in mixed precision with the projections as a matrix product
        _case("step_96_512_mixed_bf16", "step", 96, 96, 0.3125, 512, 128, mixed=True, proj=1, steps=2),
        # the largest system, mixed precision with the launch shape stored from an earlier tuning
        _case("step_120_1024_mixed", "step", 120, 120, 0.3125, 1024, 256, mixed=True, steps=1, x_shape=1),
    ]


def draw(rng):
    kind = rng.choice(["hpsi", "step", "step", "step", "batch", "etrs", "ground", "observe"])
    sizes = [12, 16, 20, 24, 32, 40, 48, 60, 64, 72, 80, 96, 120]
    if kind == "batch":
        sizes = [24, 32, 40, 48, 60, 64]
    elif kind in ("etrs", "ground"):
        sizes = [16, 24, 32, 40, 48, 60, 64, 72, 80]
    n0 = rng.choice(sizes)
    n1 = n0 if kind == "batch" or rng.random() < 0.6 else rng.choice([m for m in sizes if 0.6 <= m / n0 <= 1.7])
    h = round(rng.uniform(0.29, 0.3125 if max(n0, n1) >= 96 else 0.36), 4)
    if kind in ("hpsi", "step") and n0 <= 24:
        h = round(rng.uniform(0.33, 0.625), 4)
    points = n0 * n1 * n1
    most = {"hpsi": 400, "step": 1024, "batch": 200, "etrs": 256, "ground": 200, "observe": 400}[kind]
    most = max(8, min(most, int(4.5e8 / points)))     # at most about the orbitals of the 96-point workload
    norb = int(round(math.exp(rng.uniform(math.log(3), math.log(most)))))
    norb = max(2, min(norb, _sphere((n0, n1, n1), h)[0] // 10))     # well under the size of the basis
    volume = points * h ** 3
    natoms = max(1, min(int(volume / 150) + 1, int(round(norb * rng.uniform(0.1, 0.5))), 256))
    mixed = kind in ("step", "hpsi", "batch", "etrs") and (kind == "batch" or rng.random() < 0.5)
    proj = 1 if mixed and kind == "step" and rng.random() < 0.4 else 0
    steps = rng.choice([1, 2, 3]) if kind in ("step", "batch") else 1
    return {"kind": kind, "n0": n0, "n1": n1, "h": h, "norb": norb, "natoms": natoms, "mixed": mixed, "proj": proj,
            "steps": steps, "tune": False, "x_shape": -1}


# ------------------------------------------------------------------- inputs

class Problem:
    """One system's inputs: grid, potential and projectors (host arrays)."""

    def __init__(self, case, seed, norb=None, natoms=None):
        self.n = (case["n0"], case["n1"], case["n1"])
        self.L = tuple(case["h"] * m for m in self.n)
        self.N = int(np.prod(self.n))
        self.omega = float(np.prod(self.L))
        self.norb = norb or case["norb"]
        self.natoms = natoms or case["natoms"]
        self.seed = seed
        rng = np.random.default_rng([seed, 1])
        x = [np.arange(self.n[a]) * case["h"] for a in range(3)]
        pos = rng.random((self.natoms, 3)) * np.asarray(self.L)
        # local potential: attractive periodic Gaussians of depth 2 and width 1
        g = []
        for a in range(3):
            t = np.zeros((self.natoms, self.n[a]))
            images = int(math.ceil(10.0 / self.L[a])) + 1
            for i in range(-images, images + 1):
                t += np.exp(-0.5 * (x[a][None, :] - pos[:, a:a + 1] - i * self.L[a]) ** 2)
            g.append(t)
        yz = (g[1][:, :, None] * g[2][:, None, :]).reshape(self.natoms, -1)
        self.vloc = np.ascontiguousarray((-2.0 * g[0].T @ yz).reshape(self.n))
        # projector spheres: s and p Gaussians on the points within R_CUT
        dV = self.omega / self.N
        npts, idx, beta = [], [], []
        for R in pos:
            d = [(x[a] - R[a] + 0.5 * self.L[a]) % self.L[a] - 0.5 * self.L[a] for a in range(3)]
            w = [np.flatnonzero(np.abs(v) < R_CUT) for v in d]
            D = np.meshgrid(*[d[a][w[a]] for a in range(3)], indexing="ij")
            J = np.meshgrid(*w, indexing="ij")
            r2 = D[0] ** 2 + D[1] ** 2 + D[2] ** 2
            inside = r2 < R_CUT * R_CUT
            e = np.exp(-r2[inside] / (2.0 * SIGMA ** 2))
            b = np.stack([e] + [D[a][inside] * e for a in range(3)], axis=1)
            b /= np.sqrt(dV * np.sum(b * b, axis=0))[None, :]
            npts.append(int(inside.sum()))
            idx.append(((J[0] * self.n[1] + J[1]) * self.n[2] + J[2])[inside].astype(np.int32))
            beta.append(b)
        self.npts = np.asarray(npts, np.int32)
        self.idx = np.concatenate(idx)
        self.beta = np.ascontiguousarray(np.concatenate(beta))
        dl = rng.uniform(0.5, 2.0, size=(self.natoms, 2))
        self.d = np.ascontiguousarray(np.stack([dl[:, 0], dl[:, 1], dl[:, 1], dl[:, 1]], axis=1))
        m = [np.where(np.arange(k) < (k + 1) // 2, np.arange(k), np.arange(k) - k) for k in self.n]
        G = [2.0 * np.pi * m[a] / self.L[a] for a in range(3)]
        self.K = 0.5 * (G[0][:, None, None] ** 2 + G[1][None, :, None] ** 2 + G[2][None, None, :] ** 2)
        self.x = x

    def orbitals(self):
        """Unit-norm random orbitals, complex128 [norb, n0, n1, n1] on the GPU
        (drawn a little beyond the plane-wave sphere, as a caller's box is)."""
        gen = torch.Generator(device="cuda").manual_seed(self.seed * 1000003 + 17)
        K = self.K.ravel()
        sel = np.flatnonzero(K < 1.1 * ECUT)
        damp = torch.from_numpy(np.exp(-K[sel] / 4.0)).cuda()
        at = torch.from_numpy(sel).cuda()
        psi = torch.zeros((self.norb, self.N), dtype=torch.complex128, device="cuda")
        for o in range(0, self.norb, 128):
            nb = min(128, self.norb - o)
            z = torch.randn((nb, len(sel), 2), dtype=torch.float64, device="cuda", generator=gen)
            c = torch.view_as_complex(z) * damp
            c /= torch.linalg.vector_norm(c, dim=1, keepdim=True)
            psi[o:o + nb].index_copy_(1, at, c)
        return psi.reshape((self.norb,) + self.n)

    def system(self, case, chunk=0):
        s = ks.System(self.n, self.L, ECUT, self.norb, ks.KS_MIXED if case["mixed"] else ks.KS_FP64, chunk=chunk)
        s.set_vloc(torch.from_numpy(self.vloc).cuda())
        s.set_projectors(self.npts, self.idx, self.beta, self.d)
        return s


def _members(case, seed):
    """The systems of a case: one, or the ragged requests of a batch."""
    if case["kind"] != "batch":
        return [Problem(case, seed)]
    rng = np.random.default_rng(2)      # the same ragged counts for every seed
    out = []
    for i in range(MEMBERS):
        norb = int(max(2, round(case["norb"] * rng.uniform(0.1, 1.9))))
        natoms = int(max(1, round(case["natoms"] * rng.uniform(0.15, 1.85))))
        out.append(Problem(case, MEMBERS * seed + i, norb, natoms))
    return out


def _occ(norb):
    return torch.full((norb,), OCC, dtype=torch.float64, device="cuda")


def _f64(*shape):
    return torch.empty(shape, dtype=torch.float64, device="cuda")


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        # passes of at most 64 orbitals, as the serving loop creates its systems
        systems, states, boxes = [], [], []
        for p in _members(case, seed):
            s = p.system(case, chunk=64)
            st = ks.State(s, p.norb)
            psi = p.orbitals()
            st.upload(psi)
            systems.append(s)
            states.append(st)
            boxes.append(psi)
        return {"case": case, "batch": ks.Batch(states), "systems": systems, "states": states, "boxes": boxes}
    p = Problem(case, seed)
    s = p.system(case)
    if case["tune"]:
        s.autotune(p.norb)
    if case["proj"] or case["x_shape"] >= 0:
        i = s.info()
        s.set_tuning(i["x_group"], i["plane_group"], x_shape=case["x_shape"], projection=case["proj"])
    psi = p.orbitals()
    v = {"case": case, "system": s, "psi": psi, "occ": _occ(p.norb)}
    if kind == "hpsi":
        v["hpsi"] = torch.empty_like(psi)
    if kind == "ground":
        s.orthonormalize(psi)
        v["out"] = torch.empty_like(psi)
        v["eig"], v["resid"] = _f64(case["steps"], p.norb), _f64(case["steps"], p.norb)
    if kind in ("step", "etrs", "ground"):
        v["state"] = ks.State(s, p.norb)
        v["state"].upload(psi)       # the box then takes the downloaded orbitals
    if kind in ("step", "etrs"):
        v["rho"] = _f64(case["steps"], *p.n)
        v["norms"] = _f64(case["steps"], p.norb)
    if kind == "etrs":
        s.set_xc(ks.KS_XC_LDA)
    return v


def run(v):
    case = v["case"]
    kind, steps = case["kind"], case["steps"]
    if kind == "hpsi":
        return v["system"].ham_apply(v["psi"], v["hpsi"])
    if kind == "step":
        v["state"].propagate(DT, steps, v["occ"], v["rho"], v["norms"])
        return {"rho": v["rho"], "norms": v["norms"], "psi": v["state"].download(v["psi"])}
    if kind == "batch":
        v["batch"].propagate(DT, steps)
        return [st.download(box) for st, box in zip(v["states"], v["boxes"])]
    if kind == "etrs":
        v["state"].propagate_etrs(DT, steps, v["occ"], v["rho"], v["norms"])
        return {"rho": v["rho"], "norms": v["norms"], "psi": v["state"].download(v["psi"])}
    if kind == "ground":
        v["state"].upload(v["psi"])
        v["state"].eigensolve(steps, v["eig"], v["resid"])
        return {"eig": v["eig"], "resid": v["resid"], "psi": v["state"].download(v["out"])}
    if kind == "observe":
        s = v["system"]
        rho = s.density(v["psi"], v["occ"])
        norms, energy = s.reduce(v["psi"], v["occ"])
        vh = s.hartree(rho)
        return {"rho": rho, "norms": norms, "energy": energy, "hartree": vh, "xc": s.lda_xc(rho),
                "dipole": s.dipole(rho)}
    raise ValueError(kind)


# --------------------------------------------------------------- work, exact

def _sphere(n, h):
    """(plane waves, (m0, m1) columns, m0 planes) of the sphere K < E_cut."""
    m = [np.where(np.arange(k) < (k + 1) // 2, np.arange(k), np.arange(k) - k) * (2.0 * np.pi / (h * k)) for k in n]
    q01 = 0.5 * (m[0][:, None] ** 2 + m[1][None, :] ** 2)
    cols = int((q01 < ECUT).sum())
    planes = int((0.5 * m[0] ** 2 < ECUT).sum())
    left = 2.0 * (ECUT - q01[q01 < ECUT])
    npw = int(sum(np.searchsorted(np.sort(m[2] ** 2), left, side="left")))
    return npw, cols, planes


def work(case):
    """Each input read and each output written once; the arithmetic of the
    transforms pruned to the sphere (5 n log2 n a line), of the sphere sums and
    of the dense products."""
    n = (case["n0"], case["n1"], case["n1"])
    N = n[0] * n[1] * n[2]
    npw, cols, planes = _sphere(n, case["h"])
    line = lambda k: 5.0 * k * math.log2(k)
    fft = cols * line(n[2]) + planes * n[2] * line(n[1]) + n[1] * n[2] * line(n[0])
    pts = 4.0 / 3.0 * math.pi * (R_CUT / case["h"]) ** 3
    o, steps, kind = case["norb"], case["steps"], case["kind"]
    if kind == "batch":
        o *= MEMBERS
    kb = case["natoms"] * pts * 4 * 2 * 4
    hpsi = 2.0 * fft + kb + 8.0 * N
    state, box, field = 16.0 * npw * o, 16.0 * N * o, 8.0 * N
    tables = case["natoms"] * pts * (4 + 32)
    if kind == "hpsi":
        return {"bytes": state + box + field + tables, "flops": o * hpsi}
    if kind == "step":
        return {"bytes": state + box + field * (1 + steps) + tables, "flops": o * steps * (4.0 * hpsi + 5.0 * N)}
    if kind == "batch":
        return {"bytes": state + box + MEMBERS * (field + tables), "flops": o * steps * 4.0 * hpsi}
    if kind == "etrs":
        return {"bytes": state + box + field * (1 + steps) + tables,
                "flops": o * (steps * (8.0 * hpsi + 2.0 * (fft + 5.0 * N)) + fft + 5.0 * N)}
    if kind == "ground":
        return {"bytes": state + box + field + tables,
                "flops": steps * (o * 2.0 * hpsi + 8.0 * 4.0 * o * o * npw + 8.0 * 10.0 * o ** 3)}
    return {"bytes": 2.0 * state + 5.0 * field + tables, "flops": o * (hpsi + fft + 5.0 * N)}


class Reference:
    """The method in plain complex128 torch on full boxes."""

    def __init__(self, p):
        self.p = p
        self.K = torch.from_numpy(p.K).cuda()
        self.chi = self.K < ECUT
        self.vloc = torch.from_numpy(p.vloc).cuda()
        self.v = self.vloc
        off = np.concatenate([[0], np.cumsum(p.npts)])
        self.atoms = [(torch.from_numpy(p.idx[a:b].astype(np.int64)).cuda(),
                       torch.from_numpy(p.beta[a:b]).cuda()) for a, b in zip(off[:-1], off[1:])]
        self.d = torch.from_numpy(p.d).cuda()
        self.nb = max(1, int(1.5e8 // p.N))

    def real(self, c):
        return torch.fft.ifftn(c, dim=(-3, -2, -1), norm="forward") / math.sqrt(self.p.omega)

    def h(self, c):
        out = torch.empty_like(c)
        for o in range(0, c.shape[0], self.nb):
            x = c[o:o + self.nb]
            r = self.real(x)
            f = r * self.v
            flat, ff = r.reshape(len(x), -1), f.reshape(len(x), -1)
            for (idx, beta), d in zip(self.atoms, self.d):
                g = flat[:, idx]
                P = torch.complex(g.real @ beta, g.imag @ beta) * (self.p.omega / self.p.N) * d
                ff.index_add_(1, idx, torch.complex(P.real @ beta.T, P.imag @ beta.T))
            y = torch.fft.fftn(f, dim=(-3, -2, -1), norm="backward") * (math.sqrt(self.p.omega) / self.p.N)
            out[o:o + self.nb] = torch.where(self.chi, self.K * x + y, torch.zeros((), dtype=x.dtype, device=x.device))
        return out

    def start(self, c):
        return c.masked_fill_(~self.chi, 0)

    def taylor(self, c, dt, second=None):
        """sum_k (-i dt)^k/k! H^k c; with `second`, also the sum for that step."""
        acc, acc2, w, a, b = c.clone(), c.clone() if second else None, c, 1.0, 1.0
        for k in range(1, 5):
            w = self.h(w)
            a = a * (-1j * dt) / k
            acc += a * w
            if second:
                b = b * (-1j * second) / k
                acc2 += b * w
        return (acc, acc2) if second else acc

    def density(self, c):
        rho = torch.zeros(self.p.n, dtype=torch.float64, device="cuda")
        for o in range(0, c.shape[0], self.nb):
            r = self.real(c[o:o + self.nb])
            rho += OCC * (r.real ** 2 + r.imag ** 2).sum(0)
        return rho

    def norms(self, c):
        return torch.stack([(x.real ** 2 + x.imag ** 2).sum() for x in c])

    def hartree(self, rho):
        g = torch.fft.fftn(rho)
        g = torch.where(self.K > 0, 2.0 * math.pi * g / torch.where(self.K > 0, self.K, torch.ones_like(self.K)),
                        torch.zeros_like(g))
        return torch.fft.ifftn(g).real

    def xc(self, rho):
        rs = (3.0 / (4.0 * math.pi * rho)) ** (1.0 / 3.0)
        vx = -((3.0 / math.pi) * rho) ** (1.0 / 3.0)
        s = torch.sqrt(rs)
        q = 1.0 + 1.0529 * s + 0.3334 * rs
        low = -0.1423 / q * (1.0 + 7.0 / 6.0 * 1.0529 * s + 4.0 / 3.0 * 0.3334 * rs) / q
        ln = torch.log(rs)
        high = 0.0311 * ln + (-0.048 - 0.0311 / 3.0) + 2.0 / 3.0 * 0.0020 * rs * ln + (2.0 * -0.0116 - 0.0020) * rs / 3.0
        return vx + torch.where(rs >= 1.0, low, high)

    def dipole(self, rho):
        dV = self.p.omega / self.p.N
        x = [torch.from_numpy(v).cuda() for v in self.p.x]
        return dV * torch.stack([(rho.sum((1, 2)) * x[0]).sum(), (rho.sum((0, 2)) * x[1]).sum(),
                                 (rho.sum((0, 1)) * x[2]).sum()])

    # The dense algebra of the ground state, on the host and on the sphere's
    # coefficients alone: C is [norb, plane waves].
    def pack(self, c):
        return c.reshape(c.shape[0], -1)[:, self.chi.ravel()].cpu()

    def box(self, C):
        out = torch.zeros((C.shape[0], self.p.N), dtype=torch.complex128, device="cuda")
        out[:, self.chi.ravel()] = C.cuda()
        return out.reshape((C.shape[0],) + self.p.n)

    @staticmethod
    def orthonormal(C):
        low = np.linalg.cholesky((C.conj() @ C.T).numpy())     # S = C^H C over the orbitals
        return torch.from_numpy(np.linalg.solve(low.conj(), C.numpy()))

    def descend(self, C):
        """One steepest-descent iteration: (orbitals, Ritz values, residual norms)."""
        K = self.K[self.chi].cpu()[None, :]
        W = self.pack(self.h(self.box(C)))
        A = C.conj() @ W.T
        e, Q = torch.linalg.eigh(0.5 * (A + A.conj().T))
        top = Q.gather(0, Q.abs().argmax(0, keepdim=True))
        Q = Q * (top.conj() / top.abs())
        C, W = Q.T @ C, Q.T @ W
        r = W - e[:, None] * C
        sq = r.real ** 2 + r.imag ** 2
        res = sq.sum(1).sqrt()
        x = K / ((K * sq).sum(1) / sq.sum(1))[:, None]
        poly = 27.0 + 18.0 * x + 12.0 * x ** 2 + 8.0 * x ** 3
        p = poly / (poly + 16.0 * x ** 4) * r
        p = p - (C.conj() * p).sum(1, keepdim=True) * C
        q = p / torch.linalg.vector_norm(p, dim=1, keepdim=True)
        hq = self.pack(self.h(self.box(q)))
        off = (C.conj() * hq).sum(1)
        M = torch.zeros((C.shape[0], 2, 2), dtype=torch.complex128)
        M[:, 0, 0], M[:, 0, 1], M[:, 1, 0] = e.to(M.dtype), off, off.conj()
        M[:, 1, 1] = (q.conj() * hq).sum(1).real.to(M.dtype)
        y = torch.linalg.eigh(M)[1][:, :, 0]
        y = y * (y[:, :1].conj() / y[:, :1].abs())
        return self.orthonormal(y[:, :1] * C + y[:, 1:] * q), e, res


def exact(case, seed):
    kind, steps = case["kind"], case["steps"]
    got = []
    for p in _members(case, seed):
        ref = Reference(p)
        c = ref.start(p.orbitals())
        if kind == "hpsi":
            return ref.h(c)
        if kind in ("step", "batch"):
            rho, norms = [], []
            for _ in range(steps):
                c = ref.taylor(c, DT)
                if kind == "step":
                    rho.append(ref.density(c))
                    norms.append(ref.norms(c))
            if kind == "step":
                return {"rho": torch.stack(rho), "norms": torch.stack(norms), "psi": c}
            got.append(c)
        if kind == "etrs":
            rho, norms = [], []
            now = ref.density(c)
            for _ in range(steps):
                ref.v = ref.vloc + ref.hartree(now) + ref.xc(now)
                c, full = ref.taylor(c, 0.5 * DT, DT)
                now = ref.density(full)
                ref.v = ref.vloc + ref.hartree(now) + ref.xc(now)
                c = ref.taylor(c, 0.5 * DT)
                now = ref.density(c)
                rho.append(now)
                norms.append(ref.norms(c))
            return {"rho": torch.stack(rho), "norms": torch.stack(norms), "psi": c}
        if kind == "ground":
            C = ref.orthonormal(ref.pack(c))
            eig, res = [], []
            for _ in range(steps):
                C, e, r = ref.descend(C)
                eig.append(e)
                res.append(r)
            return {"eig": torch.stack(eig), "resid": torch.stack(res), "psi": ref.box(C)}
        if kind == "observe":
            rho = ref.density(c)
            w = ref.h(c)
            energy = OCC * sum((a.conj() * b).sum().real for a, b in zip(c, w)).reshape(1)
            return {"rho": rho, "norms": ref.norms(c), "energy": energy, "hartree": ref.hartree(rho),
                    "xc": ref.xc(rho), "dipole": ref.dipole(rho)}
    return got

"""Performance cases: what a user of this library has it do, with its inputs.

Workloads follow the repository's own configurations (2D and 3D spiral
acquisitions, solid-harmonic field terms up to third order plus an
off-resonance map, smooth coil sensitivities, multi-echo prescans) with the
sizes, shot counts, voxel sets, operand precisions and options varied.  All
calls go through the public binding (``paper_2604_09233_amd``).

    listed()            the named cases
    draw(rng)           one more case from the same ranges (no name)
    prepare(case, seed) inputs and handles on the GPU, from the seed alone
    run(state)          one pass; returns every output
    exact(case, seed)   the same outputs in 64-bit plain torch, or None
    work(case)          bytes and operations of one pass
"""
import math

import numpy as np
import torch

from paper_2604_09233_amd import autograd, nfs

DEV = "cuda:0"
DWELL = 2e-6          # s, sample spacing of the readouts
BLOCK = 1 << 28       # phase entries evaluated at a time by the 64-bit formulas


# ---------------------------------------------------------------------------
# cases
def listed():
    return [
        # The smallest call: the operator once on a 32 x 32 single-shot slice
        # (parameter searches, unit tests of a pipeline); latency and launches.
        dict(name="e_2d_32_fp32", kind="E", prec="fp32", nx=32, ny=32, nz=1, coils=4, terms=4, shots=1, k_shot=2048,
             turns=16.0, b0_hz=50.0, mask=False),
        # Adjoint of a measured data set onto the voxels of a reconstruction
        # mask: odd voxel and sample counts, the half-precision operands.
        dict(name="eh_2d_masked_fp16", kind="EH", prec="fp16", nx=128, ny=128, nz=1, coils=15, terms=16, shots=4,
             k_shot=14999, turns=4.0, b0_hz=100.0, mask=True),
        # The normal operator of the 2D 128 x 128 / 16-coil / 60000-sample
        # workload: one CG iteration's work for a caller with its own solver.
        dict(name="ehe_2d_128_fp16", kind="EHE", prec="fp16", nx=128, ny=128, nz=1, coils=16, terms=16, shots=4,
             k_shot=15000, turns=4.0, b0_hz=100.0, mask=False),
        # The forward operator of a small volume in the float32-grade form
        # (simulating data from an image).
        dict(name="e_3d_48_fp32", kind="E", prec="fp32", nx=48, ny=48, nz=24, coils=8, terms=16, shots=4, k_shot=8000,
             turns=3.0, b0_hz=150.0, mask=False),
        # The largest: the normal operator of the 3D 96 x 96 x 48 / 32-coil /
        # 572000-sample workload, which is the bulk of the headline solve.
        dict(name="ehe_3d_96_fp16", kind="EHE", prec="fp16", nx=96, ny=96, nz=48, coils=32, terms=16, shots=16,
             k_shot=35750, turns=7.0, b0_hz=150.0, mask=False),
        # A whole 2D reconstruction: 30 re-orthogonalised CG iterations.
        dict(name="cg_2d_128_fp16", kind="CG", prec="fp16", nx=128, ny=128, nz=1, coils=16, terms=16, shots=4,
             k_shot=15000, turns=4.0, b0_hz=100.0, mask=False, n_iter=30, reorth=True),
        # A whole small 3D reconstruction with bfloat16 operands and the plain
        # recurrences (the call's default).
        dict(name="cg_3d_48_bf16", kind="CG", prec="bf16", nx=48, ny=48, nz=24, coils=8, terms=16, shots=4,
             k_shot=8000, turns=3.0, b0_hz=150.0, mask=False, n_iter=10, reorth=False),
        # A multi-slice reconstruction: uneven slices solved together.
        dict(name="batch_8_slices_bf16", kind="BATCH", prec="bf16", slices=8, n_lo=96, n_hi=160, g_lo=8, g_hi=32,
             k_lo=8000, k_hi=30000, terms=16, b0_hz=100.0, n_iter=12),
        # A 2D reconstruction with its phase basis reduced first, as a caller
        # with a new geometry per scan does it: compression, data rotation,
        # solve.
        dict(name="compressed_cg_2d_128_fp16", kind="COMP", prec="fp16", nx=128, ny=128, nz=1, coils=16, terms=16,
             shots=4, k_shot=15000, turns=4.0, b0_hz=100.0, mask=False, n_iter=12, reorth=True),
        # One step of field-map and trajectory refinement: forward, loss and
        # gradients to the image, the B0 map and the field coefficients.
        dict(name="grad_2d_128_fp32", kind="GRAD", prec="fp32", nx=128, ny=128, nz=1, coils=16, terms=16, shots=4,
             k_shot=15000, turns=4.0, b0_hz=100.0, mask=False),
        # Sensitivity maps from a multi-echo prescan of a slab.
        dict(name="sens_3d_112", kind="SENS", nx=112, ny=112, nz=20, coils=8, echoes=8, alpha=10.0, tol=1e-6),
        # The k-space filter of a reconstructed volume.
        dict(name="filter_3d_96", kind="FILTER", nx=96, ny=96, nz=48),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any of the kinds above at sizes spread over their
    ranges, at most as costly as the largest listed case."""
    kind = rng.choice(["E", "EH", "EHE", "EHE", "CG", "CG", "GRAD", "GRAD", "BATCH", "COMP", "SENS", "FILTER"])
    prec = rng.choice(["fp16", "fp16", "bf16", "fp32"])
    if kind == "FILTER":
        three = rng.random() < 0.5
        return dict(kind=kind, nx=_log_int(rng, 24, 320), ny=_log_int(rng, 24, 320),
                    nz=_log_int(rng, 5, 60) if three else 1)
    if kind == "SENS":
        return dict(kind=kind, nx=_log_int(rng, 40, 130), ny=_log_int(rng, 40, 130),
                    nz=rng.choice([1, 1, _log_int(rng, 4, 22)]), coils=rng.randint(2, 12), echoes=rng.randint(4, 12),
                    alpha=10.0, tol=1e-6)
    if kind == "BATCH":
        lo = rng.randint(24, 96)
        return dict(kind=kind, prec=prec, slices=rng.randint(2, 8), n_lo=lo, n_hi=lo + rng.randint(1, 48),
                    g_lo=rng.randint(2, 8), g_hi=rng.randint(9, 32), k_lo=_log_int(rng, 800, 8000),
                    k_hi=_log_int(rng, 8001, 24000), terms=rng.choice([4, 9, 16]), b0_hz=rng.uniform(20.0, 150.0),
                    n_iter=rng.randint(4, 12))
    three = rng.random() < 0.4
    c = dict(kind=kind, prec=prec, coils=rng.choice([1, 4, 8, 12, 15, 16, 24, 32]), terms=rng.choice([4, 9, 16, 16]),
             b0_hz=rng.uniform(20.0, 150.0), mask=rng.random() < 0.4)
    if three:
        n = _log_int(rng, 16, 64)
        c.update(nx=n, ny=n, nz=_log_int(rng, 6, 32), shots=rng.randint(2, 12), turns=rng.uniform(2.0, 7.0),
                 k_shot=_log_int(rng, 800, 20000))
    else:
        n = _log_int(rng, 24, 200)
        c.update(nx=n, ny=n + rng.randint(-7, 7), nz=1, shots=rng.choice([1, 1, 2, 4]), turns=n / rng.uniform(8.0, 40.0),
                 k_shot=_log_int(rng, 1000, 24000))
    if kind in ("CG", "COMP"):
        c.update(n_iter=rng.randint(4, 20), reorth=True)
    return c


# ---------------------------------------------------------------------------
# inputs (numpy / torch on the seed alone, in float64, rounded once)
def _coords(nx, ny, nz):
    ax = [(torch.arange(n, dtype=torch.float64, device=DEV) - n / 2) / (n / 2) for n in (nx, ny)]
    az = (torch.arange(nz, dtype=torch.float64, device=DEV) - nz / 2) / (nz / 2) if nz > 1 else \
        torch.full((1,), 0.1, dtype=torch.float64, device=DEV)
    z, y, x = torch.meshgrid(az, ax[1], ax[0], indexing="ij")
    return x.reshape(-1), y.reshape(-1), z.reshape(-1)


def _harmonics(x, y, z, n):
    r2 = x * x + y * y + z * z
    t = [torch.ones_like(x), x, y, z, x * y, z * y, 3 * z * z - r2, x * z, x * x - y * y, 3 * x * x * y - y ** 3,
         x * y * z, (5 * z * z - r2) * y, 5 * z ** 3 - 3 * z * r2, (5 * z * z - r2) * x, z * (x * x - y * y),
         x ** 3 - 3 * x * y * y]
    return torch.stack(t[:n])


def _trajectory(rng, n, nz, shots, k_shot, turns, terms):
    """Spiral-out shots to the edge of k-space, small smooth field terms."""
    tau = np.arange(k_shot) / k_shot
    kmax = math.pi * n / 2
    ks = []
    for s in range(shots):
        kc = np.zeros((k_shot, terms))
        th = 2 * np.pi * (turns * tau + s / shots)
        kc[:, 1] = kmax * tau * np.cos(th)
        kc[:, 2] = kmax * tau * np.sin(th)
        if nz > 1:
            spread = nz / shots
            kc[:, 3] = math.pi * ((s - (shots - 1) / 2) * spread + spread * (tau - 0.5))
        for b in [0] + list(range(4, terms)):
            w = sum(rng.uniform(0.5, 1.0) * np.sin(2 * np.pi * (rng.uniform(1.0, 3.0) * tau + rng.uniform()))
                    for _ in range(3))
            kc[:, b] = 1e-3 * kmax * w / np.sqrt(np.mean(w * w))
        ks.append(kc)
    return np.concatenate(ks), np.tile(np.arange(k_shot) * DWELL, shots)


def _b0(rng, x, y, z, hz):
    f = torch.zeros_like(x)
    for _ in range(8):
        c, w, a = rng.uniform(-0.6, 0.6, 3), rng.uniform(0.15, 0.5), rng.choice([-1.0, 1.0])
        f += a * torch.exp(-((x - c[0]) ** 2 + (y - c[1]) ** 2 + (z - c[2]) ** 2) / (2 * w * w))
    f -= f.min()
    return 2 * math.pi * hz * (2 * f / f.max().clamp_min(1e-30) - 1)


def _coil_maps(rng, G, x, y, z, nz):
    S = torch.empty(G, x.numel(), dtype=torch.complex128, device=DEV)
    for j in range(G):
        ring, k = divmod(j, 8) if nz > 1 else (0, j)
        ang = 2 * math.pi * k / (8 if nz > 1 else G) + 0.3 * ring
        c = (1.5 * math.cos(ang), 1.5 * math.sin(ang), -0.75 + 0.5 * ring if nz > 1 else 0.0)
        u = rng.standard_normal(3)
        u /= np.linalg.norm(u)
        d = [x - c[0], y - c[1], z - c[2]]
        ph = 2 * math.pi * j / G + 0.5 * (d[0] * u[0] + d[1] * u[1] + d[2] * u[2])
        S[j] = torch.polar(torch.exp(-(d[0] ** 2 + d[1] ** 2 + d[2] ** 2) / 2), ph)
    return S


def _object(rng, x, y, z):
    """Ellipsoids times a slow phase."""
    rho = torch.zeros_like(x)
    for _ in range(10):
        c, a = rng.uniform(-0.5, 0.5, 3), rng.uniform(0.1, 0.5, 3)
        q = ((x - c[0]) / a[0]) ** 2 + ((y - c[1]) / a[1]) ** 2 + ((z - c[2]) / a[2]) ** 2
        rho += rng.uniform(0.2, 1.0) * (q <= 1.0)
    return torch.polar(rho, 0.3 * x)


def _cnoise(rng, *shape):
    a = rng.standard_normal(shape + (2,), dtype=np.float32)
    return torch.view_as_complex(torch.from_numpy(a)).to(DEV)


def _acquisition(case, rng, data):
    """Model arrays of one acquisition, its object and (if asked) its data:
    the object's points on every n-th voxel plus noise."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    x, y, z = _coords(nx, ny, nz)
    if case.get("mask"):
        keep = (x / 0.86) ** 2 + (y / 0.94) ** 2 + ((z / 1.1) ** 2 if nz > 1 else 0.0) <= 1.0
        x, y, z = x[keep], y[keep], z[keep]
    P = case["terms"]
    kc, t = _trajectory(rng, nx, nz, case["shots"], case["k_shot"], case["turns"], P)
    d = dict(fields=_harmonics(x, y, z, P).float(), b0=_b0(rng, x, y, z, case["b0_hz"]).float(),
             kcoef=torch.from_numpy(kc).float().to(DEV), t=torch.from_numpy(t).float().to(DEV),
             sens=_coil_maps(rng, case["coils"], x, y, z, nz).to(torch.complex64))
    d["rho"] = _object(rng, x, y, z).to(torch.complex64)
    if data:
        L, K, G = x.numel(), t.size, case["coils"]
        step = max(1, -(-L * K // (1 << 28)))
        sub = slice(step // 2, None, step)
        h, b, q = d["fields"][:, sub].double(), d["b0"][sub].double(), (d["sens"] * d["rho"])[:, sub] * step
        m = torch.empty(G, K, dtype=torch.complex64, device=DEV)
        blk = max(1, (1 << 25) // h.shape[1])
        for k0 in range(0, K, blk):
            ph = d["t"][k0:k0 + blk, None].double() * b
            for p in range(P):
                ph += d["kcoef"][k0:k0 + blk, p, None].double() * h[p]
            e = torch.polar(torch.ones_like(ph, dtype=torch.float32), torch.remainder(ph, 2 * math.pi).float())
            for c in range(G):
                m[c, k0:k0 + blk] = (e * q[c]).sum(1)
        sig = float(m.abs().square().mean().sqrt()) / (30 * math.sqrt(2))
        d["m"] = m + sig * _cnoise(rng, G, K)
    return d


def _slice_cases(case):
    """The slices of a batch: their sizes are part of the case."""
    rng = np.random.default_rng([case["slices"], case["n_lo"], case["n_hi"], case["k_lo"], case["k_hi"]])
    out = []
    for _ in range(case["slices"]):
        n = int(rng.integers(case["n_lo"], case["n_hi"] + 1)) // 2 * 2
        out.append(dict(nx=n, ny=n, nz=1, coils=int(rng.integers(case["g_lo"], case["g_hi"] + 1)),
                        terms=case["terms"], shots=1, k_shot=int(rng.integers(case["k_lo"], case["k_hi"] + 1)),
                        turns=n / 8.0, b0_hz=case["b0_hz"], mask=False))
    return out


def _prescan(case, rng):
    x, y, z = _coords(case["nx"], case["ny"], case["nz"])
    zz = (z / 2.5) ** 2 if case["nz"] > 1 else 0.0
    head = (x / 0.84) ** 2 + (y / 0.92) ** 2 + zz <= 1.0
    brain = (x / 0.70) ** 2 + (y / 0.78) ** 2 + zz <= 1.0
    wide = (x / 0.88) ** 2 + (y / 0.96) ** 2 + zz <= 1.0
    rho = 0.12 * head + (0.68 + 0.1 * torch.cos(6 * x) * torch.cos(5 * y)) * brain
    S = _coil_maps(rng, case["coils"], x, y, z, case["nz"])
    om = _b0(rng, x, y, z, 100.0)
    sig = float((S * rho).abs().max()) / (40 * math.sqrt(2))
    X = torch.empty(case["coils"], case["echoes"], x.numel(), dtype=torch.complex64, device=DEV)
    for n in range(case["echoes"]):
        ph = torch.polar(rho, om * (n * 2.3e-3) + 0.2 * (n % 2))
        X[:, n] = (S * ph).to(torch.complex64) + sig * _cnoise(rng, case["coils"], x.numel())
    return dict(imgs=X, mask_T=brain.float(), mask_R=wide.float())


def _volume(case, rng):
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    x, y, z = _coords(nx, ny, nz)
    rho = _object(rng, x, y, z).to(torch.complex64) + 0.02 * _cnoise(rng, x.numel())
    u = [torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device=DEV) for n in (nx, ny, nz)]
    w, v, u = torch.meshgrid(u[2], u[1], u[0], indexing="ij")
    inside = (u / (0.5 * nx)) ** 2 + (v / (0.5 * ny)) ** 2 <= 1.0
    return dict(rho=rho, f=(inside & (w.abs() <= 0.5 * nz)).reshape(-1).float())


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "FILTER":
        return _volume(case, rng)
    if kind == "SENS":
        return _prescan(case, rng)
    if kind == "BATCH":
        return [_acquisition(c, rng, True) for c in _slice_cases(case)]
    d = _acquisition(case, rng, kind in ("EH", "CG", "COMP", "GRAD"))
    if kind == "EHE":  # a CG direction: the object plus fine structure
        d["rho"] = d["rho"] + 0.5 * _cnoise(rng, d["rho"].numel())
    if kind == "GRAD":  # refinement starts from a wrong B0 map and trajectory
        d["kcoef"] = d["kcoef"] * (1 + 1e-3 * torch.from_numpy(rng.standard_normal(case["terms"])).float().to(DEV))
        d["b0"] = d["b0"] * 0.9 + 20.0
    return d


# ---------------------------------------------------------------------------
def _problem(d):
    return nfs.Problem(d["sens"], d["fields"], d["b0"], d["kcoef"], d["t"], device=DEV)


def prepare(case, seed):
    d = _inputs(case, seed)
    st = dict(case=case, d=d)
    kind = case["kind"]
    if kind == "BATCH":
        st["probs"] = [_problem(s) for s in d]
        st["ms"] = [s["m"] for s in d]
    elif kind in ("E", "EH", "EHE", "CG", "COMP"):
        st["prob"] = _problem(d)
    elif kind == "GRAD":
        for k in ("rho", "b0", "kcoef"):
            d[k] = d[k].clone().requires_grad_(True)
    torch.cuda.synchronize()
    return st


def run(st):
    c, d = st["case"], st["d"]
    kind, prec = c["kind"], c.get("prec")
    if kind == "E":
        return nfs.apply_E(st["prob"], d["rho"], prec)
    if kind == "EH":
        return nfs.apply_EH(st["prob"], d["m"], prec)
    if kind == "EHE":
        return nfs.apply_EHE(st["prob"], d["rho"], prec)
    if kind == "CG":
        rho, hist, info = nfs.cg_solve(st["prob"], d["m"], c["n_iter"], precision=prec, reorth=c["reorth"])
        return dict(rho=rho, hist=hist, info=info)
    if kind == "BATCH":
        rho, hist, info = nfs.cg_solve_batched(st["probs"], st["ms"], c["n_iter"], precision=prec, reorth=True)
        return dict(rho=rho, hist=hist, info=info)
    if kind == "COMP":
        cp, theta, _ = nfs.compress_basis(st["prob"])
        rho, hist, info = nfs.cg_solve(cp, nfs.phase_shift(d["m"], theta, -1), c["n_iter"], precision=prec,
                                       reorth=c["reorth"])
        return dict(rho=rho, hist=hist, info=info)
    if kind == "GRAD":
        for k in ("rho", "b0", "kcoef"):
            d[k].grad = None
        y = autograd.encode(d["rho"], d["b0"], d["kcoef"], d["sens"], d["fields"], d["t"], prec)
        (y - d["m"]).abs().square().sum().backward()
        return dict(y=y.detach(), g_rho=d["rho"].grad, g_b0=d["b0"].grad, g_kcoef=d["kcoef"].grad)
    if kind == "SENS":
        s32, s64, shat, info = nfs.sens_maps(d["imgs"], d["mask_T"], d["mask_R"], (c["nx"], c["ny"], c["nz"]),
                                             c["alpha"], tol=c["tol"])
        return dict(s32=s32, s64=s64, shat=shat, info=list(info))
    return nfs.apply_kspace_filter(d["rho"], d["f"], (c["nx"], c["ny"], c["nz"]))


# ---------------------------------------------------------------------------
# 64-bit formulas
class _Op:
    """E and E^H in float64, a block of samples at a time.  Complex values
    are held as real and imaginary rows, so that the products are real."""

    def __init__(self, d):
        self.R = torch.cat([d["b0"].detach().double()[None], d["fields"].double()])
        self.A = torch.cat([d["t"].double()[:, None], d["kcoef"].detach().double()], 1)
        self.S = d["sens"].to(torch.complex128)
        self.G = self.S.shape[0]
        self.K, self.L = self.A.shape[0], self.R.shape[1]
        self.blk = max(1, min(self.K, BLOCK // self.L))

    def blocks(self):
        for k0 in range(0, self.K, self.blk):
            ph = self.A[k0:k0 + self.blk] @ self.R
            yield slice(k0, k0 + ph.shape[0]), torch.cos(ph), torch.sin(ph)

    def _rows(self, rho):
        q = self.S * rho
        return torch.cat([q.real, q.imag])

    def _fwd(self, c, s, q):
        u, v, G = q @ c.T, q @ s.T, self.G
        return torch.cat([u[:G] - v[G:], u[G:] + v[:G]])

    def _back(self, c, s, m):
        u, v, G = m @ c, m @ s, self.G
        return torch.complex(u[:G] + v[G:], u[G:] - v[:G])

    def E(self, rho):
        q = self._rows(rho)
        y = torch.empty(2 * self.G, self.K, dtype=torch.float64, device=DEV)
        for k, c, s in self.blocks():
            y[:, k] = self._fwd(c, s, q)
        return torch.complex(y[:self.G], y[self.G:])

    def EH(self, m):
        m = torch.cat([m.real, m.imag])
        acc = torch.zeros_like(self.S)
        for k, c, s in self.blocks():
            acc += self._back(c, s, m[:, k].contiguous())
        return (self.S.conj() * acc).sum(0)

    def EHE(self, rho):
        q = self._rows(rho)
        acc = torch.zeros_like(self.S)
        for _, c, s in self.blocks():
            acc += self._back(c, s, self._fwd(c, s, q))
        return (self.S.conj() * acc).sum(0)


def _cg64(d, n_iter, reorth):
    op = _Op(d)
    m = d["m"].to(torch.complex128)
    r = op.EH(m)
    p, rho = r.clone(), torch.zeros_like(r)
    dd = float(m.abs().square().sum())
    al = float(r.abs().square().sum())
    hist, V = [[math.sqrt(al), 0.0, dd]], [r / math.sqrt(al)]
    for _ in range(n_iter):
        q = op.EHE(p)
        be = float((p.conj() * q).real.sum())
        rho = rho + (al / be) * p
        r = r - (al / be) * q
        dd -= al * al / be
        if reorth:
            for v in V:
                r = r - (v.conj() * r).sum() * v
        an = float(r.abs().square().sum())
        if reorth:
            V.append(r / math.sqrt(an))
        p = r + (an / al) * p
        al = an
        hist.append([math.sqrt(al), float(rho.abs().square().sum().sqrt()), dd])
    return rho, torch.tensor(hist, dtype=torch.float64, device=DEV), \
        torch.tensor([n_iter, 1], dtype=torch.int32, device=DEV)


def exact(case, seed):
    kind = case["kind"]
    if kind == "SENS":  # an iterative solution to a tolerance
        return None
    d = _inputs(case, seed)
    if kind == "FILTER":
        s = (case["nz"], case["ny"], case["nx"])
        k = torch.fft.fftn(d["rho"].to(torch.complex128).reshape(s)) * d["f"].double().reshape(s)
        return torch.fft.ifftn(k).reshape(-1)
    if kind == "BATCH":
        r = [_cg64(s, case["n_iter"], True) for s in d]
        return dict(rho=[x[0] for x in r], hist=[x[1] for x in r], info=[x[2] for x in r])
    if kind in ("CG", "COMP"):
        rho, hist, info = _cg64(d, case["n_iter"], case["reorth"])
        return dict(rho=rho, hist=hist, info=info)
    op = _Op(d)
    rho = d["rho"].detach().to(torch.complex128)
    if kind == "E":
        return op.E(rho)
    if kind == "EH":
        return op.EH(d["m"].to(torch.complex128))
    if kind == "EHE":
        return op.EHE(rho)
    y = op.E(rho)
    g = 2 * (y - d["m"].to(torch.complex128))
    g_b0 = (rho.conj() * op.EH(g * d["t"].double())).imag
    g_k = torch.stack([(g * op.E(d["fields"][b].double() * rho).conj()).imag.sum(0) for b in range(case["terms"])], 1)
    return dict(y=y, g_rho=op.EH(g), g_b0=g_b0, g_kcoef=g_k)


# ---------------------------------------------------------------------------
def _sizes(case):
    L = case["nx"] * case["ny"] * case["nz"]
    if case.get("mask"):
        L = int(L * math.pi / 4 * 0.86 * 0.94 * (0.92 if case["nz"] > 1 else 1.0))
    return L, case["shots"] * case["k_shot"], case["coils"], case["terms"]


def _op_flops(L, K, G, P):
    """One E or E^H: the phase (P + 1 terms) and the complex contraction."""
    return float(L) * K * (2 * (P + 1) + 8 * G)


def _model_bytes(L, K, G, P):
    return 4.0 * (L * (P + 1) + K * (P + 1)) + 8.0 * G * L


def work(case):
    kind = case["kind"]
    if kind == "FILTER":
        L = case["nx"] * case["ny"] * case["nz"]
        return dict(bytes=20.0 * L, flops=10.0 * L * math.log2(max(2, L)))
    if kind == "SENS":
        L, G, n = case["nx"] * case["ny"] * case["nz"], case["coils"], case["echoes"]
        return dict(bytes=8.0 * G * n * L + 8.0 * L + 40.0 * G * L, flops=8.0 * G * G * n * L)
    if kind == "BATCH":
        w = dict(bytes=0.0, flops=0.0)
        for L, K, G, P in map(_sizes, _slice_cases(case)):
            w["bytes"] += _model_bytes(L, K, G, P) + 8.0 * G * K + 8.0 * L
            w["flops"] += (2 * case["n_iter"] + 1) * _op_flops(L, K, G, P)
        return w
    L, K, G, P = _sizes(case)
    one = _op_flops(L, K, G, P)
    model = _model_bytes(L, K, G, P)
    if kind in ("E", "EH"):
        return dict(bytes=model + 8.0 * L + 8.0 * G * K, flops=one)
    if kind == "EHE":
        return dict(bytes=model + 16.0 * L, flops=2 * one)
    if kind in ("CG", "COMP"):
        return dict(bytes=model + 8.0 * L + 8.0 * G * K, flops=(2 * case["n_iter"] + 1) * one)
    # GRAD: the forward, E^H for the image and for B0, and for the field
    # coefficients the coil sum per pair with its P real products
    return dict(bytes=model + 16.0 * L + 24.0 * G * K + 4.0 * L + 4.0 * K * P,
                flops=4 * one + 2.0 * P * L * K)

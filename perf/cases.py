"""What this framework is asked to do in use, as measurable cases.

A case is a dict of plain values: the entry point (`op`), the grid, the array,
the record and the options.  `prepare` makes what a program holds before the
call (geometry, inputs, workspace), `run` makes one call through the public
binding, `work` counts what the call cannot do without, and `exact` gives the
same outputs in float64 from the equations alone (torch on the device, nothing
of the library).

The physical set-up is the one of the synthetic workloads: 0.5 mm voxels, water
/ steel / cement / rock layers, transmitters a constant step apart, receivers
at 5 mm pitch, a 500 kHz pulse in a 12 us window, the template tabulated at
640 MHz (so 64 fine positions a sample at 10 MHz, 32 at 20 MHz).

Operations
  forward       y = A x
  adjoint       x = A^T r
  pair          one of each (a caller's own iteration, an operator test)
  reconstruct   MAP reconstruction by the surrogate iteration
  icd           MAP reconstruction by grouped ICD (8 x 8 lattice)
  batch         a step of a batch of resident sessions, as a server takes it
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2202_09703_amd import umbir

MM = 1e-3
SPEED = (1480.0, 5900.0, 3000.0, 4500.0)       # water, steel, cement, rock [m/s]
DENSITY = (1000.0, 7850.0, 1900.0, 2600.0)
ALPHA = (2e-6, 0.0, 30e-6, 0.0)                # attenuation where it is asked for [s/m]
F_C, SIGMA_T, T_WIN, F_FINE = 0.5e6, 1.25e-6, 12e-6, 640e6
BETA, STEP = 8, 0.5 * MM
STORAGE = {"f32": umbir.STORAGE_F32, "f16": umbir.STORAGE_F16, "bf16": umbir.STORAGE_BF16}
PRIOR = SimpleNamespace(p=1.1, q=2.0, T=0.01, sigma0=5.0, m=0.1, a=1.0, estimate_direct=True)
SNR_DB = 15.0
LATTICE = (8, 8)          # ICD voxel groups
SESSION_ITER = 100000     # iterations a batch's sessions are created for


def _case(name, op, nx, nz, layers, scans, rx, samples, mhz=20, pitch=4, storage="f32", templates=0, iters=0,
          problems=0):
    return {"name": name, "op": op, "nx": nx, "nz": nz, "layers": layers, "scans": scans, "rx": rx,
            "samples": samples, "mhz": mhz, "pitch": pitch, "storage": storage, "templates": templates,
            "iters": iters, "problems": problems}


def listed():
    return [
        # the smallest calls: one transmitter, eight receivers, a 64 x 64 grid at 10 MHz;
        # launches and latency decide, and half of a server's requests are of this size
        _case("forward_64", "forward", 64, 64, 3, 1, 8, 256, mhz=10),
        _case("adjoint_64", "adjoint", 64, 64, 3, 1, 8, 256, mhz=10),
        # the same problem solved: what a server answers such a request with
        _case("reconstruct_64", "reconstruct", 64, 64, 3, 1, 8, 256, mhz=10, iters=20),
        # the ordinary problem, 32 scan positions of 16 receivers, each direction by itself
        _case("forward_256", "forward", 256, 256, 3, 32, 16, 2048),
        _case("adjoint_256", "adjoint", 256, 256, 3, 32, 16, 2048),
        # the ordinary problem solved (the benchmark's workload, its geometry kept)
        _case("reconstruct_256", "reconstruct", 256, 256, 3, 32, 16, 2048, iters=50),
        # the largest problem, four layers: one application each way, FP32 and FP16 storage
        _case("pair_512", "pair", 512, 512, 4, 64, 32, 4096),
        _case("pair_512_f16", "pair", 512, 512, 4, 64, 32, 4096, storage="f16"),
        # a ragged problem: nothing a power of two, an odd record, BF16 storage
        _case("pair_ragged_bf16", "pair", 331, 187, 4, 11, 19, 1531, storage="bf16"),
        # lossy water and cement: sixteen attenuated templates
        _case("pair_attenuated", "pair", 256, 256, 3, 32, 16, 2048, templates=16),
        # the paper's own solver
        _case("icd_256", "icd", 256, 256, 3, 32, 16, 2048, iters=2),
        # six uneven problems resident on the device, five iterations of each, as the
        # server steps them between admissions
        _case("batch_6", "batch", 384, 384, 4, 16, 32, 4096, iters=5, problems=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_LARGEST = 64 * 32 * 512.0 * 512.0   # (trace, voxel) pairs of the largest listed call


def draw(rng):
    while True:
        op = rng.choice(("forward", "forward", "adjoint", "adjoint", "pair", "reconstruct", "reconstruct", "icd",
                         "batch"))
        mhz = rng.choice((10, 20, 20, 20))
        nx, nz = _log_int(rng, 64, 512), _log_int(rng, 64, 512)
        layers = rng.choice((1, 2, 3, 3, 4))
        scans, rx = _log_int(rng, 1, 64), _log_int(rng, 8, 32)
        samples = _log_int(rng, 256, 4096)
        storage, templates, iters, problems = "f32", 0, 0, 0
        pairs = float(nx * nz * scans * rx)
        if op in ("forward", "adjoint", "pair", "reconstruct"):
            storage = rng.choice(("f32", "f32", "f16", "bf16"))
        if op in ("forward", "adjoint", "pair") and storage == "f32" and layers >= 3 and rng.random() < 0.25:
            templates = rng.choice((4, 8, 16))
        limit = _LARGEST
        if op == "reconstruct":
            iters = rng.randint(10, 50)
            limit = _LARGEST / 16
        elif op == "icd":
            iters = rng.randint(1, 3)
            limit = _LARGEST / 16
        elif op == "batch":
            iters, problems = 5, rng.randint(2, 6)
            limit = 384.0 * 384 * 16 * 32
        if templates:
            limit = _LARGEST / 16
        if pairs > limit:
            continue
        return {"op": op, "nx": nx, "nz": nz, "layers": layers, "scans": scans, "rx": rx, "samples": samples,
                "mhz": mhz, "pitch": rng.choice((2, 4, 6)), "storage": storage, "templates": templates,
                "iters": iters, "problems": problems}


# ---- the problem a case describes


def _card(case):
    n, nx, nz = case["layers"], case["nx"], case["nz"]
    depth = nz * STEP
    thick = (10 * MM, 8 * MM, 0.3125 * depth)[:n - 1]
    atten = ALPHA[:n] if case["templates"] else (0.0,) * n
    scans, rx = case["scans"], case["rx"]
    fs = case["mhz"] * 1e6
    half = case["pitch"] / 2
    return SimpleNamespace(
        medium=SimpleNamespace(speed=SPEED[:n], thickness=thick, atten=atten, density=DENSITY[:n]),
        grid=SimpleNamespace(nx=nx, nz=nz, dx=STEP, dz=STEP, x0=-nx * STEP / 2, z0=0.0),
        array=SimpleNamespace(tx_x=tuple((case["pitch"] * i - half * (scans - 1)) * MM for i in range(scans)),
                              rx_offset=tuple((j - (rx - 1) / 2) * 5 * MM for j in range(rx)), beta=BETA),
        acq=SimpleNamespace(n_samples=case["samples"], fs=fs, f_c=F_C, sigma_t=SIGMA_T, t_win=T_WIN,
                            oversample=int(round(F_FINE / fs)), storage=STORAGE[case["storage"]],
                            n_gamma=case["templates"]))


def _members(case):
    """The uneven problems of a batch: the case's sizes, each member's drawn
    from three tenths of them upwards."""
    rng = np.random.Generator(np.random.PCG64([case["nx"], case["nz"], case["samples"], case["problems"]]))
    out = []
    for k in range(case["problems"]):
        def part(n, least):
            return max(min(n, least), int(round(n * rng.uniform(0.3, 1.0))))
        out.append(dict(case, op="reconstruct", problems=0, nx=part(case["nx"], 64), nz=part(case["nz"], 64),
                        scans=part(case["scans"], 1), rx=part(case["rx"], 8), samples=part(case["samples"], 256)))
    return out


def _image(case, gen):
    """A reflectivity image: the layers' interfaces, a delamination at the
    second one, point reflectors."""
    nx, nz = case["nx"], case["nz"]
    x = torch.zeros(nz, nx, dtype=torch.float64, device="cuda")
    card = _card(case)
    z = [s * d for s, d in zip(card.medium.speed, card.medium.density)]
    top = 0.0
    for k, t in enumerate(card.medium.thickness):
        top += t
        row = int(round(top / STEP))
        if row < nz:
            x[row, :] = (z[k + 1] - z[k]) / (z[k + 1] + z[k])
            if k == 1:
                span = max(1, int(0.3 * nx))
                start = int(torch.randint(0, nx - span + 1, (1,), generator=gen).item())
                x[row, start:start + span] = -0.94
    n = max(5, nx // 6)
    rows = torch.randint(nz // 5, nz, (n,), generator=gen)
    cols = torch.randint(0, nx, (n,), generator=gen)
    amp = torch.rand(n, generator=gen, dtype=torch.float64) * 0.7 + 0.3
    sign = torch.randint(0, 2, (n,), generator=gen).double() * 2 - 1
    x[rows.cuda(), cols.cuda()] = (amp * sign).cuda()
    return x


def _generators(seed):
    cpu = torch.Generator().manual_seed(int(seed) % (1 << 62))
    dev = torch.Generator(device="cuda").manual_seed((int(seed) + 77) % (1 << 62))
    return cpu, dev


def _inputs(case, seed):
    """Images and traces of a seed.  forward takes an image as an iteration
    holds it (structure plus a dense background), adjoint residual traces,
    the solvers data: echoes, weak direct arrivals and noise."""
    cpu, dev = _generators(seed)
    shape = (case["scans"], case["rx"], case["samples"])
    dtype = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[case["storage"]]
    truth = _image(case, cpu)
    got = SimpleNamespace()
    if case["op"] in ("forward", "pair"):
        noise = torch.randn(truth.shape, generator=dev, dtype=torch.float64, device="cuda")
        got.x = (truth + 0.02 * noise).float()
    if case["op"] in ("adjoint", "pair"):
        got.r = torch.randn(shape, generator=dev, dtype=torch.float32, device="cuda").to(dtype)
    if case["op"] in ("reconstruct", "icd"):
        ref = _Exact(case)
        clean = ref.forward(truth, sparse=True)
        got.sigma = float(clean.square().mean().sqrt()) / 10 ** (SNR_DB / 20)
        arrivals = 0.1 + 0.2 * torch.rand(shape[:2], generator=cpu, dtype=torch.float64).cuda()
        noise = torch.randn(shape, generator=dev, dtype=torch.float64, device="cuda")
        got.y = (clean + ref.direct(arrivals) + got.sigma * noise).to(dtype)
    return got


def prepare(case, seed):
    if case["op"] == "batch":
        members = _members(case)
        sessions = []
        for k, c in enumerate(members):
            d = _inputs(c, seed + 1000 * k)
            sessions.append(umbir.Solver(umbir.build_geometry(_card(c)), PRIOR, d.sigma, d.y, SESSION_ITER))
        return SimpleNamespace(case=case, sessions=sessions, batch=umbir.Batch(sessions, umbir.BATCH_STREAMS),
                               x=[torch.empty(s.geom.image_shape, device="cuda") for s in sessions],
                               g=[torch.empty(s.geom.trace_shape[:2], device="cuda") for s in sessions])
    s = _inputs(case, seed)
    s.case = case
    s.geom = umbir.build_geometry(_card(case))
    kind = {"forward": umbir.WORK_FORWARD, "adjoint": umbir.WORK_ADJOINT, "pair": umbir.WORK_ADJOINT,
            "reconstruct": umbir.WORK_RECONSTRUCT}.get(case["op"])
    if kind is not None:
        s.work = s.geom.workspace(kind)
    if case["op"] in ("forward", "pair"):
        s.y_out = torch.empty(s.geom.trace_shape, dtype=s.geom.trace_dtype, device="cuda")
    if case["op"] in ("adjoint", "pair"):
        s.x_out = torch.empty(s.geom.image_shape, device="cuda")
    return s


def run(s):
    op = s.case["op"]
    if op == "forward":
        return umbir.forward(s.geom, s.x, s.y_out, work=s.work)
    if op == "adjoint":
        return umbir.adjoint(s.geom, s.r, s.x_out, work=s.work)
    if op == "pair":
        y = umbir.forward(s.geom, s.x, s.y_out, work=s.work)
        return {"y": y, "x": umbir.adjoint(s.geom, s.r, s.x_out, work=s.work)}
    if op == "reconstruct":
        x, g, cost = umbir.reconstruct(s.geom, PRIOR, s.sigma, s.y, s.case["iters"], work=s.work)
    elif op == "icd":
        x, g, cost = umbir.reconstruct_icd(s.geom, PRIOR, s.sigma, s.y, s.case["iters"], group=LATTICE)
    else:
        s.batch.step(s.case["iters"])
        return [t[:2] for t in (q.read(x, g, with_cost=False) for q, x, g in zip(s.sessions, s.x, s.g))]
    # the cost history comes as float64 sums of FP32 residuals: kept as a caller plots it
    return {"x": x, "g": g, "cost": cost.float()}


def work(case):
    """Compulsory work: images, traces, the one-way travel-time table and the
    templates once per application of A or A^T, and the multiply-adds of the
    operator (L_h taps per (trace, voxel) pair, or per fine position of the
    record where that is less)."""
    if case["op"] == "batch":
        each = [work(c) for c in _members(case)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    n, traces, m = case["nx"] * case["nz"], case["scans"] * case["rx"], case["samples"]
    q = F_FINE / (case["mhz"] * 1e6)
    window = T_WIN * case["mhz"] * 1e6
    elem = 4 if case["storage"] == "f32" else 2
    span = (case["scans"] - 1) * case["pitch"] / 0.5 + (case["rx"] - 1) * 10
    legs = 12.0 * case["nz"] * (2 * case["nx"] + span)
    once_b = 4.0 * n + float(elem) * traces * m + legs + 4.0 * q * window * max(1, case["templates"])
    once_f = 2.0 * window * traces * min(float(n), q * m)
    times = {"forward": 1, "adjoint": 1, "pair": 2, "reconstruct": 2 * case["iters"] + 3,
             "icd": 2 * case["iters"] + 4}[case["op"]]
    return {"bytes": times * once_b, "flops": times * once_f}


# ---- the same outputs in float64, from the equations


class _Exact:
    """A, A^T and D of a case in float64 on the device.  Delays, weights and
    templates follow the paper's Eqs. (3)-(12); entry (trace, m; voxel) is
    W I((m - D) Q), I the linear interpolant of the tabulated template."""

    def __init__(self, case):
        self.case, card = case, _card(case)
        a, g, q, med = card.array, card.grid, card.acq, card.medium
        self.nx, self.nz, self.P, self.K = g.nx, g.nz, len(a.tx_x), len(a.rx_offset)
        self.M, self.Q, self.fs = q.n_samples, q.oversample, q.fs
        self.Lh = int(round(T_WIN * q.fs))
        f64 = dict(dtype=torch.float64, device="cuda")
        lat = [int(round(2 * (g.x0 - t) / g.dx)) + 1 for t in a.tx_x]
        rxo = [int(round(2 * (g.x0 - t - o) / g.dx)) + 1 for t in a.tx_x for o in a.rx_offset]
        self.btx = torch.tensor(lat, device="cuda").repeat_interleave(self.K)
        self.brx = torch.tensor(rxo, device="cuda")
        n_off = max(max(abs(b), abs(b + 2 * (g.nx - 1))) for b in lat + rxo) + 1
        # one-way legs [nz][n_off]: bisection for the ray parameter (Snell)
        depth = (torch.arange(g.nz, **f64) + 0.5) * g.dz + g.z0
        X = torch.arange(n_off, **f64)[None, :] * (g.dx / 2)
        tops = [0.0]
        for t in med.thickness:
            tops.append(tops[-1] + t)
        eta = torch.stack([(torch.minimum(depth, torch.full_like(depth, tops[k + 1] if k + 1 < len(tops) else math.inf))
                            - tops[k]).clamp(min=0.0) for k in range(len(tops))])
        c = torch.tensor(med.speed, **f64)
        cmax = torch.where(eta > 0, c[:, None], torch.zeros_like(eta)).amax(0)
        hi = (1.0 / cmax)[:, None].expand(-1, n_off).clone()
        lo = torch.zeros_like(hi)

        def offset(k):
            x = torch.zeros_like(k)
            for l in range(len(c)):
                s = k * c[l] * (eta[l] > 0)[:, None]
                x += eta[l][:, None] * s / torch.sqrt((1 - s) * (1 + s))
            return x

        for _ in range(64):
            mid = 0.5 * (lo + hi)
            low = offset(mid) < X
            lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
        k = torch.where(X == 0, torch.zeros_like(lo), 0.5 * (lo + hi))
        T, theta, att = k * X, torch.zeros_like(k), torch.zeros_like(k)
        for l in range(len(c)):
            s = k * c[l] * (eta[l] > 0)[:, None]
            cosv = torch.sqrt((1 - s) * (1 + s))
            T += eta[l][:, None] * cosv / c[l]
            theta += torch.asin(s)
            att += med.atten[l] * eta[l][:, None] / cosv
        self.delay, self.apod = T * q.fs * self.Q, torch.cos(theta) ** a.beta  # delays in fine positions
        layer = (eta > 0).sum(0) - 1
        tau, zimp = torch.ones(g.nz, **f64), [s * d for s, d in zip(med.speed, med.density)]
        for l in range(len(c) - 1):
            tau = torch.where(layer > l, tau * (4 * zimp[l] * zimp[l + 1] / (zimp[l] + zimp[l + 1]) ** 2), tau)
        self.tau = tau
        # templates [G][Q Lh + 1]
        t = torch.arange(self.Q * self.Lh + 1, **f64) / (self.Q * q.fs) - T_WIN / 2
        bank = [torch.sin(2 * math.pi * F_C * t) * torch.exp(-t * t / (2 * SIGMA_T ** 2))]
        self.G, self.att = 1, None
        if case["templates"] and float(att.max()) > 0:
            self.G = case["templates"]
            step = 2 * float(att.max()) / (self.G - 1)
            self.att = att / step
            nodes, wts = np.polynomial.legendre.leggauss(24)
            fmax = F_C + 6 / (math.pi * SIGMA_T)
            panels = max(16, int(math.ceil(8 * fmax * T_WIN / 2)))
            edges = np.linspace(0, fmax, panels + 1)
            f = ((edges[1:] + edges[:-1])[:, None] / 2 + (edges[1] - edges[0]) / 2 * nodes[None, :]).reshape(-1)
            wf = np.tile((edges[1] - edges[0]) / 2 * wts, panels)
            spec = SIGMA_T * math.sqrt(2 * math.pi) * (np.exp(-2 * (math.pi * SIGMA_T * (f - F_C)) ** 2)
                                                       - np.exp(-2 * (math.pi * SIGMA_T * (f + F_C)) ** 2))
            f, amp = torch.tensor(f, **f64), torch.tensor(wf * spec, **f64)
            sines = torch.sin(2 * math.pi * t[:, None] * f[None, :])
            bank += [sines @ (amp * torch.exp(-gb * step * f)) for gb in range(1, self.G)]
        self.bank = torch.stack(bank)
        self.bank[:, 0] = 0.0
        self.bank[:, -1] = 0.0
        self.MQ = self.M * self.Q
        self.size = self.MQ + self.Q * self.Lh + 2
        self.n_fft = 1 << (self.size - 1).bit_length()
        m = torch.arange(self.M, **f64)
        cols = [self._interp((m - q.fs * abs(o) / med.speed[0]) * self.Q) for o in a.rx_offset]
        self.dbasis = torch.stack(cols)[None].expand(self.P, -1, -1)

    def _interp(self, z):
        last = self.Q * self.Lh
        inside = (z > 0) & (z < last)
        zc = torch.where(inside, z, torch.zeros_like(z))
        n = zc.floor().long()
        f = zc - n
        b = self.bank[0]
        return torch.where(inside, (1 - f) * b[n] + f * b[(n + 1).clamp(max=last)], torch.zeros_like(z))

    def _chunks(self, n_vox):
        step = max(1, min(self.P * self.K, int(2 ** 27 // max(n_vox * 2, self.n_fft * max(1, self.G)))))
        return [(t, min(t + step, self.P * self.K)) for t in range(0, self.P * self.K, step)]

    def _pairs(self, t0, t1, row, col):
        """Fine position J, fraction, weight and template of (trace, voxel)."""
        ia = (self.btx[t0:t1, None] + 2 * col[None, :]).abs()
        ib = (self.brx[t0:t1, None] + 2 * col[None, :]).abs()
        r = row[None, :].expand_as(ia)
        D = self.delay[r, ia] + self.delay[r, ib]
        w = self.tau[row][None, :] * self.apod[r, ia] * self.apod[r, ib]
        J = D.floor()
        phi = D - J
        J = J.clamp(max=self.MQ).long()
        if self.G == 1:
            return J, phi, w, None
        b = (self.att[r, ia] + self.att[r, ib] + 0.5).floor().clamp(max=self.G - 1).long()
        return J, phi, w, b

    def _voxels(self, vox):
        if vox is None:
            vox = torch.arange(self.nx * self.nz, device="cuda")
        return vox, vox // self.nx, vox % self.nx

    def spectra(self, absolute=False):
        b = self.bank.abs() if absolute else self.bank
        return torch.fft.rfft(b, n=self.n_fft)

    def forward(self, x, vox=None, absolute=False, sparse=False):
        """A x over the voxels `vox` (x: their values), all voxels by default."""
        if sparse:
            vox = x.reshape(-1).nonzero().reshape(-1)
            x = x.reshape(-1)[vox]
        vox, row, col = self._voxels(vox)
        x = x.reshape(-1)
        spec = self.spectra(absolute)
        out = []
        for t0, t1 in self._chunks(len(vox)):
            J, phi, w, b = self._pairs(t0, t1, row, col)
            w = (w.abs() if absolute else w) * x[None, :]
            width = self.MQ + 2
            s = torch.zeros(t1 - t0, self.G * width, dtype=torch.float64, device="cuda")
            J = J if b is None else J + b * width
            s.scatter_add_(1, J, w * (1 - phi))
            s.scatter_add_(1, J + 1, w * phi)
            s = s.view(t1 - t0, self.G, width)[:, :, :self.MQ]
            y = torch.fft.irfft((torch.fft.rfft(s, n=self.n_fft) * spec[None]).sum(1), n=self.n_fft)
            out.append(y[:, :self.MQ:self.Q].clone())
        return torch.cat(out).view(self.P, self.K, self.M)

    def adjoint(self, r, vox=None, absolute=False):
        vox, row, col = self._voxels(vox)
        spec = self.spectra(absolute).conj()
        r = r.double().reshape(self.P * self.K, self.M)
        x = torch.zeros(len(vox), dtype=torch.float64, device="cuda")
        for t0, t1 in self._chunks(len(vox)):
            up = torch.zeros(t1 - t0, self.MQ, dtype=torch.float64, device="cuda")
            up[:, ::self.Q] = r[t0:t1]
            c = torch.fft.irfft(torch.fft.rfft(up, n=self.n_fft)[:, None] * spec[None], n=self.n_fft)
            width = self.MQ + 2
            c = c[:, :, :width].clone()
            c[:, :, self.MQ:] = 0.0
            c = c.reshape(t1 - t0, self.G * width)
            J, phi, w, b = self._pairs(t0, t1, row, col)
            J = J if b is None else J + b * width
            w = w.abs() if absolute else w
            x += (w * ((1 - phi) * c.gather(1, J) + phi * c.gather(1, J + 1))).sum(0)
        return x

    def direct(self, g):
        return self.dbasis * g[:, :, None]

    # the prior (QGGMRF on the 8-neighbourhood), its cost and its surrogate

    def _cliques(self):
        edge = 1 / (4 + 2 * math.sqrt(2))
        depth = torch.arange(self.nz, dtype=torch.float64, device="cuda") + 0.5
        ms = 1 + (PRIOR.m - 1) * (depth / depth[-1]) ** PRIOR.a
        for dr, dc, bw in ((0, 1, edge), (1, 0, edge), (1, -1, edge / math.sqrt(2)), (1, 1, edge / math.sqrt(2))):
            s = (slice(0, self.nz - dr), slice(max(0, -dc), self.nx - max(0, dc)))
            r = (slice(dr, self.nz), slice(max(0, dc), self.nx - max(0, -dc)))
            sg = PRIOR.sigma0 * torch.sqrt(ms[s[0]] * ms[r[0]])[:, None]
            yield s, r, bw, sg

    def prior(self, x):
        """Cost, slope sum 2 B d and curvature sum 2 B of the prior at x."""
        cost, slope, curv = 0.0, torch.zeros_like(x), torch.zeros_like(x)
        p, T = PRIOR.p, PRIOR.T
        for s, r, bw, sg in self._cliques():
            d = x[s] - x[r]
            u = (d.abs() / (T * sg)) ** (2 - p)
            lead = T ** (p - 2) / sg ** 2
            cost = cost + (bw * d * d * lead / (p * (1 + u))).sum()
            B = bw * 0.5 * lead * (2 / p + u) / (1 + u) ** 2
            slope[s] += 2 * B * d
            slope[r] -= 2 * B * d
            curv[s] += 2 * B
            curv[r] += 2 * B
        return cost, slope, curv

    def _g_step(self, e, g):
        norm = self.dbasis.square().sum(2)
        dg = torch.where(norm > 0, (self.dbasis * e).sum(2) / norm.clamp(min=1e-300), torch.zeros_like(norm))
        return e - self.direct(dg), g + dg

    def _residual(self, y, x, g):
        return y - self.forward(x) - self.direct(g)

    def sqs(self, y, sigma, iters):
        y = y.double()
        x = torch.zeros(self.nz, self.nx, dtype=torch.float64, device="cuda")
        g = torch.zeros(self.P, self.K, dtype=torch.float64, device="cuda")
        den = self.adjoint(self.forward(torch.ones_like(x), absolute=True), absolute=True).view_as(x) / sigma ** 2
        cost = []
        for _ in range(iters):
            e = self._residual(y, x, g)
            c, slope, curv = self.prior(x)
            cost.append(e.square().sum() / (2 * sigma ** 2) + c)
            e, g = self._g_step(e, g)
            u = self.adjoint(e).view_as(x)
            x = x - (slope - u / sigma ** 2) / (den + 2 * curv)
        e = self._residual(y, x, g)
        cost.append(e.square().sum() / (2 * sigma ** 2) + self.prior(x)[0])
        return x, g, torch.stack(cost)

    def icd(self, y, sigma, sweeps):
        y = y.double()
        idx = torch.arange(self.nz * self.nx, device="cuda").view(self.nz, self.nx)
        groups = [idx[a::LATTICE[0], b::LATTICE[1]].reshape(-1) for a in range(LATTICE[0]) for b in range(LATTICE[1])]
        ones = [torch.ones(len(v), dtype=torch.float64, device="cuda") for v in groups]
        den = [self.adjoint(self.forward(o, v, absolute=True), v, absolute=True) / sigma ** 2
               for o, v in zip(ones, groups)]
        x = torch.zeros(self.nz, self.nx, dtype=torch.float64, device="cuda")
        g = torch.zeros(self.P, self.K, dtype=torch.float64, device="cuda")
        e, cost = y, []
        for _ in range(sweeps):
            cost.append(e.square().sum() / (2 * sigma ** 2) + self.prior(x)[0])
            e, g = self._g_step(e, g)
            for v, d in zip(groups, den):
                _, slope, curv = self.prior(x)
                theta = slope.reshape(-1)[v] - self.adjoint(e, v) / sigma ** 2
                h = d + curv.reshape(-1)[v]
                step = torch.where(h > 0, -theta / h.clamp(min=1e-300), torch.zeros_like(h))
                x.view(-1)[v] += step
                e = e - self.forward(step, v)
        cost.append(e.square().sum() / (2 * sigma ** 2) + self.prior(x)[0])
        return x, g, torch.stack(cost)


def exact(case, seed):
    if case["op"] == "batch":
        out = []
        for k, c in enumerate(_members(case)):
            d = _inputs(c, seed + 1000 * k)
            out.append(list(_Exact(c).sqs(d.y, d.sigma, case["iters"])[:2]))
        return out
    d = _inputs(case, seed)
    ref = _Exact(case)
    if case["op"] == "forward":
        return ref.forward(d.x.double())
    if case["op"] == "adjoint":
        return ref.adjoint(d.r).view(ref.nz, ref.nx)
    if case["op"] == "pair":
        return {"y": ref.forward(d.x.double()), "x": ref.adjoint(d.r).view(ref.nz, ref.nx)}
    # a whole solve costs two applications an iteration: left out where that is long
    pairs = case["nx"] * case["nz"] * case["scans"] * case["rx"]
    if case["op"] == "reconstruct":
        if pairs * case["iters"] > 2.5e9:
            return None
        x, g, cost = ref.sqs(d.y, d.sigma, case["iters"])
    else:
        if case["scans"] * case["rx"] * case["samples"] * case["iters"] > 2.5e6:
            return None
        x, g, cost = ref.icd(d.y, d.sigma, case["iters"])
    return {"x": x, "g": g, "cost": cost}

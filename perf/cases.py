"""Timed cases of the library's paths, through its Python entry points.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (inputs drawn from the seed, contexts with their basis loaded),
`run` is one pass of it, `work` the bytes and operations the pass cannot do
without, and `exact` the same outputs in float64 by plain torch.

Kinds
  modal      one system: push of a window of sampled steps, read, reset
  group      many uneven systems advanced together (one grouped push), reads
  shc        spectral heat current of one run: push, read, reset
  shc_group  many independent SHC runs advanced together
  virial     neighbour lists and one evaluation of Tersoff Si
  md         molecular dynamics of Tersoff Si writing the push inputs; with
             lags > 0 the SHC correlation of those steps on the fly

A pass reads a window and clears it (the paper's HNEMA output cadence), so
that every pass of a state gives the same outputs; molecular dynamics runs on
from where the last pass ended, as a trajectory does.
"""
import math

import numpy as np
import torch

from paper_2102_03691_amd import (DIRECTIONAL, GKMA, HNEMA, PREC_BF16X3, PREC_FP32, PREC_FP8X3, ModalGroup, ModalHC,
                                  ModalSHC, ModalVirial, SHCGroup, tersoff_si)

DEV = "cuda:0"
KB = 8.617333262e-5                                    # eV / K
KE = 1.66053906660e-27 * 1e10 / 1.602176634e-19        # 1 amu (A/fs)^2 in eV
SI_MASS, SPRING, SI_A = 28.0855, 10.0, 5.432           # amu, eV / A^2, A
ISOTOPES = ((27.9769265, 0.922), (28.9764947, 0.047), (29.9737702, 0.031))
PREC = {"fp32": PREC_FP32, "bf16x3": PREC_BF16X3, "fp8x3": PREC_FP8X3}
BPE = {"fp32": 4, "bf16x3": 4, "fp8x3": 2}             # bytes of a stored basis element
METHODS = {"hnema": HNEMA, "gkma": GKMA, "both": HNEMA | GKMA, "dir": HNEMA | DIRECTIONAL}


def listed():
    modal = dict(kind="modal", precision="bf16x3", t=128, methods="hnema", share=1.0, bins=500, lags=0, natural=False,
                 host=False)
    return [
        # an MD code that hands over every step as it is made, on the smallest
        # lattice: latency and launches
        dict(modal, name="step_sc4", dims="4,4,4", precision="fp32", t=1, bins=100, steps=1),
        # the default configuration (float32, no blocking), a trajectory piece of 64 steps
        dict(modal, name="steps_sc16", dims="16,16,16", precision="fp32", t=1, steps=64),
        # the headline workload: thin film, split bfloat16, T = 128
        dict(modal, name="slab_bf16x3", dims="48,48,4", bins=1000, steps=256),
        # a rod (nanotube-like) with GKMA beside HNEMA, one correlation window
        dict(modal, name="rod_gkma", dims="4,4,500", t=256, methods="both", lags=500, steps=2048),
        # odd sizes, natural isotopes, the lower part of the spectrum only,
        # host arrays, a trailing partial block
        dict(modal, name="ragged_host", dims="7,9,11", t=96, methods="both", share=0.7216, bins=37, lags=150, natural=True,
             host=True, steps=250),
        # the split by direction of motion (in-plane / flexural) in float32
        dict(modal, name="film_dir_fp32", dims="24,24,4", precision="fp32", t=64, methods="dir", bins=200, steps=128),
        # 16 uneven systems served together, e4m3 hi/lo, HNEMA and GKMA mixed
        dict(kind="group", name="uneven_fp8x3", edges="20,16,10,8,12,14,16,8,20,10,12,14,8,16,10,12",
             methods="hnema,gkma,hnema,gkma,gkma,hnema,hnema,hnema,hnema,gkma,hnema,gkma,hnema,gkma,hnema,hnema",
             precision="fp8x3", t=64, bins=100, lags=200, steps=128),
        # SHC of an 8000-atom run: 250 lags (500 fs at 2 fs)
        dict(kind="shc", name="shc_8000", atoms=8000, lags=250, t=256, steps=512),
        # 32 independent small SHC runs, averaged over by the paper
        dict(kind="shc_group", name="shc_32_small",
             atoms="216,512,1000,343,729,250,864,400,216,640,960,300,512,800,450,343,"
                   "1000,216,700,576,384,900,250,512,864,320,432,729,216,600,1000,486", lags=250, t=256, steps=256),
        # a program with its own integrator: new lists and one evaluation
        dict(kind="virial", name="virial_64k", cells="20,20,20", skin=0.0),
        # NVE production of a large block, push inputs of every step kept
        dict(kind="md", name="nve_216k", cells="30,30,30", steps=32, rebuild=16, nvt=False, lags=0, t=0),
        # the paper's HNEMD + SHC protocol on its 8000-atom block: thermostat,
        # driving force, SHC on the fly
        dict(kind="md", name="hnemd_8000", cells="10,10,10", steps=256, rebuild=50, nvt=True, lags=250, t=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["modal_step", "modal", "modal", "modal", "group", "shc", "shc_group", "virial", "md", "md"])
    if kind == "modal_step":
        e = [_log_int(rng, 3, 16) for _ in range(3)]
        return dict(kind="modal", dims=",".join(map(str, e)), precision="fp32", t=1,
                    methods=rng.choice(["hnema", "hnema", "both"]), share=rng.choice([1.0, 1.0, rng.uniform(0.3, 1.0)]),
                    bins=_log_int(rng, 3, 500), lags=_log_int(rng, 10, 300), natural=rng.random() < 0.5, host=rng.random() < 0.25,
                    steps=_log_int(rng, 1, 96))
    if kind == "modal":
        e = [_log_int(rng, 4, 18) for _ in range(3)]
        t = 32 * rng.randint(1, 8)
        return dict(kind="modal", dims=",".join(map(str, e)), precision=rng.choice(["bf16x3", "bf16x3", "fp32", "fp8x3"]), t=t,
                    methods=rng.choice(["hnema", "hnema", "gkma", "both", "dir"]),
                    share=rng.choice([1.0, 1.0, rng.uniform(0.3, 1.0)]), bins=_log_int(rng, 3, 1000), lags=_log_int(rng, 20, 600),
                    natural=rng.random() < 0.5, host=rng.random() < 0.25, steps=max(1, round(t * rng.uniform(0.5, 4.0))))
    if kind == "group":
        n = rng.randint(3, 20)
        return dict(kind="group", edges=",".join(str(rng.randint(4, 16)) for _ in range(n)),
                    methods=",".join(rng.choice(["hnema", "gkma"]) for _ in range(n)),
                    precision=rng.choice(["bf16x3", "fp8x3", "fp8x3", "fp32"]), t=32 * rng.randint(1, 4), bins=_log_int(rng, 3, 300),
                    lags=_log_int(rng, 20, 300), steps=rng.randint(40, 300))
    if kind == "shc":
        t = 64 * rng.randint(1, 8)
        return dict(kind="shc", atoms=_log_int(rng, 200, 8000), lags=_log_int(rng, 50, 500), t=t,
                    steps=max(1, round(t * rng.uniform(0.5, 2.0))))
    if kind == "shc_group":
        return dict(kind="shc_group", atoms=",".join(str(_log_int(rng, 100, 2000)) for _ in range(rng.randint(4, 48))),
                    lags=_log_int(rng, 50, 500), t=rng.choice([64, 128, 192, 256]), steps=rng.randint(50, 400))
    if kind == "virial":
        return dict(kind="virial", cells=",".join(str(_log_int(rng, 2, 20)) for _ in range(3)), skin=rng.choice([0.0, 0.0, 0.5, 1.0]))
    nvt = rng.random() < 0.5
    t = 64 * rng.randint(1, 4)
    return dict(kind="md", cells=",".join(str(_log_int(rng, 2, 16)) for _ in range(3)), steps=_log_int(rng, 8, 200),
                rebuild=rng.choice([10, 20, 50, 0]), nvt=nvt, lags=_log_int(rng, 50, 300) if nvt else 0, t=t if nvt else 0)


def _ints(text):
    return [int(x) for x in text.split(",")]


# ------------------------------------------------------------------ lattices
class _Lattice:
    """Simple-cubic lattice of L1 x L2 x L3 atoms and a real orthonormal basis:
    the plane waves (cos + sin)(2 pi k.r) / sqrt(N) times a frame of three
    polarisations per k (one along the wave vector), with the frequencies of
    nearest-neighbour springs; the `share` lowest modes of it."""

    def __init__(self, dims, share=1.0):
        self.dims = dims
        L = np.array(dims)
        self.N = int(L.prod())
        k = np.stack(np.meshgrid(*[np.arange(x) for x in dims], indexing="ij"), axis=-1).reshape(-1, 3)
        self.k = k
        s2 = np.sin(np.pi * np.minimum(k, L - k) / L) ** 2
        w0 = math.sqrt(SPRING / (SI_MASS * KE)) * 1000.0 / (2.0 * math.pi)
        f = np.repeat(2.0 * w0 * np.sqrt(np.sort(s2, axis=1).sum(axis=1)), 3)
        self.f_max = 2.0 * w0 * math.sqrt(3.0)
        q = np.sin(2.0 * np.pi * k / L) + 0.5 * (2 * k == L)
        n = np.linalg.norm(q, axis=1, keepdims=True)
        e1 = np.where(n > 1e-9, q / np.maximum(n, 1e-9), np.array([1.0, 0.0, 0.0]))
        axis = np.eye(3)[np.argmin(np.abs(e1), axis=1)]
        e2 = np.cross(e1, axis)
        e2 /= np.linalg.norm(e2, axis=1, keepdims=True)
        self.pol = np.stack([e1, e2, np.cross(e1, e2)], axis=1)          # [k, 3, 3]
        m = max(1, round(share * 3 * self.N))
        self.modes = np.arange(3 * self.N) if m == 3 * self.N else np.sort(np.argsort(f, kind="stable")[:m])
        self.freq = f[self.modes]
        self.M = len(self.modes)

    def rows(self, m0, n):
        """Rows m0 .. m0 + n - 1 of E^T, [n, 3N] float64 on the GPU."""
        m = torch.as_tensor(self.modes[m0:m0 + n], device=DEV)
        if not hasattr(self, "_dev"):
            L1, L2, L3 = self.dims
            w = torch.tensor([L2 * L3, L1 * L3, L1 * L2], device=DEV)
            k = torch.as_tensor(self.k, device=DEV)
            tab = torch.arange(self.N, device=DEV, dtype=torch.float64) * (2.0 * math.pi / self.N)
            self._dev = k * w, k, (tab.cos() + tab.sin()) / math.sqrt(self.N), torch.as_tensor(self.pol, device=DEV)
        kw, r, wave, pol = self._dev
        f = m // 3
        p = kw[f, 0, None] * r[:, 0] + kw[f, 1, None] * r[:, 1] + kw[f, 2, None] * r[:, 2]
        phi = wave[p.remainder_(self.N)]
        return (phi[:, :, None] * pol[f, m % 3][:, None, :]).reshape(len(m), 3 * self.N)

    def bins(self, nb):
        return np.minimum(np.floor(self.freq / (self.f_max / nb) + 1e-9).astype(np.int64), nb - 1)


def _masses(n, natural, seed):
    if not natural:
        return np.full(n, SI_MASS)
    m, p = np.array(ISOTOPES).T
    return m[np.random.default_rng(seed).choice(3, size=n, p=p / p.sum())]


def _steps(seed, mass, n, device=DEV):
    """Maxwell-Boltzmann velocities at 300 K [n, N, 3] and Gaussian virials [n, N, 3, 3]."""
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    sig = torch.as_tensor(np.sqrt(KB * 300.0 / (mass * KE)), device=device).float()
    v = torch.randn((n, len(mass), 3), generator=g, device=device) * sig[:, None]
    return v, torch.randn((n, len(mass), 3, 3), generator=g, device=device)


def _context(lat, mass, methods, precision, t, bins, lags, stream=None):
    h = ModalHC(0, stream)
    h.load_system(mass, lat.freq)
    h.set_bins_uniform(bins, 0.0, lat.f_max)
    h.configure(methods=methods, precision=PREC[precision], t_block=t, corr_len=lags if methods & GKMA else 0, dt=1.0)
    chunk = max(1, (1 << 26) // (3 * lat.N))
    for m0 in range(0, lat.M, chunk):
        h.load_eigvec_rows(m0, lat.rows(m0, min(chunk, lat.M - m0)))
    h.finalize()
    return h


def _read(h, methods):
    out = {}
    if methods & HNEMA:
        out["hnema"], out["total"], _ = h.read_hnema()
    if methods & DIRECTIONAL:
        out["hnema_dir"], out["total_dir"], _ = h.read_hnema_dir()
    if methods & GKMA:
        g = h.read_gkma()
        out["corr"], out["integral"], out["hcacf"] = g["corr"], g["integral"], g["hcacf"]
    return out


def _modal_parts(case):
    lat = _Lattice(_ints(case["dims"]), case["share"])
    return lat, _masses(lat.N, case["natural"], 7), METHODS[case["methods"]]


def _group_parts(case, seed):
    for q, (e, m) in enumerate(zip(_ints(case["edges"]), case["methods"].split(","))):
        lat = _Lattice((e, e, e))
        mass = _masses(lat.N, q % 2 == 1, q)
        yield lat, mass, METHODS[m], _steps(seed * 64 + q, mass, case["steps"])


# ------------------------------------------------------------------- silicon
_CELL = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0], [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]])


def _silicon(cells, seed):
    """Displaced diamond crystal: positions and box (A), masses, velocities at 300 K."""
    rng = np.random.default_rng(seed)
    c = np.stack(np.meshgrid(*[np.arange(x) for x in cells], indexing="ij"), axis=-1).reshape(-1, 1, 3)
    box = np.array(cells) * SI_A
    pos = (4 * c + _CELL).reshape(-1, 3) * (SI_A / 4) + 0.06 * rng.standard_normal((8 * len(c), 3))
    mass = _masses(len(pos), True, 5)
    vel = rng.standard_normal((len(pos), 3)) * np.sqrt(KB * 300.0 / (mass * KE))[:, None]
    return np.mod(pos, box), box, mass, vel


def _bonds(cells):
    """The four bonded atoms of every atom [N, 4] (slot q of the partner's row
    points back), from the lattice sites."""
    n = 4 * np.array(cells)
    site = (4 * np.stack(np.meshgrid(*[np.arange(x) for x in cells], indexing="ij"), axis=-1).reshape(-1, 1, 3) + _CELL).reshape(-1, 3)
    at = np.full(tuple(n), -1, dtype=np.int64)
    at[tuple(site.T)] = np.arange(len(site))
    step = np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]])
    sign = np.where(site.sum(axis=1) % 4 == 0, 1, -1)
    to = np.mod(site[:, None, :] + sign[:, None, None] * step, n)
    return torch.as_tensor(at[to[..., 0], to[..., 1], to[..., 2]], device=DEV)


def _tersoff(x, box, nbr):
    """Site energies, forces and per-atom virials (Eqs. 4 and 8) in float64."""
    p = tersoff_si()
    d = x[nbr] - x[:, None, :]
    r = (d - box * torch.round(d / box)).requires_grad_(True)
    l = r.norm(dim=2)
    s = torch.sin(0.5 * math.pi * (l - p["R"]) / p["D"])
    fc = torch.where(l < p["R"] - p["D"], torch.ones_like(l), torch.where(l > p["R"] + p["D"], torch.zeros_like(l), 0.5 - 0.5 * s))
    u = r / l[:, :, None]
    cs = torch.matmul(u, u.transpose(1, 2).contiguous())
    g = p["gamma"] * (1.0 + (p["c"] / p["d"]) ** 2 * (cs - p["h"]) ** 2 / (p["d"] ** 2 + (cs - p["h"]) ** 2))
    other = 1.0 - torch.eye(4, device=DEV, dtype=torch.float64)
    zeta = (g * fc[:, None, :] * other).sum(dim=2)
    b = (1.0 + (p["beta"] * zeta) ** p["n"]) ** (-0.5 / p["n"])
    U = 0.5 * (fc * (p["A"] * torch.exp(-p["lambda1"] * l) - b * p["B"] * torch.exp(-p["lambda2"] * l))).sum(dim=1)
    dij, = torch.autograd.grad(U.sum(), r)
    r = r.detach()
    dji = dij[nbr, torch.arange(4, device=DEV)]
    return U.detach(), (dij - dji).sum(dim=1), (r[:, :, :, None] * dji[:, :, None, :]).sum(dim=1)


_FE = (1e-5, 0.0, 0.0)      # driving force, 1 / A
_T0, _TAU = 300.0, 100.0    # thermostat, K and fs


def _drive(U, W, vel, mass):
    fe = torch.tensor(_FE, device=DEV, dtype=torch.float64)
    e = U + 0.5 * KE * mass * (vel * vel).sum(dim=1)
    return e[:, None] * fe + (fe[None, :, None] * W).sum(dim=1)


def _trajectory(case, seed):
    cells = _ints(case["cells"])
    pos, box, mass, vel = (torch.as_tensor(a, device=DEV) for a in _silicon(cells, seed))
    nbr, n, nvt = _bonds(cells), len(pos), case["nvt"]
    c, xi, eta = 0.5 / KE, 0.0, 0.0
    gkt = 3 * n * KB * _T0
    G = lambda: (float((mass[:, None] * vel * vel).sum()) * KE - gkt) / (gkt * _TAU ** 2)  # noqa: E731

    def force():
        U, F, W = _tersoff(pos, box, nbr)
        return (F + _drive(U, W, vel, mass) if nvt else F), W
    F, _ = force()
    vs, Ws = [], []
    for _ in range(case["steps"]):
        if nvt:
            xi += 0.5 * G()
            vel = vel * math.exp(-0.5 * xi)
            eta += 0.5 * xi
        vel = vel + c * F / mass[:, None]
        pos = pos + vel
        pos = pos - torch.floor(pos / box) * box
        F, W = force()
        vel = vel + c * F / mass[:, None]
        if nvt:
            vel = vel * math.exp(-0.5 * xi)
            eta += 0.5 * xi
            xi += 0.5 * G()
        vs.append(vel.float())
        Ws.append(W.float())
    out = {"pos": pos, "vel": vel, "v32": torch.stack(vs).double(), "W32": torch.stack(Ws).double()}
    if nvt:
        out["xi"], out["eta"] = xi, eta
    return out


# ----------------------------------------------------------------------- SHC
_OMEGA = np.linspace(0.0, 0.12, 240)     # rad / fs: 0 .. 19 THz


def _shc_read(s):
    K, _ = s.read_dir()
    return K


def _shc_exact(v, W, lags):
    """K[tau, mu, nu] = <sum_i W_i^{mu nu}(s) v_i^nu(s + tau)> over the available origins."""
    S = v.shape[0]
    K = torch.zeros((lags, 3, 3), dtype=torch.float64, device=DEV)
    for nu in range(3):
        late = v[:, :, nu].double()
        for mu in range(3):
            gram = W[:, :, mu, nu].double() @ late.T.contiguous()
            for tau in range(min(lags, S)):
                K[tau, mu, nu] = torch.diagonal(gram, offset=tau).sum() / (S - tau)
    return K


def _spectrum_exact(K, dt):
    """Even extension, trapezoid rule, Hann window, for every split component."""
    n = K.shape[0]
    t = torch.arange(n, device=DEV, dtype=torch.float64)
    c = torch.full((n,), 2.0, device=DEV, dtype=torch.float64)
    c[0] = c[-1] = 1.0
    if n > 1:
        c = c * 0.5 * (1.0 + torch.cos(math.pi * t / (n - 1)))
    w = torch.as_tensor(_OMEGA, device=DEV)
    return dt * (torch.cos(w[:, None] * t * dt) * c) @ K.reshape(n, -1)


# --------------------------------------------------------------- the four calls
def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "kind": kind}
    if kind == "modal":
        lat, mass, methods = _modal_parts(case)
        st["methods"] = methods
        st["h"] = _context(lat, mass, methods, case["precision"], case["t"], case["bins"], case["lags"])
        v, W = _steps(seed, mass, case["steps"])
        st["v"], st["W"] = (v.cpu().numpy(), W.cpu().numpy()) if case["host"] else (v, W)
    elif kind == "group":
        st["stream"] = torch.cuda.Stream()
        st["hs"], st["methods"], st["v"], st["W"] = [], [], [], []
        with torch.cuda.stream(st["stream"]):
            for lat, mass, methods, (v, W) in _group_parts(case, seed):
                st["hs"].append(_context(lat, mass, methods, case["precision"], case["t"], case["bins"], case["lags"],
                                         st["stream"].cuda_stream))
                st["methods"].append(methods)
                st["v"].append(v)
                st["W"].append(W)
            # the tile shape is fixed: a timed choice would change the rounding from run to run
            st["group"] = ModalGroup(st["hs"], graph=True, autotune=False)
        st["stream"].synchronize()
    elif kind == "shc":
        mass = _masses(case["atoms"], True, 3)
        st["shc"] = ModalSHC(case["atoms"], case["lags"], case["t"])
        st["v"], st["W"] = _steps(seed, mass, case["steps"])
    elif kind == "shc_group":
        st["stream"] = torch.cuda.Stream()
        st["v"], st["W"], st["runs"] = [], [], []
        with torch.cuda.stream(st["stream"]):
            for q, n in enumerate(_ints(case["atoms"])):
                v, W = _steps(seed * 64 + q, _masses(n, True, q), case["steps"])
                st["v"].append(v)
                st["W"].append(W)
                st["runs"].append(ModalSHC(n, case["lags"], case["t"], stream=st["stream"].cuda_stream))
            st["group"] = SHCGroup(st["runs"])
        st["stream"].synchronize()
    else:
        pos, box, mass, vel = _silicon(_ints(case["cells"]), seed)
        skin = 1.0 if kind == "md" else case["skin"]
        st["vir"] = ModalVirial(mass, box, tersoff_si(), max_neighbors=24 if skin > 0.5 else 16, skin=skin)
        st["pos"], st["vel"] = torch.as_tensor(pos, device=DEV), torch.as_tensor(vel, device=DEV)
        if kind == "md":
            n, S = len(pos), case["steps"]
            st["v32"] = torch.empty((S, n, 3), dtype=torch.float32, device=DEV)
            st["W32"] = torch.empty((S, n, 3, 3), dtype=torch.float32, device=DEV)
            st["th"] = (0.0, 0.0)
            st["shc"] = ModalSHC(n, case["lags"], case["t"]) if case["lags"] else None
            st["vir"].neighbors(st["pos"])
    return st


def run(st):
    case, kind = st["case"], st["kind"]
    if kind == "modal":
        st["h"].push(st["v"], st["W"])
        out = _read(st["h"], st["methods"])
        st["h"].reset()
        return out
    if kind == "group":
        with torch.cuda.stream(st["stream"]):
            st["group"].push(st["v"], st["W"])
            out = [_read(h, m) for h, m in zip(st["hs"], st["methods"])]
            for h in st["hs"]:
                h.reset()
        return out
    if kind == "shc":
        st["shc"].push(st["v"], st["W"])
        out = _shc_read(st["shc"])
        st["shc"].reset()
        return out
    if kind == "shc_group":
        with torch.cuda.stream(st["stream"]):
            st["group"].push(st["v"], st["W"])
            out = [_shc_read(s) for s in st["runs"]]
            for s in st["runs"]:
                s.reset()
        return out
    vir, pos, vel = st["vir"], st["pos"], st["vel"]
    if kind == "virial":
        vir.neighbors(pos)
        return vir.compute(pos, vel, _FE)
    out = {"pos": pos, "vel": vel, "v32": st["v32"], "W32": st["W32"]}
    if case["nvt"]:
        st["th"] = vir.md_nvt(pos, vel, 1.0, case["steps"], _FE, _T0, _TAU, thermostat=st["th"], rebuild=case["rebuild"],
                              v32=st["v32"], W32=st["W32"])
        out["xi"], out["eta"] = st["th"]
    else:
        vir.md(pos, vel, 1.0, case["steps"], rebuild=case["rebuild"], v32=st["v32"], W32=st["W32"])
    if st["shc"] is not None:
        st["shc"].push(st["v32"], st["W32"])
        out["K"] = _shc_read(st["shc"])
        out["spectrum"] = st["shc"].spectrum_dir(_OMEGA, 1.0, window=True)
        st["shc"].reset()
    return out


def _modal_work(lat, methods, precision, bins, lags, steps):
    nd = 3 if methods & DIRECTIONAL else 1
    outs = (bins * 3 * nd * 8 if methods & HNEMA else 0) + (2 * lags * bins * 9 * 8 if methods & GKMA else 0)
    corr = 2.0 * 3 * (bins + 1) * 3 * lags * steps if methods & GKMA else 0.0
    return np.array([lat.M * 3.0 * lat.N * BPE[precision] + 48.0 * lat.N * steps + outs, 24.0 * lat.N * lat.M * steps + corr])


def _shc_work(atoms, lags, steps):
    # every sample's inputs once; a product for each available (step, lag) pair
    pairs = sum(max(0, steps - tau) for tau in range(lags))
    return np.array([48.0 * atoms * steps + 72.0 * lags, 18.0 * atoms * pairs])


def work(case):
    kind = case["kind"]
    if kind == "modal":
        lat, _, methods = _modal_parts(case)
        w = _modal_work(lat, methods, case["precision"], case["bins"], case["lags"], case["steps"])
    elif kind == "group":
        w = sum(_modal_work(_Lattice((e, e, e)), METHODS[m], case["precision"], case["bins"], case["lags"], case["steps"])
                for e, m in zip(_ints(case["edges"]), case["methods"].split(",")))
    elif kind == "shc":
        w = _shc_work(case["atoms"], case["lags"], case["steps"])
    elif kind == "shc_group":
        w = sum(_shc_work(n, case["lags"], case["steps"]) for n in _ints(case["atoms"]))
    else:
        n = 8.0 * math.prod(_ints(case["cells"]))
        ops = 4 * 65.0 + 12 * 79.0           # four bonds, twelve ordered pairs of bonds per atom
        if kind == "virial":
            # positions, velocities and masses in; U, F, W, W32 and F_ext out
            w = np.array([n * (24 + 24 + 8 + 8 + 24 + 72 + 36 + 24), n * ops])
        else:
            # per step the inputs of the push out; positions, velocities and forces read and written
            w = np.array([n * (48 + 2 * 72) * case["steps"], n * ops * case["steps"]])
            if case["lags"]:
                w = w + _shc_work(n, case["lags"], case["steps"])
    return {"bytes": float(w[0]), "flops": float(w[1])}


# ------------------------------------------------------------- float64 values
def _modal_exact(lat, mass, methods, bins, lags, v, W):
    S = v.shape[0]
    sm = torch.as_tensor(np.sqrt(mass), device=DEV)
    u = (v.double() * sm[:, None]).reshape(S, -1)
    w = W.double() / sm[:, None, None]
    nd = 3 if methods & DIRECTIONAL else 1
    b = torch.as_tensor(lat.bins(bins), device=DEV)
    Jb = torch.zeros((bins, 3, nd, S), dtype=torch.float64, device=DEV)
    chunk = max(1, (1 << 26) // (3 * lat.N))
    for m0 in range(0, lat.M, chunk):
        E = lat.rows(m0, min(chunk, lat.M - m0))
        X = E @ u.T
        for mu in range(3):
            for nu in range(nd):
                if nd == 3:
                    A = E.reshape(-1, lat.N, 3)[:, :, nu].contiguous() @ w[:, :, mu, nu].T
                else:
                    A = E @ w[:, :, mu, :].reshape(S, -1).T
                Jb[:, mu, nu].index_add_(0, b[m0:m0 + E.shape[0]], X * A)
    Jt = (W.double() * v.double()[:, :, None, :]).sum(dim=1)              # [S, mu, nu]
    out = {}
    if methods & HNEMA:
        out["hnema"], out["total"] = Jb.sum(dim=2).mean(dim=2), Jt.sum(dim=2).mean(dim=0)
    if methods & DIRECTIONAL:
        out["hnema_dir"], out["total_dir"] = Jb.mean(dim=3), Jt.mean(dim=0)
    if methods & GKMA:
        J = Jt.sum(dim=2)                                                  # [S, nu]
        rows = torch.cat([Jb[:, :, 0].reshape(3 * bins, S), J.T])
        C = torch.zeros((lags, 3 * (bins + 1), 3), dtype=torch.float64, device=DEV)
        for tau in range(min(lags, S)):
            C[tau] = rows[:, tau:] @ J[: S - tau] / (S - tau)
        C = C.reshape(lags, bins + 1, 3, 3)
        I = torch.zeros_like(C)
        I[1:] = torch.cumsum(0.5 * (C[1:] + C[:-1]), dim=0)
        out["corr"], out["integral"], out["hcacf"] = C[:, :bins], I[:, :bins], C[:, bins]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "modal":
        lat, mass, methods = _modal_parts(case)
        return _modal_exact(lat, mass, methods, case["bins"], case["lags"], *_steps(seed, mass, case["steps"]))
    if kind == "group":
        return [_modal_exact(lat, mass, methods, case["bins"], case["lags"], v, W)
                for lat, mass, methods, (v, W) in _group_parts(case, seed)]
    if kind == "shc":
        return _shc_exact(*_steps(seed, _masses(case["atoms"], True, 3), case["steps"]), case["lags"])
    if kind == "shc_group":
        return [_shc_exact(*_steps(seed * 64 + q, _masses(n, True, q), case["steps"]), case["lags"])
                for q, n in enumerate(_ints(case["atoms"]))]
    if kind == "virial":
        cells = _ints(case["cells"])
        pos, box, mass, vel = (torch.as_tensor(a, device=DEV) for a in _silicon(cells, seed))
        U, F, W = _tersoff(pos, box, _bonds(cells))
        return {"U": U, "F": F, "W": W, "W32": W, "Fext": _drive(U, W, vel, mass)}
    out = _trajectory(case, seed)
    if case["lags"]:
        K = _shc_exact(out["v32"], out["W32"], case["lags"])
        out["K"], out["spectrum"] = K, _spectrum_exact(K, 1.0).reshape(-1, 3, 3)
    return out

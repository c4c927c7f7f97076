"""Performance cases of the FEWHA library: the calls that programs make on it, at the sizes of the
configured systems (8 m test and VLT-like systems, the 37 m and 39 m MAORY-like systems, the 9-layer
system with spot elongation and DM fitting) and at neighbouring, odd sizes.

A case is a dict of plain values:
  kind      what is called: an operator (apply_A, apply_AT, apply_M, rhs), "transforms" (W^{-1} and
            W^{-T} of a batch), "frame" (Context.reconstruct), "streamed" (slopes from host memory),
            "graph" (Batch.reconstruct, graph replay), "solve" (converged MAP solves of a batch) or
            "gradient" (forward and implicit backward through the MAP solve)
  system    the telescope, sensors and layers (SYSTEMS), `subaps` the subapertures per side of its
            large sensors
  batch     problems (or frames) per call; a "graph" case of system "mixed" takes half of them from
            the 39 m system and half from the 5-layer 8 m system, each with its own Cn2, r0 and sigma
  iters, closed, augment, groups, tuned, rtol   the options of the call

Slopes are those of frozen-flow von Karman screens plus Gaussian slope noise.  The reference values
(`exact`) come from Reference below: the same operators as dense float64 torch products (bilinear
sampling and the wavelet basis are separable, so each is a product with two small matrices).
"""

import functools
import math

import numpy as np
import torch

ARCSEC = math.pi / (180.0 * 3600.0)
SQ10 = math.sqrt(10.0)
SQ5 = math.sqrt(5.0 + 2.0 * SQ10)
# Daubechies-3 lowpass filter in closed form, and its highpass partner
H3 = [v / (16.0 * math.sqrt(2.0)) for v in (1 + SQ10 + SQ5, 5 + SQ10 + 3 * SQ5, 10 - 2 * SQ10 + 2 * SQ5,
                                            10 - 2 * SQ10 - 2 * SQ5, 5 + SQ10 - 3 * SQ5, 1 + SQ10 - SQ5)]
G3 = [(-1) ** i * H3[5 - i] for i in range(6)]

# D (m), obstructed area, LGS (count, ring radius in arcsec, first azimuth), NGS (the same), layer
# grids, heights (m), Cn2 weights, levels, domain side (m), spot elongation, fitted DMs, iterations
SYSTEMS = {
    "8m": dict(D=8.0, obs=0.11, lgs=(3, 40.0, 0.0), ngs=(2, 30.0, 60.0), ngs_sigma=0.05, n=(32, 32, 64),
               h=(0.0, 4000.0, 12700.0), cn2=(0.6, 0.25, 0.15), levels=3, side=12.8, subaps=20, iters=4),
    "8m_5layers": dict(D=8.0, obs=0.0, lgs=(4, 30.0, 45.0), ngs=(0, 0.0, 0.0), ngs_sigma=0.1, n=(64,) * 5,
                       h=(0.0, 2000.0, 4000.0, 8000.0, 14000.0), cn2=(0.2,) * 5, levels=4, side=12.8, subaps=40,
                       iters=6),
    "37m": dict(D=37.0, obs=0.11, lgs=(6, 45.0, 0.0), ngs=(3, 55.0, 60.0), ngs_sigma=0.1, n=(128, 64, 64),
                h=(0.0, 4000.0, 12700.0), cn2=(0.75, 0.15, 0.10), levels=5, side=64.0, subaps=74, iters=2),
    "39m": dict(D=39.0, obs=0.11, lgs=(6, 45.0, 0.0), ngs=(3, 55.0, 60.0), ngs_sigma=0.1, n=(128, 128, 256),
                h=(0.0, 4000.0, 12700.0), cn2=(0.75, 0.15, 0.10), levels=5, side=62.4, subaps=80, iters=4),
    "39m_9layers": dict(D=39.0, obs=0.11, lgs=(6, 45.0, 0.0), ngs=(0, 0.0, 0.0), ngs_sigma=0.1,
                        n=(128,) * 5 + (256,) * 4, h=tuple(2500.0 * k for k in range(9)),
                        cn2=(0.45, 0.12, 0.09, 0.08, 0.07, 0.06, 0.05, 0.045, 0.035), levels=5, side=62.4,
                        subaps=80, iters=20, elong=0.2, fit=True),
}
POOL = 3  # frames of a sequence's pool, walked forward and back


def listed():
    return [
        # one wavefront propagated through the small test system: the smallest call, all latency
        dict(name="propagate_8m", kind="apply_A", system="8m", subaps=20),
        # the normal operator by itself at full size, as a program's own solver or a diagnosis calls it
        dict(name="normal_operator_39m", kind="apply_M", system="39m", subaps=80),
        # layers from stored coefficients and back, for 32 sequences: encode and decode
        dict(name="transforms_39m_x32", kind="transforms", system="39m", subaps=80, batch=32),
        # one control step of the small system
        dict(name="frame_8m", kind="frame", system="8m", subaps=20, iters=4),
        # one control step of the 39 m system on a context with default launch shapes
        dict(name="frame_39m", kind="frame", system="39m", subaps=80, iters=4),
        # the paper's own system and solver (2 augmented iterations), latency on the graph path with
        # the launch shapes that the autotuner finds for single frames
        dict(name="frame_37m_augmented", kind="graph", system="37m", subaps=74, batch=1, iters=2, augment=2,
             tuned=True),
        # closed loop with the slopes arriving in host memory by sensor groups
        dict(name="closed_loop_39m_streamed", kind="streamed", system="39m", subaps=80, iters=4, closed=True,
             groups=3),
        # the benchmark's timed batch: 32 sequences per graph replay
        dict(name="batch_39m_x32", kind="graph", system="39m", subaps=80, batch=32, iters=4),
        # an uneven batch: 12 problems of the 39 m and 12 of the 5-layer 8 m system
        dict(name="batch_mixed_x24", kind="graph", system="mixed", subaps=80, batch=24, iters=6),
        # the 9-layer system with block noise, 20 iterations and the fitting step
        dict(name="batch_9layers_x8", kind="graph", system="39m_9layers", subaps=80, batch=8, iters=20),
        # a training step of the prior weights and heights on the small system: forward and backward
        dict(name="gradient_8m_x5", kind="gradient", system="8m", subaps=20, batch=5, rtol=1e-10),
        # converged reference solutions at full size (against which a frame's error is measured)
        dict(name="solve_39m_x2", kind="solve", system="39m", subaps=80, batch=2, rtol=1e-9),
    ]


def draw(rng):
    """One more case of the same ranges: other sensor sizes (odd ones among them), batches and options."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["operator", "operator", "transforms", "frame", "frame", "streamed", "graph", "graph", "graph",
                       "gradient", "solve"])
    system = rng.choice(["8m", "8m_5layers", "37m", "39m"])
    subaps = {"8m": lambda: rng.randint(13, 22), "8m_5layers": lambda: rng.randint(25, 42),
              "37m": lambda: rng.randint(55, 78), "39m": lambda: rng.randint(61, 84)}
    if kind == "operator":
        return dict(kind=rng.choice(["apply_A", "apply_AT", "apply_M", "rhs"]), system=system, subaps=subaps[system]())
    if kind == "transforms":
        return dict(kind="transforms", system=system, subaps=subaps[system](), batch=size(1, 32))
    if kind == "frame":
        return dict(kind="frame", system=system, subaps=subaps[system](), iters=rng.randint(2, 10))
    if kind == "streamed":
        return dict(kind="streamed", system=system, subaps=subaps[system](), iters=rng.randint(2, 6),
                    closed=rng.random() < 0.5, groups=rng.randint(1, 4))
    if kind == "graph":
        which = rng.choice(["8m", "8m_5layers", "37m", "39m", "39m", "mixed", "39m_9layers"])
        if which == "39m_9layers":
            return dict(kind="graph", system=which, subaps=rng.randint(61, 80), batch=size(1, 8),
                        iters=rng.randint(8, 20))
        if which == "mixed":
            return dict(kind="graph", system=which, subaps=rng.randint(61, 84), batch=2 * size(1, 12),
                        iters=rng.randint(2, 6))
        return dict(kind="graph", system=which, subaps=subaps[which](), batch=size(1, 33), iters=rng.randint(2, 6),
                    augment=rng.choice([0, 0, 1, 2, 3]), tuned=rng.random() < 0.3)
    if kind == "gradient":
        return dict(kind="gradient", system="8m", subaps=rng.randint(13, 22), batch=size(1, 8), rtol=1e-10)
    if rng.random() < 0.6:
        return dict(kind="solve", system="8m", subaps=rng.randint(13, 22), batch=size(1, 16), rtol=1e-10)
    return dict(kind="solve", system="39m", subaps=rng.randint(72, 84), batch=rng.randint(1, 2), rtol=1e-9)


# ---------------------------------------------------------------- systems

def _ring(count, radius, first_az):
    az = [math.radians(first_az + k * 360.0 / max(count, 1)) for k in range(count)]
    return [(radius * ARCSEC * math.cos(a), radius * ARCSEC * math.sin(a), a) for a in az]


def config(system, subaps, closed=False, augment=0, cn2=None, r0=0.157, sigma=0.1):
    """A configuration of the library (a Context's cfg) from a system of SYSTEMS."""
    s = SYSTEMS[system]
    D = s["D"]
    wfs = [dict(kind="lgs", n_subap=subaps, theta=(x, y), H=90000.0, sigma=sigma,
                launch=(0.5 * D * math.cos(a), 0.5 * D * math.sin(a)), tt_removal=True) for x, y, a in _ring(*s["lgs"])]
    wfs += [dict(kind="ngs", n_subap=2, theta=(x, y), H=None, sigma=s["ngs_sigma"] if sigma == 0.1 else sigma,
                 launch=(0.0, 0.0), tt_removal=False) for x, y, _ in _ring(*s["ngs"])]
    cfg = dict(name=system, D=D, obstruction=s["obs"], wfs=wfs,
               layers=[dict(h=h, n=n, levels=s["levels"], cn2=w) for h, n, w in zip(s["h"], s["n"], cn2 or s["cn2"])],
               domain_side=s["side"], prior=dict(alpha=1.0, r0=r0, L0=25.0, tau=0.0),
               noise=dict(alpha_eta=s.get("elong", 0.0), na_fwhm=11400.0, spot_fwhm=ARCSEC), iters=s["iters"],
               gain=0.5 if closed else 1.0, loop="closed" if closed else "open", augment=augment)
    if s.get("fit"):
        cfg["dms"] = [dict(h=0.0, n_act=83, pitch=D / 80), dict(h=4000.0, n_act=47, pitch=1.0),
                      dict(h=12700.0, n_act=47, pitch=1.0)]
        cfg["fit"] = dict(directions=[(x * ARCSEC, y * ARCSEC) for y in (-30.0, 0.0, 30.0) for x in (-30.0, 0.0, 30.0)],
                          iters=10, eps_rel=1e-6)
    return cfg


def problems(case, seed):
    """The configurations of the case's problems (those of an uneven batch differ by the seed)."""
    kw = dict(closed=case.get("closed", False), augment=case.get("augment", 0))
    n = case.get("batch", 1)
    if case["system"] != "mixed":
        return [config(case["system"], case["subaps"], **kw)] * n
    g = np.random.default_rng([seed, 5])
    out = []
    for k in range(n):
        system, subaps = ("39m", case["subaps"]) if k < n // 2 else ("8m_5layers", case["subaps"] // 2)
        w = np.maximum(g.dirichlet(np.ones(len(SYSTEMS[system]["n"]))), 1e-3)
        out.append(config(system, subaps, cn2=[float(v) for v in w], r0=float(g.uniform(0.1, 0.2)),
                          sigma=float(g.uniform(0.05, 0.3))))
    return out


# -------------------------------------------------------------- reference

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


@functools.lru_cache(maxsize=None)
def _analysis(m, device):
    A = np.zeros((m, m))
    for k in range(m // 2):
        for i in range(6):
            A[k, (2 * k + i) % m] += H3[i]
            A[m // 2 + k, (2 * k + i) % m] += G3[i]
    return torch.tensor(A, dtype=torch.float64, device=device)


def _grid_lines(t, n):
    """Bilinear sampling matrix of a grid of n nodes at positions t (node units), and its derivative in t
    (on a grid line the mean of the one-sided ones)."""
    q = np.floor(t).astype(int)
    w = t - q
    rows = np.arange(len(t))
    S, dS = np.zeros((len(t), n)), np.zeros((len(t), n))
    S[rows, q] += 1.0 - w
    S[rows, q + 1] += w
    near = np.rint(t).astype(int)
    tie = np.abs(t - near) < 1e-9
    lo, hi = np.where(tie, np.maximum(near - 1, 0), q), np.where(tie, np.minimum(near + 1, n - 1), q + 1)
    f = np.where(tie, 0.5, 1.0)
    np.add.at(dS, (rows, hi), f)
    np.add.at(dS, (rows, lo), -f)
    return S, dS


class Reference:
    """One configuration's operators in float64.  Coefficients and layers are lists of (B, n, n) tensors,
    slopes lists (one entry per group of sensors of one size) of pairs of (B, sensors, N, N) grids."""

    def __init__(self, cfg):
        self.cfg, self.dev = cfg, _device()
        D, L = cfg["D"], cfg["domain_side"]
        self.n = [l["n"] for l in cfg["layers"]]
        self.delta = [L / n for n in self.n]
        self.nc = sum(n * n for n in self.n)
        self.alpha = cfg["prior"]["alpha"]
        ten = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=self.dev)  # noqa: E731
        self.groups = []
        for N in dict.fromkeys(w["n_subap"] for w in cfg["wfs"]):
            ids = [g for g, w in enumerate(cfg["wfs"]) if w["n_subap"] == N]
            ws = [cfg["wfs"][g] for g in ids]
            x, c = -0.5 * D + np.arange(N + 1) * (D / N), -0.5 * D + (np.arange(N) + 0.5) * (D / N)
            X, Y = np.meshgrid(c, c)
            R = np.sqrt(X * X + Y * Y)
            mask = (R >= math.sqrt(cfg["obstruction"]) * 0.5 * D) & (R <= 0.5 * D)
            S = []
            for l, lay in enumerate(cfg["layers"]):
                mats = []
                for w in ws:
                    sc = 1.0 - lay["h"] / w["H"] if w["kind"] == "lgs" else 1.0
                    for ax in (1, 0):  # rows are y
                        a, da = _grid_lines((sc * x + lay["h"] * w["theta"][ax] + 0.5 * L) / self.delta[l], lay["n"])
                        dt = ((-x / w["H"] if w["kind"] == "lgs" else 0.0 * x) + w["theta"][ax]) / self.delta[l]
                        mats.append((a, da * dt[:, None]))
                S.append([ten(np.stack([m[k] for m in mats[ax::2]])) for ax in (0, 1) for k in (0, 1)])  # Sy dSy Sx dSx
            cov = np.zeros((len(ws), 3, N, N))
            for k, w in enumerate(ws):
                s2 = w["sigma"] ** 2
                cov[k, 0] = cov[k, 2] = s2
                if w["kind"] == "lgs" and cfg["noise"]["alpha_eta"] > 0:
                    fw, e2 = cfg["noise"]["na_fwhm"] / w["H"] ** 2, (cfg["noise"]["alpha_eta"] / cfg["noise"]["spot_fwhm"]) ** 2
                    bx, by = fw * (X - w["launch"][0]), fw * (Y - w["launch"][1])
                    cov[k] += s2 * e2 * np.stack([bx * bx, bx * by, by * by])
            det = cov[:, 0] * cov[:, 2] - cov[:, 1] ** 2
            inv = np.stack([cov[:, 2], -cov[:, 1], cov[:, 0]], 1) / det[:, None] * mask
            self.groups.append(dict(N=N, ids=ids, S=S, mask=torch.tensor(mask, device=self.dev), m=ten(mask * 1.0),
                                    nM=int(mask.sum()), inv=[ten(inv[:, k]) for k in range(3)],
                                    tt=ten([1.0 if w["kind"] == "lgs" and w["tt_removal"] else 0.0 for w in ws]),
                                    sigma=[w["sigma"] for w in ws]))
        pr = cfg["prior"]
        self.D = []
        for lay in cfg["layers"]:
            n, jmin = lay["n"], int(math.log2(lay["n"])) - lay["levels"]
            mx = np.maximum(*np.meshgrid(np.arange(n), np.arange(n)))
            f = 2.0 ** np.where(mx >= 1 << jmin, np.floor(np.log2(np.maximum(mx, 1))), jmin) / L
            self.D.append(ten((f * f + pr["L0"] ** -2.0) ** (11.0 / 6.0) / (0.023 * lay["cn2"] * pr["r0"] ** (-5.0 / 3.0))))
        self._J = None

    # -- layouts
    def split(self, v):
        """(B, N_c) -> list of (B, n, n)."""
        return [p.reshape(-1, n, n) for p, n in zip(v.to(self.dev, torch.float64).split([n * n for n in self.n], 1), self.n)]

    @staticmethod
    def join(x):
        return torch.cat([v.reshape(v.shape[0], -1) for v in x], 1)

    def slopes_out(self, s):
        parts = {}
        for g, (sx, sy) in zip(self.groups, s):
            for k, i in enumerate(g["ids"]):
                parts[i] = torch.cat([sx[:, k][:, g["mask"]], sy[:, k][:, g["mask"]]], 1)
        return torch.cat([parts[i] for i in sorted(parts)], 1)

    def slopes_in(self, v):
        v = v.to(self.dev, torch.float64)
        sizes = [2 * g["nM"] for w in self.cfg["wfs"] for g in self.groups if g["N"] == w["n_subap"]]
        parts = v.split(sizes, 1)
        out = []
        for g in self.groups:
            s = torch.zeros(2, v.shape[0], len(g["ids"]), g["N"], g["N"], dtype=torch.float64, device=self.dev)
            for k, i in enumerate(g["ids"]):
                s[0, :, k, g["mask"]], s[1, :, k, g["mask"]] = parts[i][:, :g["nM"]], parts[i][:, g["nM"]:]
            out.append((s[0], s[1]))
        return out

    # -- operators
    def W(self, x, scale=True):
        out = []
        for v, lay, d in zip(x, self.cfg["layers"], self.delta):
            v, m = v.clone(), lay["n"]
            for _ in range(lay["levels"]):
                A = _analysis(m, self.dev)
                v[:, :m, :m] = A @ v[:, :m, :m] @ A.T
                m //= 2
            out.append(v / d if scale else v)
        return out

    def Winv(self, c):
        out = []
        for v, lay, d in zip(c, self.cfg["layers"], self.delta):
            v = v.clone()
            for k in range(lay["levels"] - 1, -1, -1):
                m = lay["n"] >> k
                A = _analysis(m, self.dev)
                v[:, :m, :m] = A.T @ v[:, :m, :m] @ A
            out.append(v / d)
        return out

    def A(self, x, only=None):
        """Slopes of the layers x; only = l: the derivative in h_l instead."""
        out = []
        for g in self.groups:
            v = 0.0
            for l, (Sy, dSy, Sx, dSx) in enumerate(g["S"]):
                if only is None:
                    v = v + Sy @ x[l][:, None] @ Sx.mT
                elif only == l:
                    v = v + dSy @ x[l][:, None] @ Sx.mT + Sy @ x[l][:, None] @ dSx.mT
            a, b, c, d = v[..., :-1, :-1], v[..., :-1, 1:], v[..., 1:, :-1], v[..., 1:, 1:]
            out.append((0.5 * ((b - a) + (d - c)) * g["m"], 0.5 * ((c - a) + (d - b)) * g["m"]))
        return out

    def AT(self, s):
        out = [0.0] * len(self.n)
        for g, (sx, sy) in zip(self.groups, s):
            p, q = 0.5 * (sx + sy), 0.5 * (sx - sy)
            pad = torch.nn.functional.pad
            v = pad(p, (1, 0, 1, 0)) - pad(p, (0, 1, 0, 1)) + pad(q, (1, 0, 0, 1)) - pad(q, (0, 1, 1, 0))
            for l, (Sy, _, Sx, _) in enumerate(g["S"]):
                out[l] = out[l] + (Sy.mT @ v @ Sx).sum(1)
        return out

    def weigh(self, s):
        """C_hat^{-1} s."""
        out = []
        for g, (sx, sy) in zip(self.groups, s):
            t = (g["tt"] / g["nM"])[None, :, None, None]
            flat = lambda v: v - v.sum((2, 3), keepdim=True) * t * g["m"]  # noqa: B023, E731
            sx, sy = flat(sx), flat(sy)
            a, b, c = g["inv"]
            out.append((flat(a * sx + b * sy), flat(b * sx + c * sy)))
        return out

    def M(self, c):
        q = self.W(self.AT(self.weigh(self.A(self.Winv(c)))))
        return [v + self.alpha * d * x for v, d, x in zip(q, self.D, c)]

    def rhs(self, s):
        return self.W(self.AT(self.weigh(s)))

    @property
    def J(self):
        """The exact diagonal of M: a basis function u v^T has slopes that are products of one factor along
        each axis, so a band's diagonal is a few small matrix products."""
        if self._J is None:
            self._J = []
            for l, lay in enumerate(self.cfg["layers"]):
                n = lay["n"]
                diag = torch.zeros(n, n, dtype=torch.float64, device=self.dev)
                low, m = torch.eye(n, dtype=torch.float64, device=self.dev), n
                for _ in range(lay["levels"]):
                    B = low @ _analysis(m, self.dev).T
                    low, high, m = B[:, :m // 2], B[:, m // 2:], m // 2
                    diag[:m, m:2 * m] = self._band(l, low, high)
                    diag[m:2 * m, :m] = self._band(l, high, low)
                    diag[m:2 * m, m:2 * m] = self._band(l, high, high)
                diag[:m, :m] = self._band(l, low, low)
                self._J.append(diag / self.delta[l] ** 2 + self.alpha * self.D[l])
        return self._J

    def _band(self, l, U, V):
        out = 0.0
        for g in self.groups:
            Sy, _, Sx, _ = g["S"][l]
            a, b = Sy @ U, Sx @ V
            ha, da = 0.5 * (a[:, 1:] + a[:, :-1]), a[:, 1:] - a[:, :-1]
            hb, db = 0.5 * (b[:, 1:] + b[:, :-1]), b[:, 1:] - b[:, :-1]
            xx, xy, yy = g["inv"]
            d = (ha * ha).mT @ xx @ (db * db) + 2 * (ha * da).mT @ xy @ (db * hb) + (da * da).mT @ yy @ (hb * hb)
            zx, zy = ha.mT @ g["m"] @ db, da.mT @ g["m"] @ hb
            cx, cy = ha.mT @ xx @ db + da.mT @ xy @ hb, ha.mT @ xy @ db + da.mT @ yy @ hb
            k = [v.sum((1, 2))[:, None, None] / g["nM"] for v in g["inv"]]
            t = -2 * (zx * cx + zy * cy) + k[0] * zx * zx + 2 * k[1] * zx * zy + k[2] * zy * zy
            out = out + (d + t * (g["tt"] / g["nM"])[:, None, None]).sum(0)
        return out

    # -- solvers (one problem per entry of the batch dimension)
    @staticmethod
    def dot(x, y):
        return sum((a * b).sum((1, 2)) for a, b in zip(x, y))[:, None, None]

    def pcg(self, x, r, iters, rtol=0.0, keep=0):
        P, Q = [], []
        z = [a / j for a, j in zip(r, self.J)]
        p, rho = z, self.dot(r, z)
        stop = rho * rtol * rtol
        for k in range(iters):
            q = self.M(p)
            if k < keep:
                P, Q = P + [p], Q + [q]
            a = rho / self.dot(p, q).clamp_min(1e-300)
            x = [u + a * v for u, v in zip(x, p)]
            r = [u - a * v for u, v in zip(r, q)]
            z = [u / j for u, j in zip(r, self.J)]
            new = self.dot(r, z)
            p = [u + (new / rho.clamp_min(1e-300)) * v for u, v in zip(z, p)]
            rho = new
            if rtol and k % 64 == 0 and bool((rho <= stop).all()):
                break
        return x, r, P, Q

    def frame(self, state, slopes, iters):
        """One control step from a (B, n_state) state: (new state, layers, commands)."""
        cfg = self.cfg
        fit = Fitting(self) if cfg.get("fit") else None
        na, keep = (fit.n_act if fit else self.nc), cfg["augment"]
        st = state.to(self.dev, torch.float64)
        c, b0, r0, a_prev, a = st[:, :3 * self.nc + 2 * na].split([self.nc] * 3 + [na] * 2, 1)
        s = self.slopes_in(slopes)
        if cfg["loop"] == "closed":
            s = [(x + u, y + v) for (x, y), (u, v) in zip(s, self.A(self.split(a_prev)))]
        b = self.rhs(s)
        x, r, P, Q = self.pcg(self.split(c), self.split(self.join(b) - b0 + r0), iters, keep=keep)
        phi = self.Winv(x)
        step = fit.solve(phi) if fit else self.join(phi)
        new = a + cfg["gain"] * (step - a_prev) if cfg["loop"] == "closed" else (1 - cfg["gain"]) * a + cfg["gain"] * step
        parts = [self.join(x), self.join(b), self.join(r), a, new]
        if keep:
            zero = torch.zeros_like(parts[0])
            tail = torch.zeros(st.shape[0], 4, dtype=torch.float64, device=self.dev)
            tail[:, 0] = len(P)
            for v in (P, Q):
                parts += [self.join(u) for u in v] + [zero] * (keep - len(v))
            parts.append(tail)
        return torch.cat(parts, 1), self.join(phi), new


class Fitting:
    """The fitting step: CG on sum_k B_k^T M B_k + eps from zero."""

    def __init__(self, ref):
        cfg, self.ref = ref.cfg, ref
        N, D, L = cfg["wfs"][0]["n_subap"], cfg["D"], cfg["domain_side"]
        m = ref.groups[0]["mask"].cpu().numpy()
        cm = np.zeros((N + 1, N + 1), dtype=bool)
        for di in (0, 1):
            for dj in (0, 1):
                cm[di:N + di, dj:N + dj] |= m
        ten = lambda a: torch.tensor(np.asarray(a), dtype=torch.float64, device=ref.dev)  # noqa: E731
        self.mask = ten(cm * 1.0)
        x = -0.5 * D + np.arange(N + 1) * (D / N)

        def mats(h, n, unit, centre):
            return [ten(np.stack([_grid_lines((x + h * d[ax]) / unit + centre, n)[0] for d in cfg["fit"]["directions"]]))
                    for ax in (1, 0)]

        self.P = [mats(l["h"], l["n"], L / l["n"], 0.5 * l["n"]) for l in cfg["layers"]]
        self.B = [mats(d["h"], d["n_act"], d["pitch"], 0.5 * (d["n_act"] - 1)) for d in cfg["dms"]]
        self.sizes = [d["n_act"] for d in cfg["dms"]]
        self.n_act = sum(n * n for n in self.sizes)
        diag = sum(float(((Sy * Sy).mT @ self.mask @ (Sx * Sx)).sum()) for Sy, Sx in self.B)
        self.eps = cfg["fit"]["eps_rel"] * diag / self.n_act

    def forward(self, mats, x):
        return sum(Sy @ v[:, None] @ Sx.mT for (Sy, Sx), v in zip(mats, x)) * self.mask

    def adjoint(self, w):
        return torch.cat([(Sy.mT @ w @ Sx).sum(1).flatten(1) for Sy, Sx in self.B], 1)

    def solve(self, phi):
        r = self.adjoint(self.forward(self.P, phi))
        a, p, rho = torch.zeros_like(r), r, (r * r).sum(1, keepdim=True)
        for _ in range(self.ref.cfg["fit"]["iters"]):
            grids = [v.reshape(-1, n, n) for v, n in zip(p.split([n * n for n in self.sizes], 1), self.sizes)]
            q = self.adjoint(self.forward(self.B, grids)) + self.eps * p
            al = rho / (p * q).sum(1, keepdim=True)
            a, r = a + al * p, r - al * q
            new = (r * r).sum(1, keepdim=True)
            p, rho = r + new / rho * p, new
        return a


# ----------------------------------------------------------------- inputs

def screens(cfg, seed, k, count, gen):
    """`count` consecutive frames of problem k's layers: frozen-flow von Karman screens, (count, N_c) float64."""
    dev, out = gen.device, []
    g = np.random.default_rng([seed, 3, k])
    pr = cfg["prior"]
    for lay in cfg["layers"]:
        n, m = lay["n"], 2 * lay["n"]
        d = cfg["domain_side"] / n
        f = torch.fft.fftfreq(m, d=d, dtype=torch.float64, device=dev)
        f2 = f[:, None] ** 2 + f[None, :] ** 2 + pr["L0"] ** -2.0
        amp = math.sqrt(0.023 * lay["cn2"] * pr["r0"] ** (-5.0 / 3.0))
        spec = torch.randn(2, m, m, dtype=torch.float64, device=dev, generator=gen)
        spec = torch.complex(spec[0], spec[1]) * (amp * f2 ** (-11.0 / 12.0) / (m * d))
        spec[0, 0] = 0.0
        v, az = g.uniform(5.0, 20.0), g.uniform(0.0, 2.0 * math.pi)
        t = torch.arange(count, dtype=torch.float64, device=dev)[:, None, None] / 500.0
        shift = torch.exp(-2j * math.pi * t * v * (math.cos(az) * f[None, None, :] + math.sin(az) * f[None, :, None]))
        out.append((torch.fft.ifft2(spec * shift).real * m * m)[:, :n, :n].reshape(count, -1))
    return torch.cat(out, 1)


def _generator(seed):
    gen = torch.Generator(device=_device())
    gen.manual_seed(seed)
    return gen


@functools.lru_cache(maxsize=8)
def _operators(key):
    return Reference(dict(config(*key), name="shared"))


def shared(cfg):
    """The operators of the configuration's geometry (its Cn2, r0 and noise levels play no part in A and W)."""
    return _operators((cfg["name"], cfg["wfs"][0]["n_subap"]))


def inputs(case, seed):
    """Per problem: a pool of slopes (POOL, n_slopes), the state [c | b | r | a_prev | a | ...] of a running
    sequence, layers and coefficients, all float32."""
    gen, out = _generator(seed), []
    for k, cfg in enumerate(problems(case, seed)):
        ref = shared(cfg)
        phi = screens(cfg, seed, k, POOL + 1, gen)
        s = ref.slopes_out(ref.A(ref.split(phi)))
        sig = torch.cat([torch.full((2 * g["nM"],), w["sigma"], dtype=torch.float64, device=ref.dev)
                         for w in cfg["wfs"] for g in ref.groups if g["N"] == w["n_subap"]])
        s = s + sig * torch.randn(s.shape, dtype=torch.float64, device=ref.dev, generator=gen)
        # the coefficients of the frame before, a little off, as a running sequence holds them
        c = [0.95 * v * d * d for v, d in zip(ref.W(ref.split(phi[:1])), ref.delta)]
        out.append(dict(cfg=cfg, phi=phi[1:].float(), c=ref.join(c)[0].float(), slopes=s[1:].float(), before=s[:1]))
    return out


def state_of(cfg, p, ref, n_act, n_state):
    """A running sequence's state: c, its right-hand side b, the residual r = b - M c and the commands of c
    (zeros where a fitting step makes the commands)."""
    c = ref.split(p["c"][None])
    b = ref.rhs(ref.slopes_in(p["before"]))
    r = [u - v for u, v in zip(b, ref.M(c))]
    a = ref.join(ref.Winv(c)) if n_act == ref.nc else torch.zeros(1, n_act, dtype=torch.float64, device=ref.dev)
    tail = torch.zeros(1, n_state - 3 * ref.nc - 2 * n_act, dtype=torch.float64, device=ref.dev)
    return torch.cat([p["c"][None].double(), ref.join(b), ref.join(r), a, a, tail], 1)[0].float()


def upstream(case, seed, n, nc):
    """dL/dphi of a reconstruction error: noise-like, 1e-2 rad."""
    gen = _generator(seed + 77)
    return 1e-2 * torch.randn(n, nc, dtype=torch.float32, device=gen.device, generator=gen)


def closed_loop_slopes(ref, p, state):
    """Slopes as measured behind the mirrors: those of the commands a_prev taken away."""
    nc = ref.nc
    a = ref.slopes_out(ref.A(ref.split(state[None, 3 * nc:4 * nc])))
    return (p["slopes"].double() - a).float()


def sizes_of(cfg):
    nc = sum(l["n"] ** 2 for l in cfg["layers"])
    na = sum(d["n_act"] ** 2 for d in cfg["dms"]) if cfg.get("fit") else nc
    keep = cfg["augment"]
    return nc, na, 3 * nc + 2 * na + (2 * keep * nc + 4 if keep else 0)


def frames_of(case, seed):
    """Per problem (cfg, pool of slopes, state) of the frame kinds, as exact() and prepare() both take them."""
    out, refs = [], {}
    for p in inputs(case, seed):
        cfg = p["cfg"]
        key = id(cfg) if case["system"] == "mixed" else 0
        ref = refs.setdefault(key, Reference(cfg))
        nc, na, ns = sizes_of(cfg)
        st = state_of(cfg, p, ref, na, ns)
        out.append((cfg, ref, closed_loop_slopes(ref, p, st) if cfg["loop"] == "closed" else p["slopes"], st))
    return out


# ------------------------------------------------------------ the measured

TUNED_SINGLE = {"dwt_resident": 64, "pt_rows": 4, "pt_split": 1, "glob_fuse": 1}


def prepare(case, seed):
    import paper_2202_11945_amd as fw
    from paper_2202_11945_amd.autograd import FrameBatch

    kind = case["kind"]
    if kind in ("apply_A", "apply_AT", "apply_M", "rhs"):
        p = inputs(case, seed)[0]
        ctx = fw.Context(p["cfg"], device=0)
        x = {"apply_A": p["phi"], "apply_AT": p["slopes"], "rhs": p["slopes"], "apply_M": p["c"][None]}[kind][0]
        out = torch.empty(ctx.n_slopes if kind == "apply_A" else ctx.n_coeff, device="cuda")
        return dict(kind=kind, call=getattr(ctx, kind), x=x.contiguous(), out=out)
    if kind == "transforms":
        ps = inputs(case, seed)
        ctx = fw.Context(ps[0]["cfg"], device=0)
        c, n = torch.stack([p["c"] for p in ps]), len(ps)
        phi, back = torch.empty_like(c), torch.empty_like(c)
        return dict(kind=kind, batch=fw.Batch([ctx] * n), c=list(c), phi=phi, back=back, phis=list(phi), backs=list(back))
    if kind == "gradient":
        ps = inputs(case, seed)
        fb = FrameBatch(ps[0]["cfg"], len(ps))
        return dict(kind=kind, frames=fb, slopes=torch.stack([p["slopes"][0] for p in ps]), rtol=case["rtol"],
                    g=upstream(case, seed, len(ps), fb.ctx.n_coeff))
    if kind == "solve":
        ps = inputs(case, seed)
        ctx = fw.Context(ps[0]["cfg"], device=0)
        x = torch.empty(len(ps), ctx.n_coeff, device="cuda")
        return dict(kind=kind, batch=fw.Batch([ctx] * len(ps)), slopes=[p["slopes"][0].contiguous() for p in ps], x=x,
                    xs=list(x), rtol=case["rtol"])
    fr = frames_of(case, seed)
    made = {}
    for cfg, _, _, _ in fr:
        if id(cfg) not in made:
            made[id(cfg)] = fw.Context(cfg, device=0)
    ctxs = [made[id(cfg)] for cfg, _, _, _ in fr]
    # problems of one size side by side in one tensor, so that a sequence's buffers are its rows
    group = {}
    for k, ctx in enumerate(ctxs):
        group.setdefault((ctx.n_state, ctx.n_coeff), []).append(k)
    rows, outs = [None] * len(fr), []
    for (ns, nc), ks in group.items():
        st = torch.zeros(len(ks), -(-ns // 4) * 4, device="cuda")  # 16-byte aligned rows
        st = st[:, :ns].copy_(torch.stack([fr[k][3] for k in ks]))
        lay = torch.empty(len(ks), nc, device="cuda")
        dm = torch.empty(len(ks), ctxs[ks[0]].n_act, device="cuda")
        outs.append(dict(state=st, layers=lay, dm=dm))
        for j, k in enumerate(ks):
            rows[k] = (st[j], lay[j], dm[j])
    pools = [list(f[2].contiguous()) for f in fr]
    if kind == "streamed":
        pools = [[v.cpu().pin_memory() for v in p] for p in pools]
    state = dict(kind=kind, ctx=ctxs[0], pools=pools, rows=rows, outs=outs, iters=case["iters"], k=0,
                 groups=case.get("groups", 1))
    if kind == "graph":
        state["batch"] = fw.Batch(ctxs, tuning=TUNED_SINGLE if case.get("tuned") else None)
        state["states"], state["layers"], state["dms"] = ([r[i] for r in rows] for i in range(3))
    return state


def run(s):
    kind = s["kind"]
    if kind in ("apply_A", "apply_AT", "apply_M", "rhs"):
        return s["call"](s["x"], s["out"])
    if kind == "transforms":
        s["batch"].apply_Winv(s["c"], s["phis"])
        s["batch"].apply_WinvT(s["phis"], s["backs"])
        return {"layers": s["phi"], "coef": s["back"]}
    if kind == "gradient":
        from paper_2202_11945_amd.autograd import MAPLayers
        params = s["frames"].params.clone().requires_grad_()
        phi = MAPLayers.apply(params, s["slopes"], s["frames"], s["rtol"])
        phi.backward(s["g"])
        # the gradient goes to a float32 optimiser: its fields are float32
        return {"layers": phi.detach(), "grad": params.grad.float()}
    if kind == "solve":
        s["batch"].solve_map(slopes=s["slopes"], x=s["xs"], rtol=s["rtol"])
        return s["x"]
    # a sequence walks its pool forward and back, one frame a call
    i = s["k"] % (2 * POOL - 2)
    i, s["k"] = min(i, 2 * POOL - 2 - i), s["k"] + 1
    if kind == "graph":
        s["batch"].reconstruct([p[i] for p in s["pools"]], s["states"], s["layers"], s["dms"], iters=s["iters"])
    else:
        st, lay, dm = s["rows"][0]
        if kind == "streamed":
            s["ctx"].reconstruct_streamed(s["pools"][0][i], st, lay, dm, iters=s["iters"], chunks=s["groups"])
        else:
            s["ctx"].reconstruct(s["pools"][0][i], st, lay, dm, iters=s["iters"])
    return s["outs"]


def work(case):
    """Bytes: every input read and every output written once (float32).  Flops: the arithmetic of the
    operators (12 per tap set of a bilinear sample, 24 per coefficient, pass pair and level of a transform)
    and of the vector recurrences."""
    nb, nf = 0.0, 0.0
    for cfg in problems(case, 0):
        s = SYSTEMS[cfg["name"]]
        nc, na, ns = sizes_of(cfg)
        dwt = 32.0 * nc
        act, corners = 0.0, 0.0
        for w in cfg["wfs"]:
            c = (np.arange(w["n_subap"]) + 0.5) / w["n_subap"] - 0.5
            r = np.hypot(*np.meshgrid(c, c))
            act += float(((r >= 0.5 * math.sqrt(s["obs"])) & (r <= 0.5)).sum())
            corners += (w["n_subap"] + 1.0) ** 2
        prop = 12.0 * corners * len(s["n"]) + 8.0 * act
        M = 2 * dwt + 2 * prop + 8 * act + 2 * nc
        kind = case["kind"]
        if kind in ("apply_A", "apply_AT"):
            nb, nf = nb + 4 * (nc + 2 * act), nf + prop
        elif kind == "apply_M":
            nb, nf = nb + 8 * nc, nf + M
        elif kind == "rhs":
            nb, nf = nb + 4 * (nc + 2 * act), nf + dwt + prop
        elif kind == "transforms":
            nb, nf = nb + 16 * nc, nf + 2 * dwt
        elif kind in ("solve", "gradient"):
            # how many steps an iterative solve takes is the path's own choice: one operator application per
            # two digits is less than any of them takes
            solves = 2 if kind == "gradient" else 1
            nb += solves * 4 * (nc + 2 * act)
            nf += solves * M * math.ceil(-math.log10(case["rtol"]) / 2)
        else:
            it = case["iters"]
            nb += 4 * (2 * act + 2 * ns + nc + na)
            nf += dwt + prop + it * (M + 14 * nc) + dwt + 4 * nc
            if cfg.get("fit"):
                fit = 9 * 12.0 * (s["subaps"] + 1.0) ** 2
                nf += fit * (len(s["n"]) + 3) + cfg["fit"]["iters"] * (6 * fit + 10 * na)
    return {"bytes": nb, "flops": nf}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("apply_A", "apply_AT", "apply_M", "rhs"):
        p = inputs(case, seed)[0]
        ref = Reference(p["cfg"])
        if kind == "apply_A":
            return ref.slopes_out(ref.A(ref.split(p["phi"][:1])))[0].cpu()
        if kind == "apply_M":
            return ref.join(ref.M(ref.split(p["c"][None])))[0].cpu()
        s = ref.slopes_in(p["slopes"][:1])
        return ref.join(ref.AT(s) if kind == "apply_AT" else ref.rhs(s))[0].cpu()
    if kind == "transforms":
        ps = inputs(case, seed)
        ref = Reference(ps[0]["cfg"])
        phi = ref.Winv(ref.split(torch.stack([p["c"] for p in ps])))
        # the library's W^{-T} is delta^{-1} W
        return {"layers": ref.join(phi).cpu(), "coef": ref.join(ref.W(phi)).cpu()}
    if kind == "solve":
        ps = inputs(case, seed)
        ref = Reference(ps[0]["cfg"])
        b = ref.rhs(ref.slopes_in(torch.stack([p["slopes"][0] for p in ps])))
        return ref.join(ref.pcg([0 * v for v in b], b, 40000, rtol=1e-12)[0]).cpu()
    if kind == "gradient":
        ps = inputs(case, seed)
        cfg = ps[0]["cfg"]
        ref, B = Reference(cfg), len(ps)
        s = ref.slopes_in(torch.stack([p["slopes"][0] for p in ps]))
        g = ref.split(upstream(case, seed, B, ref.nc))
        b = ref.rhs(s)
        c = ref.pcg([0 * v for v in b], b, 40000, rtol=1e-13)[0]
        b = ref.W(g)
        lam = ref.pcg([0 * v for v in b], b, 40000, rtol=1e-13)[0]
        phi, psi = ref.Winv(c), ref.Winv(lam)
        dot = lambda a, b: sum(float((x * u).sum() + (y * v).sum()) for (x, y), (u, v) in zip(a, b))  # noqa: E731
        t = [float((u * d * v).sum()) for u, d, v in zip(lam, ref.D, c)]
        res = ref.weigh([(x - u, y - v) for (x, y), (u, v) in zip(s, ref.A(phi))])
        wl = ref.weigh(ref.A(psi))
        grad = [-sum(t)] + [ref.alpha * v / l["cn2"] for v, l in zip(t, cfg["layers"])]
        grad += [dot(ref.A(psi, only=l), res) - dot(wl, ref.A(phi, only=l)) for l in range(len(t))]
        return {"layers": ref.join(phi).cpu(), "grad": torch.tensor(grad, dtype=torch.float64)}
    fr = frames_of(case, seed)
    done = []
    for cfg, ref, slopes, st in fr:
        done.append(ref.frame(st[None], slopes[:1], case["iters"]))
    group = {}
    for k, (cfg, _, _, _) in enumerate(fr):
        group.setdefault((sizes_of(cfg)[2], sizes_of(cfg)[0]), []).append(k)
    return [{n: torch.cat([done[k][i] for k in ks]).cpu() for i, n in enumerate(("state", "layers", "dm"))}
            for ks in group.values()]

"""Representative calls of the library's public entry points, for timing and comparison.

Each case is a dict of plain values; ``prepare`` makes what a user's program holds before
the call (the context with its mesh and permittivity, the acquisition, the matrices),
``run`` makes one call, ``work`` counts what the call cannot do without and ``exact`` gives
the same outputs from a plain FP64 implementation of the scheme in torch.

Kinds of cases, by entry point:

forward     Context.forward_traces: many independent sources stepped on one mesh
jacobian    Context.jacobian_coarse, multigrid mode, written to device memory
gradient    Context.misfit_gradient: checkpointed reverse-time adjoint
autograd    autograd.traces: a new permittivity, its traces and the loss gradient
tv          Context.tv_invert_level: one-level TV iteration on a Jacobian-sized matrix
tv2         Context.tv_invert_two_level: the coarse-to-fine iteration
"""
from __future__ import annotations

import functools
import math
import warnings

import numpy as np
import torch

from paper_1707_04605_amd import Context
from paper_1707_04605_amd import autograd as mgrt_autograd
from synth import acquisition, body, levels, pml, regularizer
from synth.mesh import kuhn_mesh

WAVE = ("forward", "jacobian", "gradient", "autograd")


def _wave(name, kind, d, N, L, src, rec, steps, prec, **more):
    c = dict(kind=kind, d=d, N=N, L=L, src=src, rec=rec, steps=steps, prec=prec, pml=False)
    c.update(more)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a few sources on a mesh of 1,089 nodes, FP64 (a quick check of a
        # set-up, a unit test, one inner call of an interactive session); launches count
        _wave("forward_2d_smallest", "forward", 2, 32, 0, 3, 1, 600, 64),
        # the small 2D configuration as it stands: 128^2 cells, one monostatic source
        _wave("forward_2d_one_source", "forward", 2, 128, 0, 1, 1, 4000, 64),
        # an ordinary survey on a mesh whose size is no power of two, sources that do not
        # fill their batch
        _wave("forward_2d_ordinary", "forward", 2, 250, 0, 12, 1, 2000, 32),
        # the 2D batched configuration (1024^2 cells, 64 monostatic sources), an eighth of
        # its steps, traces left on the GPU
        _wave("forward_2d_large", "forward", 2, 1024, 0, 64, 1, 2000, 32, device_out=True),
        # reference-precision survey: FP64 fields, a ragged number of sources
        _wave("forward_2d_fp64", "forward", 2, 512, 0, 30, 1, 1500, 64),
        # the paper's boundary and losses: split-field PML, lossy target
        _wave("forward_2d_pml", "forward", 2, 320, 0, 16, 1, 1000, 32, pml=True),
        # 3D survey (the 3D batched configuration at half its cells per axis)
        _wave("forward_3d", "forward", 3, 64, 0, 32, 1, 800, 32),
        # the differentiation configuration at half its cells per axis, half its sources
        # and steps: the same 8,192 columns and 512 samples
        _wave("jacobian_2d", "jacobian", 2, 512, 3, 32, 1, 8000, 32, samples=512),
        # the 3D gradient configuration (bistatic, coarse level) on a smaller odd mesh
        _wave("gradient_3d", "gradient", 3, 48, 3, 16, 2, 600, 32, level="coarse"),
        # one step of a gradient-based inversion: new permittivity, traces, loss gradient
        _wave("autograd_2d", "autograd", 2, 96, 0, 5, 1, 1200, 64),
        # the TV solve on the differentiation configuration's Jacobian shape
        dict(name="tv_level", kind="tv", Nc=64, rows=32768, prec=32, iters=3),
        # coarse-to-fine on the same levels, half the data, largest third kept
        dict(name="tv_two_level", kind="tv2", Nc=64, rows=16384, prec=32, iters=3),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("forward", "forward", "forward", "forward", "jacobian", "gradient",
                       "autograd", "tv", "tv2"))
    if kind in ("tv", "tv2"):
        Nc = 2 * _logint(rng, 4, 32)
        M = 2 * Nc * Nc
        return dict(kind=kind, Nc=Nc, rows=max(32, min(32768, int(M * rng.uniform(0.7, 4.0)))),
                    prec=rng.choice((32, 64)), iters=rng.randint(2, 4))
    d = rng.choice((2, 2, 2, 3))
    prec = rng.choice((32, 32, 64))
    more = {}
    if kind == "forward":
        N, L = (_logint(rng, 24, 700), 0) if d == 2 else (_logint(rng, 8, 60), 0)
        src, rec = _logint(rng, 1, 64), rng.choice((1, 1, 2))
        more["pml"] = rng.random() < 0.2
    elif kind == "jacobian":
        L = rng.choice((2, 3))
        N = (1 << L) * (_logint(rng, 4, 48) if d == 2 else _logint(rng, 2, 4))
        src, rec = _logint(rng, 1, 32), rng.choice((1, 1, 2))
        more["samples"] = _logint(rng, 16, 256)
    elif kind == "gradient":
        L = rng.choice((1, 2))
        N = (1 << L) * (_logint(rng, 6, 80) if d == 2 else _logint(rng, 3, 10))
        src, rec = _logint(rng, 1, 32), rng.choice((1, 2))
        more["level"] = rng.choice(("coarse", "fine"))
    else:
        L, src, rec = 0, _logint(rng, 1, 16), 1
        N = _logint(rng, 20, 200) if d == 2 else _logint(rng, 8, 24)
    # up to 5e10 node updates, well below the largest listed case
    n = (N + 1) ** d * src * (1 if kind == "forward" else 3)
    top = max(200, min(8000 if kind == "jacobian" else 4000, int(5e10 / n)))
    steps = min(top, _logint(rng, 200, 4000))
    if kind == "jacobian":
        steps = max(steps, 2 * more["samples"])
    return _wave(None, kind, d, N, L, src, rec, steps, prec, **more)


# ---------------------------------------------------------------------------- inputs


@functools.lru_cache(maxsize=4)
def _mesh(d, N, L):
    return kuhn_mesh(d, N, L)


class _Problem:
    """Seeded inputs of a wave case: a star-shaped body, sources around it, a wavelet."""

    def __init__(self, case, seed):
        d, N = case["d"], case["N"]
        self.mesh = ms = _mesh(d, N, case["L"])
        rng = np.random.default_rng([seed, 17])
        tgt = body.make_body2d(seed, 4) if d == 2 else body.make_body3d(seed, 2)
        self.eps = body.element_permittivity(ms.centroids, tgt, noise=0.1, noise_seed=seed + 1)
        self.sigma = self.pml = None
        if case["pml"]:
            self.pml = pml.pml_coefficients(ms.centroids)
            self.sigma = pml.lossy_sigma(self.eps, tgt.inside(ms.centroids))
        S = case["src"]
        pts = acquisition.circle_points(S) if d == 2 else acquisition.sphere_points(S)
        a = rng.uniform(0, 2 * np.pi)
        rot = np.array([[np.cos(a), -np.sin(a)], [np.sin(a), np.cos(a)]])
        pts = pts.copy()
        pts[:, :2] = pts[:, :2] @ rot.T
        self.src = pts
        self.rec = acquisition.monostatic(pts) if case["rec"] == 1 else acquisition.bistatic_antipodal(pts)
        self.dt = acquisition.time_step(d, ms.h, float(self.eps.min()))
        self.steps = case["steps"]
        # ten nodes per wavelength at eps = 4 on this mesh, at most the configurations' f0
        self.f0 = min(acquisition.wavelet_f0(), acquisition.wavelet_f0(ms.h))
        self.wavelet = acquisition.sample_wavelet(self.dt, self.steps, self.f0)
        shape = (S, case["rec"], self.steps)
        self.residual = None
        if case["kind"] == "gradient":
            # residuals look like traces: the wavelet at random delays and strengths
            t = np.arange(self.steps) * self.dt
            at = rng.uniform(0.2, 0.9, size=shape[:2]) * t[-1]
            amp = rng.normal(size=shape[:2])
            self.residual = amp[..., None] * acquisition.gaussian_sine(
                t[None, None, :] - at[..., None] + 4.0 / self.f0, self.f0)
        if case["kind"] == "autograd":
            self.observed = 0.01 * rng.normal(size=shape)
        if case["kind"] == "jacobian":
            self.samples = acquisition.sample_steps(self.steps, case["samples"])

    def context(self):
        ms = self.mesh
        ctx = Context(0)
        bf = ms.bfacets if self.pml is None else None
        if ms.L:
            ctx.upload_mesh(ms.d, ms.coords, ms.elems, bf, None, ms.coarse_of_elem, ms.coarse_verts)
        else:
            ctx.upload_mesh(ms.d, ms.coords, ms.elems, bf)
        ctx.upload_permittivity(self.eps, self.sigma)
        if self.pml is not None:
            ctx.upload_pml(*self.pml)
        return ctx


@functools.lru_cache(maxsize=2)
def _levels(Nc):
    lv = levels.two_level(2, Nc)
    return (lv, regularizer.tv_matrix(lv.coords, lv.verts2, 0.01),
            regularizer.tv_matrix(lv.coords, lv.verts1, 0.01))


def _tv_inputs(case, seed):
    """A matrix shaped and scaled like a sampled Jacobian, on the GPU, and its data."""
    lv = _levels(case["Nc"])[0]
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if case["prec"] == 32 else torch.float64
    L = torch.randn(case["rows"], lv.M, generator=g, device="cuda", dtype=dt)
    # columns near the source orbit are seen more strongly than the middle of the body
    cen = lv.coords[lv.verts1].mean(axis=1)
    L *= torch.as_tensor(0.2 + 0.8 * np.hypot(cen[:, 0], cen[:, 1]) / 2.2, device="cuda").to(dt)
    rng = np.random.default_rng([seed, 23])
    x = np.zeros(lv.M)
    for _ in range(4):
        x[np.hypot(*(cen - rng.uniform(-0.8, 0.8, size=2)).T) < rng.uniform(0.15, 0.5)] += rng.normal()
    r = (L.double() @ torch.as_tensor(x, device="cuda")).cpu().numpy()
    r += 0.01 * np.abs(r).max() * rng.normal(size=r.shape)
    return L, r


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] in WAVE:
        s["p"] = p = _Problem(case, seed)
        s["ctx"] = p.context()
        if case["kind"] == "forward" and case.get("device_out"):
            s["out"] = torch.empty(case["src"], case["rec"], p.steps, dtype=torch.float64, device="cuda")
        if case["kind"] == "jacobian":
            s["out"] = torch.empty(case["src"] * case["rec"] * case["samples"], p.mesh.n_coarse,
                                   dtype=torch.float64, device="cuda")
        if case["kind"] == "autograd":
            s["acq"] = mgrt_autograd.Acquisition(p.src, p.rec, p.wavelet, p.dt, p.steps, case["prec"])
            s["eps"] = torch.as_tensor(p.eps, device="cuda")
            s["observed"] = torch.as_tensor(p.observed, device="cuda")
        return s
    s["ctx"] = Context(0)
    s["L"], s["r"] = _tv_inputs(case, seed)
    return s


# ------------------------------------------------------------------------------ calls


def run(state):
    case, ctx = state["case"], state["ctx"]
    kind = case["kind"]
    if kind in WAVE:
        p = state["p"]
        acq = (p.src, p.rec, p.wavelet, p.dt, p.steps)
        if kind == "forward":
            return ctx.forward_traces(*acq, precision=case["prec"], out=state.get("out"))
        if kind == "jacobian":
            return ctx.jacobian_coarse(*acq, p.samples, precision=case["prec"], out=state["out"])
        if kind == "gradient":
            return ctx.misfit_gradient(*acq, p.residual, level=case["level"], precision=case["prec"])
        eps = state["eps"].clone().requires_grad_(True)
        y = mgrt_autograd.traces(eps, ctx, state["acq"])
        loss = 0.5 * (y - state["observed"]).square().sum()
        loss.backward()
        return {"traces": y.detach(), "grad": eps.grad}
    lv, Dc, Df = _levels(case["Nc"])
    if kind == "tv":
        z, _ = ctx.tv_invert_level(state["L"], state["r"], *Df, 0.01, iters=case["iters"])
        return z
    out = ctx.tv_invert_two_level(state["L"], state["r"], lv.verts1, lv.parent, lv.M2, Dc, Df, 0.01,
                                  iters=case["iters"], n_keep=levels.keep_third(lv.M2))
    return {"x": out["x"], "zc": out["zc"], "kept": out["kept"]}


def work(case):
    """The state, the operator and the results once each; the arithmetic of every step."""
    if case["kind"] in WAVE:
        d, N, S, R, T = case["d"], case["N"], case["src"], case["rec"], case["steps"]
        n, m = (N + 1) ** d, math.factorial(d) * N ** d
        esz = case["prec"] // 8
        sweeps = {"forward": 1, "jacobian": 1 if R == 1 and case["prec"] == 32 else 1 + R,
                  "gradient": 2, "autograd": 3}[case["kind"]]
        flops = sweeps * (6.0 * d + 4) * n * S * T        # 2 d neighbours, three each
        byts = 3.0 * esz * n * S + n * (4.0 * 2 * d + 2 * esz) + 8.0 * T * (1 + S * R)
        if case["kind"] == "jacobian":
            Nc = N >> case["L"]
            K, nc, cols = case["samples"], (Nc + 1) ** d, math.factorial(d) * Nc ** d
            flops += 2.0 * S * R * nc * K * (T / 2)
            byts += 8.0 * S * R * K * cols + 2.0 * esz * S * nc * T
        elif case["kind"] != "forward":
            byts += 8.0 * S * R * T + 16.0 * m
        return dict(bytes=byts, flops=flops)
    M, rows, it = 2 * case["Nc"] ** 2, case["rows"], case["iters"]
    byts = rows * M * (case["prec"] / 8.0) + 8.0 * rows + 8.0 * it * M
    if case["kind"] == "tv":
        return dict(bytes=byts, flops=rows * float(M) ** 2 + it * M ** 3 / 3.0)
    M2 = M // 4
    K = 3 * levels.keep_third(M2)
    return dict(bytes=byts, flops=rows * (float(M2) ** 2 + it * float(K) ** 2) +
                it * (M2 ** 3 + K ** 3) / 3.0)


# ----------------------------------------------------------- plain FP64 implementation


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


class _Exact:
    """The nodal three-level leap-frog scheme in FP64 torch: sparse matrix times fields."""

    def __init__(self, p, absorbing=True):
        ms = p.mesh
        self.p, self.dev = p, _device()
        d, n, V = ms.d, ms.n, ms.d + 1
        X = ms.coords[ms.elems]                                  # (m, V, d)
        inv = np.linalg.inv(X[:, 1:] - X[:, :1])                 # columns: gradients
        grad = np.empty_like(X)
        grad[:, 1:] = np.swapaxes(inv, 1, 2)
        grad[:, 0] = -grad[:, 1:].sum(axis=1)
        self.vol = vol = np.abs(np.linalg.det(X[:, 1:] - X[:, :1])) / math.factorial(d)
        el = ms.elems.astype(np.int64)

        def lumped(w):
            return np.bincount(el.ravel(), weights=np.repeat(w * vol / V, V), minlength=n)

        mass, damp = lumped(p.eps), np.zeros(n)
        if p.sigma is not None:
            damp += lumped(p.sigma)
        if p.pml is not None:
            damp += lumped(p.pml[0])
        else:
            F = ms.coords[ms.bfacets]
            e1 = F[:, 1] - F[:, 0]
            area = np.linalg.norm(e1, axis=1) if d == 2 else \
                0.5 * np.linalg.norm(np.cross(e1, F[:, 2] - F[:, 0]), axis=1)
            damp += np.bincount(ms.bfacets.ravel(), weights=np.repeat(area / d, d), minlength=n)
        D, E = mass + 0.5 * p.dt * damp, mass - 0.5 * p.dt * damp
        dev = self.dev
        rows, cols, vals = [], [], []
        for a in range(V):
            for b in range(V):
                rows.append(el[:, a])
                cols.append(el[:, b])
                vals.append(-p.dt ** 2 * vol * (grad[:, a] * grad[:, b]).sum(axis=1) / D[el[:, a]])
        rows.append(np.arange(n))
        cols.append(np.arange(n))
        vals.append(2.0 * mass / D)
        self.A = self._csr(np.concatenate(rows), np.concatenate(cols), np.concatenate(vals), n, n)
        self.c = torch.as_tensor(-E / D, device=dev)[:, None]
        self.gain = torch.as_tensor(p.dt / D, device=dev)
        self.q = None
        if p.pml is not None:
            t, k = np.nonzero(p.pml[1] > 0)
            z = p.pml[1][t, k]
            ent = np.repeat(np.arange(t.size), V)
            g = grad[t, :, k].ravel()
            nodes = el[t].ravel()
            self.Bq = self._csr(ent, nodes, p.dt * g, t.size, n)
            load = p.dt ** 2 * np.repeat(z * vol[t], V) * g / D[nodes]
            self.Bt = self._csr(nodes, ent, load, n, t.size)
            self.decay = torch.as_tensor(1.0 - p.dt * z, device=dev)[:, None]

    def _csr(self, r, c, v, nr, nc):
        warnings.filterwarnings("ignore", message="Sparse CSR tensor support")
        a = torch.sparse_coo_tensor(torch.as_tensor(np.stack([r, c]), device=self.dev),
                                    torch.as_tensor(v, device=self.dev), (nr, nc))
        return a.coalesce().to_sparse_csr()

    def stencil(self, pts):
        """Nodes and P1 weights of points (k, d) in the Kuhn mesh: (k, d+1) each."""
        ms = self.p.mesh
        d, N = ms.d, ms.N
        u = (np.asarray(pts, dtype=np.float64).reshape(-1, d) + 1.5) / ms.h
        cell = np.clip(np.floor(u), 0, N - 1).astype(np.int64)
        f = u - cell
        order = np.argsort(-f, axis=1, kind="stable")
        fs = np.take_along_axis(f, order, axis=1)
        w = np.concatenate([1 - fs[:, :1], fs[:, :-1] - fs[:, 1:], fs[:, -1:]], axis=1)
        step = (N + 1) ** np.arange(d)
        node = [(cell * step).sum(axis=1)]
        for k in range(d):
            node.append(node[-1] + step[order[:, k]])
        return (torch.as_tensor(np.stack(node, axis=1), device=self.dev),
                torch.as_tensor(w, device=self.dev))

    def sweep(self, points, loads, visit):
        """Step len(loads[0]) steps; loads: (columns, per, steps) series at points
        (columns, per, d).  visit(l, p_l, p_{l+1})."""
        C, per, T = loads.shape
        node, w = self.stencil(points)
        col = torch.arange(C, device=self.dev).repeat_interleave(per)[:, None].expand_as(node)
        amp = (w * self.gain[node]).reshape(-1)
        where = (node.reshape(-1), col.reshape(-1))
        g = torch.as_tensor(loads, device=self.dev).reshape(C * per, T)
        g = torch.diff(g, dim=1, prepend=torch.zeros(C * per, 1, device=self.dev, dtype=torch.float64))
        V = node.shape[1]
        n = self.c.shape[0]
        p = torch.zeros(n, C, device=self.dev, dtype=torch.float64)
        pm = torch.zeros_like(p)
        q = None
        if self.p.pml is not None:
            q = torch.zeros(self.decay.shape[0], C, device=self.dev, dtype=torch.float64)
        for l in range(T):
            y = self.A @ p
            y.addcmul_(self.c, pm)
            if q is not None:
                y += self.Bt @ q
                q = self.decay * q + self.Bq @ p
            y.index_put_(where, amp * g[:, l].repeat_interleave(V), accumulate=True)
            visit(l, p, y)
            p, pm = y, p

    def forward(self, keep=None):
        """Traces (S, R, T); keep(l, p_l, p_{l+1}) sees every step."""
        p = self.p
        S, R, d = p.rec.shape
        rn, rw = self.stencil(p.rec.reshape(-1, d))
        rc = torch.arange(S, device=self.dev).repeat_interleave(R)[:, None].expand_as(rn)
        out = torch.empty(p.steps, S * R, device=self.dev, dtype=torch.float64)

        def visit(l, a, b):
            out[l] = (b[rn, rc] * rw).sum(dim=1)
            if keep:
                keep(l, a, b)
        self.sweep(p.src[:, None], np.broadcast_to(p.wavelet, (S, 1, p.steps)).copy(), visit)
        return out.T.reshape(S, R, p.steps).contiguous()

    def gradient(self, vel, residual):
        """d/d eps per fine element of <residual, traces>, vel the velocities of every step."""
        p = self.p
        T = p.steps
        acc = torch.zeros(self.c.shape[0], device=self.dev, dtype=torch.float64)

        def visit(l, a, b):
            acc.add_((b * vel[T - 1 - l]).sum(dim=1))
        self.sweep(p.rec, np.ascontiguousarray(residual[..., ::-1]), visit)
        el = torch.as_tensor(p.mesh.elems.astype(np.int64), device=self.dev)
        vol = torch.as_tensor(self.vol, device=self.dev)
        return acc[el].sum(dim=1) * vol / el.shape[1]

    def velocities(self):
        p = self.p
        vel = torch.empty(p.steps, self.c.shape[0], p.src.shape[0], device=self.dev, dtype=torch.float64)
        y = self.forward(lambda l, a, b: vel[l].copy_((a - b) / p.dt))
        return y, vel

    def jacobian(self):
        """The multigrid Jacobian: lumped coarse mass derivative, reciprocity, lagged sums."""
        p, ms = self.p, self.p.mesh
        S, R, d = p.rec.shape
        T, V = p.steps, ms.d + 1
        cn, idx = np.unique(ms.coarse_verts, return_inverse=True)
        cn = torch.as_tensor(cn.astype(np.int64), device=self.dev)
        b = torch.empty(T, cn.numel(), S, device=self.dev, dtype=torch.float64)
        self.sweep(p.src[:, None], np.broadcast_to(p.wavelet, (S, 1, T)).copy(),
                   lambda l, x, y: b[l].copy_((x[cn] - y[cn]) / p.dt))
        lam = torch.empty(T, cn.numel(), S * R, device=self.dev, dtype=torch.float64)
        unit = np.zeros((S * R, 1, T))
        unit[:, :, 0] = 1.0
        self.sweep(p.rec.reshape(-1, 1, d), unit, lambda l, x, y: lam[l].copy_(y[cn]))
        ss = torch.as_tensor(p.samples, device=self.dev)
        C = torch.empty(S * R, ss.numel(), cn.numel(), device=self.dev, dtype=torch.float64)
        for s in range(S):
            fb = torch.fft.rfft(b[:, :, s], n=2 * T, dim=0)
            for r in range(R):
                fl = torch.fft.rfft(lam[:, :, s * R + r], n=2 * T, dim=0)
                C[s * R + r] = torch.fft.irfft(fb * fl, n=2 * T, dim=0)[ss]
        X = ms.coords[ms.coarse_verts]
        cvol = np.abs(np.linalg.det(X[:, 1:] - X[:, :1])) / math.factorial(d)
        idx = torch.as_tensor(idx.reshape(-1, V).astype(np.int64), device=self.dev)
        J = sum(C[:, :, idx[:, a]] for a in range(V))
        J *= torch.as_tensor(cvol / V, device=self.dev)
        return J.reshape(-1, J.shape[-1])


def _tv_weights(v):
    top = v.abs().max()
    return torch.ones_like(v) if top == 0 else 1.0 / torch.clamp(v.abs(), min=1e-8 * float(top))


def _tv_solve(G, D, gamma, b):
    A = G + 0.01 * (D.T * gamma) @ D
    c = torch.linalg.cholesky(A)
    return torch.cholesky_solve(b[:, None], c)[:, 0]


def _exact_tv(case, seed):
    dev = "cuda"
    lv, Dc, Df = _levels(case["Nc"])
    L, r = _tv_inputs(case, seed)
    L, r = L.double(), torch.as_tensor(r, device=dev)

    def dense(csr, M):
        a = torch.sparse_csr_tensor(torch.as_tensor(csr[0]), torch.as_tensor(csr[1].astype(np.int64)),
                                    torch.as_tensor(csr[2]), (M, M))
        return a.to_dense().to(dev)

    Df = dense(Df, lv.M)
    if case["kind"] == "tv":
        G, b = L.T @ L, L.T @ r
        z, out = None, []
        for it in range(case["iters"]):
            z = _tv_solve(G, Df, torch.ones_like(b) if it == 0 else _tv_weights(Df @ z), b)
            out.append(z.cpu().numpy())
        return np.stack(out)
    Dc = dense(Dc, lv.M2)
    parent = torch.as_tensor(lv.parent.astype(np.int64), device=dev)
    Rc = torch.zeros(lv.M, lv.M2, dtype=torch.float64, device=dev)
    Rc[torch.arange(lv.M, device=dev), parent] = 1.0
    Lc = L @ Rc
    Gc, bc = Lc.T @ Lc, Lc.T @ r
    kids = np.argsort(lv.parent, kind="stable").reshape(lv.M2, -1)
    keep = levels.keep_third(lv.M2)
    zc, f, xs, zs, ks = None, None, [], [], []
    for it in range(case["iters"]):
        zc = _tv_solve(Gc, Dc, torch.ones_like(bc) if it == 0 else _tv_weights(Dc @ zc), bc)
        kept = np.sort(np.argsort(-zc.abs().cpu().numpy(), kind="stable")[:keep])
        # any basis of the zero-sum fluctuations of the kept parents spans the fine space
        k = kids[kept]
        Rf = torch.zeros(lv.M, keep * (k.shape[1] - 1), dtype=torch.float64, device=dev)
        for j in range(1, k.shape[1]):
            c = torch.arange(keep, device=dev) * (k.shape[1] - 1) + j - 1
            Rf[torch.as_tensor(k[:, j].astype(np.int64), device=dev), c] = 1.0
            Rf[torch.as_tensor(k[:, 0].astype(np.int64), device=dev), c] = -1.0
        Lf, DR = L @ Rf, Df @ Rf
        gam = torch.ones(lv.M, dtype=torch.float64, device=dev) if it == 0 else _tv_weights(Df @ f)
        f = Rf @ _tv_solve(Lf.T @ Lf, DR, gam, Lf.T @ (r - Lc @ zc))
        xs.append((Rc @ zc + f).cpu().numpy())
        zs.append(zc.cpu().numpy())
        ks.append(kept.astype(np.int32))
    return {"x": np.stack(xs), "zc": np.stack(zs), "kept": np.stack(ks)}


def exact(case, seed):
    if case["kind"] not in WAVE:
        return _exact_tv(case, seed)
    w = work(case)
    n, T, S = (case["N"] + 1) ** case["d"], case["steps"], case["src"]
    sweeps = {"forward": 1, "jacobian": 1 + case["rec"], "gradient": 2, "autograd": 2}[case["kind"]]
    # seconds of the sparse products below: launches, and bytes at about 1 TB/s
    if sweeps * T * (2e-4 + 8.0 * n * S * 10 / 1e12) > 20:
        return None
    p = _Problem(case, seed)
    ex = _Exact(p)
    kind = case["kind"]
    if kind == "forward":
        return ex.forward()
    if kind == "jacobian":
        return ex.jacobian()
    if 8.0 * n * S * T > 6e10:
        return None
    y, vel = ex.velocities()
    if kind == "autograd":
        rho = y.cpu().numpy() - p.observed
        return {"traces": y, "grad": ex.gradient(vel, rho)}
    g = ex.gradient(vel, p.residual)
    if case["level"] == "coarse":
        co = torch.as_tensor(p.mesh.coarse_of_elem.astype(np.int64), device=ex.dev)
        g = torch.zeros(p.mesh.n_coarse, device=ex.dev, dtype=torch.float64).index_add_(0, co, g)
    return g

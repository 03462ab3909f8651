"""Measured cases of the transport-matrix framework.

Each case is one pass through the public handle (``paper_1410_0204_amd.tmm.TMM``)
or the autograd function over it, on a synthetic ocean of a stated size:

* ``step``      one time step between two caller-owned states (a host program
                that couples the ocean step to something else, step by step);
* ``year``      one model year with its residual, the unit of spin-up;
* ``ensemble``  model years of a batch with per-member lengths and residuals;
* ``tangent``   the year map and its exact Jacobian-vector product, the inner
                loop of Newton-Krylov;
* ``adjoint``   misfit of a model year, its parameter and initial-state
                gradients (checkpointed discrete adjoint);
* ``gradient``  the same through ``torch.autograd``, as parameter estimation
                calls it, for several members at once.

The grids are the package's named ones (16x8x4, 32x16x8, 128x64x15,
256x128x23, 360x180x23) and others of the same make.  A case's grid and
monthly matrices are fixed by its ``grid_seed``, as a user's are; parameters,
states, directions and observations come from the seed of ``prepare``.
"""

import functools
import math

import numpy as np
import torch

import synth
from paper_1410_0204_amd import autograd, autotune, tmm

NMAT, NSTEP = 12, 2880


def _case(name, call, grid, model=synth.MODEL_NDOP, neu=2, nbgc=1, members=1, ckpt=0, grid_seed=3):
    nlon, nlat, nlayer, ncol, n = grid
    return dict(name=name, call=call, nlon=nlon, nlat=nlat, nlayer=nlayer, ncol=ncol, n=n, model=model, neu=neu,
                nbgc=nbgc, members=members, ckpt=ckpt, grid_seed=grid_seed)


TINY = (16, 8, 4, 90, 300)
SMALL = (32, 16, 8, 400, 2700)
GLOBAL = (128, 64, 15, 4448, 52749)
RAGGED = (90, 47, 19, 2111, 21347)
ENSEMBLE = (256, 128, 23, 22000, 500000)
ONE_DEGREE = (360, 180, 23, 42000, 760000)


def listed():
    return [
        # one step of a small ocean: the cost of a call
        _case("small_step", "step", SMALL, grid_seed=5),
        # spin-up year of the smallest ocean, one-tracer model
        _case("tiny_n_year", "year", TINY, model=synth.MODEL_N, neu=1, grid_seed=7),
        # spin-up year of the 2.8-degree ocean, the paper's PO4-DOP experiment
        _case("global_year", "year", GLOBAL, grid_seed=11),
        # the same with the paper's 8 internal biogeochemical steps per ocean step
        _case("global_nbgc8_year", "year", GLOBAL, nbgc=8, grid_seed=11),
        # one Newton-Krylov product with the exact tangent
        _case("global_tangent", "tangent", GLOBAL, grid_seed=11),
        # gradient of a year's misfit with the whole trajectory stored
        _case("global_adjoint", "adjoint", GLOBAL, ckpt=NSTEP, grid_seed=11),
        # the three-tracer model's gradient with a checkpoint per month
        _case("global_phy_adjoint_ckpt", "adjoint", GLOBAL, model=synth.MODEL_NDOPPHY, ckpt=240, grid_seed=11),
        # parameter estimation: gradients of four parameter vectors at once
        _case("global_members_gradient", "gradient", GLOBAL, members=4, ckpt=240, grid_seed=11),
        # a parameter study on an odd-sized ocean, members of uneven length
        _case("ragged_ensemble", "ensemble", RAGGED, members=9, grid_seed=3),
        # a parameter study of the three-tracer model
        _case("global_phy_members_year", "ensemble", GLOBAL, model=synth.MODEL_NDOPPHY, members=6, grid_seed=11),
        # steps of oceans that stream from memory: one member on the 1.0-degree grid ...
        _case("one_degree_step", "step", ONE_DEGREE, grid_seed=17),
        # ... and 64 members on the 1.4-degree grid
        _case("ensemble64_step", "step", ENSEMBLE, members=64, grid_seed=13),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: any call, grids from 16x8x4 upwards, odd sizes, every model."""
    call = rng.choice(["step", "step", "year", "year", "ensemble", "tangent", "adjoint", "gradient"])
    model = rng.choice([synth.MODEL_N, synth.MODEL_NDOP, synth.MODEL_NDOP, synth.MODEL_NDOPPHY])
    nbgc = rng.choice([1, 1, 1, 8])
    members = 1
    if call == "step":
        members = rng.choice([1, _log_int(rng, 2, 64)])
        most = 400000 if members == 1 else min(400000, 6000000 // members)
    elif call == "ensemble":
        members = _log_int(rng, 2, 24)
        most = min(52749, 300000 // members)
    elif call == "gradient":
        members = rng.randint(2, 4)
        most = 100000 // members
    else:
        most = 52749
    n = _log_int(rng, 300, most)
    nlayer = rng.randint(4, 23)
    # columns of 55 to 85 % of the full depth on average, two thirds of the grid wet
    ncol = max(1, int(n / (nlayer * rng.uniform(0.55, 0.85))))
    nlat = max(3, int(math.sqrt(ncol / 0.66 / 2.0)))
    nlon = max(4, int(math.ceil(ncol / 0.66 / nlat)))
    ckpt = rng.choice([240, 480, NSTEP if n <= 52749 else 240]) if call == "adjoint" else 240 if call == "gradient" else 0
    c = _case("", call, (nlon, nlat, nlayer, ncol, n), model=model, neu=1 if model == synth.MODEL_N else 2, nbgc=nbgc,
              members=members, ckpt=ckpt, grid_seed=rng.randint(1, 1000))
    del c["name"]
    return c


@functools.lru_cache(maxsize=2)
def _ocean(nlon, nlat, nlayer, ncol, n, model, neu, nbgc, grid_seed):
    return synth.custom(nlon, nlat, nlayer, ncol, n, model=model, neuphotic=neu, seed=grid_seed, nmat=NMAT,
                        nstep=NSTEP, nbgc=nbgc)


def _inputs(case, seed):
    """The ocean (host arrays), parameters, state, tangent direction, observations, step and lengths."""
    inp = _ocean(*(case[k] for k in ("nlon", "nlat", "nlayer", "ncol", "n", "model", "neu", "nbgc", "grid_seed")))
    nb, ntr, n, call = case["members"], inp.ntracer, inp.n, case["call"]
    r = np.random.default_rng(seed)
    u = synth.latin_hypercube(inp.model, max(nb, 2), seed)[:nb]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))

    def rand(*shape):
        return torch.rand(shape, dtype=torch.float64, device="cuda", generator=g)

    # concentrations as they are during a spin-up: PO4 around its mean, DOP and PHY small
    mean = torch.tensor([2.0, 0.05, 0.02][:ntr], dtype=torch.float64, device="cuda").repeat(nb)
    y = mean * (0.2 + 1.6 * rand(n, nb * ntr))
    v = (rand(n, nb * ntr) - 0.5) * mean if call == "tangent" else None
    obs = mean * (0.2 + 1.6 * rand(NMAT, n, nb * ntr)) if call in ("adjoint", "gradient") else None
    j = int(r.integers(0, NSTEP))
    years = np.asarray(r.permutation(np.arange(nb) % 2 + 1), dtype=np.int32)
    return inp, u, y, v, obs, j, years


def prepare(case, seed):
    inp, u, y, v, obs, j, years = _inputs(case, seed)
    nb, call = case["members"], case["call"]
    grad = call in ("adjoint", "gradient")
    t = tmm.TMM(inp.desc_arrays(), nbatch_max=nb, adjoint_nbatch_max=nb if grad else 0,
                ckpt_every=case["ckpt"] if grad else 240)
    autotune.apply_tuned(t, nb)
    t.set_params(u)
    s = dict(t=t, call=call, u=torch.as_tensor(u), y=y, v=v, obs=obs, j=j, years=years)
    if call == "step":
        s["out"] = t.state()
    return s


def run(s):
    t, call = s["t"], s["call"]
    if call == "step":
        return t.step(s["j"], s["y"], s["out"])
    if call == "year":
        return t.year(s["y"])
    if call == "ensemble":
        return t.year(s["y"], nyears=int(s["years"].max()), years_per_member=s["years"])
    if call == "tangent":
        return t.year_jvp(s["y"], s["v"], mode=tmm.TMM_JVP_TANGENT)
    if call == "adjoint":
        return t.year_adjoint(s["y"], s["obs"])
    u = s["u"].clone().requires_grad_(True)
    y = s["y"].detach().requires_grad_(True)
    J = autograd.year_misfit(u, y, t, s["obs"])
    J.sum().backward()
    return J.detach(), u.grad, y.grad


def _shape(case):
    """Rows, columns, tracers, nonzeros of Ae (five-point stencil) and of Ai (dense column blocks)."""
    ntr = synth.NTRACER[case["model"]]
    mean_depth = case["n"] / case["ncol"]
    return case["n"], ntr, 4.85 * case["n"], case["n"] * mean_depth * 1.2


def work(case):
    """Bytes: the twelve months' matrices the pass touches, once each, and the states that go in and
    out; a stored trajectory where the checkpoints keep one.  Operations: two for each nonzero,
    state column and step (four with the interpolation's share left out), the sources left out."""
    n, ntr, nnz_e, nnz_i = _shape(case)
    W = case["members"] * ntr
    state, mats = 8.0 * n * W, 8.0 * (nnz_e + nnz_i) + 4.0 * nnz_e
    step_flops = 2.0 * (nnz_e + nnz_i) * W
    call = case["call"]
    if call == "step":
        return {"bytes": 2 * state + 2 * mats, "flops": step_flops}
    if call == "year":
        return {"bytes": 2 * state + NMAT * mats, "flops": NSTEP * step_flops}
    if call == "ensemble":
        years = 1.5 if case["members"] > 1 else 1.0
        return {"bytes": 2 * state + NMAT * mats, "flops": years * NSTEP * step_flops}
    if call == "tangent":
        return {"bytes": 4 * state + NMAT * mats, "flops": 2 * NSTEP * step_flops}
    return {"bytes": (2 + NMAT + 2 * case["ckpt"]) * state + 2 * NMAT * mats, "flops": 2 * NSTEP * step_flops}


# ---------------------------------------------------------------------------
# The same results in plain torch, float64
# ---------------------------------------------------------------------------

class _Plain:
    """The time step on states padded to [column, layer, member, tracer], from the method's formulas."""

    def __init__(self, inp, u):
        d = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()  # noqa: E731
        g, tm = inp.grid, inp.tm
        C, L, n = g.ncol, g.nlayer, g.n
        self.C, self.L, self.nb, self.ntr, self.model = C, L, len(u), inp.ntracer, inp.model
        self.nbgc = inp.nbgc
        cs, nc = g.col_start.astype(np.int64), np.diff(g.col_start).astype(np.int64)
        col = np.repeat(np.arange(C), nc)
        lay = np.arange(n) - cs[col]
        place = col * L + lay                                   # row -> padded row
        self.place = d(place)
        # Ae as padded neighbour lists; the extra padded row C*L holds zeros
        rp, ci = tm.ae_rowptr.astype(np.int64), tm.ae_colidx.astype(np.int64)
        row, slot = np.repeat(np.arange(n), np.diff(rp)), np.arange(ci.size) - np.repeat(rp[:-1], np.diff(rp))
        S = int(np.diff(rp).max())
        nb = np.full((C * L, S), C * L)
        nb[place[row], slot] = place[ci]
        self.nbr = d(nb)
        at = d(place[row] * S + slot)
        # Ai as padded blocks [column, row, row]
        rp, ci = tm.ai_rowptr.astype(np.int64), tm.ai_colidx.astype(np.int64)
        row = np.repeat(np.arange(n), np.diff(rp))
        bat = d((col[row] * L + lay[row]) * L + lay[ci])
        self.month = functools.lru_cache(maxsize=3)(lambda m: (
            torch.zeros(C * L * S, dtype=torch.float64, device="cuda").index_put_((at,), d(tm.ae_val[m]), accumulate=True)
            .reshape(C * L, S),
            torch.zeros(C * L * L, dtype=torch.float64, device="cuda").index_put_((bat,), d(tm.ai_val[m]), accumulate=True)
            .reshape(C, L, L)))
        # water column geometry
        h = g.dz.astype(np.float64)
        bottom = np.cumsum(h)
        k = np.arange(L)
        self.h = d(h)
        self.zc = d(bottom - 0.5 * h)
        self.wet = d(k[None, :] < nc[:, None])
        self.eu = d(k[None, :] < np.minimum(nc, inp.neuphotic)[:, None])
        self.shallow = d(nc <= inp.neuphotic)
        self.lastlay = d(k[None, :] == nc[:, None] - 1)
        self.below = self.wet & d((k >= inp.neuphotic))[None, :]
        lp = bottom[inp.neuphotic - 1]
        self.ztop = d(np.log(np.maximum(np.concatenate([[lp], bottom[:-1]]), lp) / lp))
        self.zbot = d(np.log(np.maximum(bottom, lp) / lp))
        self.vol = d(g.area[col] * h[lay])
        self.dtd = 360.0 / NSTEP
        lat, t = np.radians(g.lat)[None, :], np.arange(NSTEP)[:, None] / NSTEP
        decl = -np.radians(23.44) * np.cos(2 * np.pi * (t + 10.0 / 360.0))
        h0 = np.arccos(np.clip(-np.tan(lat) * np.tan(decl), -1.0, 1.0))
        q = 1361.0 / np.pi * (h0 * np.sin(lat) * np.sin(decl) + np.cos(lat) * np.cos(decl) * np.sin(h0))
        self.light = d(np.maximum(q, 0.0) * 0.4)                # [step, column]

    def pad(self, y):
        z = torch.zeros(self.C * self.L, y.shape[1], dtype=y.dtype, device=y.device)
        return z.index_put((self.place,), y).reshape(self.C, self.L, self.nb, self.ntr)

    def unpad(self, p):
        return p.reshape(self.C * self.L, -1)[self.place]

    def tables(self, u):
        """Light attenuation and remineralisation fractions of each member's parameters."""
        b, kw = u[:, -1], u[:, 1]
        att = torch.exp(-self.zc[:, None] * kw)                 # [layer, member]
        top, bot = torch.exp(-self.ztop[:, None] * b), torch.exp(-self.zbot[:, None] * b)
        last = self.lastlay[:, :, None]
        deep = (top - torch.where(last, torch.zeros_like(bot), bot)) / self.h[:, None]
        deep = torch.where(self.below[:, :, None], deep, torch.zeros_like(deep))
        shallow = torch.where(last, 1.0 / self.h[:, None] + 0 * top, torch.zeros_like(top))
        return att, torch.where(self.shallow[:, None, None], shallow, deep)

    def q(self, p, u, tab, light):
        """Sources [column, layer, member, tracer] of sections 2.2.1 and 2.2.2."""
        att, rho = tab
        eu, N = self.eu[:, :, None], p[..., 0].clamp(min=0.0)
        I = light[:, None, None] * att
        f = u[:, 0] * N / (N + u[:, 2]) * I / (I + u[:, 3])
        f = torch.where(eu, f, torch.zeros_like(f))
        if self.model == synth.MODEL_N:
            Phi = (self.h[:, None] * f).sum(1, keepdim=True)
            return (-f + Phi * rho)[..., None]
        lam, sig, D = u[:, 4], u[:, 5], p[..., 1]
        if self.model == synth.MODEL_NDOP:
            Phi = (self.h[:, None] * f).sum(1, keepdim=True)
            return torch.stack([-f + lam * D + (1 - sig) * Phi * rho, sig * f - lam * D], -1)
        P, sig3 = p[..., 2], u[:, 9]
        f = f * P
        Phi = (self.h[:, None] * (sig3 * f)).sum(1, keepdim=True)
        loss = torch.where(eu, u[:, 6] * P + u[:, 7] * P * P, torch.zeros_like(P))
        return torch.stack([-f + lam * D + (1 - sig) * Phi * rho, sig * sig3 * f + loss - lam * D + u[:, 8] * P,
                            (1 - sig3) * f - loss - u[:, 8] * P], -1)

    def matrices(self, j):
        spm = NSTEP // NMAT
        m, r = divmod(j - spm // 2, spm)
        w = r / spm
        return [(1 - w) * a + w * b for a, b in zip(self.month(m % NMAT), self.month((m + 1) % NMAT))]

    def step(self, j, p, u, tab):
        ae, ai = self.matrices(j)
        j = j % NSTEP
        inc = torch.zeros_like(p)
        for _ in range(max(self.nbgc, 1)):
            inc = inc + self.dtd / max(self.nbgc, 1) * self.q(p + inc, u, tab, self.light[j])
        flat = torch.cat([p.reshape(self.C * self.L, -1), torch.zeros_like(p[0, :1].reshape(1, -1))])
        z = inc.reshape(self.C * self.L, -1)
        for s in range(self.nbr.shape[1]):
            z = z + ae[:, s, None] * flat[self.nbr[:, s]]
        z = torch.where(self.wet.reshape(-1, 1), z, torch.zeros_like(z)).reshape(self.C, self.L, -1)
        if z.numel() * self.L <= 1 << 24:
            out = (ai[..., None] * z[:, None]).sum(2)
        else:
            out = torch.zeros_like(z)
            for s in range(self.L):
                out = out + ai[:, :, s, None] * z[:, s, None]
        return out.reshape(p.shape)

    def misfit_gradient(self, p, u, obs):
        """J, its derivatives with respect to u and the start state: stored states, one step at a time back."""
        spm, tab = NSTEP // NMAT, self.tables(u)
        w = self.vol[:, None] / (NMAT * self.vol.sum())
        ys = [p]
        for j in range(NSTEP):
            ys.append(self.step(j, ys[-1], u, tab))
        J, gu, mu = torch.zeros(self.nb, dtype=torch.float64, device="cuda"), torch.zeros_like(u), torch.zeros_like(p)
        for j in range(NSTEP, -1, -1):
            y = ys.pop()
            if j and j % spm == 0:
                e = self.unpad(y) - obs[j // spm - 1]
                J += 0.5 * (w * e * e).reshape(-1, self.nb, self.ntr).sum((0, 2))
                mu = mu + self.pad(w * e)
            if j:
                with torch.enable_grad():
                    x, uu = ys[-1].requires_grad_(True), u.clone().requires_grad_(True)
                    gx, g = torch.autograd.grad(self.step(j - 1, x, uu, self.tables(uu)), (x, uu), mu)
                mu, gu = gx, gu + g
        return J, gu, mu


def exact(case, seed):
    call = case["call"]
    if not torch.cuda.is_available():
        return None
    # a year of plain torch takes seconds; its gradient several times that
    steps = {"step": 1, "year": NSTEP, "ensemble": 2 * NSTEP, "tangent": 3 * NSTEP}.get(call, 7 * NSTEP)
    if steps > 1 and steps * (3e-4 * max(case["nbgc"], 1) + 1.3e-9 * case["n"] * case["members"]) > 30:
        return None
    inp, u, y, v, obs, j, years = _inputs(case, seed)
    ud = torch.as_tensor(u).cuda()
    P = _Plain(inp, u)
    with torch.no_grad():
        p, tab = P.pad(y), P.tables(ud)
        if call == "step":
            return P.unpad(P.step(j, p, ud, tab))
        if call == "tangent":
            jv = P.pad(v)
            for k in range(NSTEP):
                p, jv = torch.func.jvp(lambda x: P.step(k, x, ud, tab), (p,), (jv,))
            return P.unpad(p), P.unpad(jv)
        if call in ("adjoint", "gradient"):
            J, gu, gy = P.misfit_gradient(p, ud, obs)
            return J, gu, P.unpad(gy)
        lengths = years if call == "ensemble" else np.ones(1, dtype=np.int32)
        resid = np.zeros((int(lengths.max()), len(lengths)))
        out = torch.empty_like(p)
        for yr in range(int(lengths.max())):
            start = p
            for k in range(NSTEP):
                p = P.step(k, p, ud, tab)
            r = (p - start).square().sum((0, 1, 3)).sqrt().cpu().numpy()
            for b in range(len(lengths)):
                if yr < lengths[b]:
                    resid[yr, b] = r[b]
                if yr + 1 == lengths[b]:
                    out[:, :, b] = p[:, :, b]
        return P.unpad(out), resid

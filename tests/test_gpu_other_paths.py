"""GPU parity of the kernels that run where the default dispatch's first choice does not, against the oracle.

* The single-launch kernels of the packed or wave-aligned layout (k_year_persistent,
  k_adjoint_persistent): packed columns (TMM_OPT_WAVE_LOCAL 0), domains of up to 512 rows, and stencils
  of seven explicit entries per row; several members side by side that stop after different numbers of
  years, their tangents and their gradients; one, two and three tracers, with and without internal BGC
  steps, blocks of 16 and of 32 rows.
* The launch-per-step kernels for batches (k_step, k_adjoint) with three tracers and with internal
  steps, which grids deeper than 32 layers and TMM_OPT_PERSISTENT 0 run.

The year is 240 steps (hand-overs every 64 steps, month changes, checkpoints) with the rates scaled to the
length of a step as in the other edge cases; the tolerances are the usual ones."""

import copy

import numpy as np
import pytest

import oracle
import synth
from tolerances import ADJOINT, MISFIT, TANGENT, YEAR, columnwise, componentwise, pointwise

pytestmark = pytest.mark.gpu

NSTEP, NB = 240, 3
N, NDOP, PHY = synth.MODEL_N, synth.MODEL_NDOP, synth.MODEL_NDOPPHY


def _tmm():
    from paper_1410_0204_amd import tmm
    return tmm


def _ocean(model, nbgc, nlayer, neu=2):
    return synth.custom(12, 8, nlayer, 70, 47 * nlayer + 5, model=model, neuphotic=neu, nstep=NSTEP, nbgc=nbgc)


def _params(inp, nb=NB):
    u = synth.latin_hypercube(inp.model, nb, seed=5).copy()
    u[:, 0] *= inp.nstep / 2880.0
    u[:, 4] *= inp.nstep / 2880.0
    return u


def test_layout_query():
    tmm = _tmm()
    for nlayer, lanes in ((16, 16), (17, 32), (33, 0)):
        t = tmm.TMM(_ocean(NDOP, 1, nlayer).desc_arrays(), nbatch_max=1)
        print(f"[gpu] layout query nlayer={nlayer}", flush=True)
        assert t.query(tmm.TMM_Q_BIN_LANES) == lanes
        assert t.query(tmm.TMM_Q_PERSISTENT) == (1 if lanes else 0)
        t.set_option(tmm.TMM_OPT_WAVE_LOCAL, 0)
        assert t.query(tmm.TMM_Q_BIN_LANES) == 0


def _widen(inp):
    """The ocean with a stencil of seven entries: every third row also reads two rows one and two thirds of
    the grid away, a hundredth of its diagonal each (the row's sum stays)."""
    inp = copy.deepcopy(inp)
    tm, n = inp.tm, inp.n
    rp, ci, av = tm.ae_rowptr, tm.ae_colidx, tm.ae_val
    rptr, cols, vals = [0], [], []
    for i in range(n):
        e = slice(rp[i], rp[i + 1])
        c, v = list(ci[e]), av[:, e].copy()
        spare = [x for x in ((i + n // 3) % n, (i + 2 * (n // 3)) % n) if x not in c] if i % 3 == 0 else []
        if spare:
            d = c.index(i)
            x = 0.01 * v[:, d]
            v[:, d] -= len(spare) * x
            v = np.concatenate([v] + [x[:, None]] * len(spare), axis=1)
            c += spare
        order = np.argsort(c, kind="stable")
        cols.append(np.asarray(c)[order])
        vals.append(v[:, order])
        rptr.append(rptr[-1] + len(c))
    tm.ae_rowptr = np.asarray(rptr, dtype=rp.dtype)
    tm.ae_colidx = np.concatenate(cols).astype(ci.dtype)
    tm.ae_val = np.ascontiguousarray(np.concatenate(vals, axis=1))
    assert int(np.diff(tm.ae_rowptr).max()) == 7
    return inp


def _col(a, b, ntr):
    return np.ascontiguousarray(a[..., b * ntr:(b + 1) * ntr])


def _check(t, inp, o, label):
    """Uneven years, tangents and gradients of the handle's members against the oracle."""
    import torch
    tmm, ntr = _tmm(), inp.ntracer
    u = _params(inp)
    t.set_params(u)
    rng = np.random.default_rng(3)
    y = inp.initial_state(NB).reshape(inp.n, NB * ntr) * rng.uniform(0.8, 1.2, size=(inp.n, NB * ntr))
    v = rng.standard_normal(y.shape) * y
    years = [1 + b % 2 for b in range(NB)]
    got = t.year(t.state(y), nyears=2, years_per_member=years)[0].cpu().numpy()
    jv = t.year_jvp(t.state(y), t.state(v), mode=tmm.TMM_JVP_TANGENT)[1].cpu().numpy()
    snaps = [o.snapshots(u[b] * 1.01, _col(y, b, ntr)) for b in range(NB)]
    obs = np.concatenate([s * (1 + 0.05 * synth.obs_noise(s.shape, seed=9)) for s in snaps], axis=-1)
    J, G, dy0 = t.year_adjoint(t.state(y), torch.as_tensor(obs).cuda())
    dy0, G = dy0.cpu().numpy(), np.asarray(G).reshape(NB, -1)
    for b in range(NB):
        yb, vb = _col(y, b, ntr), _col(v, b, ntr)
        assert pointwise(_col(got, b, ntr), o.year(u[b], yb, years[b])[0], ntr, f"{label} member {b}") <= YEAR
        assert columnwise(_col(jv, b, ntr), o.year_tangent(u[b], yb, vb)[1], ntr, f"{label} tangent {b}") <= TANGENT
        eJ, eG, eY = o.year_adjoint(u[b], yb, _col(obs, b, ntr))
        assert componentwise(np.ravel(J)[b], eJ, "J") <= MISFIT
        assert componentwise(G[b], eG, f"{label} dJ/du {b}") <= ADJOINT
        assert columnwise(_col(dy0, b, ntr), eY, ntr, f"{label} dJ/dy0 {b}") <= ADJOINT
    return got, jv


KINDS = [(N, 1, 10, 2), (NDOP, 1, 20, 2), (PHY, 1, 10, 2), (NDOP, 8, 10, 2), (PHY, 8, 20, 2), (PHY, 8, 10, 4)]


@pytest.mark.parametrize("layout", ["packed", "wide_domains", "wide_stencil"])
@pytest.mark.parametrize("model,nbgc,nlayer,neu", KINDS)
def test_packed_and_wave_aligned_layouts(model, nbgc, nlayer, neu, layout):
    tmm = _tmm()
    inp = _ocean(model, nbgc, nlayer, neu)
    if layout == "wide_stencil":
        inp = _widen(inp)
    label = f"{layout} model={model} nbgc={nbgc} nlayer={nlayer} neu={neu}"
    print(f"[gpu] {label}", flush=True)
    t = tmm.TMM(inp.desc_arrays(), nbatch_max=NB, adjoint_nbatch_max=NB, ckpt_every=48)
    if layout == "packed":
        t.set_option(tmm.TMM_OPT_WAVE_LOCAL, 0)
        t.set_option(tmm.TMM_OPT_DOMAIN_ROWS, 96)
    elif layout == "wide_domains":
        t.set_option(tmm.TMM_OPT_DOMAIN_ROWS, 512)
    # (three tracers, with their tangent, in 512-row domains outgrow the LDS: launches per step)
    fits = not (layout == "wide_domains" and model == PHY and nlayer <= 16)
    assert t.query(tmm.TMM_Q_PERSISTENT) == t.query(tmm.TMM_Q_PERSISTENT_ADJOINT) == (1 if fits else 0)
    assert t.query(tmm.TMM_Q_BIN_LANES) == 0
    assert t.query(tmm.TMM_Q_DOMAINS) > (0 if layout == "wide_domains" else 1) or not fits
    got, jv = _check(t, inp, oracle.Oracle(inp), label)
    if layout != "wide_stencil" and model != PHY and nbgc == 1:
        # one evaluation per step, one or two tracers: the binned layout gives the same bits
        s = tmm.TMM(inp.desc_arrays(), nbatch_max=NB)
        assert s.query(tmm.TMM_Q_BIN_LANES) > 0
        s.set_params(_params(inp))
        rng = np.random.default_rng(3)
        y = inp.initial_state(NB).reshape(inp.n, -1) * rng.uniform(0.8, 1.2, size=(inp.n, NB * inp.ntracer))
        v = rng.standard_normal(y.shape) * y
        years = [1 + b % 2 for b in range(NB)]
        assert np.array_equal(s.year(s.state(y), nyears=2, years_per_member=years)[0].cpu().numpy(), got)
        assert np.array_equal(s.year_jvp(s.state(y), s.state(v), mode=tmm.TMM_JVP_TANGENT)[1].cpu().numpy(), jv)


@pytest.mark.parametrize("model,nbgc,nlayer", [(N, 1, 10), (NDOP, 1, 20), (PHY, 1, 10), (NDOP, 8, 10), (N, 8, 20),
                                               (PHY, 8, 10), (PHY, 1, 33)])
def test_launch_per_step_batches(model, nbgc, nlayer):
    tmm = _tmm()
    inp = _ocean(model, nbgc, nlayer)
    label = f"per step model={model} nbgc={nbgc} nlayer={nlayer}"
    print(f"[gpu] {label}", flush=True)
    t = tmm.TMM(inp.desc_arrays(), nbatch_max=NB, adjoint_nbatch_max=NB, ckpt_every=48)
    t.set_option(tmm.TMM_OPT_PERSISTENT, 0)
    t.set_option(tmm.TMM_OPT_MEMBER_KERNEL_MIN, 0)
    _check(t, inp, oracle.Oracle(inp), label)


@pytest.mark.parametrize("rows", [64, 128])
@pytest.mark.parametrize("model", [N, NDOP, PHY])
def test_a_batch_handle_keeps_what_one_member_has(model, rows):
    """A handle for several members offers one member's years and gradients the same kernels as a handle
    for one: how many members fit the device side by side decides how many run in a launch, not whether
    the reverse sweep is one launch or the insolation stands in LDS."""
    import torch
    tmm = _tmm()
    for nstep in (2880, NSTEP):            # (the table holds the year's steps)
        inp = synth.custom(60, 48, 10, 1900, 14000, model=model, nstep=nstep)
        got = []
        for nb in (1, 4):
            print(f"[gpu] batch handle model={model} rows={rows} nstep={nstep} members={nb}", flush=True)
            t = tmm.TMM(inp.desc_arrays(), nbatch_max=nb, adjoint_nbatch_max=nb, ckpt_every=48)
            t.set_option(tmm.TMM_OPT_WAVE_LOCAL, 0)
            t.set_option(tmm.TMM_OPT_DOMAIN_ROWS, rows)
            got.append([t.query(q) for q in (tmm.TMM_Q_PERSISTENT, tmm.TMM_Q_DOMAINS, tmm.TMM_Q_PERSISTENT_ADJOINT,
                                             tmm.TMM_Q_INSOLATION_LDS)])
        print(f"[gpu] one member, batch: {got}", flush=True)
        assert got[0] == got[1]
    # and the batch's years and gradients, members side by side, give each member's own
    ntr, nb = inp.ntracer, 4
    u = _params(inp, nb)
    rng = np.random.default_rng(6)
    y = inp.initial_state(nb).reshape(inp.n, nb * ntr) * rng.uniform(0.8, 1.2, size=(inp.n, nb * ntr))
    obs = np.broadcast_to(y, (inp.nmat,) + y.shape) * rng.uniform(0.9, 1.1, size=(inp.nmat,) + y.shape)
    t.set_params(u)
    years = t.year(t.state(y))[0].cpu().numpy()
    J, G, dy0 = t.year_adjoint(t.state(y), torch.as_tensor(np.ascontiguousarray(obs)).cuda())
    dy0, G, o = dy0.cpu().numpy(), np.asarray(G).reshape(nb, -1), oracle.Oracle(inp)
    for b in (0, nb - 1):
        assert pointwise(_col(years, b, ntr), o.year(u[b], _col(y, b, ntr))[0], ntr, f"member {b}") <= YEAR
        eJ, eG, eY = o.year_adjoint(u[b], _col(y, b, ntr), _col(obs, b, ntr))
        assert componentwise(np.ravel(J)[b], eJ, "J") <= MISFIT
        assert componentwise(G[b], eG, f"dJ/du {b}") <= ADJOINT
        assert columnwise(_col(dy0, b, ntr), eY, ntr, f"dJ/dy0 {b}") <= ADJOINT


@pytest.mark.parametrize("ncol,n,domains", [(60, 200, 1), (150, 520, 2)])
def test_domains_keep_to_the_latitude_rows_of_their_table(ncol, n, domains):
    """Many latitude rows: a grid of one domain is left whole and loads its insolation step by step; one of
    several is divided so that every domain, the first one too, holds its rows' table."""
    tmm = _tmm()
    inp = synth.custom(max(2, ncol // 40), 60 if domains > 1 else 40, 4, ncol, n, model=NDOP, nstep=NSTEP)
    t = tmm.TMM(inp.desc_arrays(), nbatch_max=NB, adjoint_nbatch_max=NB, ckpt_every=48)
    print(f"[gpu] latitude rows, {t.query(tmm.TMM_Q_DOMAINS)} domains", flush=True)
    assert t.query(tmm.TMM_Q_BIN_LANES) == 16
    if domains == 1:
        assert t.query(tmm.TMM_Q_DOMAINS) == 1 and t.query(tmm.TMM_Q_INSOLATION_LDS) == 0
    else:
        assert t.query(tmm.TMM_Q_DOMAINS) > 1 and t.query(tmm.TMM_Q_INSOLATION_LDS) == 1
    _check(t, inp, oracle.Oracle(inp), f"latitude rows {n}")

"""GPU parity at the edges of the layouts that the single-launch year kernels and the one-member step
kernel choose by a grid's shape, against the oracle.

* Water columns in bins of 16 lanes (up to 16 layers), of 32 lanes (up to 32), or neither (33): the
  forward years of members that run side by side and stop after different numbers of years, and
  their gradients, per model and with internal steps.  The year is 240 steps, so that a launch crosses
  hand-overs (every 64 steps), month changes and checkpoints.
* One-member steps: tiles of exactly 128 rows and one more, columns of the most layers the streaming
  kernel takes and of one more, tiles with an odd number of block words.

The rates are scaled with the length of a step as in the other edge cases, and the tolerances are the
usual ones of a step, a year and a gradient."""

import numpy as np
import pytest

import oracle
import synth
from tolerances import ADJOINT, MISFIT, STEP, YEAR, columnwise, componentwise, pointwise

pytestmark = pytest.mark.gpu

NSTEP = 240


def _tmm():
    from paper_1410_0204_amd import tmm
    return tmm


def _params(inp, nb):
    u = synth.latin_hypercube(inp.model, nb, seed=5).copy()
    u[:, 0] *= inp.nstep / 2880.0
    u[:, 4] *= inp.nstep / 2880.0
    return u


@pytest.mark.parametrize("nlayer,model,nbgc,nb,ckpt", [
    (1, synth.MODEL_N, 1, 5, 48), (16, synth.MODEL_N, 1, 3, 240), (17, synth.MODEL_NDOP, 1, 2, 48),
    (32, synth.MODEL_NDOPPHY, 1, 2, 240), (15, synth.MODEL_NDOP, 8, 3, 48), (33, synth.MODEL_NDOP, 1, 2, 48)])
def test_members_side_by_side(nlayer, model, nbgc, nb, ckpt):
    import torch
    inp = synth.custom(12, 8, nlayer, 70, 70 if nlayer == 1 else 47 * nlayer + 5, model=model, neuphotic=min(2, nlayer),
                       nstep=NSTEP, nbgc=nbgc)
    print(f"[gpu] members nlayer={nlayer} model={model} nbgc={nbgc} members={nb}", flush=True)
    ntr, o = inp.ntracer, oracle.Oracle(inp)
    u = _params(inp, nb)
    rng = np.random.default_rng(3)
    y = inp.initial_state(nb).reshape(inp.n, nb * ntr) * rng.uniform(0.8, 1.2, size=(inp.n, nb * ntr))
    col = lambda a, b: np.ascontiguousarray(a[..., b * ntr:(b + 1) * ntr])  # noqa: E731
    t = _tmm().TMM(inp.desc_arrays(), nbatch_max=nb, adjoint_nbatch_max=nb, ckpt_every=ckpt)
    assert t.query(_tmm().TMM_Q_PERSISTENT) == (1 if nlayer <= 32 else 0)
    t.set_params(u)
    years = [1 + b % 2 for b in range(nb)]
    got, _ = t.year(t.state(y), nyears=2, years_per_member=years)
    got = got.cpu().numpy().reshape(inp.n, nb * ntr)
    for b in range(nb):
        assert pointwise(col(got, b), o.year(u[b], col(y, b), years[b])[0], ntr, f"member {b}") <= YEAR
    snaps = [o.snapshots(u[b] * 1.01, col(y, b)) for b in range(nb)]
    obs = np.concatenate([s * (1 + 0.05 * synth.obs_noise(s.shape, seed=9)) for s in snaps], axis=-1)
    J, G, dy0 = t.year_adjoint(t.state(y), torch.as_tensor(obs).cuda())
    dy0 = dy0.cpu().numpy().reshape(inp.n, nb * ntr)
    for b in range(nb):
        eJ, eG, eY = o.year_adjoint(u[b], col(y, b), col(obs, b))
        assert componentwise(np.ravel(J)[b], eJ, "J") <= MISFIT
        if nlayer > 1 or model != synth.MODEL_N:   # else the one layer keeps what it exports: q = 0, dJ/du is rounding
            assert componentwise(np.asarray(G).reshape(nb, -1)[b], eG, "dJ/du") <= ADJOINT
        assert columnwise(col(dy0, b), eY, ntr, "dJ/dy0") <= ADJOINT


@pytest.mark.parametrize("model", [synth.MODEL_N, synth.MODEL_NDOP, synth.MODEL_NDOPPHY])
@pytest.mark.parametrize("nlayer,ncol,n", [(1, 128, 128), (1, 129, 129), (3, 43, 129), (3, 43, 127), (24, 37, 888),
                                           (24, 61, 901), (25, 30, 602)])
def test_one_member_step(nlayer, ncol, n, model):
    inp = synth.custom(16, 12, nlayer, ncol, n, model=model, neuphotic=min(2, nlayer), nstep=NSTEP)
    print(f"[gpu] step nlayer={nlayer} ncol={ncol} n={n} model={model}", flush=True)
    u = _params(inp, 1)
    y = inp.initial_state() * np.random.default_rng(4).uniform(0.8, 1.2, size=(inp.n, inp.ntracer))
    t = _tmm().TMM(inp.desc_arrays(), nbatch_max=1)
    t.set_params(u)
    o = oracle.Oracle(inp)
    for j in (0, 9, NSTEP - 1):
        assert pointwise(t.step(j, t.state(y)).cpu().numpy(), o.step(u[0], j, y), inp.ntracer, f"step {j}") <= STEP, j

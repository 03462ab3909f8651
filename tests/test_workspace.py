"""What a workspace holds: the rings and tables of the single-launch kernels only where they can run, and no
more of them than can be used at once."""

import copy
import ctypes as C

import numpy as np
import pytest

import synth
from test_abi import _desc, _status
from tolerances import ADJOINT, MISFIT, TANGENT, YEAR, columnwise, componentwise, pointwise

NSTEP = 240


def _bytes(inp, members):
    d, keep = _desc(inp, nbatch_max=members, adjoint_nbatch_max=0)
    rc, n = _status(d)
    assert rc == 0
    return n


def _ring(inp):
    return 128 * ((inp.n + 63) // 64 * 64) * inp.ntracer * 8


def _widen(inp, width):
    """The ocean with one row of `width` explicit entries (zeros added)."""
    inp = copy.deepcopy(inp)
    tm = inp.tm
    i = int(np.argmax(np.diff(tm.ae_rowptr)))
    e1 = int(tm.ae_rowptr[i + 1])
    have = tm.ae_colidx[tm.ae_rowptr[i]:e1].tolist()
    extra = [c for c in range(inp.n) if c not in have][:width - len(have)]
    tm.ae_colidx = np.insert(tm.ae_colidx, e1, extra).astype(tm.ae_colidx.dtype)
    tm.ae_val = np.insert(tm.ae_val, [e1] * len(extra), 0.0, axis=1)
    tm.ae_rowptr = tm.ae_rowptr.copy()
    tm.ae_rowptr[i + 1:] += len(extra)
    return inp


def _ocean(nlayer, neu=2):
    return synth.custom(12, 8, nlayer, 70, 47 * nlayer + 5, model=synth.MODEL_NDOP, neuphotic=neu, nstep=NSTEP)


@pytest.mark.parametrize("which", ["deep", "euphotic", "stencil"])
def test_no_rings_where_no_kernel_uses_them(which):
    inp = {"deep": lambda: _ocean(33), "euphotic": lambda: _ocean(10, neu=5),
           "stencil": lambda: _widen(_ocean(10), 9)}[which]()
    assert (_bytes(inp, 24) - _bytes(inp, 1)) / 23 < 0.25 * _ring(inp)


def test_two_rings_a_member_and_no_more_members_than_run_side_by_side():
    inp = _ocean(10)
    more = (_bytes(inp, 24) - _bytes(inp, 1)) / 23
    assert 2 * _ring(inp) <= more < 2.25 * _ring(inp)
    tiny = synth.tiny(nstep=NSTEP)                      # 300 points: 65536 / 300 = 218 members
    assert (_bytes(tiny, 1024) - _bytes(tiny, 512)) / 512 < 0.25 * _ring(tiny)
    point = synth.custom(1, 1, 1, 1, 1, neuphotic=1, model=synth.MODEL_N, nstep=NSTEP)
    assert (_bytes(point, 1024) - _bytes(point, 512)) / 512 < 0.25 * _ring(point)


@pytest.mark.gpu
def test_a_workspace_with_fewer_rings_serves_too(monkeypatch):
    """Down to two rings a handle is created and gives each member's years, tangents and gradients, as the
    full workspace does; with one, the call is refused."""
    import torch
    import oracle
    from paper_1410_0204_amd import tmm
    nb = 4
    inp = _ocean(10)
    ntr, full, ring = inp.ntracer, tmm.tmm_workspace_bytes, _ring(inp)
    u = synth.latin_hypercube(inp.model, nb, seed=5).copy()
    u[:, 0] *= NSTEP / 2880.0
    u[:, 4] *= NSTEP / 2880.0
    rng = np.random.default_rng(3)
    y = inp.initial_state(nb).reshape(inp.n, nb * ntr) * rng.uniform(0.8, 1.2, size=(inp.n, nb * ntr))
    v = rng.standard_normal(y.shape) * y
    obs = np.ascontiguousarray(np.broadcast_to(y, (inp.nmat,) + y.shape) * rng.uniform(0.9, 1.1, size=y.shape))
    o = oracle.Oracle(inp)

    def col(a, b):
        return np.ascontiguousarray(a[..., b * ntr:(b + 1) * ntr])

    for fewer in (0, 3, 6):                             # eight rings, five, two
        print(f"[gpu] workspace of {8 - fewer} rings", flush=True)
        monkeypatch.setattr(tmm, "tmm_workspace_bytes", lambda d: full(d) - fewer * ring)
        t = tmm.TMM(inp.desc_arrays(), nbatch_max=nb, adjoint_nbatch_max=nb, ckpt_every=48)
        assert t.query(tmm.TMM_Q_PERSISTENT) == 1 and t.query(tmm.TMM_Q_WORKSPACE) == full(t.desc) - fewer * ring
        t.set_params(u)
        got = t.year(t.state(y))[0].cpu().numpy()
        jv = t.year_jvp(t.state(y), t.state(v), mode=tmm.TMM_JVP_TANGENT)[1].cpu().numpy()
        J, G, dy0 = t.year_adjoint(t.state(y), torch.as_tensor(obs).cuda())
        dy0, G = dy0.cpu().numpy(), np.asarray(G).reshape(nb, -1)
        for b in range(nb):
            assert pointwise(col(got, b), o.year(u[b], col(y, b))[0], ntr, f"member {b}") <= YEAR
            assert columnwise(col(jv, b), o.year_tangent(u[b], col(y, b), col(v, b))[1], ntr, f"tangent {b}") <= TANGENT
            eJ, eG, eY = o.year_adjoint(u[b], col(y, b), col(obs, b))
            assert componentwise(np.ravel(J)[b], eJ, "J") <= MISFIT
            assert componentwise(G[b], eG, f"dJ/du {b}") <= ADJOINT
            assert columnwise(col(dy0, b), eY, ntr, f"dJ/dy0 {b}") <= ADJOINT
    monkeypatch.setattr(tmm, "tmm_workspace_bytes", lambda d: full(d) - 6 * ring - 256)
    with pytest.raises(tmm.TmmError) as err:
        tmm.TMM(inp.desc_arrays(), nbatch_max=nb, adjoint_nbatch_max=nb, ckpt_every=48)
    assert err.value.status == tmm.TMM_ENOMEM

"""What a handle says of the layout its single-launch kernels run in."""

import pytest

import synth

pytestmark = pytest.mark.gpu

NSTEP = 240
NDOP = synth.MODEL_NDOP


def _tmm():
    from paper_1410_0204_amd import tmm
    return tmm


def _ocean(model, nbgc, nlayer, neu=2):
    return synth.custom(12, 8, nlayer, 70, 47 * nlayer + 5, model=model, neuphotic=neu, nstep=NSTEP, nbgc=nbgc)


def test_layout_query():
    tmm = _tmm()
    for nlayer, lanes in ((16, 16), (17, 32), (33, 0)):
        t = tmm.TMM(_ocean(NDOP, 1, nlayer).desc_arrays(), nbatch_max=1)
        print(f"[gpu] layout query nlayer={nlayer}", flush=True)
        assert t.query(tmm.TMM_Q_BIN_LANES) == lanes
        assert t.query(tmm.TMM_Q_PERSISTENT) == (1 if lanes else 0)
        t.set_option(tmm.TMM_OPT_WAVE_LOCAL, 0)
        assert t.query(tmm.TMM_Q_BIN_LANES) == 0

"""The launch configurations the autotuner tries, on a stand-in handle."""

from types import SimpleNamespace

import pytest

from paper_1410_0204_amd import autotune as A
from paper_1410_0204_amd import tmm as T


class Handle:
    def __init__(self, ntracer, persistent, nlayer=15, nbgc=1):
        self.ntracer = self.model = ntracer
        self.persistent = persistent
        self.desc = SimpleNamespace(nlayer=nlayer, nbgc=nbgc)

    def query(self, what):
        assert what == T.TMM_Q_PERSISTENT
        return self.persistent


def _in_force(cand):
    return {**A.DEFAULTS, **cand}


@pytest.mark.parametrize("nbatch", [1, 3, 24])
@pytest.mark.parametrize("ntracer", [1, 2, 3])
def test_the_single_launch_kernels_are_tried_for_every_batch(ntracer, nbatch):
    """The library runs members side by side in one launch unless an option asks for another kernel: the
    candidates hold its own choice, at the default domain size among others."""
    found = [_in_force(c) for c in A.candidates(Handle(ntracer, 1), nbatch)]
    own = [c for c in found if c[T.TMM_OPT_PERSISTENT] == 1 and c[T.TMM_OPT_MEMBER_KERNEL_MIN] == -1
           and c[T.TMM_OPT_MEMBER_TILE] == 0 and c[T.TMM_OPT_TILE_ROWS] == 0]
    assert sorted(c[T.TMM_OPT_DOMAIN_ROWS] for c in own) == sorted(A.DOMAIN_ROWS)
    assert 256 in A.DOMAIN_ROWS
    assert any(c[T.TMM_OPT_PERSISTENT] == 0 for c in found)


@pytest.mark.parametrize("nbatch", [1, 3])
def test_no_single_launch_candidate_where_it_is_not_available(nbatch):
    assert all(c[T.TMM_OPT_PERSISTENT] == 0 for c in A.candidates(Handle(2, 0), nbatch))

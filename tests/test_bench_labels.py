"""The benchmark names the kernel a handle's years and gradients run by the layout the handle reports."""

from types import SimpleNamespace

import pytest

import bench
from paper_1410_0204_amd import tmm


class Handle:
    def __init__(self, persistent, adjoint, lanes, nlayer=15, nbgc=1):
        self.q = {tmm.TMM_Q_PERSISTENT: persistent, tmm.TMM_Q_PERSISTENT_ADJOINT: adjoint, tmm.TMM_Q_BIN_LANES: lanes}
        self.desc = SimpleNamespace(nlayer=nlayer, nbgc=nbgc)

    def query(self, what):
        return self.q[what]


@pytest.mark.parametrize("handle,year,adjoint", [
    (Handle(1, 1, 16), "k_year_bins", "k_adjoint_bins"),
    (Handle(1, 1, 0), "k_year_persistent", "k_adjoint_persistent"),
    (Handle(1, 0, 0), "k_year_persistent", "k_adjoint"),
    (Handle(0, 0, 0), "k_step_stream", "k_adjoint"),
    (Handle(0, 0, 0, nbgc=8), "k_step", "k_adjoint"),
    (Handle(0, 0, 0, nlayer=33), "k_step", "k_adjoint")])
def test_kernel_names(handle, year, adjoint):
    assert bench.year_kernel(handle) == year
    assert bench.adjoint_kernel(handle) == adjoint

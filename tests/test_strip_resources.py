"""The strip and mixed tiled solvers in the compiler's resource report (CPU only): every shape the
dispatch launches is there, and none spills registers to private memory."""
import re

import pytest

from tests.test_build_resources import _resources


@pytest.fixture(scope="module")
def kernels():
    return _resources("fit.hip")


@pytest.mark.parametrize("family,shapes", [("fit_strip_kernel", [2, 4, 6, 8, 16, 32]),
                                           ("fit_tile_mixed_kernel", [64, 96, 128, 256, 512])])
def test_large_voxel_solvers_do_not_spill(kernels, family, shapes):
    found = {}
    for name, r in kernels.items():
        m = re.search(family + r"ILi(\d+)E", name)
        if m:
            found[int(m.group(1))] = r
    assert sorted(found) == shapes
    for n, r in found.items():
        assert r["ScratchSize"] == 0 and r["VGPRs Spill"] == 0, (family, n, r)

"""Register budgets of kernels whose time was seen to follow them, from the
metadata of the built library."""
import re

import pytest

from tests import codeobj

pytestmark = pytest.mark.skipif(not codeobj.available(), reason="needs the built library")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    return codeobj.kernels(tmp_path_factory.mktemp("codeobj"))


def waves(vgprs):
    """Waves per SIMD: 512 registers of a lane, in granules of 8, at most 8 waves."""
    return min(8, 512 // ((vgprs + 7) // 8 * 8))


@pytest.mark.parametrize("taps,least", [(1, 7), (2, 5), (4, 4)])
def test_tile_factored_pass_keeps_its_waves(kernels, taps, least):
    """k_grid_tf in FP32 with one output tile per block (k_grid_tf<.., taps,
    false, false>): a line of 4096 cells took 66.5 us an iteration, not 48.3, when
    its blocks carried the next control slot through their products."""
    got = {k: v for k, v in kernels.items() if re.search(r"9k_grid_tfILb[01]ELi%dELb0ELb0E" % taps, k)}
    assert len(got) == 2
    for k, v in got.items():
        assert v["spilled"] == 0 and waves(v["vgprs"]) >= least, (k, v)

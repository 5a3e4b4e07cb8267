"""The forward's limit of 8192 tiles: 2048x1024 pixels take two wavefronts a
16x16 tile, a column more takes one, whose NaN-row form stages every record and
counts positions itself.  Compared as in test_gpu_raster_bands with a batch
depth of 128 (one wavefront a tile, the select form)."""
import pytest

import test_gpu_raster_bands as bands
from _gpu_common import gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.mark.parametrize("name,n,width,height", [("cfg2", 60000, 2048, 1024), ("cfg2", 60000, 2049, 1024),
                                                 ("cfg0", 4000, 2100, 1030)])
def test_forms_match_around_the_largest_limit(name, n, width, height):
    bands.test_bands_match_whole_tiles(name, n, width, height, True)

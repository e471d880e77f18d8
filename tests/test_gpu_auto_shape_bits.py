"""The automatic launch shape keeps the rounding of a site's update at a given
size: with beta 4 and 5 the 7-point sweep has two (tiles of one site a thread,
wider tiles), and an automatic FP32 lattice follows the first below 96^3 and
the second from there, whatever tile is the fastest."""
from dataclasses import replace

import pytest
import torch

from _parity import ARRAYS, gpu_run
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beta", [4, 5])
@pytest.mark.parametrize("N,tile_y", [(33, 4), (48, 4), (64, 4), (95, 4), (96, 8), (112, 8), (160, 8)])
def test_automatic_shape_is_bitwise_the_reference_tile(N, tile_y, beta):
    w = replace(W.CFG1.resized(N), beta=beta)
    ic = W.make_inputs(w)
    ref, _ = gpu_run(w, ic, 1, dtype="f32", tile_x=64, tile_y=tile_y)
    got, _ = gpu_run(w, ic, 1, dtype="f32")
    # from one state, one step: nothing but the site arithmetic can differ
    for k, a, b in zip(ARRAYS, got.get_state()[0], ref.get_state()[0]):
        assert torch.equal(a, b), k

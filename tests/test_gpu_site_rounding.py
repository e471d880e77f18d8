"""Every copy of a site's update in the 7-point sweep rounds alike: a tile's ring
sites (computed for the sums, stored by the neighbouring tile) and the sites of
tiles of the same kind (one site a thread; wider)."""
from dataclasses import replace

import pytest
import torch

from _parity import ARRAYS, gpu_run
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu

ONE_SITE = [(64, 4), (32, 8)]
WIDE = [(32, 16), (64, 8), (64, 16), (128, 4), (128, 8)]


@pytest.mark.parametrize("beta", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_step_sums_are_those_of_the_stored_fields(dtype, beta):
    """The gradient sums of a step (lf_scalars.pend) against the same sums over
    the stored arrays: differences in the lattice's type, squares in FP64.
    The sums hold 9e5 positive FP64 terms, added in another order: 1e-13 is far
    above the rounding of such sums (some 1e-15) and far below what last bits of
    FP32 at the tile borders would make (1e-11)."""
    w = replace(W.CFG1.resized(66), beta=beta)
    ic = W.make_inputs(w)
    for tx, ty in ONE_SITE + WIDE:
        lat, _ = gpu_run(w, ic, 1, dtype=dtype, tile_x=tx, tile_y=ty, zchunk=11)
        arrays, sc = lat.get_state()
        for d, got in zip(arrays[:2], sc.pend[:2]):
            want = sum(float(((d - d.roll(1, k)).double() ** 2).sum()) for k in range(3))
            assert abs(got - want) <= 1e-13 * want, (tx, ty)
        lat.close()


@pytest.mark.parametrize("tiles", [ONE_SITE, WIDE])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("beta", [3, 4, 5, 6])
def test_tiles_of_a_kind_are_bitwise_equal(beta, dtype, tiles):
    w = replace(W.CFG1.resized(48), beta=beta)
    ic = W.make_inputs(w)
    ref = None
    for tx, ty in tiles:
        lat, _ = gpu_run(w, ic, 1, dtype=dtype, tile_x=tx, tile_y=ty, zchunk=13)
        s = lat.get_state()[0]
        lat.close()
        ref = ref or s
        for k, a, b in zip(ARRAYS, s, ref):
            assert torch.equal(a, b), (tx, ty, k)

"""The ensemble's batched energies are a lone lattice's to the bit: the same blocks
sum the same sites in the same order, and the same arithmetic forms the report."""
import pytest
import torch

from paper_0911_5692_amd import Ensemble, Lattice
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu

KEYS = ("step", "a", "ad", "hubble", "K1", "K2", "G1", "G2", "P", "rho", "R", "status")


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("stencil", [7, 27])
@pytest.mark.parametrize("sizes", [[5], [4, 33, 64, 100], [16] * 70])
def test_reports_are_bitwise_equal(sizes, stencil, dtype):
    models = [{**W.CFG1.resized(n).model(), "stencil": stencil} for n in sizes]
    zch = [max(1, n // 2) for n in sizes]
    ens = Ensemble(models, dtype=dtype, tile_x=64, tile_y=8, zchunks=zch)
    lone = {}
    for r, n in enumerate(sizes):
        ic = W.make_inputs(W.CFG1.resized(n), realization=r % 3)
        f = [torch.from_numpy(ic[k]).cuda() for k in ("f1", "f2", "u1", "u2")]
        ens.init_physical(r, *f)
        if (n, r % 3) not in lone:
            lat = Lattice(**models[r], dtype=dtype, tile_x=64, tile_y=8, zchunk=zch[r])
            lat.init_physical(*f)
            lone[n, r % 3] = lat
    for steps in (0, 2, 3):
        ens.step(steps)
        ref = {}
        for k, lat in lone.items():
            lat.step(steps)
            ref[k] = lat.energies()
        for r, (n, e) in enumerate(zip(sizes, ens.energies())):
            want = ref[n, r % 3]
            assert {k: e[k] for k in KEYS} == {k: want[k] for k in KEYS}, (r, n)
    ens.close()

"""Which block writes the scalars of a step whose scale factor the sweep forms: a
block of its own while the tiles leave room on the device (fewer blocks than
fit at once, whatever the CUs are), else the block of the first tile.  FP64 tiles
of 64 x 16 and 128 x 8 fit once or twice on a CU, so 800 blocks are more than
fit and 200 are not."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_0911_5692_amd import Lattice
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stencil", [7, 27])
@pytest.mark.parametrize("N,tx,ty,rows", [(80, 64, 16, 800), (80, 128, 8, 800), (40, 64, 8, 200), (50, 64, 16, 200)])
def test_either_writer_against_the_oracle(N, tx, ty, rows, stencil):
    assert rows == -(-N // tx) * -(-N // ty) * N
    m = {**W.CFG1.resized(N).model(), "stencil": stencil}
    ic = W.make_inputs(W.CFG1.resized(N))
    st = O.start_physical(O.Model(**m), ic["f1"], ic["f2"], ic["u1"], ic["u2"], ic["a0"])
    lat = Lattice(**m, dtype=torch.float64, tile_x=tx, tile_y=ty, zchunk=1)
    lat.init_physical(*[torch.from_numpy(ic[k]).cuda() for k in ("f1", "f2", "u1", "u2")], ic["a0"])
    for n in (1, 4):  # either parity of the buffers
        lat.step(n)
        O.evolve(st, n)
        # FP64 throughout: a few rounding errors of 2e-16 a step
        for g, r in zip(lat.fields(), (st.f1, st.f2, st.v1, st.v2)):
            g = g.cpu().numpy()
            assert np.max(np.abs(g - r)) <= 1e-12 * np.max(np.abs(r))
        assert abs(lat.energies()["ad"] - st.ad) <= 1e-12 * abs(st.ad)
    lat.close()

"""The scale-factor update formed in the sweep's own blocks against the
oracle, at the edges of its rule: one partial row, fewer rows than CUs (an
extra block writes the scalars), more (a tile's block does), the most rows a
block sums (1024), and more than that (a kernel of its own)."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_0911_5692_amd import Lattice
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stencil", [7, 27])
@pytest.mark.parametrize("N,tx,ty,zc,rows", [(5, 64, 16, 5, 1), (16, 64, 4, 1, 64), (40, 64, 8, 1, 200),
                                             (48, 64, 4, 1, 576), (64, 64, 4, 1, 1024), (66, 64, 4, 1, 2244)])
def test_update_in_the_sweep(N, tx, ty, zc, rows, stencil):
    assert rows == -(-N // tx) * -(-N // ty) * -(-N // zc)
    m = {**W.CFG1.resized(N).model(), "stencil": stencil}
    ic = W.make_inputs(W.CFG1.resized(N))
    st = O.start_physical(O.Model(**m), ic["f1"], ic["f2"], ic["u1"], ic["u2"], ic["a0"])
    lat = Lattice(**m, dtype=torch.float64, tile_x=tx, tile_y=ty, zchunk=zc)
    lat.init_physical(*[torch.from_numpy(ic[k]).cuda() for k in ("f1", "f2", "u1", "u2")], ic["a0"])
    for n in (1, 2, 8):  # either buffer parity, lone steps and longer graphs
        lat.step(n)
        O.evolve(st, n)
        # FP64 throughout: a few rounding errors of 2e-16 a step
        for g, r in zip(lat.fields(), (st.f1, st.f2, st.v1, st.v2)):
            g = g.cpu().numpy()
            assert np.max(np.abs(g - r)) <= 1e-12 * np.max(np.abs(r))
        e = lat.energies()
        assert abs(e["ad"] - st.ad) <= 1e-12 * abs(st.ad)
    lat.close()


@pytest.mark.parametrize("N", [271, 272])
def test_27_points_with_and_without_the_update(N):
    """The largest lattice whose FP32 27-point sweep in 128 x 8 tiles updates
    the scale factor, and the smallest whose sweep reads it, against 64 x 8
    tiles, which always update it."""
    m = {**W.CFG3.resized(N).model(), "stencil": 27}
    g = torch.Generator(device="cuda").manual_seed(N)
    ic = [b + 1e-3 * torch.randn((N, N, N), dtype=torch.float64, device="cuda", generator=g)
          for b in (1.0, 0.0, -0.7, 0.0)]
    res = []
    for tx in (128, 64):
        lat = Lattice(**m, dtype=torch.float32, tile_x=tx, tile_y=8, zchunk=128)
        lat.init_physical(*ic)
        lat.step(5)
        res.append((lat.fields(), lat.energies()))
        lat.close()
    (fa, ea), (fb, eb) = res
    # the same site arithmetic; the sums in another order move a by about 1e-16
    # a step, which may turn the rounding of a coefficient
    for a, b in zip(fa, fb):
        assert float((a - b).abs().max()) <= 1e-6 * float(b.abs().max())
    assert abs(ea["ad"] - eb["ad"]) <= 1e-12 * abs(eb["ad"])

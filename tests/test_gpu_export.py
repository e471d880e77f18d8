"""Field export: every choice of outputs, ragged sizes, and a lattice whose sites
are dealt to more than one launch."""
import ctypes
import itertools

import pytest
import torch

from paper_0911_5692_amd import Lattice
from paper_0911_5692_amd import workloads as W
from paper_0911_5692_amd._lib import check, lib

pytestmark = pytest.mark.gpu


def _want(lat, synchronized):
    """f = background + (d - h e), v = background + e in FP64, from the checkpoint."""
    (d1, d2, e1, e2), sc = lat.get_state()
    h = 0.5 * lat.params.dt if synchronized else 0.0
    out = []
    for i, (d, e) in enumerate(((d1, e1), (d2, e2))):
        out.append((sc.bg_f[i] - h * sc.bg_v[i]) + (d.double() - h * e.double()))
    return out + [sc.bg_v[0] + e1.double(), sc.bg_v[1] + e2.double()]


def _random_lattice(N, dtype, seed=5):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lat = Lattice(**W.CFG3.resized(N).model(), dtype=dtype)
    ic = [b + 1e-3 * torch.randn((N, N, N), dtype=torch.float32, device="cuda", generator=gen)
          for b in (1.0, 0.0, -0.7, 0.0)]
    lat.init_physical(*ic)
    return lat


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("N", [4, 7, 33])
def test_every_choice_of_outputs(N, dtype):
    lat = _random_lattice(N, dtype)
    lat.step(2)
    for sync in (0, 1):
        want = _want(lat, sync)
        for chosen in itertools.product((0, 1), repeat=4):
            out = [torch.full((N, N, N), 77.0, dtype=torch.float64, device="cuda") for _ in range(4)]
            ptr = [ctypes.c_void_p(o.data_ptr() if c else None) for o, c in zip(out, chosen)]
            check(lib().lf_get_fields(lat._ctx, *ptr, 1, sync))
            torch.cuda.synchronize()
            for o, w, c in zip(out, want, chosen):
                # a multiply-add of the export may be fused: one rounding of values of order 1
                assert float((o - (w if c else torch.full_like(w, 77.0))).abs().max()) <= 2.0 ** -52
    lat.close()


def test_more_than_one_launch():
    N = 513  # a launch takes 2^27 = 512^3 sites
    lat = _random_lattice(N, torch.float32)
    got = lat.fields(dtype=torch.float32)
    for o, w in zip(got, _want(lat, 0)):
        # rounded once to FP32
        assert float((o.double() - w).abs().max()) <= 2.0 ** -24 * float(w.abs().max())
    lat.close()

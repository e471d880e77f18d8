"""The library's own line transforms against the oracle, at the edges of their
rule: powers of two (one butterfly count for every thread), lengths with
factors 3, 5 and 7 (ragged last rows and columns, odd lengths), the smallest
size, and cutoffs that keep everything, a part and nothing."""
import numpy as np
import pytest
import torch

from oracle import spectra as OS
from oracle import vacuum as OV
from paper_0911_5692_amd import Lattice, vacuum_fields
from paper_0911_5692_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,cutoff", [(96, 0.0), (96, 200.0), (98, 30.5), (105, 0.0), (125, 70.0), (128, 0.0),
                                      (128, 64.0), (128, 0.5), (135, 20.0), (144, 0.0)])
def test_vacuum(N, cutoff, monkeypatch):
    # whole mode numbers: fftfreq(N) * N misses some by a rounding (9, 13, 18
    # at N = 125), which then decides for modes whose |n| is the cutoff
    def mode_norm(n):
        n0, n2 = np.rint(np.fft.fftfreq(n) * n), np.rint(np.fft.rfftfreq(n) * n)
        return np.sqrt(n0[:, None, None] ** 2 + n0[None, :, None] ** 2 + n2[None, None, :] ** 2)

    monkeypatch.setattr(OV, "mode_norm", mode_norm)
    L, m2, eps2 = 0.1 * N, (1.0, 40.0), 1e-6
    spec = dict(f0=(1.0, 0.0), u0=(-0.7, 0.0), m2=m2, eps2=eps2, cutoff=cutoff, seed=77 + N)
    ref = OV.vacuum_state(N, L, spec["f0"], spec["u0"], m2, eps2, spec["seed"], cutoff or None)
    eps = np.finfo(np.float64).eps
    for k, base, g in zip(("f1", "f2", "u1", "u2"), (1.0, 0.0, -0.7, 0.0), vacuum_fields(N, L, spec)):
        r = ref[k]
        fl = np.max(np.abs(r - base))
        # 1e-12 of the fluctuation, plus the rounding of base + fluctuation
        assert np.max(np.abs(g.cpu().numpy() - r)) <= 1e-12 * fl + 4 * eps * (abs(base) + fl), k


@pytest.mark.parametrize("N,dtype,nbins", [(128, torch.float32, None), (128, torch.float64, 40), (256, torch.float32, 1)])
def test_spectrum(N, dtype, nbins):
    w = W.CFG1.resized(N)
    ic = W.make_inputs(w)
    lat = Lattice(**w.model(), dtype=dtype)
    lat.init_physical(*[torch.from_numpy(ic[k]).cuda() for k in ("f1", "f2", "u1", "u2")], ic["a0"])
    lat.step(3)
    (d1, d2, e1, e2), _ = lat.get_state()
    full = lat.fields(synchronized=True)
    h = 0.5 * w.dt
    devs = [d1.double() - h * e1.double(), d2.double() - h * e2.double(), e1.double(), e2.double()]
    for which, dev, g in zip(("f1", "f2", "v1", "v2"), devs, full):
        p, c = lat.spectrum(which, nbins)
        q, d = lat.spectrum(which, nbins)
        assert np.array_equal(p, q) and np.array_equal(c, d)
        rp, rc = OS.shell_spectrum(dev.cpu().numpy(), w.L)
        n = len(p)
        assert np.array_equal(c, rc[:n])
        assert np.all(np.abs(p[1:] - rp[1:n]) <= 1e-10 * rp[1:n] + 1e-14 * np.max(rp[1:]))
        p0 = w.L ** 3 / N ** 6 * float(g.sum()) ** 2
        assert abs(p[0] - p0) <= 1e-12 * p0 + 1e-14 * np.max(rp[1:])
    lat.close()

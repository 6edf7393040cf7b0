"""P(k) shells where the binning X pass and the mode sums have their edges: the smallest and
ragged meshes (tiles partly row padding, work-groups below one wave), one bin, and more
bins than there are shells.  Against the FP64 oracle: mode counts exact, P(k) to the 1e-4 of
the whole-spectrum test, k to FP32 rounding of each mode's term (1e-6)."""

from dataclasses import fields

import numpy as np
import pytest

import oracle
from oracle.pk import power_spectrum
from paper_1703_00879_amd import cola as C
from tests.inputs import displacements

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np1d,nmesh1d,nbins", [
    (8, 8, 8), (8, 16, 2048), (12, 12, 1), (12, 24, 23), (16, 48, 42), (32, 96, 48), (64, 128, 64),
    (64, 192, 170)])
def test_power_spectrum_shells(np1d, nmesh1d, nbins):
    p = C.Params(np1d=np1d, nmesh1d=nmesh1d, box=2.0 * np1d)
    st = C.State(p)
    C.cola_prepare(p, st)
    u = displacements(np1d, p.box, 1.5, nmesh1d, seed=4, clustered=True)
    st.disp_f.copy_(torch.from_numpy(u))
    k, P, nm = C.cola_power_spectrum(p, st, nbins)
    op = oracle.Params(**{f.name: getattr(p, f.name) for f in fields(oracle.Params)})
    ko, Po, nmo = power_spectrum(u.astype(np.float64), op, nbins)
    nmo[0] -= 1   # the oracle counts the k = 0 mode in bin 0
    assert np.array_equal(nm, nmo.astype(np.int64))
    got = nm > 0
    got[0] = False
    assert np.all(P[~got] == 0) and np.all(k[~got] == 0)
    assert np.max(np.abs(P[got] / Po[got] - 1), initial=0) < 1e-4
    assert np.max(np.abs(k[got] / ko[got] - 1), initial=0) < 1e-6

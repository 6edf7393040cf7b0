"""The k-Mouflage source and the mesh read-outs, which take four cells of a row at a time: the
smallest rows, rows that are no multiple of a wave, weak to strong screening, and meshes
that start on a 4-byte boundary.  S = (rho - 1) eps against the oracle's bisection from the
same run's density and Newtonian force meshes.  Newton's root in FP32 holds |ln X| < 32 to about
2^-18 and P_X gets (m - 1) times that, so 2e-5 (m - 1) of eps, and the source two roundings more."""

import numpy as np
import pytest

from oracle.models import eps_kmouflage
from paper_1703_00879_amd import cola as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

H0C = 1.0 / 2997.92458


@pytest.mark.parametrize("m", [2, 3, 8])
@pytest.mark.parametrize("np1d,nmesh1d", [(8, 8), (12, 24), (16, 48), (48, 192)])
def test_source_and_unaligned_meshes(np1d, nmesh1d, m):
    a, lam = 0.8, 5e6
    kw = dict(np1d=np1d, nmesh1d=nmesh1d, box=2.0 * np1d)
    g = torch.Generator(device="cuda").manual_seed(np1d)
    u = torch.randn((3, np1d ** 3), device="cuda", generator=g) * 3.0
    out = {}
    for name, p in (("lcdm", C.Params(model=C.LCDM, **kw)),
                    ("km", C.Params(model=C.KMOUFLAGE, km_m=m, km_k0=1.0, km_lambda=lam, **kw))):
        st = C.State(p)
        C.cola_prepare(p, st)
        st.disp_f.copy_(u)
        n = 5 * nmesh1d ** 3
        mesh = torch.empty(n, device="cuda")
        C.cola_pm_force(p, st, a, None, mesh)
        off = torch.full((n + 2,), 7.0, device="cuda")
        C.cola_pm_force(p, st, a, None, off[1:1 + n])
        assert torch.equal(off[1:1 + n], mesh) and off[0] == 7.0 and off[-1] == 7.0
        out[name] = mesh.cpu().numpy().astype(np.float64).reshape(5, -1)
    assert np.array_equal(out["lcdm"][0], out["km"][0])   # the density, deposited twice
    F = np.sqrt((out["lcdm"][2:] ** 2).sum(0))
    eps = eps_kmouflage(F * H0C ** 2 / a ** 2, 1.0, m, lam)
    S = (out["km"][0] - 1.0) * eps
    assert np.all(np.abs(out["km"][1] - S) <= (2e-5 * (m - 1) + 1e-6) * np.abs(S) + 1e-12)

"""The scan of the tile counts on one block, a few (which add up the blocks before their own
themselves) and more than sixteen (a pass of its own), on grids whose last block is full or
not: every cell's density against an FP64 CIC deposit of the same displacements.  Offsets are
rounded to FP32 cell coordinates of up to nmesh1d cells, 2^-24 nmesh1d an axis, times the
particle's mass in cells; the sums are exact to 2^-24."""

import pytest

from paper_1703_00879_amd import cola as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("np1d,nmesh1d", [(8, 8), (48, 96), (96, 192), (128, 256), (96, 384), (128, 512)])
def test_density(np1d, nmesh1d):
    p = C.Params(model=C.LCDM, np1d=np1d, nmesh1d=nmesh1d, box=2.0 * np1d)
    g = torch.Generator(device="cuda").manual_seed(nmesh1d)
    u = torch.randn((3, np1d ** 3), device="cuda", generator=g) * 5.0
    st = C.State(p)
    C.cola_prepare(p, st)
    st.disp_f.copy_(u)
    mesh = torch.empty((5,) + (nmesh1d,) * 3, device="cuda")
    C.cola_pm_force(p, st, 0.5, None, mesh)
    ratio = nmesh1d // np1d
    q = torch.arange(np1d, device="cuda", dtype=torch.float64)
    grid = torch.stack(torch.meshgrid(q, q, q, indexing="ij")).reshape(3, -1)
    x = grid * ratio + 0.5 + u.double() * (nmesh1d / p.box)
    lo = torch.floor(x)
    d, lo = x - lo, lo.long()
    rho = torch.zeros(nmesh1d ** 3, device="cuda", dtype=torch.float64)
    for corner in range(8):
        off = [(corner >> a) & 1 for a in range(3)]
        idx = [(lo[a] + off[a]) % nmesh1d for a in range(3)]
        w = torch.ones_like(d[0])
        for a in range(3):
            w = w * (d[a] if off[a] else 1.0 - d[a])
        rho.index_add_(0, (idx[0] * nmesh1d + idx[1]) * nmesh1d + idx[2], w * ratio ** 3)
    err = (mesh[0].double().reshape(-1) - rho).abs()
    # as many particles as the fullest cell holds may be off by 3 axes' rounding each
    tol = 1e-6 + 3 * nmesh1d * 2.0 ** -24
    assert float((err / torch.clamp(rho, min=float(ratio ** 3))).max()) < 8 * tol
    assert abs(float(mesh[0].double().mean()) - 1.0) < 1e-6

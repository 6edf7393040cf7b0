"""CIC offsets that round to a whole cell.  With 1.25 cells per length unit and u = -0.4 (in
FP32 a little more than 0.4), the cell coordinate 1/2 + u/cell is -7.5e-9 in a fused
multiply-add: its floor is -1 and its FP32 distance from it 1.  Such a particle belongs to the
next cell, whatever the parity of its own, at the edges of tiles (of 16, 8 and 4 cells) and of
the mesh too.  Every cell's density against the FP64 oracle's CIC deposit: a cell gets up to
some eight particles' mass in up to 64 weights, each a product of three FP32 factors (2e-7 of
it) rounded to a unit of 2^-24, and one FP32 rounding, 4e-6 of a particle's mass in all."""

from dataclasses import fields

import numpy as np
import pytest

import oracle
from oracle.pm import cic_deposit, positions_in_cells
from paper_1703_00879_amd import cola as C

torch = pytest.importorskip("torch")


def offsets(np1d, seed):
    """Per axis and particle -0.4 (half of them) or a displacement below a cell."""
    rng = np.random.default_rng(seed)
    u = rng.uniform(-0.79, 0.79, size=(3, np1d ** 3)).astype(np.float32)
    u[rng.random(u.shape) < 0.5] = np.float32(-0.4)
    return u


@pytest.mark.gpu
@pytest.mark.parametrize("np1d,ratio", [(12, 1), (8, 1), (24, 1), (32, 1), (48, 1), (12, 2), (16, 2), (16, 3)])
def test_density_of_offsets_that_round_to_one(np1d, ratio):
    n = np1d * ratio
    p = C.Params(model=C.LCDM, np1d=np1d, nmesh1d=n, box=n / 1.25)
    st = C.State(p)
    C.cola_prepare(p, st)
    u = offsets(np1d, n)
    st.disp_f.copy_(torch.from_numpy(u))
    mesh = torch.empty((5, n, n, n), device="cuda")
    C.cola_pm_force(p, st, 0.5, None, mesh)
    op = oracle.Params(**{f.name: getattr(p, f.name) for f in fields(oracle.Params)})
    rho = cic_deposit(positions_in_cells(u.astype(np.float64), op), n, float(ratio) ** 3)
    got = mesh[0].cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - rho)) < 4e-6 * ratio ** 3

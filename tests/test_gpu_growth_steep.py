"""Growth tables of models whose coefficients vary fast with a: k-Mouflage with P_X - 1 going
as a^-42 to a^-84 or with a strong coupling, and tables whose m^2 falls as a^-40 or whose beta
rises from 0 to 1 between two close knots.  The solver's steps have to follow the model:
steps of 0.04 in ln a leave 5e-10 to 3e-6 in these tables.  Against the FP64 oracle (DOP853,
here with a relative tolerance of 1e-13 and restarted at every knot) at the tables' 1e-10."""

from dataclasses import fields

import numpy as np
import pytest

import oracle
from oracle.cola import time_grid
from oracle.growth import distinct_n2, solve_growth
from oracle.models import Model
from paper_1703_00879_amd import cola as C

torch = pytest.importorskip("torch")

LNA = np.linspace(-3.2, 0.05, 64)
KNOTS = np.linspace(-3.2, 0.05, 14)


def oracle_table(p):
    op = oracle.Params(**{f.name: getattr(p, f.name) for f in fields(oracle.Params)})
    model = Model(op)
    k = 2 * np.pi * np.sqrt(distinct_n2(p.np1d)) / p.box if op.scale_dependent else np.zeros(1)
    return solve_growth(k, time_grid(op)[0], op.omega_m, model.mu, model.gamma2_orth, op.a_ini,
                        rtol=1e-13, breaks=tuple(np.exp(op.mb_lna)))


def table(lna, beta, m2):
    return dict(model=C.MBETA, mb_lna=tuple(lna), mb_beta=tuple(beta), mb_m2=tuple(m2))


STEEP = {
    "km_6": dict(model=C.KMOUFLAGE, km_m=8, km_xn=-6.0, km_x0=0.1, km_beta=0.5),
    "km_6_strong": dict(model=C.KMOUFLAGE, km_m=8, km_xn=-6.0, km_x0=0.1, km_beta=1.5),
    "km_12": dict(model=C.KMOUFLAGE, km_m=8, km_xn=-12.0, km_x0=0.1, km_beta=1.5),
    "km_coupling": dict(model=C.KMOUFLAGE, km_m=2, km_xn=-1.0, km_x0=0.1, km_beta=10.0),
    "mb_40": table(KNOTS, 0.4 + 0.1 * np.sin(5 * KNOTS), 1e6 * np.exp(-40 * (KNOTS + 0.8))),
    "mb_rise": table(LNA, np.where(LNA < -1, 0.0, 1.0), 1e5 * np.exp(-6 * LNA)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("name", sorted(STEEP))
def test_growth_tables_of_steep_models(name):
    p = C.Params(np1d=8, nmesh1d=16, box=60.0, n_steps=10, z_init=19.0, **STEEP[name])
    st = C.State(p)
    C.cola_prepare(p, st)
    G = oracle_table(p)
    for i in range(p.n_steps + 1):
        T = C.cola_growth_table(p, st, i)
        assert T.shape == G[i].shape
        assert np.max(np.abs(T - G[i]) / np.abs(G[i])) < 1e-10

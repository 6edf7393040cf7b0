"""Scale-dependent LPT terms transformed together, where the mesh slots hold the work fields of
both, and one after the other, where particles and mesh have the same grid: the initial
displacement and two steps against the oracle at the parity tests' 1e-5."""

from dataclasses import fields

import numpy as np
import pytest

import oracle
from oracle.cola import Run
from paper_1703_00879_amd import cola as C

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", [C.FR_HS1, C.SYMMETRON])
@pytest.mark.parametrize("np1d,nmesh1d", [(8, 16), (16, 16), (12, 24), (24, 48), (16, 48), (48, 48)])
def test_steps_match_oracle(np1d, nmesh1d, model):
    p = C.Params(model=model, np1d=np1d, nmesh1d=nmesh1d, box=6.0 * np1d, n_steps=10, seed=11)
    st = C.State(p)
    C.cola_make_ic(p, st)
    r = Run(oracle.Params(**{f.name: getattr(p, f.name) for f in fields(oracle.Params)}))

    def close():
        u = st.disp_f.cpu().numpy().astype(np.float64).ravel()
        v = np.asarray(r.u, dtype=np.float64).ravel()
        return np.linalg.norm(u - v) < 1e-5 * np.linalg.norm(v)

    assert close()
    for i in range(2):
        C.cola_step(p, st, i)
        r.step()
        assert close()

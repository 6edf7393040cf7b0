"""bench.py's byte counts of the LPT passes, whose launches take one term of a step or both, and
its names of the binning's kernels."""

import importlib.util
import os

import pytest

from paper_1703_00879_amd import cola as C

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.mark.parametrize("np1d,nmesh1d,terms", [(32, 32, 1), (32, 64, 2), (512, 1024, 2),
                                                 (768, 1536, 2), (1024, 2048, 1)])
def test_lpt_bytes_per_launch(bench, np1d, nmesh1d, terms):
    p = C.Params(model=C.FR_HS1, np1d=np1d, nmesh1d=nmesh1d)
    N, Hp = np1d ** 3, np1d ** 2 * (np1d // 2 + 1)
    ab = lambda k: bench.algorithmic_bytes(k, p)  # noqa: E731
    assert ab("lpt_fft_x_inv") == 16 * Hp + terms * 16 * Hp   # the potentials are read once
    assert ab("lpt_fft_y_inv") == terms * 16 * Hp
    assert ab("lpt_fft_y_inv_yz") == terms * 24 * Hp
    assert ab("lpt_fft_c2r_z3") == terms * (24 * Hp + 12 * N)


@pytest.mark.parametrize("symbol,name", [
    ("void cola::k_bin_count<true>(float const*, cola::BinGeo, int)", "bin_count"),
    ("void cola::k_bin_count<false>(float const*, cola::BinGeo, int)", "bin_count"),
    ("void cola::k_bin_scatter<true>(float const*, cola::BinGeo)", "bin_scatter"),
    ("void cola::k_bin_scatter<false>(float const*, cola::BinGeo)", "bin_scatter"),
])
def test_binning_kernel_names(bench, symbol, name):
    assert bench._profile_name(symbol, 1024, 512) == name

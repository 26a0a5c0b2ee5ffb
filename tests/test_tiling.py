"""Waves and groups of a fast-path launch (fast_tiling, ph_internal.hpp) for every
configuration, built for the host: a named count is kept, and no workgroup is
launched without an equation."""
import ctypes

import pytest

from tests import host_cpp

SOURCE = r"""
#include "ph_internal.hpp"
using namespace ph;
extern "C" void tiling(int n_eq, int n_var, long tiles, int cfg_w, int cfg_g, int def_w, int max_w, int waves, int *out)
{
    DevTable tab;
    tab.n_eq = n_eq;
    tab.n_var = n_var;
    tab.dfast_planes = 2;
    for (int c = 0; c < 4; ++c) {  // equations of one cost
        const int W = std::min(1 << c, n_eq);
        for (int G = 1; (G - 1) * W < n_eq; ++G) {
            const float t = float((n_eq + G * W - 1) / (G * W));
            tab.fit[c].push_back(100 * t);
            tab.fit_max[c].push_back(100 * t);
        }
    }
    const EvalFit f = fast_tiling(tab, tiles, cfg_w, cfg_g, def_w, max_w, waves, size_t(n_var) * 4096, 20.0, 1.0);
    out[0] = f.W;
    out[1] = f.G;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_cpp.load(tmp_path_factory, "tiling", SOURCE)


@pytest.mark.parametrize("max_w,waves", [(4, 4), (8, 8)])
@pytest.mark.parametrize("n_eq", [1, 2, 3, 5, 8, 11, 16, 31, 32, 64])
def test_no_workgroup_without_an_equation(lib, n_eq, max_w, waves):
    out = (ctypes.c_int * 2)()
    for tiles in (1, 7, 300, 5000):
        for cfg_w in range(0, 9):
            for cfg_g in (0, 1, 2, 3, 4, 8, 16, 64):
                def_w = 1
                while 2 * def_w <= min(max_w, n_eq):
                    def_w *= 2
                lib.tiling(n_eq, min(n_eq, 32), ctypes.c_long(tiles), cfg_w, cfg_g, def_w, max_w, waves, out)
                W, G = out[0], out[1]
                case = (tiles, cfg_w, cfg_g, W, G)
                assert 1 <= W <= min(max_w, n_eq) and G >= 1, case
                assert (G - 1) * W < n_eq, case
                if cfg_w:
                    assert W == min(cfg_w, max_w, n_eq), case
                if cfg_g:
                    assert G <= cfg_g and (G == 1 or G * W <= n_eq), case
                    if not cfg_w:
                        assert W == def_w, case

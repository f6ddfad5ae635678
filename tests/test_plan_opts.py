"""hg_build_plan_opts (host only): the plan of a build with options.  The stable one is
hg_build_plan's; in any order 32-bit keys take larger partition tiles, counted in both
passes."""
import ctypes

import pytest

from paper_1907_02900_amd import hg


@pytest.mark.parametrize("kb", [32, 64])
@pytest.mark.parametrize("n,V", [(0, 100), (1, 1), (8192, 8192), (8193, 4096), (300007, 300007),
                                 (1 << 21, 1 << 21), (1 << 28, 1 << 28), (1 << 27, 1 << 25)])
def test_plans_of_both_orders(kb, n, V):
    s, a = hg.build_plan(n, V, kb), hg.build_plan(n, V, kb, any_order=True)
    for p, tile in ((s, 4096), (a, 8192 if kb == 32 else 4096)):
        assert p["tile_keys"] == tile and p["tiles"][0] == -(-n // tile)
        second = p["tiles"][0] + (1 << p["digit_bits"][0]) if p["passes"] == 2 else 0
        assert p["tiles"][1] == second
    for f in ("bucket_bits", "bins", "passes", "digit_bits", "workspace_bytes"):
        assert a[f] == s[f]


def test_options_are_checked():
    p, o = hg.PlanInfo(), hg._opts(bins=64)
    plan = hg.lib().hg_build_plan_opts
    assert plan(1 << 16, 1 << 16, 32, ctypes.byref(o), ctypes.byref(p)) == 0 and p.bins == 64
    assert plan(1 << 16, 1 << 16, 32, None, ctypes.byref(p)) == 0 and p.tile_keys == 4096
    for bad in (hg._opts(variant=hg.VARIANT_V1), hg._opts(stable=1, any_order=True),
                hg._opts(bins=100)):
        assert plan(10, 7, 32, ctypes.byref(bad), ctypes.byref(p)) == 1
    assert plan(10, 7, 32, ctypes.byref(o), None) == 1

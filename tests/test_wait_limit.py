"""LBMD_MD_WAIT_TICKS is read in full or refused, before any device call."""
import ctypes as C

import pytest

from paper_0711_2665_amd import lbmd
from paper_0711_2665_amd.workloads import BASE


@pytest.mark.parametrize("value", ["", " ", "x", "10x", "-1", "+1", "1e3", "0x10", " 7", "7 ", "1000000001",
                                   "18446744073709551616", "99999999999999999999999"])
def test_other_values_are_refused(monkeypatch, value):
    monkeypatch.setenv("LBMD_MD_WAIT_TICKS", value)
    cfg = dict(BASE)
    cfg.update(shape=(16, 16, 16), wall_axis=-1, wall_pos=0, pore_h=0, nb=0)
    d = lbmd.make_desc(cfg)
    b = lbmd.LbBuffers(*[256 * (k + 1) for k in range(6)])     # never read: the value is refused first
    ctx = C.c_void_p()
    assert lbmd.lib().lb_init(C.byref(d), C.byref(b), None, None, None, C.byref(ctx)) == lbmd.LB_ERR_ARG
    assert "LBMD_MD_WAIT_TICKS" in lbmd.lib().lb_last_error().decode()
    assert not ctx.value

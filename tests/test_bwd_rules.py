"""The backward's rules for the path of a call, as host functions of the library: calls whose times on both sides were measured
take the side that was the faster one."""
import ctypes

import pytest

from paper_1909_05840_amd.binding import LIB_PATH


def _rule(name, types):
    rule = getattr(ctypes.CDLL(LIB_PATH), name)
    rule.restype, rule.argtypes = ctypes.c_int if "teams" in name else ctypes.c_bool, types
    return rule


# us a call with the operand staged and turned: 15.2 and 18.3, 16.1 and 18.1, 17.7 and 18.2; 18.7 and 16.8, 48.2 and 43.2
@pytest.mark.parametrize("T,N,turned", [(4, 768, False), (19, 768, False), (455, 1024, False), (871, 2304, True), (4239, 2304, True), (4239, 2300, False)])
def test_short_contractions_stage_dy(T, N, turned):
    assert _rule("_ZN2qb10bwd_turnedEll", [ctypes.c_int64] * 2)(T, N) == turned

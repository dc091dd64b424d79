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


# us a call with one launch and staged: 31.1 and 23.9, 25.5 and 22.5, 27.8 and 26.5, 30.8 and 28.4, 30.5 and 28.3; 24.3 and 28.3,
# 21.9 and 24.5, 25.8 and 28.0, 8.3 and 17.3, 12.4 and 21.4
@pytest.mark.parametrize("T,N,K,dx,dw,teams", [(2067, 3072, 768, True, False, 0), (2494, 2304, 768, True, False, 0), (1364, 2304, 768, True, True, 0),
                                               (2099, 2048, 512, True, True, 0), (2316, 768, 3072, False, True, 0),
                                               (2561, 1024, 1024, True, True, 1), (1287, 2304, 768, True, True, 1), (9214, 768, 768, True, False, 1),
                                               (648, 768, 768, True, True, 2), (242, 2304, 768, True, True, 4)])
def test_calls_take_one_launch_where_it_is_the_faster_path(T, N, K, dx, dw, teams):
    assert _rule("_ZN2qb16bwd_direct_teamsElllbb", [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2)(T, N, K, dx, dw) == teams

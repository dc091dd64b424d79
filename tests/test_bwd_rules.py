"""The backward's rules for the path of a call, as host functions of the library: calls whose times on both sides were measured
take the side that was the faster one."""
import ctypes

import pytest

from paper_1909_05840_amd.binding import LIB_PATH


def _rule(name, types):
    rule = getattr(ctypes.CDLL(LIB_PATH), name)
    rule.restype, rule.argtypes = ctypes.c_bool if "turned" in name else ctypes.c_int, types
    return rule


# us a call with the operand staged and turned: 15.2 and 18.3, 16.1 and 18.1, 17.7 and 18.2; 18.7 and 16.8, 48.2 and 43.2
@pytest.mark.parametrize("T,N,turned", [(4, 768, False), (19, 768, False), (455, 1024, False), (871, 2304, True), (4239, 2304, True), (4239, 2300, False)])
def test_short_contractions_stage_dy(T, N, turned):
    assert _rule("_ZN2qb10bwd_turnedEll", [ctypes.c_int64] * 2)(T, N) == turned


# us a call with one launch and staged, when the line was fitted: 31.1 and 23.9, 25.5 and 22.5, 27.8 and 26.5, 30.8 and 28.4, 30.5 and 28.3; 24.3 and
# 28.3, 21.9 and 24.5, 25.8 and 28.0, 8.3 and 17.3, 12.4 and 21.4; since the one launch turns its operands by LDS reads 26.1 and 25.0, 21.1 and 23.3 (the line
# has not followed), 25.9 and 25.9, 25.9 and 25.8, 29.2 and 27.9; 24.3 and 29.5, 21.9 and 26.0, 25.5 and 28.1, 8.1 (7.8 with one team) and 17.0, 11.5 and 21.5
@pytest.mark.parametrize("T,N,K,dx,dw,teams", [(2067, 3072, 768, True, False, 0), (2494, 2304, 768, True, False, 0), (1364, 2304, 768, True, True, 0),
                                               (2099, 2048, 512, True, True, 0), (2316, 768, 3072, False, True, 0),
                                               (2561, 1024, 1024, True, True, 1), (1287, 2304, 768, True, True, 1), (9214, 768, 768, True, False, 1),
                                               (648, 768, 768, True, True, 2), (242, 2304, 768, True, True, 4)])
def test_calls_take_one_launch_where_it_is_the_faster_path(T, N, K, dx, dw, teams):
    assert _rule("_ZN2qb16bwd_direct_teamsElllbb", [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2)(T, N, K, dx, dw) == teams


# What dW's tiles in that many pieces (two workgroups per CU) take off a training step, us: 8, 9, 5.5, 17, 23, 16, 19, 11, 16, 15, 5; what they would
# add to it where the older kernel keeps the call: 2.2, 2.3, 0.6, 3.5, 3.2, 2.4, 1.8, 2.2, 3.3.  12288 x 3072 x 768: dY is the large operand.  One output only,
# over the older kernel: 384 tiles of dX .88 of the time, 320 1.03, 520 1.15; 72 tiles of dW of 133 steps .98, of 97 1.06
@pytest.mark.parametrize("T,N,K,dx,dw,pieces", [(12288, 768, 768, True, True, 8), (12288, 768, 3072, True, True, 2), (4169, 768, 3072, True, True, 2),
                                                (9333, 448, 1792, True, True, 4), (4325, 1024, 4096, True, True, 1), (8192, 640, 2560, True, True, 3),
                                                (10752, 512, 2048, True, True, 4), (10240, 640, 640, True, True, 8), (7680, 768, 3072, True, True, 2),
                                                (12288, 1536, 512, True, True, 6), (1916, 832, 3328, True, True, 1),
                                                (4096, 768, 3072, True, True, 0), (3072, 768, 3072, True, True, 0), (2048, 768, 3072, True, True, 0),
                                                (4608, 832, 832, True, True, 0), (743, 1024, 4096, True, True, 0), (6307, 704, 704, True, True, 0),
                                                (9728, 576, 576, True, True, 0), (9333, 1792, 448, True, True, 0), (6022, 1920, 640, True, True, 0),
                                                (12288, 3072, 768, True, True, 0),
                                                (4096, 1024, 2304, True, False, 1), (2560, 1024, 3072, True, False, 0), (8320, 1024, 1536, True, False, 0),
                                                (8512, 2304, 768, False, True, 4), (6208, 2304, 768, False, True, 0)])
def test_large_calls_take_two_workgroups_per_cu_where_they_are_faster(T, N, K, dx, dw, pieces):
    assert _rule("_ZN2qb14bwd_duo_piecesElllbb", [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2)(T, N, K, dx, dw) == pieces


# Workgroups that wait hold at most 20 of an XCD's 64 places, so that three calls at once leave some on every XCD
def test_workgroups_that_wait_leave_places_on_every_xcd():
    waiting = _rule("_ZN2qb15bwd_duo_waitingElllbb", [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2)
    seen = set()
    for N in range(128, 3072, 64):
        for K in range(192, 6144, 192):
            for T in (1000, 1700, 3000, 5000, 8200, 12288, 20000):
                for dx in (True, False):
                    seen.add(waiting(T, N, K, dx, True))
    assert max(seen) <= 20 and len(seen) > 8

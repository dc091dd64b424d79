"""The forward's rule for the kernel of a call, as a host function of the library: calls whose times on both sides were measured take the
side that was the faster one."""
import ctypes

import pytest

from paper_1909_05840_amd.binding import LIB_PATH

SLICED, STEPPED, STAGED128, TILES256, ROLES96_TWO, ROLES96_ONE, ROLES128, PLAIN128 = range(8)


# tiles of 32 x 64 over the larger ones behind the activation quantizer: .79, .92, .82, .97;  1.05 at 8 bits with a range per token
@pytest.mark.parametrize("bits,T,N,K,per_token,path", [(4, 5359, 640, 128, False, STEPPED), (4, 5359, 640, 512, False, STEPPED), (8, 7919, 512, 128, False, STEPPED),
                                                       (2, 6511, 640, 640, False, STEPPED), (8, 6511, 640, 768, True, ROLES128)])
def test_calls_of_few_neurons_take_the_small_tiles_where_they_are_faster(bits, T, N, K, per_token, path):
    rule = ctypes.CDLL(LIB_PATH)._ZN2qb8fwd_pathEiiiibb
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int] * 4 + [ctypes.c_bool] * 2
    assert rule(bits, T, N, K, per_token, False) == path

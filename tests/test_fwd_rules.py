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


def takes_list(jobs):
    from paper_1909_05840_amd.binding import _FwdJob
    rule = ctypes.CDLL(LIB_PATH)._ZN2qb14fwd_takes_listEPK10qb_fwd_jobi
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_int]
    arr = (_FwdJob * len(jobs))(*[_FwdJob(1, 1, 6.0, 1, 1, 1, bits, 1, T, N, K, None, 1) for bits, T, N, K in jobs])
    return rule(ctypes.addressof(arr), len(jobs))


def layer(hidden, T, widths):
    return [(b, T, N, K) for b in widths for N, K in ((3 * hidden, hidden), (hidden, hidden), (4 * hidden, hidden), (hidden, 4 * hidden))]


# list / other kernels, us: 439 / 412, 480 / 458, 468 / 431, 526 / 471;  898 / 846;  120 / 104, 131 / 111, 147 / 124, 84 / 79, 41 / 36, 63 / 57
@pytest.mark.parametrize("jobs", [layer(1024, 32768, [2]), layer(1024, 32768, [3]), layer(1024, 32768, [4]), layer(1024, 32768, [8]), layer(1024, 32768, [2, 4]),
                                  [(2, 32768, 1024, 4096)], [(4, 32768, 1024, 4096)], [(8, 32768, 1024, 4096)], [(2, 16384, 4096, 1024)],
                                  [(2, 16384, 768, 3072)], [(8, 16384, 3072, 768)]])
def test_batched_calls_whose_jobs_fill_rounds_of_the_largest_tiles_keep_their_launches(jobs):
    assert not takes_list(jobs)


# list / other kernels, us: 75 / 144, 147 / 172, 214 / 273, 48 / 74;  57 / 66, 60 / 69, 67 / 78;  60 / 68, 64 / 71;  57 / 69
@pytest.mark.parametrize("jobs", [layer(768, 2048, [2, 3, 4, 8]), layer(768, 4096, [2, 3, 4, 8]), layer(768, 6144, [2, 3, 4, 8]), layer(768, 1024, [2, 3, 4, 8]),
                                  layer(768, 6144, [2]), layer(768, 6144, [4]), layer(768, 6144, [8]), layer(1024, 4096, [2]), layer(1024, 4096, [4]),
                                  [(8, 32768, 1792, 448)]])
def test_batched_calls_whose_rounds_are_ragged_share_a_launch(jobs):
    assert takes_list(jobs)


SLICED_BIT = 1 << 16


# the kernel compiled for what all few-tile jobs of a launch have in common, bits | units of a step << 8; of more jobs than a launch holds those of a
# width together
@pytest.mark.parametrize("jobs,kernels", [([(8, 64, 768, 768)] * 3, [8 | SLICED_BIT]), (layer(768, 8, [4]), [4 | SLICED_BIT]), (layer(256, 8, [4, 8]), [SLICED_BIT]),
                                          ([(2, 385, 768, 768)] * 12, [2 | 2 << 8]), ([(3, 700, 768, 320), (3, 64, 64, 64)], [3 | 1 << 8]),
                                          ([(4, 640, 768, 3072)] * 2, [4 | 4 << 8]), (layer(768, 385, [8]), [0]), (layer(768, 512, [8]), [8]),
                                          (layer(768, 704, [3]), [0]), (layer(768, 128, [2, 3, 4, 8]), [0]),
                                          (layer(320, 8, [2, 3, 4, 8]) * 4, [2 | SLICED_BIT, 3 | SLICED_BIT, 4 | SLICED_BIT, 8 | SLICED_BIT]),
                                          (layer(768, 300, [2, 8]) * 3, [0, 8])])
def test_few_tile_jobs_of_one_kind_take_the_kernel_of_their_kind(jobs, kernels):
    from paper_1909_05840_amd.binding import _FwdJob
    rule = ctypes.CDLL(LIB_PATH)._ZN2qb13fwd_few_tilesEPK10qb_fwd_jobiPi
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    arr = (_FwdJob * len(jobs))(*[_FwdJob(1, 1, 6.0, 1, 1, 1, bits, 1, T, N, K, None, 1) for bits, T, N, K in jobs])
    got = (ctypes.c_int * len(jobs))()
    assert rule(ctypes.addressof(arr), len(jobs), ctypes.addressof(got)) == len(kernels) and list(got)[:len(kernels)] == kernels

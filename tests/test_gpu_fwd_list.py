"""The batched forward's launches of many linears of different widths, and the single calls that share their kernel: bit for bit the results of
the other kernels, which the oracle tests cover (whole-number sums, then the same roundings)."""
import ctypes

import pytest

torch = pytest.importorskip("torch")
import paper_1909_05840_amd as qb
from paper_1909_05840_amd import binding

CLIP, GENERAL256 = 6.0, 8
pytestmark = pytest.mark.gpu


def takes_list(jobs):
    rule = ctypes.CDLL(binding.LIB_PATH)._ZN2qb14fwd_takes_listEPK10qb_fwd_jobi
    rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_void_p, ctypes.c_int]
    arr = (binding._FwdJob * len(jobs))(*[binding._FwdJob(1, 1, CLIP, 1, 1, 1, j["bits"], j["groups"], j["Xq"].shape[0], j["N"], j["Xq"].shape[1], None, 1) for j in jobs])
    return rule(ctypes.addressof(arr), len(jobs))


def job(g, bits, T, N, K, groups, bias):
    X = torch.randn(T, K, generator=g, device="cuda")
    W = torch.randn(N, K, generator=g, device="cuda") * 0.04
    packed, h, _, rs_w = qb.qb_quantize_groupwise(W, bits, groups)
    Xq, rs_x = qb.qb_quantize_act(X, CLIP)
    b = torch.randn(N, generator=g, device="cuda") if bias else None
    return {"Xq": Xq, "rs_x": rs_x, "clip": CLIP, "packed": packed, "h": h, "rs_w": rs_w, "bits": bits, "groups": groups, "N": N, "bias": b,
            "Y": torch.full((T, N), float("nan"), device="cuda")}


# (T, N, K, groups) of every width: half a last step (K an odd number of units), one step, ragged last tiles in both directions, odd N (no
# 8-byte rows), more tiles than resident workgroups; the last two stay with the tiles of 32 x 64
@pytest.mark.parametrize("shapes,is_list", [
    ([(4200, 1282, 448, 2), (4100, 1025, 128, 1), (4099, 1501, 192, 1), (129, 3000, 64, 4)], True),
    ([(2500, 1344, 448, 64), (2500, 448, 1792, 64), (2500, 1792, 448, 64), (700, 257, 320, 1)], True),
    ([(6000, 2304, 256, 128), (6000, 768, 384, 128), (5001, 1024, 512, 128), (128, 256, 2048, 128)], True),
    ([(33, 300, 64, 4), (64, 65, 192, 1), (31, 128, 2048, 1), (1, 1, 256, 1)], False),
    ([(200, 768, 768, 128), (129, 500, 320, 4), (65, 768, 3072, 128), (32, 64, 128, 1)], False)])
def test_lists_of_all_widths_give_the_single_calls_results(shapes, is_list):
    g = torch.Generator(device="cuda").manual_seed(7)
    order = [8, 4, 2, 3]  # (the widths of a workgroup's tiles change in both directions)
    jobs = [job(g, b, *s, bias=(i + b) % 2 == 0) for i, s in enumerate(shapes) for b in order]
    assert takes_list(jobs) == is_list
    qb.qb_qlinear_fwd_batched(jobs)
    for j in jobs:
        want = qb.qb_qlinear_fwd(j["Xq"], j["rs_x"], CLIP, j["packed"], j["h"], j["rs_w"], j["bits"], j["groups"], j["N"], bias=j["bias"])
        assert torch.equal(j["Y"], want), (j["bits"], j["Xq"].shape, j["N"])


def test_a_list_of_more_jobs_than_a_launch_holds():
    g = torch.Generator(device="cuda").manual_seed(8)
    jobs = [job(g, (2, 3, 4, 8)[i % 4], 2700 + 37 * i, 1024, 448 + 64 * (i % 3), 64, False) for i in range(21)]
    assert takes_list(jobs)
    qb.qb_qlinear_fwd_batched(jobs)
    for j in jobs:
        assert torch.equal(j["Y"], qb.qb_qlinear_fwd(j["Xq"], j["rs_x"], CLIP, j["packed"], j["h"], j["rs_w"], j["bits"], j["groups"], j["N"]))


# single calls whose rule names the lists' kernel, against slices of their tokens, which take another one.  Groups: one; of 16 neurons; of 17, 89 and 113, which
# begin inside a wavefront's 64 neurons and end in the next one's or in the next tile
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("T,N,K,per_token,asym,groups", [(7680, 2048, 512, True, True, 1), (8100, 1921, 768, True, False, 1), (7600, 2048, 640, False, True, 1),
                                                         (8190, 2048, 704, False, False, 1), (7640, 2047, 832, True, True, 1),
                                                         (7680, 2048, 512, True, True, 128), (7600, 2048, 640, False, True, 128), (8190, 2048, 704, False, False, 128),
                                                         (8100, 1921, 768, True, False, 113), (8100, 1921, 768, False, True, 17), (7640, 2047, 832, True, True, 23)])
def test_single_calls_of_the_lists_kernel(bits, T, N, K, per_token, asym, groups):
    rule = ctypes.CDLL(binding.LIB_PATH)._ZN2qb8fwd_pathEiiiibb
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int] * 4 + [ctypes.c_bool] * 2
    assert rule(bits, T, N, K, per_token, asym) == GENERAL256 and rule(bits, 700, N, K, per_token, asym) != GENERAL256
    g = torch.Generator(device="cuda").manual_seed(bits)
    X = torch.randn(T, K, generator=g, device="cuda")
    # a level and a spread of its own for every group (37 and 11 have no factor in common with a group count above)
    of = torch.arange(N, device="cuda") // (N // groups)
    W = (torch.randn(N, K, generator=g, device="cuda") * 0.04 * (1 + (11 * of % groups) / groups)[:, None] + (37 * of % groups * 0.01 + 0.01)[:, None]).contiguous()
    bias = torch.randn(N, generator=g, device="cuda")
    if asym:
        packed, d, q0, rs_w = qb.qb_quantize_groupwise_asym(W, bits, groups)
        assert len(set(q0.tolist())) == groups
    else:
        packed, d, _, rs_w = qb.qb_quantize_groupwise(W, bits, groups)
    assert len(set(d.tolist())) == groups
    Xq, rs_x, *hx = qb.qb_quantize_act_dyn(X) if per_token else qb.qb_quantize_act(X, CLIP)

    def forward(sl):
        args = [Xq[sl], rs_x[sl]] + ([hx[0][sl]] if per_token else [CLIP]) + [packed, d] + ([q0] if asym else []) + [rs_w, bits, groups, N]
        call = {(True, True): qb.qb_qlinear_fwd_asym_dyn, (True, False): qb.qb_qlinear_fwd_dyn, (False, True): qb.qb_qlinear_fwd_asym, (False, False): qb.qb_qlinear_fwd}
        return call[per_token, asym](*args, bias=bias, want_a4=True)

    Y, A4 = forward(slice(0, T))
    for at in range(0, T, 700):
        at = min(at, T - 700)
        y, a4 = forward(slice(at, at + 700))
        assert torch.equal(A4[at:at + 700], a4) and torch.equal(Y[at:at + 700], y)


# Jobs that share launches of 128 x 96 and of 128 x 128 tiles, three problems in each, in a call that is no list: ragged last tiles in
# both directions, odd N, one step to sixteen
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
def test_shared_launches_of_one_width_give_the_single_calls_results(bits):
    shapes = [(4001, 767, 768, 1), (4090, 1001, 256, 2), (3500, 769, 768, 1), (3000, 1100, 256, 2), (2100, 2304, 128, 1), (3900, 770, 2048, 2)]
    g = torch.Generator(device="cuda").manual_seed(10 + bits)
    jobs = [job(g, bits, T, N, K, 1 if N % 2 else N // 2, bias=i % 2 == 0) for i, (T, N, K, _) in enumerate(shapes)]
    kind = ctypes.CDLL(binding.LIB_PATH)._ZN2qb12fwd_job_kindEPK10qb_fwd_job
    assert not takes_list(jobs)
    assert [kind(ctypes.byref(binding._FwdJob(1, 1, CLIP, 1, 1, 1, bits, 1, T, N, K, None, 1))) for T, N, K, _ in shapes] == [s[3] for s in shapes]
    qb.qb_qlinear_fwd_batched(jobs)
    for j in jobs:
        want = qb.qb_qlinear_fwd(j["Xq"], j["rs_x"], CLIP, j["packed"], j["h"], j["rs_w"], bits, j["groups"], j["N"], bias=j["bias"])
        assert torch.equal(j["Y"], want), (j["Xq"].shape, j["N"])


# few-tile jobs of one width, (T, N, K): sliced; one, two and four units of 64 features a step; different ones, more workgroups than the kernel for
# everything has places
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("shapes,kind", [([(33, 300, 512), (31, 128, 2048), (64, 65, 320)], 1 << 16), ([(700, 768, 320), (129, 500, 192), (1, 1, 64)], 1 << 8),
                                         ([(700, 768, 768), (65, 130, 128), (1, 33, 1024)], 2 << 8), ([(700, 768, 2048), (33, 97, 4096)], 4 << 8),
                                         ([(1700, 1400, 256), (700, 768, 2048), (640, 1000, 192), (33, 97, 2048)], 0)])
def test_few_tile_jobs_of_one_width_give_the_single_calls_results(bits, shapes, kind):
    g = torch.Generator(device="cuda").manual_seed(bits)
    jobs = [job(g, bits, T, N, K, 1, bias=i % 2 == 0) for i, (T, N, K) in enumerate(shapes)]
    rule = ctypes.CDLL(binding.LIB_PATH)._ZN2qb13fwd_few_tilesEPK10qb_fwd_jobiPi
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p]
    arr = (binding._FwdJob * len(jobs))(*[binding._FwdJob(1, 1, CLIP, 1, 1, 1, bits, 1, T, N, K, None, 1) for T, N, K in shapes])
    kernel = ctypes.c_int()
    assert rule(ctypes.addressof(arr), len(jobs), ctypes.addressof(kernel)) == 1 and kernel.value == bits | kind and not takes_list(jobs)
    qb.qb_qlinear_fwd_batched(jobs)
    for j in jobs:
        assert torch.equal(j["Y"], qb.qb_qlinear_fwd(j["Xq"], j["rs_x"], CLIP, j["packed"], j["h"], j["rs_w"], bits, 1, j["N"], bias=j["bias"])), (j["Xq"].shape, j["N"])


def test_more_few_tile_jobs_than_a_launch_holds():
    g = torch.Generator(device="cuda").manual_seed(9)
    jobs = [job(g, (2, 3, 4, 8)[i % 4], 8 + 31 * i, 200 + i, (320, 768, 2048)[i % 3], 1, bias=i % 2 == 0) for i in range(21)]
    assert not takes_list(jobs)
    qb.qb_qlinear_fwd_batched(jobs)
    for j in jobs:
        assert torch.equal(j["Y"], qb.qb_qlinear_fwd(j["Xq"], j["rs_x"], CLIP, j["packed"], j["h"], j["rs_w"], j["bits"], 1, j["N"], bias=j["bias"])), (j["Xq"].shape, j["N"])


def test_a_list_next_to_another_streams_kernels():
    """The lists' kernel while another stream's backward and quantizers share the CUs and the memory: the bits of the call run alone."""
    g = torch.Generator(device="cuda").manual_seed(11)
    T, G = 2048, 128
    jobs = [job(g, b, T, N, K, G, False) for b in (2, 3, 4, 8) for N, K in ((2304, 768), (768, 768), (3072, 768), (768, 3072))]
    assert takes_list(jobs)
    qb.qb_qlinear_fwd_batched(jobs)
    torch.cuda.synchronize()
    alone = [j["Y"].clone() for j in jobs]
    other = job(g, 3, 4096, 2304, 768, G, False)
    W = torch.randn(2304, 768, generator=g, device="cuda")
    dY = torch.randn(4096, 2304, generator=g, device="cuda").to(torch.bfloat16)
    ws = torch.empty(qb.qb_bwd_workspace_nbytes(4096, 2304, 768), dtype=torch.uint8, device="cuda")
    dX, dW = torch.empty(4096, 768, dtype=torch.bfloat16, device="cuda"), torch.empty(2304, 768, device="cuda")
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(4):
        for j in jobs:
            j["Y"].fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(s2):
            for _ in range(8):
                qb.qb_qlinear_bwd_ste(dY, other["Xq"], CLIP, other["packed"], other["h"], 3, G, dX=dX, dW=dW, workspace=ws)
                qb.qb_quantize_groupwise(W, 3, G)
        with torch.cuda.stream(s1):
            for _ in range(6):
                qb.qb_qlinear_fwd_batched(jobs)
        torch.cuda.synchronize()
        for j, want in zip(jobs, alone):
            assert torch.equal(j["Y"], want), (j["bits"], j["N"])

"""The backward's one-launch kernel for small calls (N a multiple of 64) at the edges of its tiles and steps, for one, two
and four teams per workgroup, and the staged path's turned operand, strips of tiles and two workgroups per CU, against the oracle
and plain fp64."""
import ctypes
import functools

import numpy as np
import pytest
import torch

import oracle
from paper_1909_05840_amd import workloads as wl
from paper_1909_05840_amd.binding import LIB_PATH

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CLIP = 6.0


def bounds(dY, W_hat, x_hat):
    """per element: bf16 rounding of the de-quantized weights and of the result; fp32 sums of exact products"""
    a = np.abs(dY.float().numpy().astype(np.float64))
    return 2.0 ** -8 * (a @ np.abs(W_hat)), 2.0 ** -12 * (a.T @ np.abs(x_hat))


def one_launch_teams(T, N, K, dx=True, dw=True):
    """teams per workgroup that the library's rule gives a call, 0 for the staged path"""
    rule = ctypes.CDLL(LIB_PATH)._ZN2qb16bwd_direct_teamsElllbb
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2
    return rule(T, N, K, dx, dw)


def duo_pieces(T, N, K, dx=True, dw=True):
    """pieces of dW's tiles that the library's rule for two workgroups per CU gives a call, 0 for another kernel"""
    rule = ctypes.CDLL(LIB_PATH)._ZN2qb14bwd_duo_piecesElllbb
    rule.restype, rule.argtypes = ctypes.c_int, [ctypes.c_int64] * 3 + [ctypes.c_bool] * 2
    return rule(T, N, K, dx, dw)


def check(dY, W_hat, Xq, dX, dW):
    """every element of dX and dW against plain fp64 within bounds() (sums on the GPU, for the host takes long)"""
    y, w = dY.to(DEV).double(), torch.as_tensor(W_hat).to(DEV).double()
    x = (2.0 * Xq.double() + 1.0) * (CLIP / 255.0)
    if dX is not None:
        ref = y @ w
        assert bool(((dX.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -8 * (y.abs() @ w.abs())).all())
    if dW is not None:
        ref = y.T @ x
        assert bool(((dW.double() - ref).abs() <= 2.0 ** -12 * (y.abs().T @ x.abs())).all())


def behind(t, elements):
    """the same values in memory that starts `elements` elements behind an allocation's start"""
    buf = torch.empty(t.numel() + elements, dtype=t.dtype, device=DEV)
    view = buf[elements:].view(t.shape)
    view.copy_(t)
    return view


# (T, N, K, groups): one step and one tile; one row beyond a step or tile, one short of it; contractions of 1..9 steps in
# one direction and up to 36 in the other, so that teams end with and without a last step (two and four teams; one team for
# the first shape); rows per group 1, 3, 6, N
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("shape", [(64, 64, 64, 64), (65, 128, 64, 1), (127, 192, 128, 64), (193, 64, 320, 8), (130, 2304, 64, 384),
                                   (577, 448, 192, 64), (1001, 448, 448, 64), (600, 768, 768, 128), (2111, 64, 128, 1)])
def test_one_launch_backward(qb, bits, shape):
    T, N, K, G = shape
    print("bwd direct", shape, bits, flush=True)
    W = wl.weight(N, K, seed=N + K + bits)
    X = wl.activation(T, K, seed=T + bits)
    X[0, 0], X[T - 1, K - 1] = CLIP, -100.0
    dY = wl.grad_output_bf16(T, N, seed=T + N)
    Wd, Xd, dYd = W.to(DEV), X.to(DEV), dY.to(DEV)
    packed, h, m, _ = qb.qb_quantize_groupwise(Wd, bits, G)
    Xq, _ = qb.qb_quantize_act(Xd, CLIP)
    dX, dW = qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G)
    sX, sW = qb.qb_qlinear_bwd_ste(behind(dYd, 4), Xq, CLIP, packed, h, bits, G)  # (8-byte aligned)
    mX, mW = qb.qb_qlinear_bwd_ste_masked(dYd, Xq, CLIP, packed, h, bits, G, X=Xd, W=Wd, m=0.5 * m)
    oX = behind(torch.empty(T, K, dtype=torch.bfloat16, device=DEV), 1)
    oW = behind(torch.empty(N, K, device=DEV), 1)
    qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G, dX=oX, dW=oW)
    torch.cuda.synchronize()
    oc, oh, om, _ = oracle.quantize_groupwise(W.numpy(), bits, G)
    oq, _ = oracle.quantize_act(X.numpy(), CLIP)
    rX, rW = oracle.qlinear_bwd_ste(wl.bf16_bits(dY), oq, CLIP, oc, oh, bits, openmp=True)
    tX, tW = bounds(dY, oracle.dequantize_groupwise(oc, oh, bits), oracle.dequantize_act(oq, CLIP))
    for a, b in ((dX, dW), (sX, sW)):
        a, b = a.float().cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
        assert (np.abs(a - rX) <= 2.0 ** -8 * np.abs(rX) + tX).all() and (np.abs(b - rW) <= tW).all()
    assert torch.equal(oX, dX) and torch.equal(oW, dW) and torch.equal(sX, dX) and torch.equal(sW, dW)
    out_x, out_w = Xd.abs() > CLIP, Wd.abs() > (0.5 * m).repeat_interleave(N // G)[:, None]
    assert bool(out_x[T - 1, K - 1]) and not bool(out_x[0, 0]) and bool(out_w.any())
    assert torch.equal(mX, torch.where(out_x, torch.zeros_like(dX), dX)) and torch.equal(mW, torch.where(out_w, torch.zeros_like(dW), dW))
    # one output only: another number of teams may be chosen, so only the bounds hold
    a, none = qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G, want_dw=False)
    none2, b = qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G, want_dx=False)
    assert none is None and none2 is None
    assert (np.abs(a.float().cpu().numpy() - rX) <= 2.0 ** -8 * np.abs(rX) + tX).all() and (np.abs(b.cpu().numpy() - rW) <= tW).all()


# (T, N, K, groups, one output only): one team, contractions of 4 to 36 steps, odd and even, with and without rows beyond a
# multiple of 64
@pytest.mark.parametrize("bits", [2, 3, 4, 8])
@pytest.mark.parametrize("shape", [(1001, 448, 1792, 64, None), (1001, 2304, 768, 128, None), (448, 320, 2560, 64, None), (300, 512, 2048, 1, None),
                                   (1500, 256, 1024, 4, "dX"), (1001, 2304, 768, 384, "dW")])
@pytest.mark.parametrize("asym", [False, True])
def test_one_team(qb, bits, shape, asym):
    T, N, K, G, only = shape
    print("bwd one team", shape, bits, asym, flush=True)
    assert one_launch_teams(T, N, K, only != "dW", only != "dX") == 1
    W, dY = wl.weight(N, K, seed=N + K + bits), wl.grad_output_bf16(T, N, seed=T + N)
    Xq, _ = qb.qb_quantize_act(wl.activation(T, K, seed=T + bits).to(DEV), CLIP)
    want = {"want_dx": only != "dW", "want_dw": only != "dX"}
    if asym:
        packed, delta, q0, _ = qb.qb_quantize_groupwise_asym((W + 0.05).to(DEV), bits, G)
        dX, dW = qb.qb_qlinear_bwd_ste_asym(dY.to(DEV), Xq, CLIP, packed, delta, q0, bits, G, **want)
        W_hat = oracle.dequantize_groupwise_asym(qb.qb_unpack_codes(packed, N, K, bits).cpu().numpy(), delta.cpu().numpy(), q0.cpu().numpy())
    else:
        packed, h, _, _ = qb.qb_quantize_groupwise(W.to(DEV), bits, G)
        dX, dW = qb.qb_qlinear_bwd_ste(dY.to(DEV), Xq, CLIP, packed, h, bits, G, **want)
        W_hat = oracle.dequantize_groupwise(qb.qb_unpack_codes(packed, N, K, bits).cpu().numpy(), h.cpu().numpy(), bits)
    check(dY, W_hat, Xq, dX, dW)


# (T, N, K) and the pieces of two workgroups per CU: rows of 22 tiles of 128 x 192 (strips of four and a last one of two), with two
# workgroups per CU and, dW alone, equal runs; rows of 13, equal runs with both products, dX alone in whole rows; of 13 of 128 x 96 (a last
# one of one), both products in strips, and with dX (four steps) in whole rows
@pytest.mark.parametrize("shape", [(6100, 200, 4096, 4), (8300, 200, 4096, 5), (700, 264, 1216, 0), (700, 200, 1216, 0), (2500, 2000, 2496, 0)])
def test_last_strip_of_tiles_is_narrower(qb, shape):
    T, N, K, pieces = shape
    print("bwd strips", shape, flush=True)
    assert one_launch_teams(T, N, K) == 0 and duo_pieces(T, N, K) == pieces and duo_pieces(T, N, K, dx=False) == 0
    dY = wl.grad_output_bf16(T, N, seed=T + N)
    packed, h, _, _ = qb.qb_quantize_groupwise(wl.weight(N, K, seed=N + K).to(DEV), 4, 8)
    Xq, _ = qb.qb_quantize_act(wl.activation(T, K, seed=T).to(DEV), CLIP)
    dX, dW = qb.qb_qlinear_bwd_ste(dY.to(DEV), Xq, CLIP, packed, h, 4, 8)
    W_hat = oracle.dequantize_groupwise(qb.qb_unpack_codes(packed, N, K, 4).cpu().numpy(), h.cpu().numpy(), 4)
    check(dY, W_hat, Xq, dX, dW)
    check(dY, W_hat, Xq, qb.qb_qlinear_bwd_ste(dY.to(DEV), Xq, CLIP, packed, h, 4, 8, want_dw=False)[0], None)
    check(dY, W_hat, Xq, None, qb.qb_qlinear_bwd_ste(dY.to(DEV), Xq, CLIP, packed, h, 4, 8, want_dx=False)[1])


# (T, N, K): N a multiple of 8 or of 64, T with and without rows beyond a multiple of 64, tiles of 128 x 96 and (the last
# three: dW alone has 256 CUs times 16 steps) 128 x 192, columns past the end of a tile.  One more column of dY makes its rows
# no multiple of 16 bytes, so that the operand is staged; the tiles and the steps of dW stay the same.  Of a dY that is not
# 16-byte aligned the operand is turned at any T.
@pytest.mark.parametrize("shape", [(65, 72, 64), (300, 136, 192), (640, 8, 128), (4099, 520, 1088), (4160, 520, 1088),
                                   (5500, 1000, 1088), (8200, 960, 768), (8256, 960, 768)])
def test_turned_operand_gives_the_staged_operands_sums(qb, shape):
    T, N, K = shape
    print("bwd turned", shape, flush=True)
    assert N % 128 != 0 and one_launch_teams(T, N, K, False, True) == 0
    dY = wl.grad_output_bf16(T, N + 1, seed=T + N).to(DEV)
    packed, h, _, _ = qb.qb_quantize_groupwise(wl.weight(N + 1, K, seed=N + K).to(DEV), 4, 1)
    Xq, _ = qb.qb_quantize_act(wl.activation(T, K, seed=T).to(DEV), CLIP)
    for last in (float("inf"), 0.0):  # rows past the last one are zeros, not the last one times zero
        dY[T - 1, 3] = last
        _, dW = qb.qb_qlinear_bwd_ste(dY[:, :N].contiguous(), Xq, CLIP, packed, h, 4, 1, want_dx=False)
        _, sW = qb.qb_qlinear_bwd_ste(dY, Xq, CLIP, packed, h, 4, 1, want_dx=False)
        _, mW = qb.qb_qlinear_bwd_ste(behind(dY[:, :N].contiguous(), 4), Xq, CLIP, packed, h, 4, 1, want_dx=False)
        assert torch.equal(dW, sW[:N]) and torch.equal(mW, sW[:N])
    ref = dY[:, :N].double().T @ ((2.0 * Xq.double() + 1.0) * (CLIP / 255.0))
    assert (dW.double() - ref).norm() <= 1e-5 * ref.norm()  # fp32 sums of exact products


# (T, N, K) and what calls for both products, dX alone and dW alone get: pieces of dW's tiles with two workgroups per CU (tiles of
# 128 x 192, sums of pieces exchanged, dX's whole tiles, some workgroups with more of them than others), 0 for the kernel of equal
# runs.  dW's tiles whole and in two to eight pieces; whole tiles only (8192 x 1024 x 1536), tiles with rows and columns past the end, T and N
# with and without a rest to a step; dY turned with N a multiple of 8 and not of 128, and staged, for both products and for dW alone
@pytest.mark.parametrize("bits", [3, 8])
@pytest.mark.parametrize("shape", [(2863, 1024, 4096, (1, 1, 0)), (5505, 768, 3072, (2, 1, 0)), (8192, 700, 704, (8, 0, 0)), (5505, 1016, 960, (6, 0, 0)),
                                   (4160, 1030, 4096, (1, 1, 0)), (12800, 512, 640, (8, 0, 0)), (8192, 1024, 1536, (4, 1, 4)), (8200, 1336, 1216, (3, 1, 4)),
                                   (8250, 1012, 1472, (3, 0, 4)), (9001, 504, 1728, (5, 0, 0))])
def test_two_workgroups_per_cu(qb, shape, bits):
    T, N, K, pieces = shape
    print("bwd two workgroups per CU", shape, bits, flush=True)
    assert (duo_pieces(T, N, K), duo_pieces(T, N, K, dw=False), duo_pieces(T, N, K, dx=False)) == pieces
    W, X, dY = wl.weight(N, K, seed=N + K + bits), wl.activation(T, K, seed=T), wl.grad_output_bf16(T, N, seed=T + N)
    G = 2
    Wd, Xd, dYd = W.to(DEV), X.to(DEV), dY.to(DEV)
    packed, h, m, _ = qb.qb_quantize_groupwise(Wd, bits, G)
    Xq, _ = qb.qb_quantize_act(Xd, CLIP)
    dX, dW = qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G)
    W_hat = oracle.dequantize_groupwise(qb.qb_unpack_codes(packed, N, K, bits).cpu().numpy(), h.cpu().numpy(), bits)
    check(dY, W_hat, Xq, dX, dW)
    # the same bits again, from inputs that lie elsewhere, into outputs that ask for single stores, and behind a clamp mask
    oX = behind(torch.empty(T, K, dtype=torch.bfloat16, device=DEV), 1)
    oW = behind(torch.empty(N, K, device=DEV), 1)
    qb.qb_qlinear_bwd_ste(behind(dYd, 4), Xq, CLIP, packed, h, bits, G, dX=oX, dW=oW)
    assert torch.equal(oX, dX) and torch.equal(oW, dW)
    mX, mW = qb.qb_qlinear_bwd_ste_masked(dYd, Xq, CLIP, packed, h, bits, G, X=2.0 * Xd, W=Wd, m=0.5 * m)
    out_x, out_w = (2.0 * Xd).abs() > CLIP, Wd.abs() > (0.5 * m).repeat_interleave(N // G)[:, None]
    assert bool(out_x.any()) and bool(out_w.any())
    assert torch.equal(mX, torch.where(out_x, torch.zeros_like(dX), dX)) and torch.equal(mW, torch.where(out_w, torch.zeros_like(dW), dW))
    check(dY, W_hat, Xq, qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G, want_dw=False)[0], None)
    dW = qb.qb_qlinear_bwd_ste(dYd, Xq, CLIP, packed, h, bits, G, want_dx=False)[1]
    check(dY, W_hat, Xq, None, dW)
    qb.qb_qlinear_bwd_ste(behind(dYd, 4), Xq, CLIP, packed, h, bits, G, dW=oW, want_dx=False)
    mW = qb.qb_qlinear_bwd_ste_masked(dYd, Xq, CLIP, packed, h, bits, G, X=2.0 * Xd, W=Wd, m=0.5 * m, want_dx=False)[1]
    assert torch.equal(oW, dW) and torch.equal(mW, torch.where(out_w, torch.zeros_like(dW), dW))


def test_two_workgroups_per_cu_on_three_streams(qb):
    """Calls whose workgroups wait for each other's sums and fill a CU's LDS, on three streams at once: each result is, bit for
    bit, that of the same call alone."""
    calls = []
    for T, N, K, dx, pieces in [(5505, 768, 3072, True, 2), (9001, 504, 1728, True, 5), (8200, 1336, 1216, False, 4)]:
        assert duo_pieces(T, N, K, dx) == pieces
        print("bwd two workgroups per CU, streams", T, N, K, flush=True)
        packed, h, _, _ = qb.qb_quantize_groupwise(wl.weight(N, K, seed=N).to(DEV), 4, 2)
        Xq, _ = qb.qb_quantize_act(wl.activation(T, K, seed=T).to(DEV), CLIP)
        out = {"dW": torch.empty(N, K, device=DEV)}
        if dx:
            out["dX"] = torch.empty(T, K, dtype=torch.bfloat16, device=DEV)
        args = dict(workspace=torch.empty(qb.qb_bwd_workspace_nbytes(T, N, K), dtype=torch.uint8, device=DEV), want_dx=dx, **out)
        call = functools.partial(qb.qb_qlinear_bwd_ste, wl.grad_output_bf16(T, N, seed=T + N).to(DEV), Xq, CLIP, packed, h, 4, 2, **args)
        call()
        calls.append((call, out, {n: o.clone() for n, o in out.items()}))
    streams = [torch.cuda.Stream() for _ in calls]  # default priority
    for _ in range(5):
        for _, out, _ in calls:
            for o in out.values():
                o.fill_(float("nan"))
        torch.cuda.synchronize()
        for (call, _, _), st in zip(calls, streams):
            with torch.cuda.stream(st):
                for _ in range(3):
                    call()
        torch.cuda.synchronize()
        for _, out, alone in calls:
            assert all(torch.equal(out[n], alone[n]) for n in out)


# 192 rows of a wide tile's second operand span more than 2^32 bytes: the tile's last columns come out as the others do
def test_rows_far_apart(qb):
    T, N, K = 12000000, 8, 192
    print("bwd rows far apart", T, N, K, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    Xq = torch.randint(-128, 128, (T, K), generator=g, device=DEV, dtype=torch.int8)
    dY = torch.randn(T, N, generator=g, device=DEV).to(torch.bfloat16)
    packed, h, _, _ = qb.qb_quantize_groupwise(wl.weight(N, K, seed=1).to(DEV), 4, 1)
    _, dW = qb.qb_qlinear_bwd_ste(dY, Xq, CLIP, packed, h, 4, 1, want_dx=False)
    ref = torch.zeros(N, K, dtype=torch.float64, device=DEV)
    for t in range(0, T, 1000000):
        ref += dY[t:t + 1000000].double().T @ ((2.0 * Xq[t:t + 1000000].double() + 1.0) * (CLIP / 255.0))
    # fp32 sums of exact products in 256 runs of up to 733 steps of 64: rounding errors add up like a random walk, 2^-24 * sqrt(733) of
    # partial sums as large as the result and smaller
    assert ((dW.double() - ref).norm(dim=0) <= 1e-5 * ref.norm(dim=0)).all()


# one launch, staged (turned where dY is not aligned), turned, neither
@pytest.mark.parametrize("shape", [(129, 128, 192), (16, 192, 64), (300, 136, 192), (320, 136, 192), (6001, 1024, 768), (77, 50, 64)])
@pytest.mark.parametrize("off_y,off_x,off_w", [(4, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 4), (3, 7, 12)])
def test_where_the_inputs_lie_does_not_change_a_bit(qb, shape, off_y, off_x, off_w):
    T, N, K = shape
    print("bwd alignment", shape, off_y, off_x, off_w, flush=True)
    dY = wl.grad_output_bf16(T, N, seed=T + N).to(DEV)
    Xq, _ = qb.qb_quantize_act(wl.activation(T, K, seed=T).to(DEV), CLIP)
    for bits in (3, 8):
        packed, h, _, _ = qb.qb_quantize_groupwise(wl.weight(N, K, seed=N + K).to(DEV), bits, 2)
        dX, dW = qb.qb_qlinear_bwd_ste(dY, Xq, CLIP, packed, h, bits, 2)
        aX, aW = qb.qb_qlinear_bwd_ste(behind(dY, off_y), behind(Xq, off_x), CLIP, behind(packed, off_w), h, bits, 2)
        assert torch.equal(aX, dX) and torch.equal(aW, dW)


@pytest.mark.parametrize("shape", [(65, 128, 64, 2), (577, 448, 192, 64)])
def test_one_launch_backward_asymmetric(qb, shape):
    T, N, K, G = shape
    bits = 4
    W = wl.weight(N, K, seed=N + K) + 0.05
    X = wl.activation(T, K, seed=T)
    dY = wl.grad_output_bf16(T, N, seed=T + N)
    packed, delta, q0, _ = qb.qb_quantize_groupwise_asym(W.to(DEV), bits, G)
    Xq, _ = qb.qb_quantize_act(X.to(DEV), CLIP)
    dX, dW = qb.qb_qlinear_bwd_ste_asym(dY.to(DEV), Xq, CLIP, packed, delta, q0, bits, G)
    torch.cuda.synchronize()
    oc, od, oq0, _ = oracle.quantize_groupwise_asym(W.numpy(), bits, G)
    oq, _ = oracle.quantize_act(X.numpy(), CLIP)
    rX = oracle.qlinear_bwd_dx_asym(wl.bf16_bits(dY), oc, od, oq0, openmp=True)
    _, rW = oracle.qlinear_bwd_ste(wl.bf16_bits(dY), oq, CLIP, oc, np.ones(G, np.float32), bits, want_dx=False, openmp=True)
    tX, tW = bounds(dY, oracle.dequantize_groupwise_asym(oc, od, oq0), oracle.dequantize_act(oq, CLIP))
    assert (np.abs(dX.float().cpu().numpy() - rX) <= 2.0 ** -8 * np.abs(rX) + tX).all()
    assert (np.abs(dW.cpu().numpy() - rW) <= tW).all()

"""The activation quantizers with a row in a wavefront's registers, at the edges of its registers and of the rows per wavefront, and the batched
call's runs of rows, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_05840_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CLIP = 6.0
SPECIAL = [0.0, -0.0, 6.0, -6.0, 6.0000005, -6.0000005, 100.0, -1e30, float("inf"), float("-inf")]


def rows(T, K, special=True):
    X = wl.activation(T, K, seed=T + K)
    if special:
        X[T // 2, :len(SPECIAL)] = torch.tensor(SPECIAL)
        X[T - 1, K - 1] = -6.5
    return X


# one to eight float4 a lane, full and with one lane in the last; a row a wavefront, two (the last wavefront with one) and three
@pytest.mark.parametrize("T,K", [(1, 64), (3, 256), (8193, 320), (5, 512), (16385, 64), (7, 768), (641, 768), (8192, 832), (642, 1024), (2049, 1088), (2051, 1472), (2050, 1792), (2049, 1984)])
def test_rows_in_registers(qb, T, K):
    X = rows(T, K)
    Xq, rs = qb.qb_quantize_act(X.to(DEV), CLIP)
    oq, ors = oracle.quantize_act(X.numpy(), CLIP)
    assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all()
    X = rows(T, K, special=False)
    X[T // 2, K - 1] = -37.0
    X[T - 1] = 0.0 if T > 3 else X[T - 1]
    X[0] = 1e-38
    Xq, rs, hx = qb.qb_quantize_act_dyn(X.to(DEV))
    oq, ors, ohx = oracle.quantize_act_dyn(X.numpy())
    assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all() and (hx.cpu().numpy().view(np.uint32) == ohx.view(np.uint32)).all()
    Xq, rs, hx, c = qb.qb_quantize_act_dyn_tensor(X.to(DEV))
    oq, ors = oracle.quantize_act(X.numpy(), float(X.abs().max()))
    assert float(c) == float(X.abs().max()) and (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all()


# (T, K) of a call's tensors: fewer rows than wavefronts, rows of one to four chunks whose runs end inside a tensor, at its last row and in the next one
@pytest.mark.parametrize("shapes", [[(1, 64)], [(5, 64), (3, 3072), (1, 1088), (2, 1024)], [(3001, 1088), (1, 3072), (4097, 320)], [(2000, 256)] * 3 + [(2000, 3136)],
                                    [(700, 64 * (i + 1)) for i in range(16)], [(100, 128)] * 19])
def test_batched_runs_of_rows(qb, shapes):
    Xs = [rows(T, K, special=K > 64) for T, K in shapes]
    got = qb.qb_quantize_act_batched([{"X": X.to(DEV), "clip": CLIP + i} for i, X in enumerate(Xs)])
    for i, (X, (Xq, rs)) in enumerate(zip(Xs, got)):
        oq, ors = oracle.quantize_act(X.numpy(), CLIP + i)
        assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all(), shapes[i]


# tensors whose rows go round the wavefronts one by one: all of one chunk, one row to a wavefront; few values in short rows and long ones; more rows than
# wavefronts and 3840 values and more to each, the last rows of a tensor and the first of the next one in the same round
@pytest.mark.parametrize("shapes", [[(7, 768), (8000, 64), (185, 1024)], [(5, 32768), (2, 64), (1, 1088)], [(300, 64), (41, 3072), (7, 1088)],
                                    [(13501, 1088), (1, 3072), (21001, 832), (1, 320)]])
def test_batched_rows_in_turn(qb, shapes):
    n, values = sum(T for T, _ in shapes), sum(T * K for T, K in shapes)
    assert n <= 8192 and (max(K for _, K in shapes) <= 1024 or values < 3 << 20) or n > 8192 and values >= 3840 * 8192
    Xs = [rows(T, K, special=K > 64) for T, K in shapes]
    got = qb.qb_quantize_act_batched([{"X": X.to(DEV), "clip": CLIP + i} for i, X in enumerate(Xs)])
    for i, (X, (Xq, rs)) in enumerate(zip(Xs, got)):
        oq, ors = oracle.quantize_act(X.numpy(), CLIP + i)
        assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all(), shapes[i]

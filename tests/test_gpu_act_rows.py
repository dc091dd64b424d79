"""The activation quantizers with a workgroup per row, at the edges of their rule (rows, columns) and of the row kernel (columns that
do not fill its threads, rows longer than its registers), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_1909_05840_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CLIP = 6.0


# (T, K): K just above and at 512, 1024, 2048, T at 640, 2048 and one beyond (a wavefront per row again); 64 and 128 columns past a
# multiple of 1024; rows of 4096 values fill the registers, 4160 and 32768 are loaded again
@pytest.mark.parametrize("shape", [(1, 576), (640, 576), (641, 576), (5, 512), (3, 1024), (2048, 1088), (2049, 1088), (7, 1152), (2, 1984),
                                   (2050, 2048), (17, 2112), (9, 4096), (33, 4160), (2, 32768)])
def test_rows_by_whole_workgroups(qb, shape):
    T, K = shape
    print("act rows", shape, flush=True)
    X = wl.activation(T, K, seed=T + K)
    X[0, :8] = torch.tensor([0.0, -0.0, 6.0, -6.0, 100.0, -100.0, float("inf"), float("-inf")])
    X[T - 1, K - 1] = -6.5
    Xq, rs = qb.qb_quantize_act(X.to(DEV), CLIP)
    oq, ors = oracle.quantize_act(X.numpy(), CLIP)
    assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all()
    X[0, 6:8] = 1.0
    X[T // 2, K - 1] = -37.0  # the range is the last thread's
    if T > 2:
        X[1] = 0.0
        X[2, :] = 1e-38
    Xq, rs, hx = qb.qb_quantize_act_dyn(X.to(DEV))
    oq, ors, ohx = oracle.quantize_act_dyn(X.numpy())
    assert (Xq.cpu().numpy() == oq).all() and (rs.cpu().numpy() == ors).all()
    assert (hx.cpu().numpy().view(np.uint32) == ohx.view(np.uint32)).all()


# more rows of 2048 values than a grid of workgroups covers (34 GB): the wavefronts that walk rows, against slices of the same rows
@pytest.mark.parametrize("per_token", [False, True])
def test_rows_beyond_a_grid(qb, per_token):
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    T, K, part = (1 << 22) + 3, 2048, 1 << 20
    g = torch.Generator(device="cuda").manual_seed(1)
    rows = torch.randn(part, K, generator=g, device="cuda") * 3
    X = torch.empty(T, K, device="cuda")
    for at in range(0, T, part):
        X[at:at + part] = rows[:min(part, T - at)]
    quantize = (lambda x: qb.qb_quantize_act_dyn(x)) if per_token else (lambda x: qb.qb_quantize_act(x, 6.0))
    want, got = quantize(rows), quantize(X)
    for at in range(0, T, part):
        n = min(part, T - at)
        for w, v in zip(want, got):
            assert torch.equal(v[at:at + n], w[:n]), at
    del X, got
    torch.cuda.empty_cache()

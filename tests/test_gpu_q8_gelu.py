"""The 8-bit output behind GELU takes quick steps where they cannot change a code: every code against the exact steps (erff,
true division), evaluated by torch on the same pre-activations, with pre-activations in GELU's flat tail, on the tie of zero,
wide ones, and ranges from far too small to far too large."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CLIP = 6.0


# (T, N, K): tiles of 128 x 96 with ragged edges, 128 x 128, two workgroups per CU
@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("shape", [(65, 72, 128), (300, 640, 256), (3000, 1152, 128)])
@pytest.mark.parametrize("shift,spread,clip_out", [(0.0, 1.0, 6.0), (-5.2, 0.3, 6.0), (-4.9, 0.05, 2.5), (-30.0, 10.0, 6.0), (0.0, 0.0, 1.0), (1.0, 40.0, 1e3),
                                                   (-4.0, 1.0, 1e-5), (-5.3, 0.2, 60.0)])
def test_gelu_codes_are_those_of_the_exact_steps(qb, bits, shape, shift, spread, clip_out):
    T, N, K = shape
    g = torch.Generator(device=DEV)
    g.manual_seed(T + N + bits)
    W = torch.randn(N, K, generator=g, device=DEV) * 0.04
    packed, h, _, rs_w = qb.qb_quantize_groupwise(W, bits, 8)
    Xq, rs_x = qb.qb_quantize_act(torch.randn(T, K, generator=g, device=DEV), CLIP)
    h = h * (spread / 0.5)  # (the pre-activations' deviation is about sqrt(128) * 0.04 = 0.5 without it)
    bias = torch.full((N,), shift, device=DEV)
    Yq, rs_y = qb.qb_qlinear_fwd_q8(Xq, rs_x, CLIP, packed, h, rs_w, bits, 8, N, clip_out, bias=bias, act=1)
    _, A4 = qb.qb_qlinear_fwd(Xq, rs_x, CLIP, packed, h, rs_w, bits, 8, N, want_a4=True)
    f = lambda x: torch.tensor(x, dtype=torch.float32, device=DEV)
    scale = (f(CLIP) / f(255.0)) * h.repeat_interleave(N // 8)[None, :]
    y = scale * A4.to(torch.float32) + bias[None, :]
    v = (f(0.5) * y) * (f(1.0) + torch.erf(y * f(0.70710678118654752)))
    c = f(clip_out)
    delta = f(2.0) * (c / f(255.0))
    code = torch.round((torch.maximum(torch.minimum(v, c), -c) + c) / delta)
    want = (code.to(torch.int32) - 128).to(torch.int8)
    assert torch.equal(Yq, want), int((Yq != want).sum())
    assert torch.equal(rs_y, Yq.to(torch.int32).sum(1, dtype=torch.int32))

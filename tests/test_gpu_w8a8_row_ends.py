"""The ends of the per-row W8A8 product's large tiles: rows of y that begin at whole words and that do not (odd N, or y one half into
an allocation), last columns and rows that do not fill a tile."""
import pytest
import torch

import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, rel_err, to_dev
from plan_util import w8a8_plan

pytestmark = pytest.mark.gpu

TOL = 2e-3  # exact integer sums, two products in binary32, the result's rounding to fp16 (2^-11)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("M,N", [(1279, 28670), (2030, 28666), (2030, 28669), (2048, 28672)])
def test_large_tiles(M, N, shift):
    K = 256
    assert w8a8_plan(M, N, K, True) == (0, 0)
    w = synth.weight(19, "ends/w/%d" % N, N, K, 0.05)
    x = synth.activations(19, "ends/x/%d" % M, M, K)
    wd, xd = to_dev(w), to_dev(x)
    cb, sb, zb = fq.fq_packed_sizes(N, K, 8, K)
    c, s, z = (torch.empty(n, dtype=t, device=DEV) for n, t in ((cb, torch.uint8), (sb // 4, torch.float32), (zb, torch.uint8)))
    fq.fq_quantize(wd, N, K, 8, K, c, s, z)
    layer = fq.Layer(N, K, K)
    layer.attach(8, c, s, z)
    xq = torch.empty(M, K, dtype=torch.int8, device=DEV)
    sx = torch.empty(M, dtype=torch.float32, device=DEV)
    xsum = torch.empty(K // 128, M, dtype=torch.int32, device=DEV)
    room = torch.full((M * N + 8,), float("nan"), dtype=torch.float16, device=DEV)
    y = room[shift:shift + M * N].view(M, N)
    fq.fq_quantize_act(xd, M, K, xq, sx, xsum)
    fq.fq_linear_w8a8(layer, xq, sx, xsum, M, y)
    torch.cuda.synchronize()
    # the same integers and scales in binary64
    q = c.view(N, K).double() - z.double().view(N, 1)
    ref = ((xq.double() @ q.t()) * s.double().view(1, N) * sx.double().view(M, 1)).cpu().numpy()
    assert rel_err(y.cpu().numpy(), ref) <= TOL
    assert rel_err(y[-5:, -67:].cpu().numpy(), ref[-5:, -67:]) <= TOL
    assert torch.isnan(room[:shift]).all() and torch.isnan(room[shift + M * N:]).all()

"""The quantizers that take a whole row's range -- activations per token, weights with one scale per row -- at the row
lengths where their register-held form changes and at numbers of rows around a run of eight, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu

LENGTHS = [128, 384, 2048, 2176, 4096, 4224, 8192, 8320, 16384, 16512, 32768, 32896]


@pytest.mark.parametrize("K", LENGTHS)
@pytest.mark.parametrize("M", [1, 7, 9, 24])
def test_activations(M, K):
    x = synth.activations(31, "rowq/%d/%d" % (M, K), M, K)
    x[M // 2, K - 1] = 3.0 * np.abs(x).max()       # the largest entry is the last vector's
    x[0, :] = 0
    xq = torch.full((M + 1, K), 77, dtype=torch.int8, device=DEV)
    sx = torch.full((M + 1,), 7.0, dtype=torch.float32, device=DEV)
    xsum = torch.full((K // 128 + 1, M), 7, dtype=torch.int32, device=DEV)
    fq.fq_quantize_act(to_dev(x), M, K, xq, sx, xsum)
    torch.cuda.synchronize()
    q_ref, s_ref = oracle.quantize_act(x)[:2]
    assert np.array_equal(xq[:M].cpu().numpy(), q_ref) and np.array_equal(sx[:M].cpu().numpy(), s_ref)
    assert np.array_equal(xsum[:-1].cpu().numpy(), q_ref.astype(np.int32).reshape(M, K // 128, 128).sum(2).T)
    assert (xq[M] == 77).all() and sx[M] == 7.0 and (xsum[-1] == 7).all()


@pytest.mark.parametrize("K", LENGTHS)
@pytest.mark.parametrize("sym", [False, True])
def test_weights_with_one_scale_per_row(K, sym):
    w = synth.weight(32, "rowq/w%d" % K, 5, K, 0.02, outlier_p=0.001)
    w[1, K - 1], w[2, 0], w[3, :] = 2.0, -2.0, 0
    codes = torch.full((6, K), 7, dtype=torch.uint8, device=DEV)
    scales = torch.full((6,), 7.0, dtype=torch.float32, device=DEV)
    zeros = torch.full((6,), 7, dtype=torch.uint8, device=DEV)
    (fq.fq_quantize_sym if sym else fq.fq_quantize)(to_dev(w), 5, K, 8, K, codes, scales, zeros)
    torch.cuda.synchronize()
    c_ref, s_ref, z_ref = (oracle.quantize_sym if sym else oracle.quantize)(w, 8, K)
    assert np.array_equal(codes[:5].cpu().numpy(), c_ref.reshape(5, K))
    assert np.array_equal(scales[:5].cpu().numpy(), s_ref.reshape(-1)) and np.array_equal(zeros[:5].cpu().numpy(), z_ref.reshape(-1))
    assert (codes[5] == 7).all() and scales[5] == 7.0 and zeros[5] == 7

"""The quantizers' shortened division (csrc/fq_div.h) where it could show: against the codes of Sec. 2.2 Eq. (2)
evaluated with one IEEE division per weight."""
import numpy as np
import pytest
import torch

import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_quantize, to_dev

pytestmark = pytest.mark.gpu


def _quantize_sym(w_dev, bits, group=128):
    N, K = w_dev.shape
    cb, sb, zb = fq.fq_packed_sizes(N, K, bits, group)
    c, s, z = (torch.empty(n, dtype=t, device=DEV) for n, t in ((cb, torch.uint8), (sb // 4, torch.float32), (zb, torch.uint8)))
    fq.fq_quantize_sym(w_dev, N, K, bits, group, c, s, z)
    return c.view(N, -1), s.view(N, -1), z.view(N, -1)


def _quantize_act(x):
    M, K = x.shape
    xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                    (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
    fq.fq_quantize_act(to_dev(x), M, K, xq, sx, xsum)
    return xq.cpu().numpy(), sx.cpu().numpy(), xsum.cpu().numpy()


@pytest.mark.parametrize("where", [np.inf, -np.inf])
def test_groups_that_hold_an_infinity(where):
    # The scale is infinite: finite entries divide to 0, the infinite one to NaN, which the clamp takes to the
    # lowest level.  (Unspecified by the interface; what a division gives.)
    rng = np.random.default_rng(3)
    w = rng.normal(0, 0.02, size=(3, 256)).astype(np.float16)
    w[1, 5] = where
    w[1, 133] = where
    w_dev = to_dev(w)
    for bits in (4, 8):
        c, s, z = (t.cpu().numpy() for t in _quantize_sym(w_dev, bits))
        codes = np.stack([c & 15, c >> 4], 2).reshape(3, 256) if bits == 4 else c
        want = np.full(256, 1 << (bits - 1), dtype=np.uint8)
        want[[5, 133]] = 1
        assert np.array_equal(codes[1], want) and np.all(np.isinf(s[1])) and np.isfinite(s[[0, 2]]).all()
        c, s, z = (t.cpu().numpy() for t in gpu_quantize(w_dev, bits))
        assert not c[1].any() and not z[1].any() and np.all(np.isinf(s[1]))
    c, s, _ = (t.cpu().numpy() for t in _quantize_sym(w_dev, 8, 256))
    want = np.full(256, 128, dtype=np.uint8)
    want[[5, 133]] = 1
    assert np.array_equal(c[1], want) and np.isinf(s[1, 0])
    xq, sx, xsum = _quantize_act(w)
    want = np.zeros(256, dtype=np.int8)
    want[[5, 133]] = -127
    assert np.array_equal(xq[1], want) and np.isinf(sx[1]) and list(xsum[:, 1]) == [-127, -127]
    out = torch.empty_like(w_dev)
    fq.fq_fake_quantize(w_dev, 3, 256, 3, 128, True, out)
    y = out.cpu().numpy()[1].astype(np.float32)
    assert np.isneginf(y[[5, 133]]).all() and np.isnan(np.delete(y, [5, 133])).all()

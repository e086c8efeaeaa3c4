"""The quantizers' shortened division (csrc/fq_div.h) where it could show: against the codes of Sec. 2.2 Eq. (2)
evaluated with one IEEE division per weight."""
import numpy as np
import pytest
import torch

import oracle
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


HALVES = np.arange(0x7C00, dtype=np.uint16).view(np.float16)  # 0 and every positive finite half, ascending


def _nearest_to_turnover(cand, s, z, count):
    """The `count` candidates whose quotient by s, plus z, lies closest to where the rounding to an integer turns over."""
    t = cand.astype(np.float64) / s + z
    return cand[np.argsort(np.abs(t - np.floor(t) - 0.5), kind="stable")[:count]]


def _symmetric_groups(bits):
    """A group for every third 11-bit largest magnitude, filled with the weights closest to a turnover."""
    lo = np.float16(1.0).view(np.uint16)
    w = np.empty((342, 128), dtype=np.float16)
    for m in range(342):
        amax = np.uint16(lo + min(3 * m + bits % 3, 1023)).view(np.float16)
        cand = HALVES[HALVES <= amax][-10 * 1024:]
        s = np.float64(np.float32(2) * np.float32(amax) / np.float32(2 ** bits - 2))
        near = _nearest_to_turnover(cand, s, 0.0, 127)
        w[m] = np.append(near * np.where(np.arange(len(near)) % 2, -1, 1).astype(np.float16), amax)
    return w


def _asymmetric_groups(bits, n=1024):
    rng = np.random.default_rng(bits)
    pos, neg = HALVES[(HALVES > 1e-4) & (HALVES < 8)], HALVES[(HALVES > 1e-4) & (HALVES < 8)]
    w = np.empty((n, 128), dtype=np.float16)
    for i in range(n):
        hi, lo = rng.choice(pos), -rng.choice(neg)
        if i % 8 == 0:
            lo = np.float16(0.0)
        s = np.float32(hi) - np.float32(lo)
        s = np.float64(s / np.float32(2 ** bits - 1))
        z = np.rint(-np.float64(lo) / s)
        cand = np.concatenate([rng.choice(HALVES[HALVES <= hi], 3000), -rng.choice(HALVES[HALVES <= -lo], 3000)])
        w[i] = np.append(_nearest_to_turnover(cand, s, z, 126), [lo, hi])
    return w


@pytest.mark.parametrize("bits", [2, 3, 4, 5, 6, 7, 8])
def test_codes_next_to_a_turnover(bits):
    for sym, w in ((True, _symmetric_groups(bits)), (False, _asymmetric_groups(bits))):
        w_dev = to_dev(w)
        if bits in (2, 3, 4, 8):
            c, s, z = (t.cpu().numpy() for t in (_quantize_sym if sym else gpu_quantize)(w_dev, bits))
            c_ref, s_ref, z_ref = (oracle.quantize_sym if sym else oracle.quantize)(w, bits)
            assert np.array_equal(c.reshape(c_ref.shape), c_ref) and np.array_equal(z.reshape(z_ref.shape), z_ref)
            assert np.array_equal(s.reshape(s_ref.shape).view(np.uint32), s_ref.view(np.uint32))
        out = torch.empty_like(w_dev)
        fq.fq_fake_quantize(w_dev, w.shape[0], 128, bits, 128, sym, out)
        assert np.array_equal(out.cpu().numpy().view(np.uint16), oracle.fake_quantize(w, bits, sym=sym).view(np.uint16))


@pytest.mark.parametrize("sym", [False, True])
def test_row_codes_of_every_half_of_a_range(sym):
    # one scale per row: every half between the row's ends
    rng = np.random.default_rng(8)
    ends = HALVES[(HALVES > 1e-3) & (HALVES < 64)]
    K, rows = 65536, 24
    w = np.zeros((rows, K), dtype=np.float16)
    for i in range(rows):
        hi, lo = rng.choice(ends), rng.choice(ends)
        every = np.concatenate([HALVES[HALVES <= hi], -HALVES[HALVES <= lo]])
        w[i, :len(every)] = every
    fn, ref = (fq.fq_quantize_sym, oracle.quantize_sym) if sym else (fq.fq_quantize, oracle.quantize)
    c, s, z = (torch.empty(n, dtype=t, device=DEV) for n, t in ((rows * K, torch.uint8), (rows, torch.float32), (rows, torch.uint8)))
    fn(to_dev(w), rows, K, 8, K, c, s, z)
    c_ref, s_ref, z_ref = ref(w, 8, K)
    assert np.array_equal(c.cpu().numpy().reshape(rows, K), c_ref) and np.array_equal(z.cpu().numpy(), z_ref.reshape(-1))
    assert np.array_equal(s.cpu().numpy().view(np.uint32), s_ref.reshape(-1).view(np.uint32))


def test_activation_codes_of_every_half():
    # every 11-bit largest magnitude, and with it every half down to 2^-10 of it, of both signs
    lo = int(np.float16(1.0).view(np.uint16))
    some = HALVES[lo - 10 * 1024:lo + 1024]
    x = np.concatenate([some, -some])[None, :].repeat(1024, 0)
    amax = HALVES[lo:lo + 1024][:, None]
    x = np.clip(x, -amax, amax)
    x[:, 0] = amax[:, 0]
    xq, sx, xsum = _quantize_act(x)
    s = (np.float32(2) * amax.astype(np.float32)) / np.float32(254)
    assert np.array_equal(sx.view(np.uint32), s[:, 0].view(np.uint32))
    for i in range(0, 1024, 128):
        want = np.rint(x[i:i + 128].astype(np.float32) / s[i:i + 128])  # one division per activation
        assert np.array_equal(xq[i:i + 128], want.astype(np.int8))
    assert np.array_equal(xsum, xq.reshape(1024, -1, 128).sum(2, dtype=np.int32).T)

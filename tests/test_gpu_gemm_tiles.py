"""Every instance of the matrix-core products at shapes that reach it: the tiles of fq_linear above 32 rows (csrc/fq_prompt.hip:
64, 96 and 128 tokens, one segment of K and several; csrc/fq_prefill.hip: whole and half tiles, scales one and
four groups at a time) and of fq_linear_w8a8 (csrc/fq_w8a8_prompt.hip: 64, 128 and 192
tokens; csrc/fq_w8a8.hip: 128 and 192 tokens, whole and half tiles with one scale per row).  Each case asks the
library's own rule that it does reach the instance; tokens and rows are ragged, numbers of groups odd and even.
Sampled rows over all tokens and sampled tokens over all rows, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_quantize, make_layer, rel_err, to_dev
from plan_util import part_bank, prompt_plan, w8a8_large_blocks, w8a8_plan

pytestmark = pytest.mark.gpu

# the operand is rounded to half twice, 2^-11 relative each, and the result once: 2e-3 of the largest output
TOL = 2e-3
CUS = 256


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _rows(N):
    """Rows at the edges of blocks of 32 and tiles of 128 and 256, first, in the middle and last."""
    at = [b + d for b in (0, 32, 128, 256, N // 512 * 256, (N - 1) // 256 * 256, (N - 1) // 32 * 32) for d in (-1, 0)]
    return sorted({r for r in at + [N // 3, N // 2 + 7, N - 1] if 0 <= r < N})


def _tokens(M):
    at = [b + d for b in (0, 32, 64, 96, 128, 192, 256, (M - 1) // 64 * 64) for d in (-1, 0)]
    return sorted({m for m in at + [M - 1] if 0 <= m < M})


def _weight(name, N, K, skew):
    w = synth.weight(17, name, N, K, 0.02, outlier_p=0.001)
    if skew:  # most of a group on one side: zero points far from the middle, a different one for every other row
        w[::2] += np.float16(0.03)
        w[1::2] -= np.float16(0.02)
    return w


def _check(y, M, N, ref):
    """ref(tokens, row0, rows): the oracle's outputs."""
    assert np.isfinite(y.astype(np.float32)).all()
    everyone = np.arange(M)
    for n in _rows(N):
        assert rel_err(y[:, n:n + 1], ref(everyone, n, 1)) <= TOL, n
    tokens = _tokens(M)
    got, want = y[tokens], ref(np.array(tokens), 0, N)
    for i, m in enumerate(tokens):
        assert rel_err(got[i:i + 1], want[i:i + 1]) <= TOL, m


def _linear_case(name, bits, M, N, K, scale=None):
    w = _weight(name + "/w", N, K, bits != 16)
    if scale is not None:
        w = (w.astype(np.float32) * scale(np.arange(N)[:, None], np.arange(K)[None, :])).astype(np.float16)
    x = synth.activations(17, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    x_dev = to_dev(x)
    ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2)]
    for y in ys:
        fq.fq_linear(layer, bits, x_dev, M, y)
    torch.cuda.synchronize()
    assert torch.equal(ys[0], ys[1])
    host = None if bits == 16 else [t.cpu().numpy() for t in packed[bits]]

    def ref(tokens, row0, rows):
        if bits == 16:
            return oracle.linear(x[tokens], w, None, None, 16, row0=row0, rows=rows)
        return oracle.linear(x[tokens], *host, bits, row0=row0, rows=rows)
    return ys[0].cpu().numpy(), ref


PROMPT = ([(b, 3, 1, 65, 18001, 640) for b in (2, 4, 8)] + [(16, 3, 1, 65, 9001, 640)] +
          [(b, 4, 1, 97, 18001, 1280) for b in (2, 4, 8, 16)] +
          [(2, 3, 12, 65, 129, 1536), (4, 3, 15, 65, 129, 1920), (8, 3, 13, 65, 129, 1664), (16, 3, 8, 65, 385, 1024)] +
          [(2, 4, 5, 193, 3001, 5760), (4, 4, 5, 97, 6001, 5760), (8, 4, 5, 193, 3001, 5760), (16, 4, 7, 600, 385, 2688)])


@pytest.mark.parametrize("bits,mt,segments,M,N,K", PROMPT)
def test_prompt_tiles(bits, mt, segments, M, N, K):
    if _cus() == CUS:
        assert prompt_plan(M, N, K, bits) == (mt, segments)
    y, ref = _linear_case("tiles/%d/%dx%dx%d" % (bits, M, N, K), bits, M, N, K)
    _check(y, M, N, ref)


# rounds of whole tiles with half tiles behind them, half tiles alone, whole tiles alone; K / 128 a multiple of 4 or not
LARGE = [(515, 25001, 384), (193, 18001, 2048), (385, 18001, 512), (515, 28641, 2176)]


@pytest.mark.parametrize("bits", [2, 4, 8, 16])
@pytest.mark.parametrize("M,N,K", LARGE)
def test_large_tiles(M, N, K, bits):
    if _cus() == CUS:
        assert prompt_plan(M, N, K, bits) == (0, 0)
    y, ref = _linear_case("large/%d/%dx%dx%d" % (bits, M, N, K), bits, M, N, K)
    _check(y, M, N, ref)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("M,N,K", [(385, 18001, 512), (193, 18001, 2048)])
def test_large_tiles_small_and_uneven_magnitudes(M, N, K, bits):
    # the operand carries the group's scale as a half: scales below the normal range of a half, rows 2^-20 apart
    # in magnitude in one tile, groups of a row apart too; every row against its own magnitude
    y, ref = _linear_case("uneven/%d/%d" % (bits, K), bits, M, N, K,
                          lambda n, k: 0.01 * 2.0 ** (-6.0 * (n % 3 == 1) + 5.0 * (n % 3 == 2) - 3.0 * (k >= K // 2)))
    everyone = np.arange(M)
    for n in _rows(N):
        assert rel_err(y[:, n:n + 1], ref(everyone, n, 1)) <= TOL, n


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("M,N,K", [(385, 18001, 512), (193, 18001, 2048)])
def test_large_tiles_integer_case_exact(M, N, K, bits):
    # integer weights whose groups span 0 .. 2^bits - 1 (s = 1) and small integer activations: the integer matrix
    # product, exact in binary16
    rng = np.random.default_rng(bits)
    w = rng.integers(0, 3, size=(N, K)).astype(np.int8 if bits < 8 else np.int16)
    w[:, 0::128] = 0
    w[:, 1::128] = 2 ** bits - 1
    x = rng.integers(-1, 2, size=(M, K)) * (rng.random((M, K)) < 0.25)
    x[:, 1::128] = 0
    layer, packed = make_layer(w.astype(np.float16), (bits,))
    assert torch.all(packed[bits][1] == 1.0) and torch.all(packed[bits][2] == 0)
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV)
    fq.fq_linear(layer, bits, to_dev(x.astype(np.float16)), M, y)
    expect = to_dev(x.astype(np.float32)) @ to_dev(w.astype(np.float32)).t()  # integers far below 2^24: exact
    assert expect.abs().max().item() <= 2048
    assert torch.equal(y.float(), expect)


def _w8a8_case(name, per_row, M, N, K, reps=2):
    group = K if per_row else 128
    w = _weight(name + "/w", N, K, True)
    x = synth.activations(17, name + "/x", M, K)
    x = np.abs(x) * np.where(np.arange(M) % 3 == 0, 1, 0.25).astype(np.float16)[:, None]  # group sums far from 0
    layer, packed = make_layer(w, (8,), group)
    xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                    (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
    fq.fq_quantize_act(to_dev(x), M, K, xq, sx, xsum)
    ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV) for _ in range(reps)]
    for y in ys:
        fq.fq_linear_w8a8(layer, xq, sx, xsum, M, y)
    torch.cuda.synchronize()
    assert all(torch.equal(y, ys[0]) for y in ys)
    c, s, z = (t.cpu().numpy() for t in packed[8])
    q, sc = xq.cpu().numpy(), sx.cpu().numpy()
    return ys[0].cpu().numpy(), lambda tokens, row0, rows: oracle.linear_w8a8(q[tokens], sc[tokens], c, s, z, group, row0=row0,
                                                                              rows=rows)


W8A8 = [(False, 2, 1, 65, 18001, 640), (False, 2, 1, 65, 18001, 1280), (False, 2, 7, 65, 4097, 11648), (False, 2, 7, 65, 4097, 12800),
        (False, 3, 1, 150, 18001, 640), (False, 3, 1, 150, 18001, 1280), (False, 3, 3, 129, 6001, 8064),
        (False, 3, 3, 129, 6001, 11008),
        (True, 2, 1, 65, 18001, 640), (True, 2, 1, 65, 18001, 1280), (True, 2, 4, 65, 6001, 5504),
        (True, 3, 1, 150, 13001, 640), (True, 3, 1, 150, 13001, 1280), (True, 3, 3, 129, 6001, 6656), (True, 3, 5, 129, 4097, 8064)]


@pytest.mark.parametrize("per_row,tm,segments,M,N,K", W8A8)
def test_w8a8_prompt_tiles(per_row, tm, segments, M, N, K):
    if _cus() == CUS:
        assert w8a8_plan(M, N, K, per_row) == (tm, segments)
    y, ref = _w8a8_case("w8/%d/%dx%dx%d" % (per_row, M, N, K), per_row, M, N, K)
    _check(y, M, N, ref)


@pytest.mark.parametrize("per_row,blocks,M,N,K", [(False, 2, 193, 18001, 384), (False, 2, 400, 28641, 1280), (False, 3, 257, 25001, 384),
                                                  (False, 3, 1153, 15001, 1280), (True, 0, 1000, 18001, 256), (True, 0, 385, 25001, 384),
                                                  (True, 0, 193, 18001, 256)])
def test_w8a8_large_tiles(per_row, blocks, M, N, K):
    if _cus() == CUS:
        assert w8a8_plan(M, N, K, per_row) == (0, 0) and (per_row or w8a8_large_blocks(M, N) == blocks)
    y, ref = _w8a8_case("w8large/%d/%dx%dx%d" % (per_row, M, N, K), per_row, M, N, K)
    _check(y, M, N, ref)


@pytest.mark.parametrize("kind,M,N,K", [(2, 193, 3001, 5760), (4, 97, 6001, 5760), (8, 193, 3001, 5760), (16, 600, 385, 2688),
                                        ("group", 65, 4097, 11648), ("group", 129, 6001, 8064), ("group", 33, 300, 1408),
                                        ("row", 65, 6001, 5504), ("row", 129, 4097, 8064), ("row", 33, 300, 2816)])
def test_same_bits_with_and_without_partial_sums(kind, M, N, K):
    """A stream with an array for the segments' sums, streams without one and captured calls: the same bits."""
    if _cus() == CUS:
        assert (prompt_plan(M, N, K, kind) if isinstance(kind, int) else w8a8_plan(M, N, K, kind == "row"))[1] > 1
    name = "bits/%s/%dx%dx%d" % (kind, M, N, K)
    w, x = _weight(name + "/w", N, K, kind != 16), to_dev(synth.activations(17, name + "/x", M, K))
    layer, _ = make_layer(w, (kind if isinstance(kind, int) else 8,), K if kind == "row" else 128)
    if isinstance(kind, int):
        def call(y, **stream):
            fq.fq_linear(layer, kind, x, M, y, **stream)
    else:
        xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                        (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
        fq.fq_quantize_act(x, M, K, xq, sx, xsum)

        def call(y, **stream):
            fq.fq_linear_w8a8(layer, xq, sx, xsum, M, y, **stream)
    want, y = (torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV) for _ in range(2))
    assert part_bank(torch.cuda.current_stream().cuda_stream) >= 0
    call(want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(6)]
    without = [s for s in streams if part_bank(s.cuda_stream) < 0]
    assert without
    for s in streams[:1] + without[:2]:
        y.fill_(float("nan"))
        torch.cuda.synchronize()
        call(y, stream=s)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(y)
    for _ in range(3):
        y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


@pytest.mark.parametrize("M,N,K", [(300, 5120, 13824), (200, 11008, 4096), (700, 5120, 5120), (33, 1000, 4096), (150, 18001, 1280)])
def test_w8a8_sums_of_groups_with_outliers(M, N, K):
    # Groups with an outlier have their zero point off the middle: what the codes (less 128) and what the zero points bring
    # are both large there and cancel, group by group.  Each is added to the result's sum with one rounding, the zero
    # points' factor s (128 - z) is rounded once: errors of rms 2^-23 / sqrt(12) of what is rounded, independent of each
    # other.  Their rms is worked out for every result from the sums in binary64, and of some million results none
    # may be off by more than six times that beyond its rounding to fp16.
    g = torch.Generator(device=DEV).manual_seed(5)
    w = torch.randn(N, K, generator=g, dtype=torch.float16, device=DEV) * K ** -0.5
    w.view(-1)[torch.randint(0, N * K, (N * K // 1000,), generator=g, device=DEV)] *= 20.0
    x = torch.randn(M, K, generator=g, dtype=torch.float16, device=DEV)
    codes, scales, zeros = gpu_quantize(w, 8)
    layer = fq.Layer(N, K)
    layer.attach(8, codes, scales, zeros)
    xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                    (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
    y = torch.empty((M, N), dtype=torch.float16, device=DEV)
    fq.fq_quantize_act(x, M, K, xq, sx, xsum)
    fq.fq_linear_w8a8(layer, xq, sx, xsum, M, y)
    total = torch.zeros(M, N, dtype=torch.float64, device=DEV)
    var = torch.zeros_like(total)
    q, xd = codes.view(N, K).double() - 128, xq.double()
    for i in range(K // 128):
        k = slice(128 * i, 128 * i + 128)
        scale = scales[:, i].double()
        total += (xd[:, k] @ q[:, k].t()) * scale
        var += total ** 2
        part = xsum[i].double().unsqueeze(1) * (scale * (128 - zeros[:, i].double()))
        total += part
        var += total ** 2 + part ** 2
    exact = total * sx.double().unsqueeze(1)
    rms = var.sqrt() * (2.0 ** -23 / 12 ** 0.5) * sx.double().unsqueeze(1)
    ulp = 2.0 ** (torch.floor(torch.log2(exact.abs().clamp_min(2.0 ** -14))) - 10)
    assert (((y.double() - exact).abs() - ulp / 2) / rms).max().item() <= 6.0

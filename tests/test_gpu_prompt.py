"""fq_linear for prompts of some tens to some hundreds of rows (csrc/fq_prompt.hip): tokens at the edges of
its blocks of 32 and of its tiles, rows at the edges of 128, one to many groups of K (its scales come
eight groups at a time, its steps three to a turn), one and several segments of K, against the oracle; and
that the result is the same bits wherever the partial sums of the segments are kept.  The same for the W8A8
product (csrc/fq_w8a8_prompt.hip) with groups of 128 and with one scale per row.  Few rows: most shapes here take
the smallest tiles, 64 tokens; the others are in test_gpu_gemm_tiles.py."""
import ctypes
import threading

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_linear, make_layer, rel_err, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(33, 127, 128), (64, 129, 256), (65, 1, 1152), (96, 640, 2176), (97, 300, 1024), (128, 512, 8192),
          (129, 257, 1280), (200, 384, 4224), (333, 1000, 2048), (40, 2048, 5504)]


@pytest.mark.parametrize("bits", [2, 4, 8, 16])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_prompt_matches_oracle(M, N, K, bits):
    name = "prompt/%dx%dx%d" % (M, N, K)
    w = synth.weight(11, name + "/w", N, K, 0.02, outlier_p=0.001)
    w[N // 2, :128] = 0.0  # an all-zero group: scale 1
    x = synth.activations(11, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    y = gpu_linear(layer, bits, x)
    if bits == 16:
        ref = oracle.linear(x, w, None, None, 16)
    else:
        c, s, z = (t.cpu().numpy() for t in packed[bits])
        ref = oracle.linear(x, c, s, z, bits)
    assert np.isfinite(y.astype(np.float32)).all()
    # the operand is rounded to half twice, 2^-11 relative each (csrc/fq_prefill.hip): 2e-3 of the largest output
    assert rel_err(y, ref) <= 2e-3


@pytest.mark.parametrize("per_row", [False, True])
@pytest.mark.parametrize("M,N,K", SHAPES + [(1, 640, 1152), (192, 384, 2816), (193, 128, 896)])
def test_w8a8_prompt_matches_oracle(M, N, K, per_row):
    name = "prompt8/%dx%dx%d" % (M, N, K)
    group = K if per_row else 128
    w = synth.weight(12, name + "/w", N, K, 0.02, outlier_p=0.001)
    x = synth.activations(12, name + "/x", M, K)
    layer, packed = make_layer(w, (8,), group)
    xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                    (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
    y = torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV)
    fq.fq_quantize_act(to_dev(x), M, K, xq, sx, xsum)
    fq.fq_linear_w8a8(layer, xq, sx, xsum, M, y)
    torch.cuda.synchronize()
    c, s, z = (t.cpu().numpy() for t in packed[8])
    ref = oracle.linear_w8a8(xq.cpu().numpy(), sx.cpu().numpy(), c.reshape(N, K), s.reshape(N, -1), z.reshape(N, -1), group)
    # exact integers inside a group, binary32 sums of groups: the rounding of the result to fp16, 2^-11, and the
    # W8A8 tests' bound of 2e-3
    assert rel_err(y.cpu().numpy(), ref) <= 2e-3


def test_same_bits_with_and_without_partial_sums():
    """The default stream and some others own an array for the segments' sums; further streams and
    captured calls add the segments inside one workgroup, in the same order."""
    M, N, K = 100, 512, 8192
    layer, _ = make_layer(synth.weight(11, "prompt/banks/w", N, K, 0.02), (4,))
    x = to_dev(synth.activations(11, "prompt/banks/x", M, K))
    want = torch.empty((M, N), dtype=torch.float16, device=DEV)
    fq.fq_linear(layer, 4, x, M, want)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(6)]
    ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV) for _ in streams]
    for _ in range(4):  # overlapping calls
        for st, y in zip(streams, ys):
            fq.fq_linear(layer, 4, x, M, y, stream=st)
    torch.cuda.synchronize()
    for y in ys:
        assert torch.equal(y, want)
    graph, y = torch.cuda.CUDAGraph(), torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV)
    with torch.cuda.graph(graph):
        fq.fq_linear(layer, 4, x, M, y)
    for _ in range(3):
        y.fill_(float("nan"))
        graph.replay()
        fq.fq_linear(layer, 4, x, M, ys[0])
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(ys[0], want)


def test_threads_on_one_stream():
    """Two host threads, one stream, products split along K: each thread's parts are added before the other's
    product overwrites them."""
    N, K, reps = 512, 8192, 60
    jobs = []
    for j, M in enumerate((100, 64)):
        layer, _ = make_layer(synth.weight(11, "prompt/threads/w%d" % j, N, K, 0.02), (4,))
        x = to_dev(synth.activations(11, "prompt/threads/x%d" % j, M, K))
        want = torch.empty((M, N), dtype=torch.float16, device=DEV)
        fq.fq_linear(layer, 4, x, M, want)
        jobs.append((layer, x, M, want, [torch.empty_like(want) for _ in range(reps)]))
    torch.cuda.synchronize()
    stream = torch.cuda.current_stream().cuda_stream

    def work(layer, x, M, want, ys):
        for y in ys:
            fq.fq_linear(layer, 4, x, M, y, stream=stream)

    threads = [threading.Thread(target=work, args=job) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for _, _, _, want, ys in jobs:
        assert all(torch.equal(y, want) for y in ys)


def test_null_stream_beside_a_captured_blocking_stream():
    """While a stream that synchronizes with the null stream is being captured, the runtime answers no question
    about the null stream, but takes launches on it: the calls run, without partial sums in memory."""
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL([line.split()[-1] for line in f if "libamdhip64" in line][0])
    M, N, K = 100, 512, 8192
    layer, _ = make_layer(synth.weight(11, "prompt/null/w", N, K, 0.02), (4, 8))
    x = to_dev(synth.activations(11, "prompt/null/x", M, K))
    xq, sx, xsum = (torch.empty(s, dtype=t, device=DEV) for s, t in
                    (((M, K), torch.int8), ((M,), torch.float32), ((K // 128, M), torch.int32)))
    fq.fq_quantize_act(x, M, K, xq, sx, xsum, stream=0)
    want, y = (torch.empty((2, M, N), dtype=torch.float16, device=DEV) for _ in range(2))

    def calls(out):
        fq.fq_linear(layer, 4, x, M, out[0], stream=0)
        fq.fq_linear_w8a8(layer, xq, sx, xsum, M, out[1], stream=0)

    calls(want)
    torch.cuda.synchronize()
    stream, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(stream), 0) == 0  # 0: blocking
    try:
        assert hip.hipStreamBeginCapture(stream, 2) == 0               # 2: relaxed
        try:
            calls(y)
        finally:
            assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    finally:
        assert hip.hipStreamDestroy(stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(y, want)

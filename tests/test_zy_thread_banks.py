"""hipStreamPerThread is one handle for as many streams as there are threads: every thread has a copy of the static scratch of its
own (few rows of entropy, the output layer), distinct from the copies of streams, and threads beyond the copies get the same
results without.  (Uses up the process's copies for threads, which no other file uses.)"""
import threading

import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, to_dev
from plan_util import stream_bank

pytestmark = pytest.mark.gpu

PER_THREAD = 2  # hipStreamPerThread


def _in_threads(n, fn):
    out, errors = [None] * n, []

    def go(i):
        try:
            out[i] = fn(i)
        except Exception as e:  # noqa: BLE001 (shown below)
            errors.append(e)
    threads = [threading.Thread(target=go, args=(i,)) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    return out


def test_threads_share_no_copy():
    torch.cuda.synchronize()
    streams = [stream_bank(torch.cuda.current_stream().cuda_stream)]
    mine = stream_bank(PER_THREAD)
    assert mine >= fq.FQ_SCRATCH_BANKS and stream_bank(PER_THREAD) == mine
    got = _in_threads(4, lambda i: (torch.cuda.set_device(0), stream_bank(PER_THREAD), stream_bank(PER_THREAD)))
    assert all(a == b >= fq.FQ_SCRATCH_BANKS for _, a, b in got)
    assert len({a for _, a, _ in got} | {mine} | set(streams)) == 6


def test_calls_of_many_threads():
    # more threads than copies, all on hipStreamPerThread at once; 1e-4 is the bound the entropies are held to everywhere
    n, R, V, K, M, Vh = 20, 5, 32000, 1024, 2, 5000
    a, b = synth.logits_pair(6, "threads/ent", R, V)
    H_ref, KL_ref = oracle.entropy_kl(a, b)
    w, x = synth.weight(6, "threads/w", Vh, K, 0.03), synth.activations(6, "threads/x", M, K)
    logits_ref = x.astype(np.float64) @ w.astype(np.float64).T
    e = np.exp(logits_ref - logits_ref.max(1, keepdims=True))
    p = e / e.sum(1, keepdims=True)
    HL_ref, AM_ref = -(p * np.log(p)).sum(1), logits_ref.argmax(1)
    # each thread's rows are shifted by one, so that another's partial results show
    rolls = [np.roll(np.arange(R), i) for i in range(n)]
    da, db, dw, dx = [to_dev(a[r]) for r in rolls], [to_dev(b[r]) for r in rolls], to_dev(w), [to_dev(np.roll(x, i, 0)) for i in range(n)]
    outs = [(torch.zeros(R, device=DEV), torch.zeros(R, device=DEV), torch.zeros(M, device=DEV),
             torch.zeros(M, dtype=torch.int32, device=DEV)) for _ in range(n)]
    torch.cuda.synchronize()

    def calls(i):
        torch.cuda.set_device(0)
        H, KL, HL, AM = outs[i]
        for _ in range(8):
            fq.fq_entropy_kl(da[i], db[i], R, V, H, KL, stream=PER_THREAD)
            fq.fq_lm_head_entropy(dx[i], dw, M, Vh, K, None, HL, AM, stream=PER_THREAD)
        torch.cuda.synchronize()
        return stream_bank(PER_THREAD)
    banks = _in_threads(n, calls)
    torch.cuda.synchronize()
    given = [k for k in banks if k >= 0]
    assert len(given) == len(set(given)) and -1 in banks
    for i, r in enumerate(rolls):
        H, KL, HL, AM = (t.cpu().numpy() for t in outs[i])
        assert np.all(np.abs(H - H_ref[r]) <= 1e-4 * np.abs(H_ref[r]) + 1e-7), (i, banks[i])
        assert np.all(np.abs(KL - KL_ref[r]) <= 1e-4 * np.abs(KL_ref[r]) + 1e-7), (i, banks[i])
        assert np.all(np.abs(HL - np.roll(HL_ref, i)) <= 1e-4 * np.abs(np.roll(HL_ref, i))), (i, banks[i])
        assert np.array_equal(AM, np.roll(AM_ref, i)), (i, banks[i])

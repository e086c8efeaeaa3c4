"""Entropy and KL at the sizes where rows change from whole workgroups to pieces that meet in scratch (64 | 65, 160 | 161,
256 | 257, 350 | 351, 512 | 513 rows; 4096 | 4097, 10240 | 10241 and 65535 | 65536 entries) and where a lane's last round is partly
empty, against the oracle; and calls of more rows than 64 that overlap on more streams than have scratch, and under capture."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, to_dev

pytestmark = pytest.mark.gpu


def _inputs(tag, R, V, half):
    # a few distinct rows, repeated: what is tested does not depend on a row's neighbours
    a, b = synth.logits_pair(5, "rows/%s" % tag, min(R, 7), V)
    if half:
        a, b = a.astype(np.float16), b.astype(np.float16)
    H, KL = oracle.entropy_kl(a.astype(np.float32), b.astype(np.float32))
    i = np.arange(R) % a.shape[0]
    ti = torch.from_numpy(i).to(DEV)
    return to_dev(a).index_select(0, ti), to_dev(b).index_select(0, ti), H[i], KL[i]


def _close(got, ref):
    # the bound the entry points are held to everywhere: 1e-4 of the value
    return np.all(np.abs(got.cpu().numpy() - ref) <= 1e-4 * np.abs(ref) + 1e-7)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("R,V", [(1, 4096), (65, 4097), (1, 10240), (65, 10240), (1, 10241), (3, 10244), (9, 32000), (21, 32001), (64, 32000), (65, 32000), (64, 65536),
                                 (65, 65536), (160, 12291), (161, 12292), (256, 65535), (257, 65536), (350, 11264), (351, 11265),
                                 (512, 10248), (513, 10248), (1, 3), (2, 1023), (5, 4097), (2, 33792)])
def test_rows_and_pieces(R, V, half):
    a, b, H_ref, KL_ref = _inputs("%d/%d" % (R, V), R, V, half)
    H = torch.full((R,), float("nan"), device=DEV)
    KL = torch.full((R,), float("nan"), device=DEV)
    call = fq.fq_entropy_kl_f16 if half else fq.fq_entropy_kl
    for _ in range(2):  # the second call finds the tickets as the first left them
        call(a, b, R, V, H, KL)
        assert _close(H, H_ref) and _close(KL, KL_ref)
        H.fill_(float("nan"))
        KL.fill_(float("nan"))
    call(a, None, R, V, H, None)
    assert _close(H, H_ref)


@pytest.mark.parametrize("value", [-np.inf, np.finfo(np.float32).min])
@pytest.mark.parametrize("R,V", [(2, 32001), (30, 32000), (3, 4096), (100, 32000), (520, 12000)])
def test_masked_entries_carry_no_mass(R, V, value):
    # every third entry, and the first half of the row: lanes that have seen nothing else when they meet their first logit
    a, b, _, _ = _inputs("mask", R, V, False)
    for t in (a, b):
        t[:, 7::3] = float(value)
        t[:, :V // 2] = float(value)
    H_ref, KL_ref = oracle.entropy_kl(a[:7].cpu().numpy(), b[:7].cpu().numpy())
    i = np.arange(R) % min(R, 7)
    H = torch.zeros(R, device=DEV)
    KL = torch.zeros(R, device=DEV)
    fq.fq_entropy_kl(a, b, R, V, H, KL)
    assert _close(H, H_ref[i]) and _close(KL, KL_ref[i])


def test_overlapping_streams_and_capture():
    R, V, n = 100, 20000, 11  # more streams than have scratch for so many rows
    sets = [_inputs("streams/%d" % s, R, V, False) for s in range(n)]
    H = [torch.full((4, R), float("nan"), device=DEV) for _ in range(n)]
    KL = [torch.full((4, R), float("nan"), device=DEV) for _ in range(n)]
    streams = [torch.cuda.Stream() for _ in range(n)]
    torch.cuda.synchronize()
    for i in range(4):
        for s in range(n):
            fq.fq_entropy_kl(sets[s][0], sets[s][1], R, V, H[s][i], KL[s][i], stream=streams[s])
    torch.cuda.synchronize()
    for s in range(n):
        for i in range(4):
            assert _close(H[s][i], sets[s][2]) and _close(KL[s][i], sets[s][3]), (s, i)
            assert torch.equal(H[s][i], H[s][0]) and torch.equal(KL[s][i], KL[s][0]), (s, i)
    Hg = torch.full((R,), float("nan"), device=DEV)
    KLg = torch.full((R,), float("nan"), device=DEV)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fq.fq_entropy_kl(sets[0][0], sets[0][1], R, V, Hg, KLg)
    for _ in range(3):
        Hg.fill_(float("nan"))
        KLg.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert _close(Hg, sets[0][2]) and _close(KLg, sets[0][3])


@pytest.mark.parametrize("V", [2 ** 31 - 1001, 2 ** 31 - 1, 2 ** 31 - 4])
def test_a_row_of_nearly_two_to_the_31_entries(V):
    # uniform, so that the sums are whole numbers: the entropy is ln V in binary32 (a lost piece of 32 would show at 1.5e-3)
    a = torch.zeros(V, dtype=torch.float16, device=DEV)
    H = torch.full((1,), float("nan"), device=DEV)
    fq.fq_entropy_kl_f16(a, None, 1, V, H, None)
    assert abs(H.item() - np.log(V)) <= 2e-7 * np.log(V)


@pytest.mark.parametrize("R,V,half", [(65, 12000, False), (160, 32001, True), (384, 20002, False), (65, 65536, False), (100, 65537, False),
                                      (128, 70000, True), (256, 65540, True), (300, 66001, False), (512, 65544, True), (450, 65545, False)])
@pytest.mark.parametrize("kl", [True, False])
def test_the_same_bits_with_and_without_scratch(R, V, half, kl):
    # the current stream has a copy of the scratch; hipStreamPerThread (2) and a captured call have none
    a, b, H_ref, KL_ref = _inputs("bits/%d" % V, R, V, half)
    call = fq.fq_entropy_kl_f16 if half else fq.fq_entropy_kl
    out = [[torch.full((R,), float("nan"), device=DEV), torch.full((R,), float("nan"), device=DEV) if kl else None] for _ in range(3)]
    torch.cuda.synchronize()
    call(a, b if kl else None, R, V, *out[0])
    call(a, b if kl else None, R, V, *out[1], stream=2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(a, b if kl else None, R, V, *out[2])
    graph.replay()
    torch.cuda.synchronize()
    assert _close(out[0][0], H_ref) and (not kl or _close(out[0][1], KL_ref))
    for i in (1, 2):
        assert torch.equal(out[0][0], out[i][0]) and (not kl or torch.equal(out[0][1], out[i][1])), i

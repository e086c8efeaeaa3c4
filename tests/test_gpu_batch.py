"""The small-batch kernel of single calls and stage-sized plans (csrc/fq_batch.hip) at its edges, and what its rules
leave to the register-fed kernel (csrc/fq_skinny.hip) at 4, 8 and 16 bits: rows around its
tiles of 16, batch rows around 16, inputs of one group, an odd number of groups, and more than one
panel of x in LDS (4096 inputs up to 16 batch rows, 2048 above), runs longer than the six tiles a workgroup
holds at a time, entries that share x and entries that do not, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_linear, make_layer, rel_err, to_dev
from plan_util import batch_serves, batch_serves_linear

pytestmark = pytest.mark.gpu

TOL = 2e-3  # exact integers times fp16 in binary32: what shows is the result's rounding to fp16, 2^-11


def _ref(w, packed, bits, x):
    if bits == 16:
        return oracle.linear(x, w, None, None, 16)
    c, s, z = (t.cpu().numpy() for t in packed[bits])
    return oracle.linear(x, c, s, z, bits)


@pytest.mark.parametrize("bits", [4, 8, 16])
@pytest.mark.parametrize("M,N,K", [(2, 1, 128), (16, 17, 384), (17, 15, 1152), (32, 48, 2048), (31, 33, 2176), (16, 40, 4096),
                                   (15, 64, 4224), (5, 16, 11008), (18, 256, 4480)])
def test_single_call(M, N, K, bits):
    name = "batch/%dx%dx%d" % (M, N, K)
    w = synth.weight(13, name + "/w", N, K, 0.02, outlier_p=0.001)
    x = synth.activations(13, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    assert rel_err(gpu_linear(layer, bits, x), _ref(w, packed, bits, x)) <= TOL


@pytest.mark.parametrize("bits", [4, 8, 16])
@pytest.mark.parametrize("M,N,K", [(7, 11205, 384), (20, 8201, 1152)])
def test_partial_tile_behind_others_of_its_run(M, N, K, bits):
    # two or three tiles of 16 rows per workgroup on 256 compute units, the last one partly filled; odd numbers of
    # groups (at 4 bits half a 128-byte line is left over); and the same bits from every call
    name = "batch/ragged/%dx%d" % (N, K)
    w = synth.weight(13, name + "/w", N, K, 0.02)
    x = synth.activations(13, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    y = gpu_linear(layer, bits, x)
    assert rel_err(y, _ref(w, packed, bits, x)) <= TOL
    for _ in range(3):
        assert np.array_equal(gpu_linear(layer, bits, x).view(np.uint16), y.view(np.uint16))


@pytest.mark.parametrize("bits", [4, 8, 16])
@pytest.mark.parametrize("M,N,K", [(2, 12289, 128), (16, 20000, 512), (17, 13000, 384), (9, 131071, 256), (24, 131080, 128)])
def test_single_call_left_to_the_register_fed_kernel(M, N, K, bits):
    # short rows over more than three tiles of 16 per compute unit, and 512 rows per compute unit: its 64- and
    # 128-row tiles, the last one partly filled
    assert not batch_serves_linear(N, K, bits, M)
    name = "batch/short/%dx%d" % (N, K)
    w = synth.weight(13, name + "/w", N, K, 0.02)
    x = synth.activations(13, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    assert rel_err(gpu_linear(layer, bits, x), _ref(w, packed, bits, x)) <= TOL


@pytest.mark.parametrize("M", [3, 16, 32])
def test_plan_of_mixed_entries(M):
    # short rows over many tiles, slivers beside them: the register-fed kernel
    shapes = [(30000, 256), (48, 256), (17, 384), (300, 2304), (5, 256)]
    bits = [4, 16, 8, 4, 8]
    shared = {1: 0, 4: 0}  # entries that read entry 0's x
    assert not batch_serves([(N, K, (4, 8, 16)) for N, K in shapes], M)
    layers, xs, ys, ws, packs = [], [], [], [], []
    for i, (N, K) in enumerate(shapes):
        w = synth.weight(13, "batch/plan/w%d" % i, N, K, 0.02)
        layer, packed = make_layer(w, (4, 8, 16))
        x = xs[shared[i]] if i in shared else to_dev(synth.activations(13, "batch/plan/x%d/%d" % (i, M), M, K))
        layers.append(layer), xs.append(x), ws.append(w), packs.append(packed)
        ys.append(torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV))
    wsp = torch.empty(fq.Plan.workspace_bytes(len(shapes)), dtype=torch.uint8, device=DEV)
    plan = fq.Plan(layers, xs, ys, M, wsp)
    plan.run(torch.tensor(bits, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    for i in range(len(shapes)):
        ref = _ref(ws[i], packs[i], bits[i], xs[i].cpu().numpy())
        assert rel_err(ys[i].cpu().numpy(), ref) <= TOL, i
    assert plan.status() == (0, 0)
    # a width that is not served leaves the entry's y alone and is reported
    before = ys[2].clone()
    plan.run(torch.tensor([8, 4, 2, 16, 4], dtype=torch.int32, device=DEV))
    assert plan.status() == (0, 1) and torch.equal(ys[2], before)
    assert rel_err(ys[3].cpu().numpy(), _ref(ws[3], packs[3], 16, xs[3].cpu().numpy())) <= TOL


def test_plan_of_long_runs():
    # the same over rows that are not short, on the small-batch kernel: seven tiles of 16 per workgroup and more (30000
    # rows on 256 compute units), x in one panel and in several
    shapes = [(30000, 4096), (48, 4096), (17, 384), (300, 8320), (5, 256)]
    bits = [4, 16, 8, 4, 8]
    layers, ws, packs = [], [], []
    for i, (N, K) in enumerate(shapes):
        w = synth.weight(13, "batch/long/w%d" % i, N, K, 0.02)
        layer, packed = make_layer(w, (4, 8, 16))
        layers.append(layer), ws.append(w), packs.append(packed)
    for M in (3, 16, 32):
        assert batch_serves([(N, K, (4, 8, 16)) for N, K in shapes], M)
        xs = [to_dev(synth.activations(13, "batch/long/x%d/%d" % (i, M), M, K)) for i, (_, K) in enumerate(shapes)]
        xs[1] = xs[0]
        for pattern in (bits, [8, 4, 16, 8, 4]):
            ys = [torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV) for N, _ in shapes]
            wsp = torch.empty(fq.Plan.workspace_bytes(len(shapes)), dtype=torch.uint8, device=DEV)
            plan = fq.Plan(layers, xs, ys, M, wsp)
            plan.run(torch.tensor(pattern, dtype=torch.int32, device=DEV))
            torch.cuda.synchronize()
            assert plan.status() == (0, 0)
            for i, (N, K) in enumerate(shapes):
                y, x = ys[i].cpu().numpy(), xs[i].cpu().numpy()
                assert not np.isnan(y.astype(np.float32)).any()
                for row0 in range(0, N, 3700):  # some rows out of every stretch
                    n = min(60, N - row0)
                    if pattern[i] == 16:
                        ref = oracle.linear(x, ws[i], None, None, 16, row0=row0, rows=n)
                    else:
                        ref = oracle.linear(x, *(t.cpu().numpy() for t in packs[i][pattern[i]]), pattern[i], row0=row0, rows=n)
                    assert rel_err(y[:, row0:row0 + n], ref) <= TOL, (M, i, row0)


@pytest.mark.parametrize("M", [3, 20])
def test_plan_of_more_entries_than_the_small_batch_kernel_takes(M):
    # 70 entries of a few rows: the register-fed kernel with K split between the wavefronts
    shapes = [(17 + i % 5 * 16, (128, 384, 1152)[i % 3]) for i in range(70)]
    assert not batch_serves([(N, K, (4, 8, 16)) for N, K in shapes], M)
    bits = [(4, 8, 16)[i % 7 % 3] for i in range(70)]
    layers, xs, ys, refs = [], [], [], []
    for i, (N, K) in enumerate(shapes):
        w = synth.weight(13, "batch/many/w%d" % i, N, K, 0.02)
        x = synth.activations(13, "batch/many/x%d/%d" % (i, M), M, K)
        layer, packed = make_layer(w, (4, 8, 16))
        layers.append(layer), xs.append(to_dev(x)), refs.append(_ref(w, packed, bits[i], x))
        ys.append(torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV))
    wsp = torch.empty(fq.Plan.workspace_bytes(70), dtype=torch.uint8, device=DEV)
    plan = fq.Plan(layers, xs, ys, M, wsp)
    plan.run(torch.tensor(bits, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert plan.status() == (0, 0)
    for i in range(70):
        assert rel_err(ys[i].cpu().numpy(), refs[i]) <= TOL, i


@pytest.mark.parametrize("M", [16, 32])
@pytest.mark.parametrize("K,share", [(1920, True), (2048, True), (4096, True), (4224, True), (4096, False)])
def test_plan_whose_workgroups_cross_entries(K, share, M):
    # x requested ahead of the table from 2048 inputs on where all entries read it, kept for the next entry up to one
    # panel (4096 or 2048 inputs), and neither; the widths changing in between
    rows, bits = [2100, 1000, 4500, 8192], [4, 16, 8, 4]
    name = "batch/cross/%d" % K
    layers, xs, ys, ws, packs = [], [], [], [], []
    shared = to_dev(synth.activations(13, name + "/x", M, K))
    for i, N in enumerate(rows):
        w = synth.weight(13, name + "/w%d" % i, N, K, 0.02)
        layer, packed = make_layer(w, (bits[i],))
        layers.append(layer), ws.append(w), packs.append(packed)
        xs.append(shared if share or i == 1 else to_dev(synth.activations(13, name + "/x%d" % i, M, K)))
        ys.append(torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV))
    space = torch.empty(fq.Plan.workspace_bytes(len(rows)), dtype=torch.uint8, device=DEV)
    plan = fq.Plan(layers, xs, ys, M, space)
    plan.run(torch.tensor(bits, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    for i in range(len(rows)):
        ref = _ref(ws[i], packs[i], bits[i], xs[i].cpu().numpy())
        assert rel_err(ys[i].cpu().numpy(), ref) <= TOL, i

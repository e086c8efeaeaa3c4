"""The small-batch kernel (csrc/fq_batch.hip) over 2- and 3-bit copies at its edges: tiles of 16 rows partly filled, batch rows
around 16, one group, odd numbers of groups, part panels and several panels of x, several tiles to a workgroup, runs longer than six,
plans whose entries of every width share one x, slabs of a 3-bit prompt; against the oracle.  Every call is asked for its route."""
import numpy as np
import pytest
import torch

import oracle
import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_linear, make_layer, rel_err, to_dev
from plan_util import batch_serves, batch_serves_narrow, batch_serves_slab

pytestmark = pytest.mark.gpu

TOL = 2e-3  # exact integers times fp16 in binary32: what shows is the result's rounding to fp16, 2^-11


def _ref(w, packed, bits, x):
    if bits == 16:
        return oracle.linear(x, w, None, None, 16)
    c, s, z = (t.cpu().numpy() for t in packed[bits])
    return oracle.linear(x, c, s, z, bits)


@pytest.mark.parametrize("bits", [2, 3])
@pytest.mark.parametrize("M,N,K", [(2, 1, 128), (16, 17, 384), (17, 15, 1152), (32, 48, 2048), (31, 33, 2176), (16, 40, 4096),
                                   (15, 64, 4224), (5, 16, 11008), (18, 256, 4480), (7, 8191, 384), (7, 11205, 4096), (20, 8209, 6144),
                                   (32, 8225, 5120), (9, 30000, 4096)])
def test_single_call(M, N, K, bits):
    assert batch_serves_narrow(N, K, bits, M)
    name = "narrow/%dx%dx%d" % (M, N, K)
    w = synth.weight(17, name + "/w", N, K, 0.02, outlier_p=0.001)
    x = synth.activations(17, name + "/x", M, K)
    layer, packed = make_layer(w, (bits,))
    y = gpu_linear(layer, bits, x)
    assert rel_err(y, _ref(w, packed, bits, x)) <= TOL
    assert np.array_equal(gpu_linear(layer, bits, x).view(np.uint16), y.view(np.uint16))


@pytest.mark.parametrize("M", [2, 16, 32])
@pytest.mark.parametrize("K,share", [(1152, True), (4096, True), (4224, True), (4096, False)])
def test_plan_whose_workgroups_cross_entries_of_all_widths(K, share, M):
    # (short rows come here up to two tiles per compute unit)
    rows, widths = [1100, 500, 2400, 1600, 17, 2400] if K < 2048 else [2100, 1000, 4500, 3000, 17, 4000], (2, 3, 4, 8, 16)
    assert batch_serves([(N, K, widths) for N in rows], M, own_x=not share)
    name = "narrow/cross/%d" % K
    layers, xs, ys, ws, packs = [], [], [], [], []
    shared = to_dev(synth.activations(17, name + "/x", M, K))
    for i, N in enumerate(rows):
        w = synth.weight(17, name + "/w%d" % i, N, K, 0.02)
        layer, packed = make_layer(w, widths)
        layers.append(layer), ws.append(w), packs.append(packed)
        xs.append(shared if share or i == 1 else to_dev(synth.activations(17, name + "/x%d" % i, M, K)))
        ys.append(torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV))
    space = torch.empty(fq.Plan.workspace_bytes(len(rows)), dtype=torch.uint8, device=DEV)
    plan = fq.Plan(layers, xs, ys, M, space)
    for pattern in ([2, 16, 3, 8, 2, 4], [3, 2, 4, 3, 8, 16]):
        for y in ys:
            y.fill_(float("nan"))
        plan.run(torch.tensor(pattern, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        assert plan.status() == (0, 0)
        for i in range(len(rows)):
            assert rel_err(ys[i].cpu().numpy(), _ref(ws[i], packs[i], pattern[i], xs[i].cpu().numpy())) <= TOL, (pattern, i)


def test_a_width_without_a_copy_is_reported():
    w = synth.weight(17, "narrow/status/w", 100, 512, 0.02)
    x = synth.activations(17, "narrow/status/x", 4, 512)
    layer, packed = make_layer(w, (2, 8))
    y = torch.full((4, 100), float("nan"), dtype=torch.float16, device=DEV)
    space = torch.empty(fq.Plan.workspace_bytes(1), dtype=torch.uint8, device=DEV)
    plan = fq.Plan([layer], [to_dev(x)], [y], 4, space)
    assert batch_serves([(100, 512, (2, 8))], 4)
    plan.run(torch.tensor([3], dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert plan.status() == (0, 1) and torch.isnan(y).all()
    plan.run(torch.tensor([2], dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert rel_err(y.cpu().numpy(), _ref(w, packed, 2, x)) <= TOL


@pytest.mark.parametrize("M", [33, 34, 100])
def test_slabs_of_a_three_bit_prompt(M):
    # (a last slab of one row takes the register-fed kernel)
    assert batch_serves_slab(1000, 2176, 32) and batch_serves_slab(1000, 2176, 2)
    w = synth.weight(17, "narrow/slab/w", 1000, 2176, 0.02)
    x = synth.activations(17, "narrow/slab/x/%d" % M, M, 2176)
    layer, packed = make_layer(w, (3,))
    assert rel_err(gpu_linear(layer, 3, x), _ref(w, packed, 3, x)) <= TOL

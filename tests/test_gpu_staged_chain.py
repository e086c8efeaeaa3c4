"""Stage-ordered plans whose stages wait for the rows they read (no grid barrier), and plans that look like them but go
through the barrier: chains through a part of a y, two stages back, through buffers used again, past an entry that has no
copy at its bit-width, past rows that a launch refuses, rows that are NaNs, and rows that never
come.  Against the same stages as plans of their own, in turn: bit for bit."""
import pytest
import torch

import synth
import paper_2506_12024_amd as fq
from gpu_util import DEV, gpu_quantize, make_layer, to_dev

pytestmark = pytest.mark.gpu


def _plan(layers, xs, ys, stage):
    ws = torch.empty(fq.StagedPlan.workspace_bytes(len(layers), max(stage) + 1), dtype=torch.uint8, device=DEV)
    return fq.StagedPlan(layers, xs, ys, stage, 1, ws)


def _layer(tag, N, K, widths=(2, 3, 4, 8, 16), nan_row=None):
    w = synth.weight(21, "stgc/" + tag, N, K, K ** -0.5)
    if nan_row is not None:
        w = w.copy()
        w.view("uint16")[nan_row] = 0xFFFF
    return make_layer(w, widths)[0]


# how each linear finds its x: ("y", entry, first) or ("new", tag); its y: None for a buffer of its own, else entry whose y it reuses
CHAIN = [(0, 515, 512, ("new", "a"), None), (1, 1100, 512, ("y", 0, 0), None), (1, 384, 512, ("y", 0, 0), None),
         (2, 640, 1024, ("y", 1, 8), None), (3, 37, 640, ("y", 3, 0), None), (3, 12400, 640, ("y", 3, 0), None),
         (4, 515, 12288, ("y", 5, 16), None), (5, 130, 512, ("y", 6, 0), None)]


def _variant(name):
    c = list(CHAIN)
    if name == "two_back":        # stage 4 reads what stage 2 wrote: through the barrier there, polled elsewhere
        c[6] = (4, 515, 640, ("y", 3, 0), None)
    if name == "reused":          # stage 5 writes where stage 1 did: barriers everywhere
        c[7] = (5, 130, 512, ("y", 6, 0), 2)
    if name == "outside":         # an entry whose x is none of the plan's
        c[4] = (3, 37, 640, ("new", "b"), None)
    return c


@pytest.mark.parametrize("name", ["chain", "two_back", "reused", "outside", "unattached", "nan"])
def test_chains_match_their_stages_one_by_one(name):
    ents = _variant(name)
    widths = [(4, 8) if name == "unattached" and i == 3 else (2, 3, 4, 8, 16) for i in range(len(ents))]
    layers = [_layer("%d" % i, N, K, widths[i], 5 if name == "nan" and i == 1 else None)
              for i, (_, N, K, _, _) in enumerate(ents)]
    new = {t: torch.zeros(1, 640, dtype=torch.float16, device=DEV) for t in ("a", "b")}

    def buffers():
        ys, xs = [], []
        for st, N, K, (kind, src, *first), again in ents:
            xs.append(new[src][:, :K].contiguous() if kind == "new" else ys[src][:, first[0]:first[0] + K])
            ys.append(ys[again][:, :N] if again is not None else torch.zeros(1, N, dtype=torch.float16, device=DEV))
        return xs, ys

    new["a"].copy_(to_dev(synth.activations(21, "stgc/a", 1, 640)))
    new["b"].copy_(to_dev(synth.activations(21, "stgc/b", 1, 640)))
    xs, ys = buffers()
    xr, yr = buffers()
    stage = [e[0] for e in ents]
    plan = _plan(layers, xs, ys, stage)
    sets = [[i for i, v in enumerate(stage) if v == st] for st in range(max(stage) + 1)]
    ones = [_plan([layers[i] for i in set_], [xr[i] for i in set_], [yr[i] for i in set_], [0] * len(set_)) for set_ in sets]
    for rep, pattern in enumerate([(4, 8), (8, 4, 16), (2, 3, 4), (16,), (4,)]):
        bits = [16 if name == "nan" and i == 1 else pattern[i % len(pattern)] for i in range(len(ents))]
        if name == "unattached":
            bits[3] = 16 if rep % 2 else 8      # every other time nobody writes stage 2's y: its old content is read
        for b in range(rep % 2 + 1):
            plan.run(torch.tensor(bits, dtype=torch.int32, device=DEV))
        for set_, one in zip(sets, ones):
            one.run(torch.tensor([bits[i] for i in set_], dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        for i in range(len(ents)):
            a, b = ys[i].view(torch.int16), yr[i].view(torch.int16)
            if name == "nan":
                a, b = torch.where(ys[i].isnan(), 0, a), torch.where(yr[i].isnan(), 0, b)
                assert torch.equal(ys[i].isnan(), yr[i].isnan()), (rep, i)
            assert torch.equal(a, b), (rep, i)
        assert plan.status()[0] == 0
    if name == "nan":
        assert ys[1].isnan().any()


def test_rows_of_a_share_that_is_refused_are_not_waited_for():
    # 40000 short rows beside 1500 long ones: a workgroup would be dealt more of the short ones than it holds results
    # for, so they keep what they held, a 0xFFFF half in every one of them among the rest; their reader goes on all the same
    def layer(N, K, bits):
        w = torch.randn(N, K, dtype=torch.float16, device=DEV) * K ** -0.5
        return fq.Layer(N, K).attach(bits, *((w,) if bits == 16 else gpu_quantize(w, bits)))

    torch.manual_seed(3)
    shapes, bits, stage = [(128, 128), (40000, 128), (1500, 32768), (256, 1024)], [4, 4, 16, 8], [0, 1, 1, 2]
    layers = [layer(N, K, b) for (N, K), b in zip(shapes, bits)]
    ys = [torch.zeros(1, N, dtype=torch.float16, device=DEV) for N, _ in shapes]
    xs = [torch.randn(1, K, dtype=torch.float16, device=DEV) for _, K in shapes[:3]] + [ys[1][:, :1024]]
    plan = _plan(layers, xs, ys, stage)
    plan.set_wait_limit(1 << 16)
    bits_dev = torch.tensor(bits, dtype=torch.int32, device=DEV)
    ys[1].view(torch.int16).fill_(-1)
    plan.run(bits_dev)
    torch.cuda.synchronize()
    assert plan.status() == (0, 2)
    assert (ys[1].view(torch.int16) == -1).all() and ys[3].isnan().all()
    ys[1].copy_(torch.randn(1, 40000, dtype=torch.float16, device=DEV))
    held, ref = ys[1].clone(), torch.zeros_like(ys[3])
    plan.run(bits_dev)
    _plan([layers[3]], [xs[3]], [ref], [0]).run(bits_dev[3:])
    torch.cuda.synchronize()
    assert plan.status() == (0, 2) and torch.equal(ys[1], held) and torch.equal(ys[3], ref)


def test_a_wait_for_rows_that_runs_out_returns_and_the_next_launch_is_whole():
    # Forced from the host: in the plan's table the third linear's x, which the kernel waits for, is put to a buffer that nobody
    # writes.  Every launch gives up there, and not at a barrier; with the x put back the plan is whole.
    shapes, stage = [(1024, 1024), (1152, 1024), (1024, 1024), (512, 1024)], [0, 1, 2, 3]
    layers = [_layer("gu%d" % i, N, K, (8,)) for i, (N, K) in enumerate(shapes)]
    ys = [torch.zeros(1, N, dtype=torch.float16, device=DEV) for N, _ in shapes]
    xs = [to_dev(synth.activations(21, "stgc/gu", 1, 1024)), ys[0], ys[1][:, 16:1040], ys[2]]
    ws = torch.zeros(fq.StagedPlan.workspace_bytes(4, 4), dtype=torch.uint8, device=DEV)
    plan = fq.StagedPlan(layers, xs, ys, stage, 1, ws)
    words = ws.view(torch.int64)
    at = (words == xs[2].data_ptr()).nonzero().flatten().tolist()
    assert len(at) == 1
    never = torch.full((1, 1024), -1, dtype=torch.int16, device=DEV)
    words[at[0]] = never.data_ptr()
    bits = torch.full((4,), 8, dtype=torch.int32, device=DEV)
    plan.set_wait_limit(1 << 12)
    for n in range(3):
        ys[3].fill_(7)
        plan.run(bits)
        torch.cuda.synchronize()
        assert plan.status() == (n + 1, 0)
        assert ys[0].isfinite().all() and ys[1].isfinite().all()
        assert (ys[2].view(torch.int16) == -1).all() and (ys[3] == 7).all()
    words[at[0]] = xs[2].data_ptr()
    plan.set_wait_limit(1 << 21)
    refs = [torch.zeros_like(y) for y in ys]
    for i in range(4):
        x = xs[0] if i == 0 else refs[i - 1][:, 16:1040] if i == 2 else refs[i - 1]
        _plan([layers[i]], [x], [refs[i]], [0]).run(bits[:1])
    for _ in range(2):
        plan.run(bits)
        torch.cuda.synchronize()
        assert plan.status() == (3, 0)
        for y, r in zip(ys, refs):
            assert torch.equal(y.view(torch.int16), r.view(torch.int16))

"""A model of the stage-ordered kernel's boundaries (csrc/fq_staged.hip) in single steps, wavefront by wavefront, under
random schedules (CPU only): the grid barrier, the boundary at which the data is the signal, and how a launch ends when
either wait runs out.

A workgroup is some compute wavefronts and a service wavefront that share LDS: a count of rows left there, the stage ahead of
which the workgroup leaves, and a workgroup barrier (which counts the wavefronts that have not ended).  Memory holds the
arrival count (one counter here: that many count alike is test_staged_protocol_model.py's), the abort flag, the sticky count
of launches that gave up, the count of finished workgroups, and the rows.  A step is one access to memory or LDS;
the schedule picks whose is next, and lets some wavefronts fall far behind.  What the kernel relies on:
  - no wavefront goes on with an x of which a row is unwritten or of an earlier launch,
  - rows are all written by a launch that nobody gave up,
  - whoever gives up, everyone ends, and the words are clean for the next launch, which is whole."""
import random

import pytest

UNWRITTEN = -1
NEVER = 1 << 30


class Launch:
    def __init__(self, G, CW, polled, share, reads, sync, rows, number, limit, marks=True):
        self.G, self.CW, self.polled, self.share, self.reads = G, CW, polled, share, reads
        self.sync, self.rows, self.number, self.limit, self.marks = sync, rows, number, limit, marks
        self.S = len(polled)
        self.left = [0] * G                      # LDS: rows announced, by wavefronts and stages
        self.leave = [NEVER] * G                 # LDS: the stage ahead of which the workgroup leaves
        self.alive = [CW + 1] * G
        self.arrived, self.passed = [0] * G, [0] * G
        self.stale = []

    # -- one workgroup's barrier; waits in steps
    def barrier(self, b):
        mine = self.passed[b]
        self.arrived[b] += 1
        self.release(b)
        while self.passed[b] == mine:
            yield

    def release(self, b):
        if self.arrived[b] and self.arrived[b] == self.alive[b]:
            self.arrived[b] = 0
            self.passed[b] += 1

    def leaves(self, b, s):
        return self.leave[b] <= s if self.marks else self.leave[b] != NEVER

    def give_up(self, b, s, round_):
        up = 0
        if round_ >= self.limit:
            up, self.sync["abort"] = self.sync["abort"], 1
            yield
            if up == 0:
                self.sync["gave_up"] += 1
                yield
            up = 1
        elif round_ % 4 == 3:
            up = self.sync["abort"]
            yield
        if up:
            self.leave[b] = s
            yield
        return up

    def stage_x(self, b, s):
        """Reads of the x of stage s: polled, or plain behind the barrier."""
        if not self.share[s][b] or s == 0:
            return
        need = self.reads[s]
        for round_ in range(NEVER):
            seen = []
            for r in need:
                seen.append(self.rows[s - 1][r])
                yield
            if self.polled[s] and UNWRITTEN in seen:
                if (yield from self.give_up(b, s, round_)):
                    return
                continue
            self.stale += [(s, b, v) for v in seen if v != self.number]
            return

    def wait_stage(self, met):
        for it in range(NEVER):
            if self.sync["abort"]:
                return False
            yield
            if self.sync["arrivals"] >= (met + 1) * self.G:
                return True
            yield
            if it >= self.limit:
                up, self.sync["abort"] = self.sync["abort"], 1
                yield
                if up == 0:
                    self.sync["gave_up"] += 1
                return False

    def service(self, b):
        yield from self.barrier(b)
        for s in range(1, self.S):
            if s + 1 < self.S and self.polled[s + 1] and self.share[s][b]:
                self.rows[s][b] = UNWRITTEN
                yield
        met = 0
        for s in range(self.S):
            while self.left[b] < self.CW * (s + 1):
                yield
            if self.share[s][b]:
                self.rows[s][b] = self.number
                yield
            if s + 1 == self.S:
                break
            if not self.polled[s + 1]:
                self.sync["arrivals"] += 1
                yield
                reached = yield from self.wait_stage(met)
                met += 1
                if not reached:
                    self.leave[b] = s + 1
                yield from self.barrier(b)
                if not reached:
                    break
            yield from self.stage_x(b, s + 1)
            yield from self.barrier(b)
            yield
            if self.leaves(b, s + 1):
                break
        self.sync["done"] += 1
        last = self.sync["done"] == self.G
        yield
        if last:
            for word in ("arrivals", "abort", "done"):
                self.sync[word] = 0
                yield

    def compute(self, b):
        for s in range(self.S):
            if s:
                if not self.polled[s]:
                    yield from self.barrier(b)
                    yield
                    if self.leaves(b, s):
                        return
                while self.left[b] < self.CW * s:
                    yield
            yield from self.stage_x(b, s)
            yield from self.barrier(b)
            yield
            if self.leaves(b, s):
                return
            self.left[b] += 1
            yield

    def run(self, rng, late=()):
        waves = [(b, g) for b in range(self.G) for g in [self.service(b)] + [self.compute(b) for _ in range(self.CW)]]
        slow = {id(g): rng.choice([0.02, 0.3]) for _, g in rng.sample(waves, rng.randint(0, min(4, len(waves))))}
        running = [w for w in waves if w[0] not in late]
        waiting = [w for w in waves if w[0] in late]
        for _ in range(400000):
            if not running:
                running, waiting = waiting, []   # workgroups that found no room until the others had ended
                if not running:
                    return
            w = rng.choice(running)
            if rng.random() > slow.get(id(w[1]), 1.0):
                continue
            try:
                next(w[1])
            except StopIteration:
                running.remove(w)
                self.alive[w[0]] -= 1
                self.release(w[0])
        raise AssertionError("a wavefront never ended")


def _plan(rng):
    """Stages with and without the barrier, who has a share of each and which rows a stage reads."""
    G, S = rng.randint(1, 4), rng.randint(3, 6)
    polled = [False, False] + [rng.random() < 0.7 for _ in range(S - 2)]
    share = [[rng.random() < 0.8 for _ in range(G)] for _ in range(S)]
    for s in share:
        s[rng.randrange(G)] = True
    reads = [[]] + [[b for b in range(G) if share[s - 1][b]] for s in range(1, S)]
    return G, rng.randint(1, 3), polled, share, reads


def _clean(sync):
    return (sync["arrivals"], sync["abort"], sync["done"]) == (0, 0, 0)


def _play(seed, marks=True):
    """A whole launch, some with waits that may run out, a whole one.  Returns (gave up, a polled wait ran out, clean)."""
    rng = random.Random(seed)
    G, CW, polled, share, reads = _plan(rng)
    sync = {"arrivals": 0, "abort": 0, "gave_up": 0, "done": 0}
    rows = [[UNWRITTEN] * G for _ in polled]
    at_polled = False
    for number in range(5):
        whole = number in (0, 4)
        before = sync["gave_up"]
        late = () if whole or G == 1 or rng.random() < 0.6 else (rng.randrange(G),)
        run = Launch(G, CW, polled, share, reads, sync, rows, number, NEVER if whole else rng.choice([0, 0, 3, 12]), marks)
        run.run(rng, late)
        if not _clean(sync):
            return sync["gave_up"], at_polled, False
        assert run.stale == [], (seed, number)
        if sync["gave_up"] == before:
            assert all(rows[s][b] == number for s in range(len(polled)) for b in range(G) if share[s][b]), (seed, number)
        else:
            assert not whole and sync["gave_up"] == before + 1
            at_polled = at_polled or any(v != NEVER and polled[v] for v in run.leave)
    return sync["gave_up"], at_polled, True


@pytest.mark.parametrize("part", range(8))
def test_launches_end_clean_whoever_gives_up(part):
    gave_up = at_polled = 0
    for seed in range(40 * part, 40 * part + 40):
        n, polled, clean = _play(seed)
        assert clean, seed
        gave_up += n
        at_polled += polled
    assert gave_up > 10 and at_polled > 5


def test_the_model_tells_a_flag_without_its_stage():
    # The leave word as a plain flag: a service wavefront that looks at it late, when its compute wavefronts have given up
    # at the next stage, counts its workgroup out while they may still raise the abort flag.
    assert not all(_play(seed, marks=False)[2] for seed in range(400))

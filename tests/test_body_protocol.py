"""The order of events in the one-launch body on the CPU: models of its waves under random schedules, with rolls closed at any number of
workgroups.  A layer at a time (csrc/conv_body.hip): two teams of four waves a workgroup, barriers, words, both forms of looking.  Two
layers a unit (csrc/conv_body_pairs.h): eight waves, words by step, two tensors in turn, units that stay in LDS or not, thirds of weights.
Every schedule has to end with all units stored, and every patch, skip value, weight and bias that a wave reads has to be
the right layer's, stored and acknowledged before the read and not written anew before it is used.

They follow the kernels by hand, so a change of a kernel's order of events belongs here too."""
import random

import pytest

WAVES = 4


class Stuck(Exception):
    pass


def schedule(rng, G, alive):
    """Runs the waves of G workgroups, {(workgroup, ..): events}, to their ends."""
    waits = dict.fromkeys(alive)
    speed = {k: rng.choice((1, 1, 1, 8)) * rng.choice((1, 4)) for k in alive}
    slow = rng.choice((None, None, *range(G)))               # a workgroup that hardly runs
    while alive:
        able = [k for k in alive if waits[k] is None or waits[k]()]
        if not able:
            raise Stuck(sorted(alive))
        for k in rng.choices(able, [speed[k] * (1 if k[0] != slow else 0.02) for k in able], k=3):
            if k not in alive or (waits[k] is not None and not waits[k]()):
                continue
            try:
                waits[k] = next(alive[k])
            except StopIteration:
                del alive[k]


class Launch:
    def __init__(self, rng, topology, layers, G, images, rows, cols, few, mistake=None):
        self.rng, self.topology, self.layers, self.G, self.few, self.mistake = rng, topology, layers, G, few, mistake
        self.rows, self.cols, self.units = rows, cols, images * rows * cols
        self.done = [[0] * WAVES for _ in range(self.units)]
        # version of a buffer's rows: layers stored there so far, when the store is issued and when it is acknowledged
        self.issued, self.acked = ({b: [[0] * WAVES for _ in range(self.units)] for b in "hat"} for _ in range(2))

    # ---- which buffers a layer uses ----
    def skips(self, l):
        return self.topology != "plain" and bool(l % 2 or (self.topology == "edsr" and l == self.layers - 1))

    def reads(self, l):
        if self.topology == "plain":
            return "h" if l == 0 else "a" if l % 2 else "t"
        return "t" if l % 2 else "h" if l == 0 else "a"

    def writes(self, l):
        return ("t" if l % 2 else "a") if self.topology == "plain" else ("a" if l % 2 else "t")

    def skip(self, l):
        return "a" if l % 2 and l != 1 else "h"

    # ---- units and their neighbours ----
    def at(self, layer, idx, ahead):
        idx += ahead
        while idx >= self.units and layer < self.layers:
            idx, layer = idx - self.units, layer + 1
        return layer, idx

    def around(self, idx):
        n, c = divmod(idx, self.rows * self.cols)
        y, x = divmod(c, self.cols)
        return [(n * self.rows + v) * self.cols + u for v in (y - 1, y, y + 1) for u in (x - 1, x, x + 1) if 0 <= v < self.rows and 0 <= u < self.cols]

    def ready(self, u):
        layer, idx = u
        if self.mistake == "no wait":
            return True
        return not 0 < layer < self.layers or all(w >= layer for i in self.around(idx) for w in self.done[i])

    def check(self, buf, version, idxs, waves, table, what):
        for i in idxs:
            for w in waves:
                assert table[buf][i][w] == version, (what, buf, i, w, table[buf][i][w], version)

    def patch(self, u, table, what):
        buf = self.reads(u[0])
        self.check(buf, 0 if buf == "h" else u[0], self.around(u[1]), range(WAVES), table, what)

    def run(self):
        groups = [Group(self, g) for g in range(self.G)]
        schedule(self.rng, self.G, {(g, t, w): groups[g].wave(t, w) for g in range(self.G) for t in range(2) for w in range(WAVES)})
        for layer in range(self.layers):
            last = max(l for l in range(self.layers) if self.writes(l) == self.writes(layer))
            self.check(self.writes(layer), last + 1, range(self.units), range(WAVES), self.acked, "end")
        assert all(w == self.layers for d in self.done for w in d)


class Group:
    def __init__(self, launch, number):
        self.L, self.number = launch, number
        self.weights, self.patches, self.bias = [None] * WAVES, [[None] * WAVES for _ in range(2)], [None, None]
        self.ready, self.again, self.sync = [[0, 0], [0, 0]], [0, 0], [0, 0]
        self.passed = {(t, w): 0 for t in range(2) for w in range(WAVES)}       # barriers that each wave that has not ended has come to

    def wave(self, team, w):
        """The events of one wave.  Yields where other waves may run; what it yields, if anything, says when it can go on."""
        L, layers, units, few = self.L, self.L.layers, self.L.units, self.L.few
        G = min(L.G, units)
        if self.number >= G:
            return

        def barrier():
            self.passed[team, w] += 1
            return lambda n=self.passed[team, w]: min(self.passed.values()) >= n

        cur = L.at(0, self.number, team * G)
        prev, loaded, due, resident, bias_layer, turn, syncs = cur, False, False, -1, -1, 0, 0

        def mark(u):                                         # the stores are acknowledged by now, and may not have been before
            L.acked[L.writes(u[0])][u[1]][w] = u[0] + 1
            L.done[u[1]][w] = u[0] + 1

        if team == 1:
            yield barrier()
            resident = 0
            yield barrier()
        while True:
            if due and (cur[0] >= layers or not loaded):
                mark(prev)
                due = False
                yield
            if cur[0] >= layers:
                break
            if not loaded or cur[0] != resident:
                if cur[0] != resident:
                    self.weights[w] = None                   # on their way to LDS
                    yield
                if not loaded:
                    yield (lambda u=cur: L.ready(u))
                    L.patch(cur, L.acked, "patch")
                    yield
                    L.patch(cur, L.issued, "patch, used")
                    self.patches[team][w] = cur
                if w == 0:
                    self.bias[team] = cur[0]
                bias_layer = cur[0]
                if cur[0] != resident:
                    self.weights[w] = cur[0]
                syncs += WAVES
                self.sync[team] += 1
                yield (lambda n=syncs: self.sync[team] >= n)
            resident = cur[0]
            # ---- computes ----
            skip = L.skips(cur[0])
            if skip:
                version = cur[0] - 1 if L.skip(cur[0]) == "a" else 0
                L.check(L.skip(cur[0]), version, [cur[1]], [w], L.acked, "skip")
            assert self.bias[team] == cur[0]
            assert self.weights == [cur[0]] * WAVES and self.patches[team] == [cur] * WAVES, (self.weights, self.patches[team], cur)
            yield
            nu = L.at(*cur, 2 * G)
            front = cur[0] + (cur[1] + G >= units)
            if due:
                mark(prev)
            yield
            if not few and w == 0:
                self.ready[team][(turn & 1) ^ 1] = int(L.ready(nu))
                yield
            yield barrier()
            assert self.weights == [cur[0]] * WAVES and self.patches[team] == [cur] * WAVES
            yield barrier()
            # ---- the other team computes ----
            ready0, ready1 = (0, 0) if few else (self.ready[team ^ 1][(turn + team) & 1], self.ready[team][(turn & 1) ^ 1])
            at_end, none = front >= layers, nu[0] >= layers
            early = bool(not none and ready1)
            fetch = early
            self.patches[team][w] = "staging"
            again = not early and w == 0 and L.ready(nu)
            if early:
                L.patch(nu, L.acked, "early patch")
            yield
            if skip:
                L.check(L.skip(cur[0]), version, [cur[1]], [w], L.issued, "skip, used")
            L.issued[L.writes(cur[0])][cur[1]][w] = cur[0] + 1
            yield
            if not early and not none:
                if w == 0:
                    self.again[team] = turn * 2 + 2 + int(again)
                yield (lambda n=turn + 1: self.again[team] >> 1 == n)
                fetch = bool(self.again[team] & 1)
                if fetch:
                    L.patch(nu, L.acked, "patch after a second look")
                yield
                mark(cur)
                yield
            told = not early and not none
            prev, cur, turn, due = cur, nu, turn + 1, False
            if not told:
                if at_end or none or (not ready0 and L.mistake != "no word"):
                    mark(prev)
                    if at_end:
                        break
                else:
                    due = True
                yield
            resident = front
            yield barrier()
            if fetch:
                L.patch(cur, L.issued, "patch, used")
                self.patches[team][w] = cur
            loaded = fetch
            if cur[0] < layers and cur[0] != bias_layer:
                if w == 0:
                    self.bias[team] = cur[0]
                bias_layer = cur[0]
            yield barrier()
        del self.passed[team, w]                             # barriers do not wait for waves that have ended


@pytest.mark.parametrize("topology,layers", [("edsr", 3), ("edsr", 9), ("res", 2), ("res", 6), ("plain", 2), ("plain", 5)])
@pytest.mark.parametrize("few", [False, True])
def test_every_schedule_ends_and_reads_what_the_layer_before_stored(topology, layers, few):
    rng = random.Random(f"{topology} {layers} {few}")
    for _ in range(12):
        G, images, rows, cols = rng.randint(1, 6), rng.randint(1, 3), rng.randint(1, 4), rng.randint(1, 3)
        Launch(rng, topology, layers, G, images, rows, cols, few).run()


def test_the_model_tells_a_missing_word_and_a_missing_wait():
    def fails(mistake):
        rng, seen = random.Random(mistake), set()
        for _ in range(40):
            try:
                Launch(rng, "edsr", 5, 3, 1, 1, 4, False, mistake).run()
            except (Stuck, AssertionError) as e:
                seen.add(type(e))
        return seen
    assert Stuck in fails("no word") and AssertionError in fails("no wait") and not fails(None)


class Pairs:
    """Two layers a unit: G workgroups for images x rows x cols units, SLOTS thirds of a layer's weights in LDS."""
    ALL = 8                                                  # waves of a workgroup

    def __init__(self, rng, topology, layers, G, images, rows, cols, slots, mistake=None):
        self.rng, self.layers, self.steps, self.slots, self.mistake = rng, layers, (layers + 1) // 2, slots, mistake
        self.rows, self.cols, self.units = rows, cols, images * rows * cols
        self.G = min(G, self.units)
        self.stay = self.G >= self.units
        self.last = "t" if topology == "edsr" or (topology == "plain" and layers % 2 == 0) else "a"
        self.done = [0] * self.units
        # version of a wave's share of a unit: steps that had stored it, or its rows and columns that others read
        self.issued, self.acked = ({b: [[0] * self.ALL for _ in range(self.units)] for b in "hat"} for _ in range(2))
        self.whole = {b: [False] * self.units for b in "hat"}

    around = Launch.around

    def out(self, s):
        other = {"a": "t", "t": "a"}[self.last]
        return other if (self.steps - 1 - s) % 2 and self.mistake != "one tensor" else self.last

    def check(self, s, idxs, table, what):
        buf, version = ("h", 0) if s == 0 else (self.out(s - 1), s)
        for i in idxs:
            assert table[buf][i] == [version] * self.ALL, (what, s, i, table[buf][i], version)

    def run(self):
        groups = [PairGroup(self, g) for g in range(self.G)]
        schedule(self.rng, self.G, {(g, w): groups[g].wave(w) for g in range(self.G) for w in range(self.ALL)})
        assert self.done == [self.steps] * self.units and all(self.whole[self.last])
        assert all(v == [self.steps] * self.ALL for v in self.acked[self.last])


class PairGroup:
    def __init__(self, launch, number):
        self.L, self.number, self.stored = launch, number, 0
        self.inner, self.ring = ([None] * launch.ALL for _ in range(2))      # of the patch's place, by the wave that writes them: (what, step, unit)
        self.slot = [[None] * launch.ALL for _ in range(launch.slots)]       # the third of weights there, each wave's part of it
        self.passed = [0] * launch.ALL

    def wave(self, w):
        L, S, units, steps = self.L, self.L.slots, self.L.units, self.L.steps
        flying = []                                          # thirds that this wave has requested: (slot, number)

        def barrier():
            self.passed[w] += 1
            return lambda n=self.passed[w]: min(self.passed) >= n

        def request(number, slot):
            self.slot[slot][w] = None
            flying.append((slot, number))

        def arrived(but=0):                                  # all but the last `but` thirds.  What else is outstanding makes the wait longer, never shorter
            while len(flying) > but:
                slot, number = flying.pop(0)
                self.slot[slot][w] = number

        layer_no, par = 0, 0                                 # layers so far: thirds are numbered 3 * layer_no + k, those of the layer behind 3 more

        def slot_of(k):
            return k if S == 3 else (k + par) & 1

        def products(what, patch):
            nonlocal layer_no, par
            for k in range(3):
                assert self.slot[slot_of(k)] == [3 * layer_no + k] * L.ALL, (self.slot, layer_no, k)
                if patch:
                    assert self.inner == self.ring == [what] * L.ALL, (self.inner, self.ring, what)
                yield
                arrived(S - 2 if L.mistake != "weights" else S - 1)
                yield barrier()
                if S == 3:
                    request(3 * layer_no + 3 + k, k)
                elif k == 0:
                    request(3 * layer_no + 2, slot_of(0))
                else:
                    request(3 * layer_no + 2 + k, slot_of(k))
            yield
            assert self.inner == self.ring == [what] * L.ALL
            layer_no, par = layer_no + 1, par ^ 1

        for k in range(S):
            request(k, k)
        s, u, count = 0, self.number, 0
        while s < steps:
            s_next, u_next = (s, u + L.G) if u + L.G < units else (s + 1, self.number)
            two, own = 2 * s + 1 < L.layers, L.stay and s > 0
            yield
            if s and L.mistake != "no wait":
                yield (lambda: all(L.done[i] >= s for i in L.around(u)))
            others = [i for i in L.around(u) if not own or i != u]
            L.check(s, others, L.acked, "patch")
            yield
            L.check(s, others, L.issued, "patch, used")
            if s and not own:                                # the unit itself, from memory
                assert L.whole[L.out(s - 1)][u]
            self.ring[w] = ("in", s, u)
            if not own:
                self.inner[w] = ("in", s, u)
            arrived()
            yield barrier()
            if two:
                yield from products(("in", s, u), True)
                yield barrier()                              # the skip is read
                self.inner[w] = self.ring[w] = ("between", s, u)
                yield barrier()
            yield from products(("between" if two else "in", s, u), True)
            L.issued[L.out(s)][u][w] = s + 1
            yield barrier()
            if L.stay and s + 1 < steps:
                self.inner[w] = ("in", s + 1, u)
            yield
            L.acked[L.out(s)][u][w] = s + 1
            L.whole[L.out(s)][u] = not L.stay or s + 1 == steps
            self.stored += 1
            if self.stored == (count + 1) * L.ALL or (L.mistake == "early word" and self.stored == count * L.ALL + 1):
                L.done[u] = s + 1
            count += 1
            s, u = s_next, u_next


@pytest.mark.parametrize("topology,layers", [("edsr", 3), ("edsr", 9), ("res", 2), ("res", 8), ("plain", 2), ("plain", 3), ("plain", 5), ("plain", 6)])
@pytest.mark.parametrize("slots", [2, 3])
def test_two_layers_a_unit_in_every_schedule(topology, layers, slots):
    rng = random.Random(f"{topology} {layers} {slots}")
    for k in range(12):
        images, rows, cols = rng.randint(1, 3), rng.randint(1, 4), rng.randint(1, 3)
        units = images * rows * cols
        G = units if k % 2 else rng.randint(1, min(units, 6))              # the whole roll, or one that closed early
        if units <= 12:
            Pairs(rng, topology, layers, G, images, rows, cols, slots).run()


def test_the_model_of_two_layers_a_unit_tells_mistakes():
    def fails(mistake, G):
        rng, seen = random.Random(mistake), set()
        for _ in range(30):
            try:
                Pairs(rng, "edsr", 7, G, 1, 1, 4, rng.choice((2, 3)), mistake).run()
            except (Stuck, AssertionError) as e:
                seen.add(type(e))
        return seen
    for G in (4, 3):
        assert not fails(None, G)
        for mistake in ("no wait", "one tensor", "early word", "weights"):
            assert AssertionError in fails(mistake, G), (mistake, G)

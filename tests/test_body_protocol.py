"""The order of events in the one-launch body (csrc/conv_body.hip) on the CPU: a model of its waves - two teams of four a
workgroup, barriers, rolls closed at any number of workgroups, words, both forms of looking - under random schedules.
Every schedule has to end with all units stored, and every patch, skip value, weight and bias that a wave reads has to be
the right layer's, stored and acknowledged before the read and not written anew before it is used.

It follows the kernel by hand, so a change of the kernel's order of events belongs here too."""
import random

import pytest

WAVES = 4


class Stuck(Exception):
    pass


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

    # ---- schedule ----
    def run(self):
        groups = [Group(self, g) for g in range(self.G)]
        alive = {(g, t, w): groups[g].wave(t, w) for g in range(self.G) for t in range(2) for w in range(WAVES)}
        waits = dict.fromkeys(alive)
        speed = {k: self.rng.choice((1, 1, 1, 8)) * self.rng.choice((1, 4)) for k in alive}
        slow = self.rng.choice((None, None, *range(self.G)))                # a workgroup that hardly runs
        while alive:
            able = [k for k in alive if waits[k] is None or waits[k]()]
            if not able:
                raise Stuck(sorted(alive))
            for k in self.rng.choices(able, [speed[k] * (1 if k[0] != slow else 0.02) for k in able], k=3):
                if k not in alive or (waits[k] is not None and not waits[k]()):
                    continue
                try:
                    waits[k] = next(alive[k])
                except StopIteration:
                    del alive[k]
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

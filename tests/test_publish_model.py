"""How a workgroup takes its tasks' inputs and publishes their outputs, on a
model of the memory they pass through.

The engine's protocol, wavefront by wavefront: the first claims a queue slot,
waits for its task id and executes one agent-scope acquire, before a barrier;
the task's stores follow; every wavefront waits for its own stores; a barrier;
the first wavefront executes one agent-scope release, counts the task off with
a relaxed atomic, and if it was the group's last, a second fence and relaxed
stores of the next group's task ids.

The memory: a store is on its way (in no order with the wavefront's others, and
whatever barriers it passes) until it reaches the L1 of its compute unit and,
dirty, the L2 of its XCD; entries are evicted from either at any time; loads
read the nearest copy, however old.  Waiting ends when the wavefront's own
stores have arrived.  A release waits for those too, then writes the L2's dirty
entries back; an acquire drops the L1 and the L2's clean entries.  Atomics act
on memory.  A random scheduler picks what happens next.  Every task checks that
it reads what the tasks of the group before it wrote; addresses are used again
by every second group, so that old values lie about.  Leaving out any one of
the steps must be noticed."""

from __future__ import annotations

import random

import pytest

WAVES, WORDS = 3, 2   # wavefronts per workgroup, words each writes per task


class Memory:
    def __init__(self, rng, n_xcd, n_cu):
        self.rng, self.words, self.atomics = rng, {}, {}
        self.speed = rng.choice((0.02, 0.1, 0.5))  # how soon stores arrive
        self.l2 = [{} for _ in range(n_xcd)]     # address -> (value, dirty)
        self.l1 = [{} for _ in range(n_cu)]      # address -> value
        self.flying = {}                         # wavefront -> [(address, value)]

    def xcd(self, cu):
        return cu % len(self.l2)

    def load(self, cu, a):
        if a not in self.l1[cu]:
            l2 = self.l2[self.xcd(cu)]
            if a not in l2:
                l2[a] = (self.words.get(a), False)
            self.l1[cu][a] = l2[a][0]
        return self.l1[cu][a]

    def arrive(self, wave):
        q = self.flying[wave]
        a, v = q.pop(self.rng.randrange(len(q)))
        if a in self.l1[wave[0]]:
            self.l1[wave[0]][a] = v
        self.l2[self.xcd(wave[0])][a] = (v, True)

    def write_back(self, x):
        for a, (v, dirty) in self.l2[x].items():
            if dirty:
                self.words[a] = v
                self.l2[x][a] = (v, False)

    def acquire(self, cu):
        self.l1[cu].clear()
        l2 = self.l2[self.xcd(cu)]
        for a in [a for a, (_, dirty) in l2.items() if not dirty]:
            del l2[a]

    def something(self):
        """A store arrives or an entry is evicted."""
        ready = [w for w, q in self.flying.items() if q]
        if ready and self.rng.random() < self.speed:
            self.arrive(self.rng.choice(ready))
        elif self.rng.random() < 0.2:
            x = self.rng.randrange(len(self.l2))
            if self.l2[x]:
                a = self.rng.choice(list(self.l2[x]))
                v, dirty = self.l2[x].pop(a)
                if dirty:
                    self.words[a] = v
            cu = self.rng.randrange(len(self.l1))
            if self.l1[cu]:
                del self.l1[cu][self.rng.choice(list(self.l1[cu]))]

    def add(self, a, n):
        old = self.atomics[a]
        self.atomics[a] = old + n
        return old


class Wrong(Exception):
    pass


def run(seed, n_wg, without=None):
    rng = random.Random(seed)
    m = Memory(rng, rng.randint(1, 2), n_wg)
    # chains of groups of tasks: (chain, position, task) -> id
    chains = [[rng.randint(1, 4) for _ in range(rng.randint(2, 5))]
              for _ in range(rng.randint(1, 3))]
    tasks = [(c, g, i) for c, gs in enumerate(chains) for g, n in enumerate(gs) for i in range(n)]
    ident = {t: k for k, t in enumerate(tasks)}
    roots = [ident[c, 0, i] for c, gs in enumerate(chains) for i in range(gs[0])]
    m.atomics = {"head": 0, "tail": len(roots)}
    for k in range(len(tasks)):
        m.atomics["q", k] = roots[k] if k < len(roots) else -1
    for c, gs in enumerate(chains):
        for g in range(1, len(gs)):
            m.atomics["pending", c, g] = gs[g - 1]
    done = []
    arrived = [0] * n_wg
    generation = [0] * n_wg
    shared = [None] * n_wg

    def barrier(cu):
        g = generation[cu]
        arrived[cu] += 1
        if arrived[cu] == WAVES:
            arrived[cu], generation[cu] = 0, g + 1
        while generation[cu] == g:
            yield

    def wait(wave):
        while m.flying[wave]:
            yield

    def release(wave):
        yield from wait(wave)
        if without != "release":
            m.write_back(m.xcd(wave[0]))
        yield

    def wavefront(cu, w):
        wave = (cu, w)
        m.flying[wave] = []
        while True:
            if w == 0:
                slot = m.add("head", 1)
                yield
                t = -1
                if slot < len(tasks):
                    while (t := m.atomics["q", slot]) < 0:
                        yield
                shared[cu] = t
                if without != "acquire":
                    m.acquire(cu)
                yield
            yield from barrier(cu)
            t = shared[cu]
            yield from barrier(cu)
            if t < 0:
                return
            c, g, i = tasks[t]
            if g:
                for j in range(chains[c][g - 1]):
                    for v in range(WAVES):
                        for k in range(WORDS):
                            yield
                            if m.load(cu, (c, (g - 1) % 2, j, v, k)) != (c, g - 1, j, v, k):
                                raise Wrong(f"task {t} reads an old value")
            for k in range(WORDS):
                m.flying[wave].append(((c, g % 2, i, w, k), (c, g, i, w, k)))
                yield
            if w == 0:
                done.append(t)
            if without != "wait":
                yield from wait(wave)
            yield from barrier(cu)
            if w == 0:
                yield from release(wave)
                if g + 1 < len(chains[c]) and m.add(("pending", c, g + 1), -1) == 1:
                    n = chains[c][g + 1]
                    base = m.add("tail", n)
                    yield from release(wave)
                    m.acquire(cu)
                    for j in range(n):
                        m.atomics["q", base + j] = ident[c, g + 1, j]
                        yield

    live = [wavefront(cu, w) for cu in range(n_wg) for w in range(WAVES)]
    steps = 0
    while live:
        steps += 1
        assert steps < 200000, "the grid does not drain"
        if rng.random() < 0.3:
            m.something()
            continue
        x = rng.choice(live)
        try:
            next(x)
        except StopIteration:
            live.remove(x)
    assert sorted(done) == list(range(len(tasks))), "every task runs once"


@pytest.mark.parametrize("n_wg", [1, 2, 4])
def test_every_task_reads_what_its_predecessors_wrote(n_wg):
    for seed in range(150):
        run(seed, n_wg)


@pytest.mark.parametrize("without", ["wait", "release", "acquire"])
def test_a_missing_step_is_noticed(without):
    noticed = 0
    for seed in range(60):
        try:
            run(seed, 4, without)
        except Wrong:
            noticed += 1
    assert noticed >= 5, noticed

"""The untimed steps of bench.py capture every graph that its timed region replays, for any
number of steps and whichever buffer they start from (a host model of cpic_evolve's stretches
and buffers in their pipelined form)."""
import math

import pytest

import bench


class Event:
    def __init__(self, n, cur, piped):
        self.n, self.cur, self.piped, self.graphs, self.captured = n, cur, piped, set(), 0

    def step(self, k):
        self.n += k
        self.cur ^= k & 1

    def evolve(self, tau):
        f = tau / bench.DTAU_FM
        left = math.ceil(f - 1e-9 * f) - self.n
        while left > 0:
            k = min(left, 16, 16 - self.n % 16)
            piped = self.piped and k >= 2
            key = (piped, self.n % 16 == 0, self.cur, k)
            self.captured += key not in self.graphs
            self.graphs.add(key)
            self.cur ^= (k % 3 != 0) if piped else k & 1
            self.n += k
            left -= k


@pytest.mark.parametrize("piped", [False, True])
def test_timed_region_captures_nothing(piped):
    for steps in list(range(1, 300)) + [400, 500, 600]:
        for first in range(16):
            for cur in (0, 1):
                w, n_kt = bench.plan_steps(steps, 5 + first, 69)
                ctx = Event(w + n_kt, cur, piped)
                bench.capture_graphs(ctx, steps)
                n = ctx.n
                bench.skip_watch(ctx, steps)
                assert ctx.n <= n + 48 and (steps > 51 or ctx.n // 64 == (ctx.n + steps) // 64)
                assert ctx.n + steps <= 1024
                ctx.captured = 0
                ctx.evolve((ctx.n + steps) * bench.DTAU_FM * (1 - 1e-12))
                assert ctx.captured == 0, (steps, first, cur)

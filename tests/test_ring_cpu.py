"""The ring kernels' host geometry and their exchange protocol, on the CPU."""
from __future__ import annotations

import random

import pytest

from paper_2607_16100_amd import llcoll as ll

AR, RS, AG, BCAST, REDUCE = range(5)
ENTRIES, PACKET, FLAG = 4, 1024, 64


@pytest.mark.parametrize("mode", [AR, RS, AG, BCAST, REDUCE])
def test_ring_shape_fits_its_area(mode):
    """Slots and completion flags end inside the area, every tile has a wave,
    and no wave is left over beyond a workgroup's rounding."""
    rng = random.Random(mode)
    served = 0
    for _ in range(4000):
        p, per_wg, max_wg = rng.randrange(2, 9), rng.choice([1, 2, 4]), rng.randrange(0, 700)
        tiles = int(2 ** rng.uniform(0, 22)) if rng.random() < 0.95 else 0
        area = int(2 ** rng.uniform(6, 33))
        st, (t, waves, slot, flags) = ll.ll_ring_shape(p, mode, tiles, area, per_wg, max_wg)
        if st != ll.LL_OK:
            assert st == ll.LL_ERR_UNSUPPORTED
            continue
        served += 1
        assert t == tiles and 0 < waves <= max_wg * per_wg and waves % per_wg == 0
        assert flags == slot * (p - 1) and slot * (p - 1) < 1 << 32
        assert flags + (p - 1) * waves * FLAG <= area
        steps = -(-tiles // waves)
        if mode == BCAST:
            assert slot >= tiles * PACKET
        elif mode != AG:
            assert slot >= waves * ENTRIES * PACKET
        # the waves of a rank take the same number of steps, give or take one
        assert waves - per_wg < -(-tiles // steps)
    assert served > 500
    assert ll.ll_ring_shape(1, mode, 1, 1 << 20, 2, 8)[0] == ll.LL_ERR_INVALID
    assert ll.ll_ring_shape(8, 5, 1, 1 << 20, 2, 8)[0] == ll.LL_ERR_INVALID


class Wave:
    """One rank's wave: publish tile s, then wait for and consume tile s - 1."""

    def __init__(self, rank, p, steps, epoch):
        self.rank, self.p, self.steps, self.epoch, self.s, self.published = rank, p, steps, epoch, 0, False

    def flag(self, s):
        return self.epoch if s // ENTRIES % 2 == 0 else 0

    def done(self):
        return self.s > self.steps

    def advance(self, ring, got):
        """One action; False if the wave has to wait.  ring[d][s][position] =
        (flag, tile) in rank d's slot from rank s."""
        if not self.published:
            if self.s < self.steps:
                for d in range(self.p):
                    if d != self.rank:
                        ring[d][self.rank][self.s % ENTRIES] = (self.flag(self.s), self.s)
            self.published = True
            return True
        if self.s > 0:
            t = self.s - 1
            for q in range(self.p):
                if q != self.rank and (q, t) not in got:
                    flag, tile = ring[self.rank][q][t % ENTRIES]
                    if flag != self.flag(t):
                        continue
                    assert tile == t, f"rank {self.rank} took tile {tile} of rank {q} for tile {t}"
                    got.add((q, t))
            if any((q, t) not in got for q in range(self.p) if q != self.rank):
                return False
        self.s, self.published = self.s + 1, False
        return True


def run_call(rng, ring, p, steps, epoch, wave=Wave):
    """One call's waves (one a rank) on the ring, in a random order."""
    waves = [wave(r, p, steps, epoch) for r in range(p)]
    got = [set() for _ in range(p)]
    bias = [rng.random() ** 3 + 1e-3 for _ in range(p)]  # some ranks run far more often than others
    stuck = 0
    while not all(w.done() for w in waves):
        w = rng.choices(waves, bias)[0]
        if w.done():
            continue
        stuck = 0 if w.advance(ring, got[w.rank]) else stuck + 1
        assert stuck < 100_000, "the waves wait for each other"
    assert all(len(g) == (p - 1) * steps for g in got)


class LibraryWave(Wave):
    """The same with the flag values of the library."""

    def flag(self, s):
        return ll.ll_ring_flag(self.epoch, s)


@pytest.mark.parametrize("p", [2, 3])
def test_a_call_runs_after_one_with_a_later_epoch(p):
    """A call captured into a graph runs when the graph does, perhaps after
    calls with later epochs: it must find none of its own flags in the ring,
    whatever the steps of those calls, so a call writes no flag but its own
    epoch and 0, which is no call's epoch."""
    rng = random.Random(p)
    for steps in (1, 4, 5, 8, 9, 13):
        ring = [[[(0, -1)] * ENTRIES for _ in range(p)] for _ in range(p)]
        run_call(rng, ring, p, steps, 8, LibraryWave)
        assert {f for d in ring for s in d for f, _ in s} <= {0, 8}
        run_call(rng, ring, p, 9, 7, LibraryWave)
    for epoch in (1, 2, 0xFFFFFFFF):
        assert [ll.ll_ring_flag(epoch, s) for s in range(13)] == [Wave(0, 2, 13, epoch).flag(s) for s in range(13)]


@pytest.mark.parametrize("p", [2, 3, 8])
def test_ring_protocol_under_any_schedule(p):
    """Whatever the order in which the ranks' waves run, every wave consumes
    the right tile from every peer (no position is overwritten before it was
    read, no stale flag is taken for a current one) and all of them finish.
    Calls follow each other on one ring with growing epochs, epoch 1 first."""
    rng = random.Random(p)
    for trial in range(60):
        ring = [[[(0, -1)] * ENTRIES for _ in range(p)] for _ in range(p)]
        epoch = 1
        for call in range(4):
            run_call(rng, ring, p, rng.choice([0, 1, 2, 3, 4, 5, 8, 9, 13, 17]), epoch)
            epoch += rng.choice([1, 1, 2, 7])


def test_three_positions_are_too_few():
    """The schedule test can fail: with three positions a fast rank overwrites
    a tile that a slow peer has not read."""
    global ENTRIES
    keep, ENTRIES = ENTRIES, 3
    try:
        with pytest.raises(AssertionError):
            test_ring_protocol_under_any_schedule(3)
    finally:
        ENTRIES = keep

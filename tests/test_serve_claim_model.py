"""CPU model of how serve_loop's workgroups find, claim and report tiles, with device
copies of the descriptors, step by step under any interleaving.

Every access to shared memory by thread 0 of a workgroup, and every write of the
host's admit / reap, is one step of a generator; a scheduler picks the next step.
What the kernel does, in its order:
  * the publication count is relayed: one workgroup in a few reads the host's word and
    raises the device's, the others read that and the host's only now and then;
  * a request's claim word (tag, tiles handed out) that still carries an older tag is
    re-tagged by compare-and-swap, tried until it succeeds or the word's tag is no
    longer older; the winner has tile 0, reads the host's descriptor and stores the
    device copy (marker, fields, number);
  * the others wait for the copy a bounded number of times, then read the host's
    descriptor seqlock-style, and hand out the remaining tiles by fetch_add;
  * an add that lands after the slot was re-tagged has taken a tile of the later
    request, which is run.
Checked at the end of a run: every tile of every request ran once, with its own
request's descriptor; every request was completed once, after all its tiles; no add
found an older tag; nothing hung.

``retry=False`` tries the compare-and-swap once.  It also fails when a workgroup that
lags on the slot's completed request lands its add between the load and the swap: the
word then still carries the older tag, and the add that follows takes a tile of no
request at all (the kernel would stop serving with a device error).
"""
import collections
import random

import pytest

WRITING = float("inf")  # the descriptor's "being rewritten" marker (kDescWriting)
FIELDS = ("ntiles", "target", "rid")


class Sim:
    def __init__(self, ntiles, slots, retry=True, copy_tries=3):
        self.ntiles_of, self.slots, self.retry, self.copy_tries = list(ntiles), slots, retry, copy_tries
        # host memory
        self.published = 0
        self.desc = [dict(seq=-1, ntiles=0, target=0, rid=-1) for _ in range(slots)]
        self.complete = [0] * slots
        self.slot_total = [0] * slots
        # device memory, cleared before the first launch
        self.pub = 0
        self.claim = [(0, 0)] * slots
        self.done = [0] * slots
        self.ready = [0] * slots
        self.copy = [dict(ntiles=0, target=0, rid=-1) for _ in range(slots)]
        # what happened
        self.runs = collections.Counter()
        self.finalized = collections.Counter()
        self.errors = []
        self.at = {}  # worker -> its last step
        self.seen = set()  # (worker, step) taken so far

    def host(self):
        for seq, nt in enumerate(self.ntiles_of):
            s = seq % self.slots
            while seq >= self.slots and self.complete[s] < seq - self.slots + 1:
                yield "host_wait"
            d = self.desc[s]
            d["seq"] = WRITING
            yield "host"
            self.slot_total[s] += nt
            for name, value in zip(FIELDS, (nt, self.slot_total[s], seq)):
                d[name] = value
                yield "host"
            d["seq"] = seq
            yield "host"
            self.published = seq + 1
            yield "host"

    def worker(self, wid):
        slots, n_req = self.slots, len(self.ntiles_of)
        seq, pub, nt_seq, ntiles, idle = 0, 0, None, 0, 0
        nxt, nxt_seq, cur, cur_seq, open_count = None, None, None, None, 0

        def report():
            nonlocal open_count
            s = cur_seq % slots
            self.done[s] += open_count
            open_count = 0
            if self.done[s] == cur["target"]:
                rid = cur["rid"]
                missing = [t for t in range(self.ntiles_of[rid]) if self.runs[(rid, t)] == 0]
                if missing:
                    self.errors.append("request %d completed before tiles %s ran" % (rid, missing))
                self.finalized[rid] += 1
                self.complete[s] = cur_seq + 1

        while True:
            yield ("top", seq)
            if seq >= n_req:
                return
            if seq >= pub:
                p = self.pub
                yield "read"
                if p <= pub and (wid == 0 or idle % 8 == 7):
                    p = self.published
                    yield "read"
                    if p > pub:
                        self.pub = max(self.pub, p)
                        yield "relay"
                pub = max(pub, p)
            if seq >= pub:
                idle += 1
                continue
            idle = 0
            s = seq % slots
            yield ("before_load", seq)
            v = self.claim[s]
            yield ("loaded", seq)
            won = False
            while v[0] < seq and (self.retry or nt_seq != seq):
                if self.claim[s] == v:
                    self.claim[s] = (seq, 1)
                    won = True
                    yield "swapped"
                    break
                v = self.claim[s]
                yield ("swap_failed", seq)
                if not self.retry:
                    break
            got, moved_on = None, False
            if won:
                nxt = {}
                for name in FIELDS:
                    nxt[name] = self.desc[s][name]
                    yield "read"
                self.ready[s] = 0
                yield "marker"
                for name in FIELDS:
                    self.copy[s][name] = nxt[name]
                    yield "write"
                self.ready[s] = seq + 1
                yield "number"
                nt_seq = nxt_seq = seq
                ntiles = nxt["ntiles"]
                got = (seq, 0)
            else:
                if nt_seq != seq:
                    for _ in range(self.copy_tries if seq else 0):
                        a = self.ready[s]
                        yield "read"
                        if a == seq + 1:
                            nxt = {}
                            for name in FIELDS:
                                nxt[name] = self.copy[s][name]
                                yield "read"
                            b = self.ready[s]
                            yield "read"
                            nxt_seq = None
                            if b == seq + 1:
                                nt_seq = nxt_seq = seq
                                ntiles = nxt["ntiles"]
                                break
                        t = self.claim[s][0]
                        yield "read"
                        if t != seq:
                            break
                if nt_seq != seq:
                    a = self.desc[s]["seq"]
                    yield "read"
                    nt = self.desc[s]["ntiles"]
                    yield "read"
                    b = self.desc[s]["seq"]
                    yield "read"
                    if not (a == seq and b == seq):
                        if open_count and cur_seq == seq:
                            report()
                        seq += 1
                        continue
                    nt_seq, ntiles = seq, nt
                v = self.claim[s]
                yield ("before_add", seq)
                if v[0] > seq or v[1] >= ntiles:
                    moved_on = True
                else:
                    ws, wc = self.claim[s]
                    self.claim[s] = (ws, wc + 1)
                    yield ("added", seq)
                    if ws < seq:
                        self.errors.append("workgroup %d added to request %d's word with tag %d" % (wid, seq, ws))
                        return
                    if ws == seq:
                        got = (seq, wc) if wc < ntiles else None
                        moved_on = got is None
                    else:  # a later request took the slot: tile wc is one of its
                        later = seq = ws
                        pub = max(pub, later + 1)
                        while True:
                            ds = self.desc[s]["seq"]
                            yield "read"
                            if ds != WRITING and ds < later:
                                continue
                            a = self.desc[s]["seq"]
                            yield "read"
                            lnt = self.desc[s]["ntiles"]
                            yield "read"
                            b = self.desc[s]["seq"]
                            yield "read"
                            held = a == later and b == later
                            if held or ds != later:
                                break
                        nt_seq, ntiles = (later, lnt) if held else (None, 0)
                        got = (later, wc) if held and wc < lnt else None
                        moved_on = got is None
            if got is not None:
                if got[0] != cur_seq:
                    if nxt_seq == got[0]:
                        cur = dict(nxt)
                    else:
                        cur = {}
                        for name in FIELDS:
                            cur[name] = self.desc[s][name]
                            yield "read"
                    cur_seq = got[0]
                open_count += 1
                if cur["rid"] != got[0]:
                    self.errors.append("workgroup %d ran tile %d of request %d with request %d's descriptor"
                                       % (wid, got[1], got[0], cur["rid"]))
                self.runs[(cur["rid"], got[1])] += 1
                yield "tile"
            elif moved_on:
                if open_count and cur_seq == seq:
                    report()
                seq += 1

    def check(self, hung):
        errs = list(self.errors)
        if hung:
            errs.append("hung: requests not completed %s" % [r for r in range(len(self.ntiles_of)) if not self.finalized[r]])
        for r, nt in enumerate(self.ntiles_of):
            errs += ["request %d tile %d ran %d times" % (r, t, self.runs[(r, t)]) for t in range(nt) if self.runs[(r, t)] != 1]
            if self.finalized[r] != 1:
                errs.append("request %d completed %d times" % (r, self.finalized[r]))
        return errs


def run(sim, nworkers, rng, holds=(), stall=0.0, max_steps=200000):
    """Random interleaving.  holds: (worker, step, wake) keeps that worker at that step
    until wake(sim).  stall: the chance that a worker is held after a step, for up to
    2,000 steps of the others."""
    gens = {"host": sim.host()}
    gens.update({w: sim.worker(w) for w in range(nworkers)})
    until = {}  # worker -> step number it sleeps to
    for step in range(max_steps):
        if sim.errors or not gens:
            break
        held = {w for w, tag, wake in holds if sim.at.get(w) == tag and not wake(sim)}
        runnable = [k for k in gens if k not in held and until.get(k, 0) <= step]
        if not runnable:
            awake = [k for k in gens if k not in held]
            if not awake:
                break
            until.clear()
            continue
        key = rng.choice(runnable)
        try:
            sim.at[key] = next(gens[key])
            sim.seen.add((key, sim.at[key]))
        except StopIteration:
            del gens[key]
            continue
        if key != "host" and rng.random() < stall:
            until[key] = step + rng.randint(1, 2000)
    return sim.check(hung=bool(gens))


def late_add_case(retry, seed):
    """One slot.  Worker 1 sleeps between its load of request 0's word and its add while
    worker 2 runs that request and the host republishes the slot; its add then lands
    between worker 0's load of the word, still tagged 0, and worker 0's swap."""
    sim = Sim([3, 7, 2], slots=1, retry=retry)
    holds = [
        (0, ("before_load", 0), lambda s: s.published >= 2),             # takes no part in request 0
        (2, ("before_load", 0), lambda s: s.at.get(1) == ("before_add", 0)),
        (1, ("before_add", 0), lambda s: (0, ("loaded", 1)) in s.seen),  # its add waits for worker 0's load
        (0, ("loaded", 1), lambda s: (1, ("added", 0)) in s.seen),       # its swap waits for that add
    ] + [(w, ("before_load", 1), lambda s: s.seen & {(0, ("added", 1)), (0, "swapped")}) for w in (1, 2)]
    return run(sim, 3, random.Random(seed), holds)


@pytest.mark.parametrize("seed", range(5))
def test_a_late_add_breaks_the_single_try(seed):
    errs = late_add_case(False, seed)
    assert any("with tag 0" in e for e in errs), errs


@pytest.mark.parametrize("seed", range(20))
def test_a_late_add_with_the_swap_retried(seed):
    assert late_add_case(True, seed) == []


@pytest.mark.parametrize("slots,nworkers", [(1, 2), (1, 4), (2, 3), (3, 5), (4, 8)])
@pytest.mark.parametrize("stall", [0.0, 0.02])
def test_random_interleavings(slots, nworkers, stall):
    for seed in range(40):
        rng = random.Random(7919 * slots + 101 * nworkers + seed)
        ntiles = [rng.randint(1, 7) for _ in range(12)]
        errs = run(Sim(ntiles, slots, copy_tries=rng.choice([1, 3, 64])), nworkers, rng, stall=stall)
        assert errs == [], (seed, ntiles, errs)

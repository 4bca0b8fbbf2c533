"""Model check of the pipelined event loop's protocol (ssa_kernel_pl, ssa_kernel_ph).

The waves of a workgroup are step machines whose steps are the kernel's LDS
accesses, in the kernel's order; a random scheduler interleaves them. The waits
that the kernel places make each wave's accesses take effect in program order,
which is what the model assumes. A slot of the ring carries, in the place of a
draw, the (trajectory, event) that it was made for, and in the place of a state
the (trajectory, event) that the event wave computed, so the checks are direct:
whatever the clock and row waves use has to be of the trajectory that the lane
holds, of the right event, and of the batch that they work on. Every trajectory
has to run exactly once and every wave has to leave.

The counters of the kernel carry the lower words of batch numbers. They have
`BITS` bits here instead of 32, so that trajectories run through their wrap many
times. `whole=False` is the protocol with lower words throughout, which the
first wrap without a restart breaks: it shows that the model sees the fault.
"""
import random

import pytest

BITS = 8
LOW = (1 << BITS) - 1
TAG = LOW >> 2          # a ready word holds two flags beside the batch
B = 4                   # events of a batch


class Broken(AssertionError):
    pass


def need(ok, what):
    if not ok:
        raise Broken(what)


def signed(v):
    v &= LOW
    return v - LOW - 1 if v >> (BITS - 1) else v


class Shared:
    def __init__(self, nb, lanes):
        self.nb = nb
        self.ready = [0] * nb
        self.flags = [None] * nb
        self.next = self.done_e = self.done_c = self.gen = self.leave = 0
        self.done_s = -64 & LOW       # nothing is drawn before the first claim
        self.sw = [0, 0]
        self.upper = [0, 0]
        self.rmask = self.live = frozenset()
        self.t_id, self.t_off, self.t_x, self.t_k = ([None] * lanes for _ in range(4))
        self.draw = [[None] * lanes for _ in range(nb)]
        self.result = [[None] * lanes for _ in range(nb)]


def draw_wave(sh, lanes, whole):
    gen, b64, sw = 0, 0, 0
    ids, offs = [None] * lanes, [0] * lanes
    while True:
        b = sh.next
        sh.next = (b + 1) & LOW
        yield
        b64 += (b - b64) & LOW
        while True:
            done, leave = sh.done_s, sh.leave
            yield
            if leave:
                return
            if signed(b - done) < sh.nb:
                break
        g = sh.gen
        yield
        if g != gen:
            gen = g
            hi = sh.sw[1]
            yield
            sw = (hi << BITS) + sh.sw[0]
            for i in range(lanes):
                yield
                ids[i] = sh.t_id[i]
                yield
                offs[i] = sh.t_off[i]
        for i in range(lanes):
            yield
            sh.draw[b64 % sh.nb][i] = (ids[i], None if offs[i] is None else offs[i] + b64 * B)
        yield
        top = b >> (BITS - 1)
        if b & (LOW >> 1) == 1 << (BITS - 2):
            sh.upper[top ^ 1] = (b64 >> BITS) + top
            yield
        mark = b64 == sw if whole else b == sw & LOW
        sh.ready[b64 % sh.nb] = ((b + 1) & TAG) << 1 | mark
        yield


def event_wave(sh, lanes, whole, rng, careful):
    held = [None] * lanes      # (trajectory, its next event)

    def acquire(b):
        while True:
            v, leave = sh.ready[b % sh.nb], sh.leave
            yield
            if v >> 1 == (b + 1) & TAG:
                return v & 1
            if leave:
                return None

    mark = yield from acquire(0)
    if mark is None:
        return
    b = 0
    while True:
        slot = b % sh.nb
        if mark:
            rm = sh.rmask
            yield
            for i in rm:
                held[i] = sh.t_x[i]
                yield
        out = []
        for i in range(lanes):
            got = sh.draw[slot][i]
            yield
            out.append((held[i], got, b))
            if held[i] is not None:
                held[i] = (held[i][0], held[i][1] + B)
        sh.done_e = b & LOW        # the batch before is in place
        yield
        mark = yield from acquire(b + 1)
        if mark is None:
            return
        if rng.random() < careful:   # the batch again, with draws formed from the tables
            for i in range(lanes):
                tid = sh.t_id[i]
                yield
                off = sh.t_off[i]
                yield
                low = b & LOW
                upper = sh.upper[low >> (BITS - 1)] if whole else 0
                yield
                n = None if off is None else off + ((upper << BITS) + low) * B
                out[i] = (out[i][0], (tid, n), b)
        for i in range(lanes):
            sh.result[slot][i] = out[i]
            yield
        b += 1


def clock_wave(sh, lanes, whole, queue, lengths, starts, ran):
    act, hold = set(), set()
    held = [None] * lanes
    st = dict(sw=0, gen=0, pending=False, changed=False)

    def claim(at):
        fresh = set()
        for i in range(lanes):
            if i in act or i in hold or not queue:
                continue
            t = queue.pop(0)
            off = starts[t] - at * B
            held[i] = [t, starts[t]]
            for table, v in ((sh.t_k, t), (sh.t_id, t), (sh.t_off, off), (sh.t_x, (t, starts[t]))):
                table[i] = v
                yield
            fresh.add(i)
            hold.add(i)
        st.update(sw=at, gen=st["gen"] + 1, pending=True, changed=False)
        sh.rmask = frozenset(fresh)
        yield
        sh.live = frozenset(act | hold)
        yield
        sh.sw[0] = at & LOW
        yield
        sh.sw[1] = at >> BITS
        yield
        sh.gen = st["gen"]
        yield

    yield from claim(0)
    sh.done_s = 0
    yield
    b = e_done = 0
    while act or hold or queue:
        if signed(e_done - b) <= 0:
            sh.done_c = b & LOW
            while True:
                yield
                e_done = sh.done_e
                if signed(e_done - b) > 0:
                    break
        restart = st["pending"] and b & LOW == st["sw"] & LOW    # (pending: at most a ring ahead)
        if restart:
            act |= hold
            hold.clear()
            st["pending"] = False
        slot = b % sh.nb
        was = frozenset(act)
        got = []
        for i in range(lanes):
            got.append(sh.result[slot][i])
            yield
        e_now = sh.done_e
        yield
        sh.done_c = b & LOW
        e_done = e_now
        for i in sorted(act):
            t, n = held[i]
            state, drawn, batch = got[i]
            need(batch == b, f"the clock wave takes batch {batch} for {b}")
            need(state == (t, n), f"state of {state} for trajectory {t}, event {n}")
            need(drawn == (t, n), f"draw of {drawn} for trajectory {t}, event {n}")
            held[i][1] = n + B
            if n + B > starts[t] + lengths[t]:
                need(t not in ran, f"trajectory {t} ended twice")
                ran.add(t)
                act.discard(i)
                st["changed"] = True
        sh.flags[slot] = (b, was, [h and h[0] for h in held], restart)
        yield
        if st["changed"] and not st["pending"]:
            done = sh.done_s
            yield
            later = b - ((b - done) & LOW) > st["sw"] if whole else signed(done - st["sw"]) > 0
            if later:
                yield from claim(b + sh.nb)
        b += 1
    sh.done_c = b & LOW
    yield
    sh.leave = 1
    yield


def row_wave(sh, lanes):
    held = [None] * lanes
    b = c_done = 0
    while True:
        while signed(c_done - b) <= 0:
            leave = sh.leave
            yield
            c_done = sh.done_c
            yield
            if signed(c_done - b) > 0:
                break
            if leave:
                return
        batch, was, trajectories, restart = sh.flags[b % sh.nb]
        yield
        need(batch == b, f"the row wave takes batch {batch} for {b}")
        if restart:
            rm = sh.rmask
            yield
            for i in rm:
                held[i] = sh.t_k[i]
                yield
        for i in was:
            state, _, at = sh.result[b % sh.nb][i]
            yield
            need(at == b and state[0] == held[i] == trajectories[i], f"rows of {state} for {held[i]}")
        sh.done_s = (b + 1) & LOW
        yield
        b += 1


def simulate(seed, nb, lengths, whole=True, lanes=3, draws=3, careful=0.2):
    rng = random.Random(seed)
    sh = Shared(nb, lanes)
    starts = [rng.choice((0, 7, 1 << 40)) for _ in lengths]
    ran = set()
    waves = [clock_wave(sh, lanes, whole, list(range(len(lengths))), lengths, starts, ran),
             event_wave(sh, lanes, whole, rng, careful), row_wave(sh, lanes)]
    waves += [draw_wave(sh, lanes, whole) for _ in range(draws)]
    speed = [rng.choice((0.1, 1.0, 1.0, 5.0)) for _ in waves]
    live = list(range(len(waves)))
    for step in range(40_000_000):
        if not live:
            break
        w = rng.choices(live, [speed[i] for i in live])[0]
        try:
            for _ in range(rng.choice((1, 1, 2, 8))):
                next(waves[w])
        except StopIteration:
            live.remove(w)
        if step % 4096 == 0:
            speed = [rng.choice((0.1, 1.0, 1.0, 5.0)) for _ in waves]
        need(whole or step < 3_000_000, "a wave waits for a counter that has wrapped")
    need(not live, "a wave never leaves")
    need(ran == set(range(len(lengths))), "a trajectory has not run")


@pytest.mark.parametrize("seed", range(12))
@pytest.mark.parametrize("nb", [4, 5, 6, 16])
def test_every_trajectory_gets_its_own_draws(nb, seed):
    rng = random.Random(100 * nb + seed)
    simulate(seed, nb, [rng.choice((0, 1, B - 1, B, 5 * B, rng.randrange(40 * B))) for _ in range(rng.randrange(1, 25))])


@pytest.mark.parametrize("nb", [4, 16])
@pytest.mark.parametrize("batches", [LOW // 2 - 1, LOW // 2 + 3, LOW - 1, LOW + 1, LOW + 2, 2 * LOW + 40])
def test_trajectories_that_outlast_the_counters(nb, batches):
    """No restart while the counters wrap, or one just before and after: a lane is restarted
    at its own batch number, not at the one that looks like it."""
    simulate(3, nb, [batches * B, 2 * B, (batches + 9) * B + 1, B, batches * B])


@pytest.mark.parametrize("batches", [LOW + 2, 2 * LOW + 40])
def test_the_model_sees_a_restart_by_lower_words(batches):
    with pytest.raises(Broken):
        simulate(3, 4, [batches * B, batches * B, batches * B], whole=False)


@pytest.mark.parametrize("careful", [1.0])
def test_the_model_sees_an_event_index_by_lower_words(careful):
    with pytest.raises(Broken):
        simulate(5, 6, [(LOW + 60) * B, 3 * B], whole=False, lanes=1, careful=careful)

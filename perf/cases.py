"""Timed workloads of the ensemble direct method, from the smallest calls to the largest.

Every case is one call of a public entry point (`ssa_ensemble_run`, or
`ssa_ensemble_run_noalloc` on buffers that the caller keeps) on a network of
`workloads.py` or `experiments.py`. A case names

  network   what is simulated (`NETWORKS` below)
  mode      the precision configuration
  n_traj    trajectories; with sets > 1, of all parameter sets together
  sets      parameter sets of the sweep (1: the network's own constants)
  t_end     horizon
  n_snap    evenly spaced snapshot rows (1: the end state alone)
  entry     "run" or "noalloc"
  record    entries of the event record of a trajectory (0: none)
  block, grid, chunks, window, place
            launch options as `ssa_ensemble_run` takes them (0: its own choice)

Inputs of a seed: the Philox key of the run and, in a sweep, the rate table.
"""
import numpy as np
import torch

from paper_2605_00479_amd import ssa
from paper_2605_00479_amd import workloads as wl

OPEN_BASE = (50.0, 0.1, 0.001, 0.5)
PAPER_REPRESSILATOR = dict(alpha0=1.0, alpha=216.0, K=1.0, h=2, dm=1.0, beta=5.0, dp=1.0)

# name -> [(model, initial counts, events of a trajectory in one unit of time)]
NETWORKS = {
    "birth_death": lambda: [(wl.birth_death(), (0,), 19.0)],
    "schlogl": lambda: [(wl.schlogl(), (250,), 4300.0)],
    "telegraph": lambda: [(wl.telegraph(), (1, 0, 0), 13.0)],
    "telegraph_bimodal": lambda: [(wl.telegraph(0.05, 0.05, 20.0, 1.0), (1, 0, 0), 20.0)],
    "telegraph_sweep": lambda: [(wl.telegraph(0.01, 0.1, 5.0, 1.0), (1, 0, 0), 2.0)],
    "dimer_sweep": lambda: [(wl.dimer_open(*OPEN_BASE), (0, 0), 870.0)],
    "dimer_closed": lambda: [(wl.dimer_closed(1e-3, 0.1), (100, 0), 4.0)],
    "repressilator": lambda: [(wl.repressilator(**PAPER_REPRESSILATOR), (0, 0, 0, 5, 0, 0), 400.0)],
    "five": lambda: [(wl.birth_death(), (0,), 19.0), (wl.schlogl(), (250,), 5000.0), (wl.telegraph(), (1, 0, 0), 11.0),
                     (wl.dimer_open(*OPEN_BASE), (0, 0), 200.0),
                     (wl.repressilator(), (0, 0, 0, 0, 0, 20), 250.0)],
}

# per-trajectory event caps (about 64 times the mean count over the network's longest horizon here)
CAPS = {"birth_death": 250_000, "schlogl": 3_000_000, "telegraph": 500_000, "telegraph_bimodal": 2_000_000,
        "telegraph_sweep": 500_000, "dimer_sweep": 3_000_000, "dimer_closed": 500_000, "repressilator": 5_000_000,
        "five": 20_000_000}


def _case(name, network, mode, n_traj, t_end, n_snap, sets=1, entry="run", record=0, block=0, grid=0, chunks=1,
          window=0, place=0):
    c = dict(network=network, mode=mode, n_traj=n_traj, t_end=t_end, n_snap=n_snap, sets=sets, entry=entry,
             record=record, block=block, grid=grid, chunks=chunks, window=window, place=place)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a call of a serving loop: a few hundred short trajectories into buffers the caller
        # keeps, no multiple of a wave; launches and host work are most of it
        _case("serve_257", "birth_death", "FP64", 257, 2.0, 3, entry="noalloc"),
        # the smallest ensemble the experiments accept, one call that allocates its outputs
        _case("dimer_closed_64", "dimer_closed", "FP32", 64, 100.0, 1),
        # the birth-death configuration: fewer waves than the chip has SIMDs
        _case("birth_death_10k", "birth_death", "FP64", 10_000, 100.0, 1),
        # Schloegl at the paper's ensemble size: long chains, a seventh of the chip's lanes
        _case("schlogl_10k", "schlogl", "FP64", 10_000, 10.0, 1),
        # the Schloegl configuration in mixed precision, more trajectories than lanes
        _case("schlogl_100k", "schlogl", "MIX_F16_SR", 100_000, 10.0, 101),
        # the paper's bimodal telegraph table in uniform bfloat16
        _case("telegraph_50k", "telegraph_bimodal", "UNI_BF16_SR", 50_000, 200.0, 1),
        # the telegraph configuration with propensity normalisation: a saturated chip, many refills
        _case("telegraph_1m", "telegraph", "UNI_F16_SR_NORM", 1_000_000, 200.0, 201),
        # dwell times: an event record beside the end state, round to nearest
        _case("dwell_20k", "telegraph_bimodal", "MIX_F16_RTN", 20_000, 1000.0, 1, record=96),
        # the repressilator table (Hill laws, six species) in uniform fp16
        _case("repressilator_10k", "repressilator", "UNI_F16_SR", 10_000, 100.0, 1),
        # a sweep over 256 parameter sets in binary64 as a program calls it without tuning
        _case("dimer_sweep_64k", "dimer_sweep", "FP64", 256 * 256, 25.0, 26, sets=256),
        # the benchmark's sweep in the launch its tuner picks
        _case("dimer_sweep_1m", "dimer_sweep", "MIX_F16_SR", 4096 * 256, 50.0, 51, sets=4096, block=512, grid=256,
              chunks=2, window=7, place=197),
        # five networks of unequal work in one launch
        _case("five_100k", "five", "MIX_BF16_SR", 100_000, 50.0, 51),
    ]


# network -> modes, trajectories (least, most), horizon (shortest, longest)
_RANGES = {
    "birth_death": (("FP64", "MIX_F16_SR"), (1, 300_000), (1.0, 200.0)),
    "schlogl": (("FP64", "MIX_F16_SR", "MIX_F16_RTN", "MIX_BF16_SR"), (64, 100_000), (0.2, 10.0)),
    "telegraph": (("FP64", "UNI_F16_SR_NORM", "UNI_BF16_SR"), (64, 1_000_000), (5.0, 200.0)),
    "telegraph_bimodal": (("MIX_F16_RTN", "UNI_BF16_SR"), (64, 50_000), (20.0, 1000.0)),
    "telegraph_sweep": (("UNI_F16_SR", "FP64"), (90, 180_000), (20.0, 400.0)),
    "dimer_sweep": (("FP64", "MIX_F16_SR"), (256, 200_000), (1.0, 25.0)),
    "dimer_closed": (("FP32", "MIX_BF16_SR"), (64, 300_000), (5.0, 100.0)),
    "repressilator": (("UNI_F16_SR", "FP64"), (64, 10_000), (5.0, 100.0)),
    "five": (("MIX_BF16_SR", "FP64"), (500, 100_000), (1.0, 50.0)),
}


def _log_uniform(rng, lo, hi):
    return float(np.exp(rng.uniform(np.log(lo), np.log(hi))))


def draw(rng):
    """One more call: any network, precision and size of the ranges, odd sizes as often as round ones."""
    network = rng.choice(sorted(_RANGES))
    modes, (lo, hi), (t_lo, t_hi) = _RANGES[network]
    mode = rng.choice(modes)
    n = int(round(_log_uniform(rng, lo, hi)))
    t_end = round(_log_uniform(rng, t_lo, t_hi), 2)
    n_snap = rng.choice((1, 1, 3, rng.randint(2, 120)))
    sets = 1
    if network == "dimer_sweep":
        sets = max(1, n // rng.choice((16, 64, 256)))
    if network == "telegraph_sweep":
        sets = 9
    record = rng.choice((0, 16, 96)) if network == "telegraph_bimodal" else 0
    chunks = rng.choice((1, 1, 1, 2, 4)) if n_snap >= 8 else 1
    # (the fixed scratch memory of the allocation-free entry holds the carry state of any size here)
    entry = rng.choice(("run", "run", "noalloc"))
    return _case(None, network, mode, n, t_end, n_snap, sets=sets, entry=entry, record=record, chunks=chunks)


def _counts(case):
    """Trajectories of each network of the launch."""
    parts = len(NETWORKS[case["network"]]())
    n = case["n_traj"] // parts
    return [n] * (parts - 1) + [case["n_traj"] - n * (parts - 1)]


def prepare(case, seed):
    items = []
    for (spec, x0, _), n in zip(NETWORKS[case["network"]](), _counts(case)):
        it = {"model": ssa.Model(spec), "x0": np.array(x0, np.int32), "n_traj": n}
        if case["sets"] > 1:
            sets = case["sets"]
            if case["network"] == "dimer_sweep":
                it["set_rates"] = wl.dimer_sweep_rates(sets, seed, OPEN_BASE)
            else:
                k_on = np.logspace(-3, -1, sets) * (1.0 + 1e-3 * (seed % 97))
                it["set_rates"] = np.stack([k_on, np.full(sets, 0.1), np.full(sets, 5.0), np.full(sets, 1.0)], axis=1)
            it["traj_per_set"] = -(-n // sets)
        if case["record"]:
            it["record"] = (0b11, case["record"])
        items.append(it)
    t_end = case["t_end"]
    snap_t = np.array([t_end]) if case["n_snap"] == 1 else wl.snapshot_grid(t_end, case["n_snap"])
    state = {"items": items, "args": (t_end, snap_t, seed, case["mode"]), "entry": case["entry"],
             "kw": dict(max_events=CAPS[case["network"]], n_chunks=case["chunks"], block_size=case["block"],
                        grid_size=case["grid"], first_window=case["window"], placement=case["place"])}
    if case["entry"] == "noalloc":
        dev = torch.device("cuda", torch.cuda.current_device())
        state["out"] = []
        for it in items:
            e, n_sp = it["n_traj"], it["model"].n_species
            o = (torch.empty((snap_t.size, n_sp, e), dtype=torch.int32, device=dev),
                 torch.empty(e, dtype=torch.int64, device=dev),
                 torch.empty(e, dtype=torch.float64, device=dev),
                 torch.empty(e, dtype=torch.uint8, device=dev))
            if case["record"]:
                # rows past a trajectory's count are not written: they stay zero
                o += (torch.zeros((e, case["record"]), dtype=torch.float64, device=dev),
                      torch.zeros((e, case["record"]), dtype=torch.uint8, device=dev),
                      torch.empty(e, dtype=torch.int32, device=dev))
            state["out"].append(o)
        # that entry takes a kernel that an ordinary run has loaded: one event of each trajectory
        few = [dict(it, n_traj=1) for it in items]
        ssa.ssa_ensemble_run(few, t_end, [t_end], seed, case["mode"], max_events=1).wait()
    return state


def _named(o):
    return dict(zip(("snap", "n_events", "t_last", "status", "rec_t", "rec_j", "rec_n"), o))


def _counted(o):
    """An item's outputs with the record's entries past a trajectory's count, which are undefined, as zero."""
    if len(o) > 4:
        t, j, n = o[4:]
        kept = torch.arange(t.shape[1], device=t.device)[None, :] < n[:, None]
        o = o[:4] + (torch.where(kept, t, 0.0), torch.where(kept, j, 0), n)
    return _named(o)


def run(state):
    if state["entry"] == "noalloc":
        ssa.ssa_ensemble_run_noalloc(state["items"], *state["args"], state["out"], **state["kw"])
        return [_named(o) for o in state["out"]]
    # the run is given back once its outputs are taken, as the experiments do
    r = ssa.ssa_ensemble_run(state["items"], *state["args"], **state["kw"])
    return [_counted(r.tensors(i)) for i in range(len(state["items"]))]


def work(case):
    """Outputs written once, rates read once; an event is one Philox4x32-10 call (10 rounds of two
    32 x 32 products, four exclusive ors and two key additions), a logarithm (about 25 operations), a
    division, and per reaction its propensity, a sum, a comparison and its part of the update."""
    nbytes, flops = 0.0, 0.0
    for (spec, _, rate), n in zip(NETWORKS[case["network"]](), _counts(case)):
        m = spec.n_reactions
        nbytes += n * (4.0 * case["n_snap"] * spec.n_species + 17.0) + 8.0 * case["sets"] * m
        if case["record"]:
            nbytes += n * (9.0 * min(case["record"], 0.05 * case["t_end"]) + 4.0)
        events = n * (1.0 + rate * case["t_end"])
        per_reaction = 4.0 + float(spec.order.sum()) / m + float((spec.law != wl.LAW_MASS_ACTION).mean()) * 6.0
        flops += events * (10 * 8.0 + 25.0 + 10.0 + m * per_reaction)
    return {"bytes": nbytes, "flops": flops}


def _philox(n, ident, seed):
    """Words 0..3 of Philox4x32-10 at counter (n, 0, ident, 0), as uint64 arrays."""
    low = np.uint64(0xFFFFFFFF)
    c0, c1 = np.asarray(n, np.uint64), np.zeros_like(ident)
    c2, c3 = ident.copy(), np.zeros_like(ident)
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = c0 * np.uint64(0xD2511F53), c2 * np.uint64(0xCD9E8D57)
        c0, c1, c2, c3 = ((p1 >> np.uint64(32)) ^ c1 ^ np.uint64(k0), p1 & low,
                          (p0 >> np.uint64(32)) ^ c3 ^ np.uint64(k1), p0 & low)
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def exact(case, seed):
    """The direct method in numpy's binary64 with its own logarithm, one array step an event of every
    trajectory: the clock of the last event. Counts and statuses are whole numbers, and a reduced-precision
    trajectory is not an approximation of a binary64 one: those have no such value."""
    if case["mode"] != "FP64" or case["network"] != "birth_death" or case["n_traj"] > 20_000:
        return None
    kb, kd = 10.0, 0.1
    n_traj, t_end = case["n_traj"], case["t_end"]
    ident = np.arange(n_traj, dtype=np.uint64)
    x, t = np.zeros(n_traj), np.zeros(n_traj)
    t_last = np.zeros(n_traj)
    live = np.arange(n_traj)
    event = 0
    while live.size:
        w0, w1, w2, w3 = _philox(event, ident[live], seed)
        u1 = (((w0 << np.uint64(21)) | (w1 >> np.uint64(11))).astype(np.float64) + 1.0) * 2.0 ** -53
        u2 = (((w2 << np.uint64(21)) | (w3 >> np.uint64(11))).astype(np.float64) + 1.0) * 2.0 ** -53
        total = kb + kd * x[live]
        t_new = t[live] - np.log(u1) / total
        fires = t_new <= t_end
        live, t_new, up = live[fires], t_new[fires], (kb > u2 * total)[fires]
        x[live] += np.where(up, 1.0, -1.0)
        t[live] = t_last[live] = t_new
        event += 1
    return [{"snap": None, "n_events": None, "t_last": t_last, "status": None}]

"""What a program that uses this framework has it do, as cases that can be timed.

Five kinds of work, each through the package's public entry points:

  sample      first-passage runs of one instance or of a batch (``run``, ``run_batch``, ``run_single_abi``): every
              potential, closed-form and learned biases, host and device results, with and without a dump of the runs;
  records     the replay of sampled runs into training records (``proposal_records``);
  loss_grad   the training objective and its gradient from records (``proposal_loss_grad``);
  train       a whole training round: sampling, replay and Adam steps (``train_proposal``);
  forward     the learned bias at given points (``mlp_forward``).

Sizes are those of ``workloads.py``, ``bench.py`` and the tests, with fewer runs where a pass would take seconds.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2206_11234_amd as fpt
from paper_2206_11234_amd.api import RECORD_DTYPE

PHI_END = math.sqrt(2.0)
N_PARAMS = 4481
POTENTIALS = {"quadratic": fpt.POT_QUADRATIC, "bump": fpt.POT_QUADRATIC_BUMP, "flat": fpt.POT_FLAT}
BIASES = {"none": fpt.BIAS_NONE, "noise": fpt.BIAS_NOISE_SCALED, "power": fpt.BIAS_POWER, "learned": fpt.BIAS_MLP}

# The far-tail setting of the learned proposal: m = 1, phi_in = 6, reflecting wall at 8.
DIFFUSION = {"pot": "quadratic", "m": 1.0, "phi_in": 6.0, "phi_uv": 8.0, "dN": 1e-3}


def listed():
    return [
        # a first look at a new setting: some hundred direct runs, results in host memory
        dict(name="direct_first_look", kind="sample", pot="quadratic", m=0.01, phi_in=5.0, phi_uv=0.0, dN=1e-3, bias="none",
             A=0.0, p=1, n_inst=1, n_traj=500, n_bins=100, dump=0, entry="abi"),
        # direct sampling at the paper's smallest useful size, every run dumped for a scatter plot
        dict(name="direct_dumped", kind="sample", pot="quadratic", m=0.01, phi_in=5.0, phi_uv=0.0, dN=1e-3, bias="none",
             A=0.0, p=1, n_inst=1, n_traj=10_000, n_bins=100, dump=10_000, entry="run"),
        # the paper's 2e5 runs: drift-dominated, its optimised power-law bias
        dict(name="drift_power_bias", kind="sample", pot="quadratic", m=0.001, phi_in=math.sqrt(42.0), phi_uv=0.0, dN=1e-3,
             bias="power", A=5e-6, p=3, n_inst=1, n_traj=200_000, n_bins=150, dump=0, entry="run"),
        # the paper's 2e5 runs: diffusion-dominated, wall at the start, noise-scaled bias
        dict(name="diffusion_wall", kind="sample", pot="quadratic", m=1.0, phi_in=math.sqrt(42.0), phi_uv=math.sqrt(42.0),
             dN=1e-3, bias="noise", A=0.4, p=1, n_inst=1, n_traj=200_000, n_bins=160, dump=0, entry="run"),
        # the fixed-bias sweep of the benchmark: six instances in one launch, its launch shape
        dict(name="fixed_bias_sweep", kind="sample", pot="sweep", bias="noise", n_inst=6, n_traj=100_000, n_bins=200, dump=0,
             entry="run", block=512, wg_per_cu=2),
        # multi-bias reconstruction on the bump potential: seven amplitudes, 500 bins each, dN = 1e-4
        dict(name="bump_multi_bias", kind="sample", pot="bump", m=0.05, phi_in=8.0, phi_uv=12.0, dN=1e-4, bias="noise", A=0.0,
             p=1, n_inst=7, n_traj=10_000, n_bins=500, dump=0, entry="run", block=512, wg_per_cu=2),
        # a parameter scan: 64 different instances in one launch
        dict(name="scan_64", kind="sample", pot="scan", bias="noise", n_inst=64, n_traj=2_000, n_bins=200, dump=0, entry="run",
             pick=0),
        # the learned proposal's evaluation runs, network every 16 steps, the benchmark's launch shape
        dict(name="learned_every_16", kind="sample", **DIFFUSION, bias="learned", A=0.9, p=16, n_inst=1, n_traj=100_000,
             n_bins=200, dump=0, entry="run", block=256, wg_per_cu=3),
        # one network aimed at three targets in one launch, evaluated every 4 steps
        dict(name="learned_batch_every_4", kind="sample", **DIFFUSION, bias="learned", A=0.6, p=4, n_inst=3, n_traj=20_000,
             n_bins=200, dump=0, entry="run"),
        # the replay of one round's window runs into records, one in four kept
        dict(name="replay_window", kind="records", **DIFFUSION, A=0.9, every=16, stride=4, pool=20_000, n_paths=600,
             centre=60.0),
        # the second-moment objective and its gradient from the records of one small round
        dict(name="second_moment_gradient", kind="loss_grad", n_paths=700, groups=1_400, objective=0, every=16, stride=1),
        # one round of training at a far window: sample, replay, 40 Adam steps on the cross entropy
        dict(name="training_round", kind="train", **DIFFUSION, A=0.9, every=16, stride=4, n_sample=30_000, n_paths=4_000,
             steps=40, centre=60.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw(rng):
    kind = rng.choice(["sample"] * 7 + ["records", "loss_grad", "train", "forward"])
    if kind == "loss_grad":
        objective = rng.choice([0, 1])
        return dict(kind=kind, n_paths=_log_int(rng, 40, 4_000), groups=_log_int(rng, 60, 3_000), objective=objective,
                    every=rng.choice([4, 8, 16]), stride=1 if objective == 0 else rng.choice([1, 4]))
    if kind == "forward":
        return dict(kind=kind, n=_log_int(rng, 1_000, 4_000_000), every=16)
    if kind == "records":
        return dict(kind=kind, **DIFFUSION, A=round(rng.uniform(0.7, 1.0), 3), every=rng.choice([4, 8, 16]),
                    stride=rng.choice([1, 4]), pool=20_000, n_paths=_log_int(rng, 48, 250), centre=rng.choice([20.0, 40.0, 60.0]))
    if kind == "train":
        return dict(kind=kind, **DIFFUSION, A=round(rng.uniform(0.7, 1.0), 3), every=rng.choice([8, 16]), stride=4,
                    n_sample=_log_int(rng, 8_000, 30_000), n_paths=_log_int(rng, 500, 4_000), steps=rng.randint(5, 40),
                    centre=rng.choice([20.0, 40.0, 60.0]))
    pot = rng.choice(["quadratic", "quadratic", "quadratic", "bump", "flat", "scan", "sweep", "learned", "learned"])
    c = dict(kind=kind, pot=pot, bias="noise", n_inst=1, n_traj=_log_int(rng, 100, 300_000), n_bins=rng.randint(60, 500), dump=0,
             entry=rng.choice(["run", "run", "abi", "noalloc"]))
    if pot == "scan":
        c.update(n_inst=rng.randint(2, 64), pick=rng.randrange(1 << 16), n_traj=_log_int(rng, 200, 4_000), entry="run")
    elif pot == "sweep":
        c.update(n_inst=6, n_traj=_log_int(rng, 1_000, 100_000), entry="run")
    elif pot == "learned":
        c.update(DIFFUSION, bias="learned", A=round(rng.uniform(0.4, 0.95), 3), p=rng.choice([1, 4, 8, 16]),
                 n_inst=rng.choice([1, 1, 1, 3]), n_traj=_log_int(rng, 500, 60_000))
        # one host-buffer entry takes closed-form launch shapes only; the static scratch holds tables of about 300 bins
        if c["n_inst"] > 1 or c["n_bins"] > 300 or c["entry"] == "abi":
            c["entry"] = "run"
    elif pot == "flat":
        c.update(m=1.0, phi_in=1.0, phi_uv=1.5, dN=1e-2, A=round(rng.uniform(-2.0, 0.0), 3), p=1)
    elif pot == "bump":
        c.update(m=0.05, phi_in=round(rng.uniform(5.0, 9.0), 3), phi_uv=12.0, dN=rng.choice([1e-3, 1e-4]),
                 A=round(rng.uniform(0.0, 4.0), 3), p=1, n_traj=_log_int(rng, 100, 100_000))
    else:
        phi = round(rng.uniform(3.0, 10.0), 3)
        m = rng.choice([0.001, 0.01, 0.1, 1.0])
        c.update(m=m, phi_in=phi, phi_uv=rng.choice([0.0, phi, phi + 2.0]) if m < 1.0 else phi + rng.choice([0.0, 1.0]),
                 dN=rng.choice([1e-3, 5e-4]), bias=rng.choice(["none", "noise", "power"]),
                 A=round(rng.uniform(0.1, 0.5), 3) if m == 1.0 else round(rng.uniform(0.5, 3.0), 3), p=rng.choice([1, 2, 3]))
        if c["bias"] == "power":
            c["A"] = round(c["A"] * m / 15.4 / phi ** (c["p"] - 1), 9)      # of the noise-scaled bias's size at the start
    if rng.random() < 0.3 and c["n_inst"] == 1 and c["entry"] != "abi":
        c["dump"] = min(c["n_traj"], 20_000)
    return c


def draw(rng):
    while True:
        c = _draw(rng)
        if work(c)["flops"] <= _MOST:
            return c


# ---------------------------------------------------------------------------
# instances
# ---------------------------------------------------------------------------
def _moments(c):
    """Mean and standard deviation of N under the drift that the runs are drawn with: backward recursion of
    T'(y) = int_y^uv (2/S^2) e^(Phi(z) - Phi(y)) dz, Phi' = 2 mu / S^2 (mu the whole drift), and of the variance's
    derivative, whose source is 2 T'^2.  Without a wall the upper end lies a few units above the start."""
    end = 0.0 if c["pot"] == "flat" else PHI_END
    top = c["phi_uv"] or c["phi_in"] + 3.0
    x = np.linspace(end, top, 8_001)
    h = x[1] - x[0]
    mid = 0.5 * (x[1:] + x[:-1])
    S = np.full_like(mid, math.sqrt(1.0 / 3.0) / (2 * math.pi)) if c["pot"] == "flat" else c["m"] * mid / (2 * math.pi * math.sqrt(6.0))
    mu = np.zeros_like(mid) if c["pot"] == "flat" else -2.0 / mid
    if c["bias"] in ("noise", "learned"):
        mu = mu + c["A"] * S
    elif c["bias"] == "power":
        mu = mu + c["A"] * mid ** c["p"]
    a = 2.0 * mu / S ** 2
    grow = np.exp(np.clip(a * h, -700.0, 700.0))
    cell = np.where(np.abs(a * h) < 1e-9, h, (grow - 1.0) / np.where(a == 0.0, 1.0, a))
    d1 = d2 = 0.0
    mean = var = 0.0
    grow, cell, add = grow.tolist(), cell.tolist(), ((2.0 / S ** 2) * cell).tolist()
    for i in range(len(mid) - 1, -1, -1):
        d1 = d1 * grow[i] + add[i]
        if d1 > 1e100:
            return 1e12, 1e12
        d2 = d2 * grow[i] + 2.0 * d1 * d1 * cell[i]
        if x[i] < c["phi_in"] - 0.5 * h:
            mean += d1 * h
            var += d2 * h
    return mean, math.sqrt(var)


def _k_max(mean, dN):
    return int(min(1 << 20, 64 * math.ceil(mean / dN)))


def _single(c):
    """The settings of a case of one potential, without its amplitude: N's mean and spread give bins and step cap."""
    mean, sd = _moments(c)
    plain, _ = _moments(dict(c, bias="none"))
    k_max = _k_max(plain, c["dN"])
    hi = min(mean + 10.0 * sd, k_max * c["dN"])
    lo = min(max(mean - 6.0 * sd, 0.05 * mean), 0.25 * hi) if mean - 6.0 * sd < 0.05 * mean else mean - 6.0 * sd
    return dict(pot=POTENTIALS[c["pot"]], m=c["m"], phi_in=c["phi_in"], phi_end=0.0 if c["pot"] == "flat" else PHI_END,
                phi_uv=c["phi_uv"] or math.inf, dN=c["dN"], k_max=k_max, V0=1.0, a=0.02, phi0=4.0, w=0.1,
                edges=np.geomspace(lo, max(hi, 1.01 * lo), c["n_bins"] + 1)), mean / c["dN"]


def _network(c, seed):
    """A network of trained size whose bias stays near A: Glorot-uniform hidden layers, a small last one."""
    rng = np.random.default_rng(seed)
    v = np.zeros(N_PARAMS, np.float32)
    v[0:192] = rng.uniform(-0.3, 0.3, 192)
    v[192:256] = rng.uniform(-0.1, 0.1, 64)
    v[256:4352] = rng.uniform(-0.216, 0.216, 4096)
    v[4352:4416] = rng.uniform(-0.1, 0.1, 64)
    v[4416:4480] = rng.uniform(-0.02, 0.02, 64)
    v[4480] = c.get("A", 0.9)
    b = v.view(np.uint32).astype(np.uint64)
    bits = ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint16)
    return SimpleNamespace(bf16_bits=lambda: bits, values=(bits.astype(np.uint32) << 16).view(np.float32), in_mean=(5.0, 196.0, 196.0),
                           in_inv_scale=(0.4, 0.005, 0.01), out_scale=1.0, eval_every=int(c.get("every", c.get("p", 16))))


def _instances(c, seed=0):
    """(instances, expected steps of all their runs)."""
    out, steps = [], 0.0
    if c["pot"] == "sweep":       # drift-dominated A = 1, 2, 4 without a wall, then diffusion-dominated with one
        for m, phi, uv in ((0.01, 10.0, 0.0), (1.0, 6.0, 8.0)):
            base = dict(c, pot="quadratic", m=m, phi_in=phi, phi_uv=uv, dN=1e-3, p=1)
            for A in (1.0, 2.0, 4.0):
                s, k = _single(dict(base, A=A))
                out.append(dict(s, bias=fpt.BIAS_NOISE_SCALED, A=A))
                steps += _capped(k, s["k_max"])
    elif c["pot"] == "scan":      # phi_in in [3, 12], masses, amplitudes, wall or none, two steps
        rng = random.Random(c["pick"])
        for _ in range(c["n_inst"]):
            phi = rng.uniform(3.0, 12.0)
            m, A = rng.choice((0.01, 0.1, 0.5, 1.0)), float(rng.randrange(7))
            b = dict(c, pot="quadratic", m=m, A=A, phi_in=phi, phi_uv=rng.choice((0.0, phi + 2.0)), dN=rng.choice((1e-3, 5e-4)), p=1)
            n_cl = (phi ** 2 - PHI_END ** 2) / 4.0
            k_max = _k_max(n_cl, b["dN"])
            out.append(dict(pot=POTENTIALS["quadratic"], m=m, A=A, bias=fpt.BIAS_NOISE_SCALED if A else fpt.BIAS_NONE, phi_in=phi,
                            phi_end=PHI_END, phi_uv=b["phi_uv"] or math.inf, dN=b["dN"], k_max=k_max,
                            edges=np.geomspace(0.25 * n_cl, k_max * b["dN"], c["n_bins"] + 1)))
            drift = A * m / (2.0 * math.pi * math.sqrt(6.0))
            far = drift * phi ** 2 >= 2.0             # the bias outweighs the drift: runs reach the cap
            steps += k_max if far else min(n_cl if not drift else -math.log((2.0 - drift * phi ** 2) / (2.0 - drift * PHI_END ** 2)) /
                                           (2.0 * drift), k_max * b["dN"]) / b["dN"]
    else:
        s, k = _single(c)
        for i in range(c["n_inst"]):
            more = {}
            if c["bias"] == "learned":
                if i == 0:
                    net = _network(c, seed)
                more = dict(mlp=net, target_N=196.0 - 20.0 * i)
            A = c["A"] + (i if c["n_inst"] > 1 and c["bias"] != "learned" else 0.0)
            bias = BIASES[c["bias"]] if A or c["bias"] == "learned" else fpt.BIAS_NONE
            out.append(dict(s, bias=bias, A=A, p=c["p"], **more))
            steps += _capped(k, s["k_max"])
    for i, s in enumerate(out):
        s.update(n_traj=c["n_traj"], stream=i)
    return [SimpleNamespace(**s) for s in out], steps * c["n_traj"]


def _capped(k, k_max):
    """Mean of min(k, k_max) for a roughly exponential k."""
    return k * -math.expm1(-k_max / k) if k > 0.05 * k_max else k


def _learned_instance(c, seed, n_traj):
    net = _network(c, seed)
    return SimpleNamespace(pot=fpt.POT_QUADRATIC, m=c["m"], phi_in=c["phi_in"], phi_end=PHI_END, phi_uv=c["phi_uv"], dN=c["dN"],
                           k_max=555_712, n_traj=n_traj, stream=3, bias=fpt.BIAS_MLP, mlp=net, target_N=c["centre"],
                           edges=np.linspace(0.0, 400.0, 201))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _made_records(c, seed):
    """Records as a replay gives them: fields between the end and the wall, k in steps of the group, H a sum of n
    increments r dN + sqrt(dN) xi, ln w_0 spread over a few units."""
    rng = np.random.default_rng(seed)
    per = rng.integers(c["groups"] // 2, c["groups"] + 1, c["n_paths"])
    off = np.zeros(c["n_paths"] + 1, np.uint64)
    off[1:] = np.cumsum(per)
    n = int(off[-1])
    path = np.repeat(np.arange(c["n_paths"], dtype=np.uint32), per)
    rec = np.zeros(n, RECORD_DTYPE)
    rec["phi"] = rng.uniform(1.5, 8.0, n).astype(np.float32)
    rec["k"] = ((np.arange(n) - off[path].astype(np.int64)) * (c["every"] * c["stride"])).astype(np.uint32)
    sd = math.sqrt(1e-3 * c["every"])
    rec["H"] = (0.9e-3 * c["every"] + sd * rng.standard_normal(n)).astype(np.float32)
    rec["pn"] = (path << np.uint32(5)) | np.uint32(c["every"])
    return SimpleNamespace(rec=rec, off=off), 2.0 * rng.standard_normal(c["n_paths"]) - 60.0


def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind == "sample":
        instances, _ = _instances(c, seed)
        return {"case": c, "instances": instances, "seed": seed}
    if kind == "loss_grad":
        recs, lw0 = _made_records(c, seed)
        net = _network(c, seed)
        theta = net.values + np.random.default_rng(seed + 1).normal(0.0, 1e-4, N_PARAMS).astype(np.float32)
        return {"case": c, "net": net, "theta": theta.astype(np.float32), "recs": recs, "lw0": lw0}
    if kind == "forward":
        rng = np.random.default_rng(seed)
        return {"case": c, "net": _network(c, seed), "phi": rng.uniform(1.4, 8.0, c["n"]).astype(np.float32),
                "N": rng.uniform(0.0, 300.0, c["n"]).astype(np.float32)}
    inst = _learned_instance(c, seed, c["pool"] if kind == "records" else c["n_sample"])
    if kind == "train":
        return {"case": c, "inst": inst, "seed": seed, "theta": inst.mlp.values}
    # the runs of a pool that ended in the window, as a sampling pass with a dump leaves them
    _, dump, _ = fpt.run(inst, seed, block=256, wg_per_cu=1, chunk=1, dump_n=c["pool"])
    lo, hi = (c["centre"] + 6.0 * s for s in (-1, 1))
    ids = np.nonzero((dump.status == fpt.ST_ENDED) & (dump.k * c["dN"] > lo) & (dump.k * c["dN"] <= hi))[0]
    ids = ids[_with_sum(-(-dump.k[ids].astype(np.int64) // (c["every"] * c["stride"])), c["n_paths"],
                        round(c["n_paths"] * c["centre"] / c["dN"] / (c["every"] * c["stride"])))]
    return {"case": c, "inst": inst, "seed": seed, "ids": ids.astype(np.uint64), "k": dump.k[ids].astype(np.uint64)}


def _with_sum(sizes, n, total):
    """n of the runs whose record counts sum to the same total for every seed: the first ones, then those that steer the
    sum back, then a pair that closes it."""
    steer = min(40, n - 2)
    take = list(range(n - 2 - steer))
    left = dict.fromkeys(range(n - 2 - steer, len(sizes)))
    total -= int(sizes[take].sum())
    for i in range(steer):
        rest = np.fromiter(left, int)
        j = int(rest[np.argmin(np.abs(sizes[rest] - total / (steer + 2 - i)))])
        take.append(j)
        total -= int(sizes[j])
        del left[j]
    rest = np.fromiter(left, int)
    a, b = np.nonzero(np.triu(sizes[rest][:, None] + sizes[rest][None, :] == total, 1))
    return np.array(take + [int(rest[a[0]]), int(rest[b[0]])])


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
_ROWS = ("lse_w", "lse_w2", "jk_lse_w", "mean_lnw", "m2_lnw", "m3_lnw", "m4_lnw", "log_p", "rel_err_jk", "rel_err_kish", "log_p_ln",
         "rel_err_ln_lo", "rel_err_ln_hi", "normal_p")
_WHOLE = ("lse_w_all", "lse_w2_all", "lse_wk", "lse_wk2", "sum_k2", "pearson_r")


def _tables(results, dumps):
    """All tables of all results, each kind in an array of its own."""
    out = {f: np.concatenate([getattr(r, f).ravel() for r in results]) for f in _ROWS}
    out.update({f: np.array([getattr(r, f) for r in results]) for f in _WHOLE})
    out["ess"] = np.concatenate([r.ess() for r in results])
    out["accepted"] = np.array([int(r.lognormal_accepted()) for r in results])
    out["counts"] = np.concatenate([r.counts for r in results]).view(np.int64)
    if dumps:
        out["dump"] = [[d.k.astype(np.int64), d.lw, d.phi, d.status] for d in dumps]
    return out


def run(state):
    c, kind = state["case"], state["case"]["kind"]
    if kind == "sample":
        shape = {k: c[k] for k in ("block", "wg_per_cu") if k in c}
        if c["entry"] == "abi":
            return _tables([fpt.run_single_abi(state["instances"][0], state["seed"])], None)
        if shape:
            shape["chunk"] = 1
        if c["dump"]:
            shape["dump_n"] = c["dump"]
        results, dumps, _ = fpt.run_batch(state["instances"], state["seed"], noalloc=c["entry"] == "noalloc", **shape)
        return _tables(results, dumps)
    if kind == "loss_grad":
        stride = c["stride"]
        return fpt.proposal_loss_grad(state["net"], 196.0, 1e-3, state["theta"], state["recs"], state["lw0"], 2e5,
                                      objective=c["objective"], temper=0.5, rec_weight=float(stride))
    if kind == "forward":
        return fpt.mlp_forward(state["net"], 196.0, state["phi"], state["N"])
    if kind == "records":
        r = fpt.proposal_records(state["inst"], state["seed"], state["ids"], state["k"], c["every"], c["stride"])
        return [r.rec[f] for f in ("phi", "k", "H", "pn")] + [r.k.astype(np.int64), r.lw, r.status]
    theta, _, reports = fpt.train_proposal(state["inst"], state["seed"], state["theta"], window=(c["centre"] - 6.0, c["centre"] + 6.0),
                                           n_sample=c["n_sample"], rounds=1, steps=c["steps"], max_paths=c["n_paths"], lr=1e-3,
                                           objective=1, temper=0.5, stride=c["stride"])
    return [theta] + [{k: r[k] for k in ("n_window", "n_used", "n_records", "loss_first", "loss_last", "kish_window")} for r in reports]


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
_STEP = 50.0              # flops of a step: noise, drift, weight, boundaries
_NET = 2.0 * N_PARAMS     # one evaluation of the network


def work(case):
    c, kind = case, case["kind"]
    if kind == "sample":
        instances, steps = _instances(c)
        rows = sum(len(i.edges) + 3 for i in instances)
        flops = steps * _STEP + (steps / c["p"] * _NET if c["bias"] == "learned" else 0.0)
        return {"bytes": rows * 16 * 16 + rows * 16 * 8 + 20.0 * c["dump"] * len(instances), "flops": flops}
    if kind == "loss_grad":
        n = 0.75 * c["n_paths"] * c["groups"]
        return {"bytes": 16.0 * n + 16.0 * c["n_paths"] + 12.0 * N_PARAMS, "flops": 3.0 * _NET * n}
    if kind == "forward":
        return {"bytes": 12.0 * c["n"], "flops": _NET * c["n"]}
    k = c["centre"] / c["dN"]
    records = c["n_paths"] * k / (c["every"] * c["stride"])
    flops = c["n_paths"] * k * (_STEP + _NET / c["every"])
    if kind == "records":
        return {"bytes": 16.0 * records, "flops": flops}
    _, steps = _instances(dict(c, bias="learned", p=c["every"], n_inst=1, n_traj=c["n_sample"], n_bins=10))
    return {"bytes": 16.0 * records * (c["steps"] + 2),
            "flops": flops + steps * (_STEP + _NET / c["every"]) + records * _NET * (3.0 * c["steps"] + 2.0)}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _net64(theta, inputs):
    """r and the layers' outputs of the network in 64 bits; `theta` with gradients where they are asked for."""
    W1, b1, W2, b2, w3, b3 = (theta[a:b] for a, b in ((0, 192), (192, 256), (256, 4352), (4352, 4416), (4416, 4480), (4480, 4481)))
    h = torch.tanh(inputs @ W1.reshape(64, 3).T + b1)
    h = torch.tanh(h @ W2.reshape(64, 64).T + b2)
    return h @ w3 + b3


def _inputs64(net, phi, N, target, dev):
    x = torch.stack([torch.as_tensor(np.asarray(v, np.float64), device=dev) for v in (phi, N, np.full(len(phi), target))], 1)
    mean = torch.tensor([float(np.float32(v)) for v in net.in_mean], dtype=torch.float64, device=dev)
    inv = torch.tensor([float(np.float32(v)) for v in net.in_inv_scale], dtype=torch.float64, device=dev)
    return (x - mean) * inv


def exact(case, seed):
    """Sampling, replay and training have no value in 64 bits: where a run stops is decided by binary32 steps, and another
    rounding gives other runs."""
    c = case
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if c["kind"] == "forward":
        s = prepare(c, seed)
        theta = torch.as_tensor(s["net"].values.astype(np.float64), device=dev)
        with torch.no_grad():
            return _net64(theta, _inputs64(s["net"], s["phi"], s["N"], 196.0, dev)).cpu().numpy()
    if c["kind"] != "loss_grad":
        return None
    s = prepare(c, seed)
    rec, n_paths = s["recs"].rec, c["n_paths"]
    dN = float(np.float32(1e-3))
    lw0 = torch.as_tensor(s["lw0"], device=dev)
    theta = torch.as_tensor(s["theta"].astype(np.float64), device=dev).requires_grad_(True)
    path = torch.as_tensor((rec["pn"] >> 5).astype(np.int64), device=dev)
    n = torch.as_tensor((rec["pn"] & 31).astype(np.float64), device=dev)
    H = torch.as_tensor(rec["H"].astype(np.float64), device=dev)
    x = _inputs64(s["net"], rec["phi"], rec["k"].astype(np.float64) * dN, 196.0, dev)
    parts = [slice(i, i + (1 << 17)) for i in range(0, rec.size, 1 << 17)]

    def terms(p):
        r = _net64(theta, x[p])
        return (-r * H[p] + r * r * n[p] * (0.5 * dN)) * c["stride"]

    lw = torch.zeros(n_paths, dtype=torch.float64, device=dev)
    with torch.no_grad():
        for p in parts:
            lw.index_add_(0, path[p], terms(p))
        a = 0.5 * lw0 + (lw if c["objective"] == 0 else 0.0)
        weight = torch.softmax(a, 0)
        loss = (torch.logsumexp(a, 0) - math.log(2e5)) if c["objective"] == 0 else (weight * lw).sum()
    for p in parts:
        (weight[path[p]] * terms(p)).sum().backward()
    return float(loss), theta.grad.cpu().numpy(), lw.cpu().numpy()


_MOST = max(work(c)["flops"] for c in listed())

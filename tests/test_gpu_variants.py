"""The variants of the step, record and training kernels at the edges of the rules that choose them:
walls in some of a batch's instances, every exponent of the power-law bias alone and mixed, runs far from
and at the bump, path counts around a wave's 8, 16, 32 and 64 slots, records around a tile of 64.

Step counts, fields and log-weights are the oracle's bit for bit.  The learned sampler rounds its own way
on the matrix cores, and is compared with itself: a run does not depend on its launch.  The training
network sums 64 terms in binary32, so ln w_theta (a sum of terms r H) and the gradient carry a relative
error of at most about 64 2^-24 = 4e-6 of the sum of the terms' sizes: 1e-4 and 1e-3 of the largest
component bound them, as for the records of whole runs."""
import dataclasses
import math

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import assert_dump_matches, assert_histogram_matches, to_model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fpt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_11234_amd as F
    return F


def _check(fpt, insts, seed=11, **kw):
    n = max(i.n_traj for i in insts)
    results, dumps, _ = fpt.run_batch(insts, seed, dump_n=n, **kw)
    for inst, res, dump in zip(insts, results, dumps):
        tr = O.simulate(to_model(inst), seed, inst.n_traj)
        assert_dump_matches(dump, tr)
        assert_histogram_matches(res, O.histogram(tr, inst.dN, inst.edges))


def _diffusion(wall, n, stream=0, **kw):
    return W.Instance("walls", m=1.0, phi_in=4.0, phi_uv=5.0 if wall else math.inf, phi_esc=0.0 if wall else 6.0,
                      bias=W.BIAS_NOISE_SCALED, A=1.0, dN=1e-3, n_traj=n, stream=stream, edges=np.linspace(0.1, 30, 31), **kw)


@pytest.mark.parametrize("walls", [(True,), (False,), (True, True), (False, False), (True, False), (False, True, True)])
def test_walls_and_escapes(fpt, walls):
    print(f"[case] walls {walls}", flush=True)
    _check(fpt, [_diffusion(w, 90 + 37 * i, stream=i) for i, w in enumerate(walls)])


@pytest.mark.parametrize("ps", [(0,), (1,), (2,), (3,), (4,), (5,), (1, 1), (1, 2), (4, 5, 0)])
def test_power_exponents(fpt, ps):
    print(f"[case] exponents {ps}", flush=True)
    # r = A phi^p / S at phi = 3 of the order of 1e-2 for every p: A = 3e-5 3^-p
    _check(fpt, [W.Instance("power", m=0.01, phi_in=3.0, bias=W.BIAS_POWER, A=3e-5 * 3.0 ** -p, p=p, dN=1e-3, n_traj=70 + i,
                            stream=i, edges=np.linspace(1.6, 1.9, 31)) for i, p in enumerate(ps)])


@pytest.mark.parametrize("a,w,wall,A", [(0.02, 0.1, True, 0.0), (0.02, 0.1, False, 2.0), (-0.02, 0.2, True, 1.0), (0.05, 0.3, True, 3.0),
                                        (0.02, 1e-3, True, 1.0), (0.0, 0.1, False, 1.0)])
@pytest.mark.parametrize("n", [5, 300])
def test_bump_far_and_near(fpt, a, w, wall, A, n):
    """Runs start far from the bump (80 in (phi - phi0)^2 / 2 w^2 is 12.6 w), cross it and end beyond it."""
    print(f"[case] a={a} w={w} wall={wall} A={A} n={n}", flush=True)
    _check(fpt, [W.Instance("bump", pot=W.POT_QUADRATIC_BUMP, m=0.05, a=a, phi0=3.0, w=w, phi_in=5.0,
                            phi_uv=6.0 if wall else math.inf, bias=W.BIAS_NOISE_SCALED if A else W.BIAS_NONE, A=A, dN=1e-3,
                            n_traj=n, k_max=20000, edges=np.linspace(1, 12, 31))])


def test_bump_batch(fpt):
    """Instances whose bumps lie elsewhere share a launch, so that a wave's runs differ in which are far."""
    print("[case] bump batch", flush=True)
    _check(fpt, [W.Instance("bump", pot=W.POT_QUADRATIC_BUMP, m=0.5, a=0.05, phi0=p0, w=0.05, phi_in=4.0, phi_uv=6.0,
                            bias=W.BIAS_NOISE_SCALED, A=1.0, dN=1e-3, n_traj=120, stream=i, k_max=20000, edges=np.linspace(0.5, 12, 31))
                 for i, p0 in enumerate((2.0, 3.0, 4.0, 9.0))])


@pytest.mark.parametrize("every", [1, 4, 16])
def test_learned_runs_do_not_depend_on_the_launch(fpt, every):
    """8, 16, 32 or 64 runs a wave (2048 waves of 8 and 16 runs end at 16384 and 32768), half networks and
    draws ahead or not: a run's every bit is that of the full launch."""
    n_full = 70000
    inst = dataclasses.replace(W.c4_instance(W.c4_params(3, eval_every=every), n_traj=n_full), phi_in=2.5, k_max=2000)
    _, full, _ = fpt.run(inst, 2, dump_n=n_full)
    for n in (1, 7, 9, 513, 16384, 16385, 33000):
        print(f"[case] every={every} n={n}", flush=True)
        _, few, _ = fpt.run(W.with_runs(inst, n), 2, dump_n=n)
        for name in ("k", "lw", "status"):
            assert np.array_equal(getattr(few, name)[:n], getattr(full, name)[:n]), (n, name)


@pytest.mark.parametrize("n_paths", [1, 8, 9, 63, 65, 300])
@pytest.mark.parametrize("proposal,group", [("fixed", 1), ("fixed", 4), ("fixed", 16), ("network", 1), ("network", 4),
                                            ("network", 8), ("network", 16)])
def test_records_of_few_paths(fpt, n_paths, proposal, group):
    print(f"[case] {n_paths} paths {proposal} group {group}", flush=True)
    base = dataclasses.replace(W.c2(1)[3], phi_in=2.5, k_max=3000)
    v = np.zeros(W.MlpParams.N_PARAMS, np.float32)
    v[4480] = 0.5
    inst = base if proposal == "fixed" else dataclasses.replace(
        base, bias=W.BIAS_MLP, A=0.0, target_N=196.0, mlp=W.MlpParams(v, out_scale=2.0, eval_every=group))
    ids = np.arange(n_paths, dtype=np.uint64) * np.uint64(3)
    o = O.records(to_model(inst), 0, ids, group)
    g = fpt.proposal_records(inst, 0, ids, o.k, group)
    assert np.array_equal(g.k, o.k) and np.array_equal(g.lw, o.lw) and np.array_equal(g.status, o.status)
    assert np.array_equal(g.off, o.off) and g.rec.tobytes() == o.rec.tobytes()


def _records(fpt, n_rec, n_paths, seed=4):
    """Records of n_paths paths, some without any."""
    rng = np.random.default_rng(seed)
    cut = np.sort(rng.integers(0, n_rec + 1, n_paths - 1))
    off = np.concatenate([[0], cut, [n_rec]]).astype(np.uint64)
    rec = np.zeros(n_rec, O.RECORD_DTYPE)
    rec["phi"] = rng.uniform(1.5, 8.0, n_rec)
    rec["k"] = rng.integers(0, 200000, n_rec)
    rec["H"] = rng.normal(0.0, 0.06, n_rec)
    owner = np.repeat(np.arange(n_paths), np.diff(off.astype(np.int64)))
    rec["pn"] = (owner.astype(np.uint32) << 5) | rng.integers(1, 17, n_rec).astype(np.uint32)
    z = np.zeros(n_paths)
    return O.Records(rec, off, z.astype(np.uint64), z, z.astype(np.int32)), rng.normal(-3.0, 1.0, n_paths)


@pytest.mark.parametrize("n_rec", [0, 1, 63, 64, 65, 255, 257, 4097])
@pytest.mark.parametrize("objective", [0, 1])
def test_loss_and_gradient_of_ragged_records(fpt, n_rec, objective):
    print(f"[case] {n_rec} records, objective {objective}", flush=True)
    recs, lw0 = _records(fpt, n_rec, 5)
    p = W.c4_params(7, scale=1.5, out_scale=0.8)
    theta = p.values_f32()
    inst = W.c4_instance(p, n_traj=1)
    loss, grad, lwt = fpt.proposal_loss_grad(p, inst.target_N, inst.dN, theta, recs, lw0, 100.0, objective)
    loss_o, grad_o, lwt_o = O.loss_grad(to_model(inst), theta.astype(np.float64), recs, lw0, 100.0, objective)
    assert np.all(np.abs(lwt - lwt_o) <= 1e-4 * np.maximum(1.0, np.abs(lwt_o)))
    assert abs(loss - loss_o) <= 1e-4 * max(1.0, abs(loss_o))
    assert np.abs(grad - grad_o).max() <= 1e-3 * np.abs(grad_o).max()


@pytest.mark.parametrize("where,pn", [(0, 5 << 5 | 4), (4000, 17), (4096, 1 << 5), (77, 0xFFFFFFFF)])
def test_records_out_of_range_are_refused(fpt, where, pn):
    recs, lw0 = _records(fpt, 4097, 5)
    p = W.c4_params(7)
    good = fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), recs, lw0, 100.0)
    recs.rec["pn"][where] = pn
    recs.rec["pn"][where + 1:where + 2] = 0        # the first one is named
    with pytest.raises(Exception, match=f"record {where}:"):
        fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), recs, lw0, 100.0)
    recs, _ = _records(fpt, 4097, 5)
    again = fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), recs, lw0, 100.0)
    assert again[0] == good[0] and np.array_equal(again[1], good[1]) and np.array_equal(again[2], good[2])


def test_bump_too_narrow_for_binary32(fpt):
    """A bump so narrow that (phi - phi0) / w^2 overflows binary32 away from it: its term in the drift is
    infinity times zero there, and a run that gets that far from it never ends.  Such a launch takes no
    group without the bump."""
    print("[case] w=8e-20", flush=True)
    _check(fpt, [W.Instance("bump", pot=W.POT_QUADRATIC_BUMP, m=0.05, a=0.05, phi0=4.0, w=8e-20, phi_in=5.0, phi_uv=6.0,
                            bias=W.BIAS_NOISE_SCALED, A=1.0, dN=1e-2, n_traj=n, k_max=1000, edges=np.linspace(1, 12, 31)) for n in (5, 300)])


@pytest.mark.parametrize("first,second", [(524288 + 3, 524288 + 200), (262144 + 7, 2 * 524288 + 9)])
def test_records_out_of_range_beyond_one_grid(fpt, first, second):
    """The check's threads (2048 a CU, 524 288 on 256 CUs) take several records each: the lowest one out of
    range is named whichever round it falls in."""
    print(f"[case] bad records {first} {second}", flush=True)
    recs, lw0 = _records(fpt, 2 * 524288 + 333, 5)
    p = W.c4_params(7)
    recs.rec["pn"][[first, second]] = 17
    with pytest.raises(Exception, match=f"record {first}:"):
        fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), recs, lw0, 100.0)


def test_log_weights_over_several_pieces(fpt):
    """More records than one piece of the evaluation holds (2^24): ln w_theta of a path is the same bits in
    whichever piece its records lie."""
    print("[case] 2^24 records and more", flush=True)
    few, lw0 = _records(fpt, 100_000, 40)
    copies = 200
    rec = np.tile(few.rec, copies)
    rec["pn"] += np.repeat(np.arange(copies, dtype=np.uint32) * np.uint32(40 << 5), few.rec.size)
    off = np.concatenate([[0]] + [few.off[1:] + np.uint64(c * few.rec.size) for c in range(copies)]).astype(np.uint64)
    assert rec.size > 1 << 24
    p = W.c4_params(7)
    z = np.zeros(40 * copies)
    many = O.Records(rec, off, z.astype(np.uint64), z, z.astype(np.int32))
    _, grad, lwt = fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), few, lw0, 100.0, 1)
    _, grad_n, lwt_n = fpt.proposal_loss_grad(p, 196.0, 1e-3, p.values_f32(), many, np.tile(lw0, copies), 100.0, 1)
    assert np.array_equal(lwt_n.reshape(copies, 40), np.broadcast_to(lwt, (copies, 40)))
    # the weights of each path are those of the few paths over the number of copies: the same gradient, with
    # the binary32 sums of a workgroup 200 times as long (2e5 terms of either sign, within 2^-24 each)
    assert np.abs(grad_n - grad).max() <= 1e-3 * np.abs(grad).max()


@pytest.mark.parametrize("every", [1, 4, 8, 16])
@pytest.mark.parametrize("n_inst", [1, 3])
def test_learned_teams_against_full_waves(fpt, every, n_inst):
    """A launch whose waves hold 64 runs each and refill (one workgroup of four waves per CU, more runs than
    its lanes) evaluates the network on two blocks of 32 columns and draws each lane's normals itself, until
    its waves drain into teams; launches of few runs are teams of 8, 16 and 32 from the start.  A run's every
    bit is the same in both, for one instance and for several of different lengths."""
    n_full = 70000 // n_inst + 1
    base = dataclasses.replace(W.c4_instance(W.c4_params(3, eval_every=every), n_traj=n_full), phi_in=2.5, k_max=2000)
    insts = [dataclasses.replace(base, stream=i, target_N=196.0 - 20.0 * i, k_max=2000 - 300 * i) for i in range(n_inst)]
    print(f"[case] every={every} instances={n_inst} full", flush=True)
    _, full, _ = fpt.run_batch(insts, 2, dump_n=n_full, block=256, wg_per_cu=1, chunk=1)
    for n in (9, 5461, 11000, 22000):
        print(f"[case] every={every} instances={n_inst} n={n}", flush=True)
        _, few, _ = fpt.run_batch([W.with_runs(i, n) for i in insts], 2, dump_n=n)
        for a, b in zip(few, full):
            for name in ("k", "lw", "phi", "status"):
                assert np.array_equal(getattr(a, name)[:n], getattr(b, name)[:n]), (n, name)


@pytest.mark.parametrize("n_paths", [16385, 32769, 65537])
@pytest.mark.parametrize("proposal,group,stride", [("fixed", 1, 1), ("fixed", 4, 3), ("fixed", 16, 1), ("bump", 4, 1), ("bump", 16, 2),
                                                   ("network", 1, 2), ("network", 4, 1), ("network", 8, 1), ("network", 16, 2)])
def test_records_of_many_paths(fpt, n_paths, proposal, group, stride):
    """16, 32 and 64 paths a wave (8 a wave last up to 16384 paths, each further doubling one more), ragged
    last waves among them."""
    print(f"[case] {n_paths} paths {proposal} group {group} stride {stride}", flush=True)
    inst = dataclasses.replace(W.c2(1)[3], phi_in=1.6, dN=1e-2, k_max=90)
    if proposal == "bump":
        inst = W.Instance("bump", pot=W.POT_QUADRATIC_BUMP, m=0.5, a=0.05, phi0=1.7, w=0.02, phi_in=2.0, phi_uv=6.0,
                          bias=W.BIAS_NOISE_SCALED, A=1.0, dN=1.5e-2, n_traj=1, k_max=90)
    elif proposal == "network":
        v = np.zeros(W.MlpParams.N_PARAMS, np.float32)
        v[4480] = 0.5
        inst = dataclasses.replace(inst, bias=W.BIAS_MLP, A=0.0, target_N=196.0, mlp=W.MlpParams(v, out_scale=2.0, eval_every=group))
    _check_records(fpt, inst, n_paths, group, stride)


@pytest.mark.parametrize("n_paths", [9, 300])
@pytest.mark.parametrize("group,stride", [(4, 1), (8, 4), (16, 3)])
@pytest.mark.parametrize("a,w,wall", [(0.05, 0.05, True), (-0.02, 0.2, False)])
def test_records_at_the_bump(fpt, n_paths, group, stride, a, w, wall):
    """Paths that start far from the bump, cross it and end beyond it."""
    print(f"[case] {n_paths} paths group {group} stride {stride} a={a} w={w}", flush=True)
    _check_records(fpt, W.Instance("bump", pot=W.POT_QUADRATIC_BUMP, m=0.05, a=a, phi0=3.0, w=w, phi_in=5.0,
                                   phi_uv=6.0 if wall else math.inf, bias=W.BIAS_NOISE_SCALED, A=1.0, dN=2e-3, n_traj=1, k_max=9000),
                   n_paths, group, stride)


def _check_records(fpt, inst, n_paths, group, stride):
    ids = np.arange(n_paths, dtype=np.uint64) * np.uint64(3)
    o = O.records(to_model(inst), 0, ids, group, stride)
    g = fpt.proposal_records(inst, 0, ids, o.k, group, stride)
    assert np.array_equal(g.k, o.k) and np.array_equal(g.lw, o.lw) and np.array_equal(g.status, o.status)
    assert np.array_equal(g.off, o.off) and g.rec.tobytes() == o.rec.tobytes()


@pytest.mark.parametrize("objective", [0, 1])
def test_loss_and_gradient_beyond_one_grid(fpt, objective):
    """More records than the evaluation's and the backward pass's grids hold at once (196 608 and 65 536 on
    256 CUs), so that workgroups and waves take second and third tiles, with a ragged last one.

    A gradient component is a sum over records of coef_e times a factor of at most F (below), each formed
    from sums of 64 binary32 terms and added up along a chain of some hundred more: 256 2^-24 of the sum of
    the terms' sizes bounds its error."""
    print(f"[case] second tiles, objective {objective}", flush=True)
    n_rec = 196608 + 65
    recs, lw0 = _records(fpt, n_rec, 40)
    p = W.c4_params(7, scale=1.5, out_scale=0.8)
    theta = p.values_f32()
    inst = W.c4_instance(p, n_traj=1)
    loss, grad, lwt = fpt.proposal_loss_grad(p, inst.target_N, inst.dN, theta, recs, lw0, 100.0, objective)
    loss_o, grad_o, lwt_o = O.loss_grad(to_model(inst), theta.astype(np.float64), recs, lw0, 100.0, objective)
    th = theta.astype(np.float64)
    W2, w3 = th[256:4352].reshape(64, 64), th[4416:4480]
    r_max = abs(p.out_scale) * (np.abs(w3).sum() + abs(th[4480]))
    a = lw0 + (lwt_o if objective == 0 else 0.0)
    c = np.exp(a - a.max())
    c /= c.sum()
    n = (recs.rec["pn"] & 31).astype(np.float64)
    H = np.abs(recs.rec["H"].astype(np.float64))
    size = (r_max * n * inst.dN + H) * abs(p.out_scale)
    x = 1.0 + max(np.abs((recs.rec["phi"] - p.in_mean[0]) * p.in_inv_scale[0]).max(),
                  np.abs((recs.rec["k"] * inst.dN - p.in_mean[1]) * p.in_inv_scale[1]).max(),
                  abs((inst.target_N - p.in_mean[2]) * p.in_inv_scale[2]))
    F = max(1.0, np.abs(w3).max(), (np.abs(w3) @ np.abs(W2)).max() * x)
    owner = (recs.rec["pn"] >> 5).astype(np.int64)
    eps = 256.0 * 2.0 ** -24
    # ln w_theta: sums of r H and r^2 n dN / 2
    term = r_max * H + r_max ** 2 * n * inst.dN
    assert np.all(np.abs(lwt - lwt_o) <= eps * np.bincount(owner, term, len(lw0)))
    assert abs(loss - loss_o) <= eps * np.bincount(owner, term, len(lw0)).max() * (1.0 if objective == 0 else 2.0)
    # the path weights follow ln w_theta
    shift = 2.0 * np.abs(lwt - lwt_o).max() if objective == 0 else 0.0
    assert np.abs(grad - grad_o).max() <= (eps + shift) * F * float((c[owner] * size).sum())

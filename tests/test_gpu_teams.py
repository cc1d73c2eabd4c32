"""Launches with fewer runs than lanes: waves that take 64, 32, 16 or 8 runs and whose idle lanes draw
normals ahead, and the drain of a full launch.  Every run bit for bit and every count as the oracle has
them, at the run counts around which the launch shape changes (2048 waves of 8, 16 and 32 runs on 256
compute units) and at ragged ones."""
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


def _well(n_traj, k_max=1 << 20, stream=0):
    # S = 1, unit well: about 1e3 steps a run, widely spread
    return W.Instance("flat", pot=W.POT_FLAT, V0=3 * (2 * math.pi) ** 2, phi_in=1.0, phi_end=0.0, phi_uv=1.5, dN=1e-3,
                      bias=W.BIAS_NOISE_SCALED, A=-1.0, n_traj=n_traj, k_max=k_max, stream=stream, edges=np.linspace(0.05, 3.0, 61))


@pytest.mark.parametrize("n_traj,shape", [
    (1, {}), (7, {}), (65, {}), (4097, {}), (16384, {}), (16385, {}), (32769, {}), (65537, {}),
    (1000, dict(block=64, wg_per_cu=1, chunk=1)),      # one wave per CU at most: 8 runs a wave
    (16400, dict(block=64, wg_per_cu=1, chunk=1)),     # 256 waves of 64 and a refill
    (3000, dict(block=1024, wg_per_cu=1, chunk=4)),
])
def test_few_runs_match_oracle(fpt, n_traj, shape):
    inst = _well(n_traj)
    print(f"[case] n={n_traj} shape={shape}", flush=True)
    res, dump, _ = fpt.run(inst, 3, dump_n=n_traj, **shape)
    tr = O.simulate(to_model(inst), 3, n_traj)
    assert_dump_matches(dump, tr)
    assert_histogram_matches(res, O.histogram(tr, inst.dN, inst.edges))


@pytest.mark.parametrize("k_max", [1, 2, 3, 4, 5, 31, 32, 33])
def test_cap_inside_a_group(fpt, k_max):
    """The step cap at every place of a group of four and of a batch of eight groups."""
    inst = _well(300, k_max=k_max)
    print(f"[case] k_max={k_max}", flush=True)
    res, dump, _ = fpt.run(inst, 3, dump_n=300)
    tr = O.simulate(to_model(inst), 3, 300)
    assert_dump_matches(dump, tr)
    assert_histogram_matches(res, O.histogram(tr, inst.dN, inst.edges))


def test_mixed_batch_spread_over_waves(fpt):
    """A batch whose longest instance is a small part of it (first ids spread over the waves), with an
    instance without runs and different caps."""
    insts = [_well(40, stream=0), dataclasses.replace(_well(900, stream=1), A=-3.0), _well(0, stream=2),
             dataclasses.replace(_well(1500, stream=3), k_max=9)]
    print("[case] mixed batch", flush=True)
    results, dumps, _ = fpt.run_batch(insts, 5, dump_n=1500)
    for inst, res, dump in zip(insts, results, dumps):
        tr = O.simulate(to_model(inst), 5, inst.n_traj)
        if inst.n_traj:
            assert_dump_matches(dump, tr)
        assert_histogram_matches(res, O.histogram(tr, inst.dN, inst.edges))


@pytest.mark.parametrize("shape", [dict(block=b) for b in (64, 512, 576, 768, 1024)] + [dict(wg_per_cu=w) for w in (1, 2, 4, 8)] +
                         [dict(block=1024, chunk=2), dict(block=640, n_traj=300_000)])
def test_part_of_a_shape_given(fpt, shape):
    """Block sizes and workgroups per CU given on their own: the library chooses the other to fit."""
    shape = dict(shape)
    inst = _well(shape.pop("n_traj", 300), k_max=400)
    print(f"[case] shape={shape} n={inst.n_traj}", flush=True)
    n = min(inst.n_traj, 2000)
    res, dump, _ = fpt.run(inst, 3, dump_n=n, **shape)
    assert_dump_matches(dump, O.simulate(to_model(inst), 3, n))
    assert res.n_traj == inst.n_traj and int(res.count.sum()) == inst.n_traj

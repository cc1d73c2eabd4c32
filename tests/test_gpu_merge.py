"""The merge of the per-workgroup tables at the edges of its split: cells in blocks of 32, slices
in 16 ranges, finalize rows in fours with subsets in sixteens.  Against the oracle's histogram of
the same runs, with the tolerances of the parity tests (binary64 sums in another order)."""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W
from helpers import assert_histogram_matches, to_model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fpt():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2206_11234_amd as F
    return F


@pytest.mark.parametrize("n_bins,n_sub,wg_per_cu,n_traj", [
    ((1, 1), 2, 1, 700),           # 5-row tables: cells end inside the first block
    ((28, 27), 16, 2, 3000),       # 32 and 31 rows
    ((29, 60), 17, 4, 3000),       # one row past a block, subsets one past the finalize lanes
    ((200, 3), 64, 2, 3000),       # the most subsets
    ((2, 2), 3, 1, 1),             # one run
])
def test_merge_matches_oracle(fpt, n_bins, n_sub, wg_per_cu, n_traj):
    print(f"[case] bins={n_bins} n_sub={n_sub} wg={wg_per_cu} n={n_traj}", flush=True)
    insts = [W.Instance(f"flat{i}", pot=W.POT_FLAT, V0=3 * (2 * math.pi) ** 2, phi_in=1.0, phi_end=0.0, phi_uv=1.5, dN=1e-3,
                        bias=W.BIAS_NOISE_SCALED, A=-0.7 - i, n_traj=n_traj, stream=i, edges=np.linspace(0.05, 3.0, b + 1))
             for i, b in enumerate(n_bins)]
    results, _, _ = fpt.run_batch(insts, 0, n_sub=n_sub, block=256, wg_per_cu=wg_per_cu, chunk=1)
    for inst, res in zip(insts, results):
        tr = O.simulate(to_model(inst), 0, inst.n_traj)
        assert_histogram_matches(res, O.histogram(tr, inst.dN, inst.edges, n_sub))

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


def _flat(n_traj, n_bins, **kw):
    return W.Instance("flat", pot=W.POT_FLAT, V0=3 * (2 * math.pi) ** 2, phi_in=1.0, phi_end=0.0, phi_uv=1.5, dN=1e-3,
                      bias=W.BIAS_NOISE_SCALED, A=-1.0, n_traj=n_traj, edges=np.linspace(0.05, 3.0, n_bins + 1), **kw)


def test_moments_are_folded_in_workgroup_order(fpt):
    """The power sums of ln w of a bin are those of one chain over the workgroups, bit for bit: the errors
    of the lognormal estimate are exponentials of the variance and show its last bit where bins hold few,
    widely spread runs.  256 workgroups of 64 lanes (per CU one) with a run to each lane take the run ids
    64 by 64; a bin with at most one run per workgroup has sums that no order within one can change."""
    cus = fpt.device_cus()
    inst = _flat(64 * cus, 2000)
    print("[case] moments in workgroup order", flush=True)
    res, dump, _ = fpt.run(inst, 1, dump_n=inst.n_traj, block=64, wg_per_cu=1, chunk=1)
    rows = O.bin_rows(dump.k.astype(np.uint64), dump.status, inst.dN, inst.edges)
    seen = 0
    for r in range(res.n_bins):
        t = np.nonzero(rows == r)[0]
        if t.size < 3 or np.unique(t // 64).size < t.size:
            continue
        x = [float(dump.lw[i]) for i in t]              # ascending ids: ascending workgroups
        s1 = s2 = s3 = s4 = 0.0
        for v in x:
            d = v - x[0]
            s4 += d * d * d * d
            s3 += d * d * d
            s2 += d * d
            s1 += d
        n = float(len(x))
        mu, e2, e3, e4 = s1 / n, s2 / n, s3 / n, s4 / n
        want = (x[0] + mu, e2 - mu * mu, e3 - 3.0 * mu * e2 + 2.0 * mu * mu * mu,
                e4 - 4.0 * mu * e3 + 6.0 * mu * mu * e2 - 3.0 * mu * mu * mu * mu)
        assert (res.mean_lnw[r], res.m2_lnw[r], res.m3_lnw[r], res.m4_lnw[r]) == want, (r, t.size)
        seen += 1
    assert seen > 200, seen


def test_sum_of_squared_steps_is_the_exact_sum_rounded(fpt):
    """Runs of up to 2^21 - 1 steps: the sum of k^2 over them is beyond binary64's integers."""
    inst = _flat(40_000, 30, k_max=2 ** 21 - 1)
    inst.dN, inst.A, inst.bias = 1e-6, 0.0, W.BIAS_NONE
    print("[case] sum k^2", flush=True)
    res, dump, _ = fpt.run(inst, 1, dump_n=inst.n_traj)
    exact = sum(int(k) * int(k) for k in dump.k)
    assert exact > 2 ** 55
    assert res.sum_k2 == float(exact)
    assert res.total_steps == int(dump.k.astype(np.int64).sum())


@pytest.mark.parametrize("extra", [-2, -1, 0, 1, 2])
@pytest.mark.parametrize("block,wg_per_cu", [(64, 1), (256, 1)])
def test_tables_at_the_edge_of_lds(fpt, block, wg_per_cu, extra):
    """The largest tables that share a CU's 160 KiB with the lanes' stopped runs (16 B each), and the first
    that go to global memory: 240 B a row with 16 subsets, 128 B an instance, in units of 256 B."""
    lanes = fpt.device_cus() * wg_per_cu * block
    rows = (160 * 1024 // wg_per_cu // 256 * 256 - 16 * block - 128) // 240
    inst = W.Instance("flat", pot=W.POT_FLAT, V0=3 * (2 * math.pi) ** 2, phi_in=1.0, phi_end=0.0, phi_uv=1.5, dN=1e-2,
                      bias=W.BIAS_NOISE_SCALED, A=-1.0, n_traj=lanes + 100, k_max=2000, edges=np.linspace(0.05, 3.0, rows - 4 + extra + 1))
    print(f"[case] block {block} x {wg_per_cu}, {rows + extra} rows", flush=True)
    res, _, _ = fpt.run(inst, 4, block=block, wg_per_cu=wg_per_cu, chunk=1)
    assert_histogram_matches(res, O.histogram(O.simulate(to_model(inst), 4, inst.n_traj), inst.dN, inst.edges))

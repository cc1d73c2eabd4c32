// fpt_kernels.hip -- persistent first-passage kernels for gfx950 (CDNA4).
//
// fpt_step: one lane per trajectory.  Each lane repeats groups of four
// Euler-Maruyama steps of the biased Langevin equation (arXiv:2206.11234,
// Sec. 2.2 eq. eq_euler_maruyam_modified) from one Philox call, updates the
// binary64 log-weight (Sec. 2.2 eq. eq_importance_sampling_bias_w, with the
// minus sign of the likelihood ratio), and stops at first passage
// (Sec. 2.1).  Finished lanes are retired at group boundaries: a wave ballot
// finds them, one atomic per wave claims new trajectory ids from the shared
// queue (mbcnt-style prefix ranks hand them out) and the lanes restart.  The
// kernel is persistent: it runs until the queue is drained.
//
// Each retiring run is binned in N = k dN (right-closed bins, Sec. 2.1) and
// accumulated into its workgroup's table: counts per (jackknife subset, row),
// log-sum-exp of w per (subset, row) and of w^2 per row (the weighted
// estimator of Sec. 2.2 and its jackknife, Sec. 2.1), and power sums of ln w
// about a per-row shift (the moments used by the lognormal estimator of
// Sec. 2.4).  The table sits in LDS when it fits and is copied to the
// workgroup's global slice at the end; otherwise it lives in that slice.
//
// fpt_merge / fpt_finalize: fold the per-workgroup slices in workgroup order
// (binary64 log-sum-exp for the weight sums, integer sums for counts,
// binomial re-basing for the moments) and evaluate the per-bin estimators.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "fpt_kernels.h"
#include "fpt_team.h"

namespace fpt {

#define FPT_NAN_BITS 0x7FF8000000000000ull
#define FPT_NEG_INF_BITS 0xFFF0000000000000ull

__device__ __forceinline__ double lse2(double a, double b) {
    if (__builtin_isinf(a) && a < 0) return b;
    if (__builtin_isinf(b) && b < 0) return a;
    const double m = fmax(a, b);
    return m + log1p(exp(-fabs(a - b)));
}

template <typename T>
__device__ __forceinline__ void atomic_lse(T *p, double x) {
    unsigned long long *a = reinterpret_cast<unsigned long long *>(p);
    unsigned long long old = __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (true) {
        const double cur = __longlong_as_double(static_cast<long long>(old));
        const double nv = lse2(cur, x);
        const unsigned long long want = static_cast<unsigned long long>(__double_as_longlong(nv));
        if (want == old) return;
        const unsigned long long prev = atomicCAS(a, old, want);
        if (prev == old) return;
        old = prev;
    }
}

__device__ __forceinline__ void atomic_add_f64(double *p, double x) {
    __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

struct Tab {
    double *scal, *jk_lse, *lse_w2, *shift, *s1, *s2, *s3, *s4;
    uint32_t *cnt;
};

__device__ __forceinline__ Tab make_tab(unsigned char *base, const TableLayout &L) {
    Tab T;
    T.scal = reinterpret_cast<double *>(base + L.off_scal);
    T.jk_lse = reinterpret_cast<double *>(base + L.off_jk_lse);
    T.lse_w2 = reinterpret_cast<double *>(base + L.off_lse_w2);
    T.shift = reinterpret_cast<double *>(base + L.off_shift);
    T.s1 = reinterpret_cast<double *>(base + L.off_s1);
    T.s2 = reinterpret_cast<double *>(base + L.off_s2);
    T.s3 = reinterpret_cast<double *>(base + L.off_s3);
    T.s4 = reinterpret_cast<double *>(base + L.off_s4);
    T.cnt = reinterpret_cast<uint32_t *>(base + L.off_cnt);
    return T;
}

// Initial contents: -inf for log-sums, NaN ("no shift yet") for shifts, 0 elsewhere.
__device__ __forceinline__ void init_table(unsigned char *base, const TableLayout &L) {
    unsigned long long *w = reinterpret_cast<unsigned long long *>(base);
    const uint32_t n_words = L.slice_bytes / 8;
    for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) {
        const uint32_t off = i * 8;
        unsigned long long v = 0ull;
        if (off < L.off_jk_lse) {
            const uint32_t f = ((off - L.off_scal) / 8) & 15u;
            v = (f == 2 || f == 3) ? FPT_NEG_INF_BITS : 0ull;
        } else if (off < L.off_shift) {
            v = FPT_NEG_INF_BITS;           // jk_lse, lse_w2
        } else if (off < L.off_s1) {
            v = FPT_NAN_BITS;               // shift
        }
        w[i] = v;
    }
}

// Wave-wide log-sum-exp over lanes (all 64 take part): one exponential and one logarithm.
__device__ __forceinline__ double wave_lse(double x) {
    double m = x;
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) m = fmax(m, __shfl_xor(m, h, 64));
    if (__builtin_isinf(m) && m < 0) return __any(x != x) ? NAN : m;
    double s = (__builtin_isinf(x) && x < 0) ? 0.0 : exp(x - m);
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) s += __shfl_xor(s, h, 64);
    return m + log(s);
}

// A lane's log-sums of w k and w k^2 over the runs it retired of one instance.
struct LaneAcc {
    int inst;
    double wk, wk2;
};

__device__ __forceinline__ void acc_reset(LaneAcc &a, int inst) {
    a.inst = inst;
    a.wk = a.wk2 = -INFINITY;
}

__device__ __forceinline__ void acc_commit_direct(const Tab &T, const LaneAcc &a) {
    double *s = T.scal + static_cast<size_t>(a.inst) * 16;
    atomic_lse(s + 2, a.wk);
    atomic_lse(s + 3, a.wk2);
}

extern __shared__ __align__(16) unsigned char fpt_lds[];

// SINGLE: one instance of the batch has runs, so its constants are uniform across the workgroup
// (the compiler keeps them in scalar registers) and queue ids are its trajectory ids.
template <int POT, int BIAS, bool LDS, bool SINGLE = false>
__device__ __forceinline__ void fpt_step_body(const StepArgs &a) {
    unsigned char *lds = fpt_lds;
    unsigned char *gslice = a.slices + static_cast<size_t>(blockIdx.x) * a.lay.slice_bytes;
    unsigned char *base = LDS ? lds : gslice;
    init_table(base, a.lay);
    __syncthreads();
    const Tab T = make_tab(base, a.lay);
    const uint32_t RT = a.lay.n_rows;
    const uint32_t J = a.lay.n_sub;

    const uint32_t lane = __lane_id();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));

    // lane state
    StepConsts C{};
    uint32_t j_cap = 0;
    int cur_inst = -1;
    RunState R{0.0f, 0u, 0.0};
    PhiloxRun noise{};
    Stopped *const F = reinterpret_cast<Stopped *>(fpt_lds + (LDS ? a.lay.slice_bytes : 0u)) + threadIdx.x;
    uint64_t t = 0;
    // the wave's lanes, as masks: those whose runs go on, those that have a run (stopped or not) and
    // those that want one
    uint64_t running = 0, active = 0, need = ~0ull >> (64 - a.lane_cap);
    LaneAcc acc;
    acc_reset(acc, -1);
    // this wave's reserved queue range
    uint64_t res_lo = 0, res_hi = 0;
    // The first ids are handed out by position, the others from the queue (StepArgs::spread).
    const uint64_t n_waves = static_cast<uint64_t>(gridDim.x) * (blockDim.x / 64);
    const uint64_t n_first = n_waves * a.lane_cap;
    bool first = true;
    bool drained = n_first >= a.v_total;   // no id is left in the queue
    Team team;
    F4 batch{};                 // learned bias: the team's current batch of normals
    int batch_at = 0;           // and the group of it that comes next
    // Power-law bias: the exponent where the wave's instances share one of 1 .. 4, whose group is
    // compiled for it; a loop over an exponent per lane costs a step 24 instructions and its overlap
    // with the next (2e5 runs with p = 3: 5.2 against 4.6 ms, in the loop of that time; now 4.1).
    int p_wave = 0;
    // Whether the wave's runs all have a wall, all have none, or differ: two instructions a step
    // without the reflection, three a group without the escape test.  Both choices are made where a
    // run has stopped or been handed out, and the groups between follow each other in a loop of one
    // branch: with the choice, the refill's tests and the teams' around each group, six instances of
    // 1e5 runs took 186 ms (chosen by group, 214), now 166.
    int walls = WALL_ANY;
    BumpFar far{a.bump_far};    // bump potential: see group4
    auto specialised = [&](auto f) {
        auto with = [&](auto p, auto wall) { f([&](const F4 &z) { (void)group4<POT, BIAS, p(), wall()>(C, j_cap, z, 0.0f, R, running, F, far); }); };
        using std::integral_constant;
        constexpr integral_constant<int, 0> p_any;
        constexpr integral_constant<int, WALL_ANY> wall_any;
        if constexpr (BIAS == BIAS_POWER) {
            switch (p_wave) {
            case 1: with(integral_constant<int, 1>{}, wall_any); break;
            case 2: with(integral_constant<int, 2>{}, wall_any); break;
            case 3: with(integral_constant<int, 3>{}, wall_any); break;
            case 4: with(integral_constant<int, 4>{}, wall_any); break;
            default: with(p_any, wall_any); break;
            }
        } else if constexpr (POT == POT_QUADRATIC_BUMP) {
            with(p_any, wall_any);
        } else {
            if (walls == WALL_NONE) with(p_any, integral_constant<int, WALL_NONE>{});
            else if (walls == WALL_ALL) with(p_any, integral_constant<int, WALL_ALL>{});
            else with(p_any, wall_any);
        }
    };
    const uint32_t odd_mask = normals_mask();
    // learned proposal: one copy of the network's A operands per workgroup
    __shared__ bf16x8 tile_lds[BIAS == BIAS_MLP ? MLP_N_FRAG * 64 : 1];
    if constexpr (BIAS == BIAS_MLP) {
        if (threadIdx.x < 64) {
            MlpTiles tiles;
            mlp_load_tiles(a.mlp_params, tiles);
            mlp_store_tiles_lds(tiles, tile_lds);
        }
        __syncthreads();
    }
    MlpConsts mc{};
    int single_inst = 0;
    auto load_instance = [&](int ii) {
        const InstDev &I = a.inst[ii];
        C = I.c;
        if constexpr (BIAS == BIAS_MLP) mc = I.mlp;
        cur_inst = ii;
        j_cap = cap_groups(C.k_max);
    };
    if constexpr (SINGLE) {
        // the one instance with runs (others in the batch, if any, have none)
        single_inst = static_cast<int>(a.order[0]);
        load_instance(single_inst);
    }

    while (true) {
        // ---- refill: hand new trajectory ids to lanes that need one
        const bool refill = need != 0;
        if (refill) {
            const bool mine = (need >> lane) & 1u;
            uint64_t v = ~0ull;
            if (first) {
                first = false;
                // neighbouring waves go to different workgroups; the ones of a CU start their order at
                // different waves, so that the longest runs' waves lie evenly over its SIMDs too
                const uint32_t wpw = blockDim.x / 64;
                const uint32_t w = (threadIdx.x / 64 + blockIdx.x / a.cus * a.turn) % wpw;
                const uint64_t wave = static_cast<uint64_t>(w) * gridDim.x + blockIdx.x;
                v = a.spread ? lane * n_waves + wave : wave * a.lane_cap + lane;
            } else if (!drained) {
                const uint32_t n_need = __popcll(need);
                const uint32_t rank = __popcll(need & lt_mask);
                const uint64_t avail = res_hi - res_lo;
                if (avail >= n_need) {
                    v = res_lo + rank;
                    res_lo += n_need;
                } else {
                    const uint64_t short_by = n_need - avail;
                    const uint64_t amt = short_by * a.chunk;
                    const int leader = __ffsll(static_cast<unsigned long long>(need)) - 1;
                    unsigned long long b = 0;
                    if (static_cast<int>(lane) == leader) b = atomicAdd(a.queue, static_cast<unsigned long long>(amt));
                    b = n_first + __shfl(b, leader, 64);
                    v = (rank < avail) ? res_lo + rank : b + (rank - avail);
                    res_lo = b + short_by;
                    res_hi = b + amt;
                }
                drained = __any(mine && v >= a.v_total);   // a wave's ids ascend: no later one is in range
            }
            const bool got = mine && v < a.v_total;
            const uint64_t given = __ballot(got);
            need = 0;
            active |= given;
            running |= given;
            {
                if (got) {
                    int ii = single_inst;
                    if constexpr (SINGLE) {
                        t = v;                 // the only instance with runs starts the queue
                    } else {
                        int lo = 0, hi = a.n_inst;
                        while (hi - lo > 1) {
                            const int mid = (lo + hi) >> 1;
                            if (a.vbeg_sorted[mid] <= v) lo = mid; else hi = mid;
                        }
                        ii = static_cast<int>(a.order[lo]);
                        t = v - a.vbeg_sorted[lo];
                    }
                    if (!SINGLE && ii != cur_inst) load_instance(ii);
                    t += a.inst[ii].t_first;   // the run's id: Philox counter and jackknife subset
                    if (acc.inst != ii) {
                        if (acc.inst >= 0) acc_commit_direct(T, acc);
                        acc_reset(acc, ii);
                    }
                    noise = philox_run(t, a.inst[ii].stream, a.key0, a.key1);
                    R = RunState{C.phi_in, 0u, 0.0};
                }
            }
        }
        if (!active) break;
        if (refill) {
            // lanes without a run do not count
            if constexpr (BIAS <= BIAS_NOISE_SCALED && POT != POT_QUADRATIC_BUMP) {
                const uint64_t walled = __ballot(C.two_uv < INFINITY) & active;
                walls = walled == 0 ? WALL_NONE : walled == active ? WALL_ALL : WALL_ANY;
            }
            if constexpr (BIAS == BIAS_POWER) {
                const int p0 = __builtin_amdgcn_readlane(C.p, __ffsll(static_cast<unsigned long long>(active)) - 1);
                p_wave = (__ballot(C.p != p0) & active) == 0 ? p0 : 0;
            }
        }
        // few runs and no more to come: the idle lanes draw normals ahead for them
        const int n_act = __popcll(running);
        const bool teamed = drained && n_act <= 32;

        // ---- a pass: groups of four Euler-Maruyama steps, each from one Philox call
        if constexpr (BIAS != BIAS_MLP) {
            if (teamed) {
                // To the end of the wave's last run: nothing is refilled or retired before it.  A wave
                // alone on its SIMD issues an instruction per 5 cycles, so the count is the time: 42 a step
                // in the loop over any G, 30 in the stretch for G = 8 (500 direct runs: 518 and 457 us).
                specialised([&](auto group) {
                    while (running) {
                        team_form(team, running, lt_mask, lane, noise, 8);
                        const int n_g = team.groups();              // 2, 4 or 8 groups a batch
                        uint32_t j = lane_read(team.slot_lane, R.j) + (lane >> team.shift);
                        F4 z = normals4(j, team.noise, a.key0, a.key1, odd_mask);
                        F4 zn = team_fetch(team, z, 0);
                        if (n_g == 8) {
                            // as below, with every group's place in the batch a constant
                            do {
                                j += 8;
                                const F4 zb = normals4(j, team.noise, a.key0, a.key1, odd_mask);
#pragma unroll
                                for (int g = 0; g < 8; ++g) {
                                    const F4 zg = zn;
                                    zn = g < 7 ? team_fetch8(team, z, g + 1) : team_fetch8(team, zb, 0);
                                    group(zg);
                                }
                                z = zb;
                            } while (running);
                        } else do {
                            // a batch ahead: its draw fills the gaps in this one's chain of steps, and
                            // its first group is fetched before this one's last steps
                            j += static_cast<uint32_t>(n_g);
                            const F4 zb = normals4(j, team.noise, a.key0, a.key1, odd_mask);
                            for (int g = 0; g < n_g; g += 2) {
                                const F4 z0 = zn;
                                const F4 z1 = team_fetch(team, z, g + 1);
                                group(z0);
                                const bool last = g + 2 == n_g;
                                zn = team_fetch(team, last ? zb : z, last ? 0 : g + 2);
                                group(z1);
                            }
                            z = zb;
                        } while (running && !team_halves(team.shift, __popcll(running), 8));
                    }
                });
            } else {
                // until a run stops: nothing else changes what is compiled in or hands out new runs
                specialised([&](auto group) {
                    const uint64_t before = running;
                    do group(normals4(R.j, noise, a.key0, a.key1, odd_mask));
                    while (running == before);
                });
            }
        } else {
            // the network is evaluated by all 64 lanes together, outside divergent code.  One
            // pass covers max(4, E) steps for the evaluation interval E (1, 4, 8 or 16): runs
            // start at k = 0 and refill only between passes, so every lane of the wave is at a
            // multiple of the pass length here and the evaluation points of all lanes coincide.
            const int E = a.mlp_every;
            const int n_q = E > 4 ? E >> 2 : 1;
            // A team's runs fit one block of 32 columns, slot c in lane c: half the network's work (16
            // and 8 slots: a third and a quarter); its batches of normals last over G / (E / 4) passes
            // where G is larger.  A lone wave of 8 runs takes 321 cycles a step at E = 16 and 722 at E = 4;
            // asking before each group whether a batch is due, 360 and 856.
            int g_mask = 0;
            auto team_next = [&](uint32_t q) {      // the normals of the q-th group from here
                if (batch_at == 0) batch = team_draw(team, lane, R.j + q, a.key0, a.key1, odd_mask);
                const F4 z = team_fetch(team, batch, batch_at);
                batch_at = (batch_at + 1) & g_mask;
                return z;
            };
            auto network = [&](auto in_team, float phi_, float N_) {
                const MlpIn x = mlp_input(mc, phi_, N_);
                if constexpr (!decltype(in_team)::value) {
                    return mc.out_scale * mlp_forward_lds(tile_lds, x);
                } else {
                    const MlpIn xs{lane_read(team.slot_lane, x.lo), lane_read(team.slot_lane, x.hi)};
                    const float o = decltype(in_team)::value == 8 ? mlp_block_lds<8>(tile_lds, xs, 0)
                                    : team.shift == 4             ? mlp_block_lds<16>(tile_lds, xs, 0)
                                                                  : mlp_block_lds<32>(tile_lds, xs, 0);
                    return mc.out_scale * lane_read(team.fetch0, o);
                }
            };
            // One evaluation per pass of E = 4, 8 or 16 steps.  The pass's normals do not depend
            // on the network, so they are drawn before it and the scheduler interleaves their
            // vector work with the evaluation's matrix-core chains (they are the normals of
            // counters k/4 .. k/4 + E/4 - 1, the ones the steps would draw; a lane whose run ends
            // early leaves the rest unused).  The evaluation runs at a raised wave priority, so
            // that it finishes sooner while the SIMD's other waves fill the gaps with steps.
            auto pass = [&](auto in_team, auto nq_tag) {
                constexpr int NQ = decltype(nq_tag)::value;
                F4 zz[NQ];
                if constexpr (decltype(in_team)::value == 8) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) zz[q] = team_fetch8(team, batch, batch_at + q);
                } else if constexpr (decltype(in_team)::value) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) zz[q] = team_next(q);
                } else {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) {
                        zz[q] = normals4(R.j + q, noise, a.key0, a.key1, odd_mask);
                        // four draws at once would not fit the registers
                        if (q == 1) __builtin_amdgcn_sched_barrier(0);
                    }
                }
                __builtin_amdgcn_s_setprio(2);
                const float r_mlp = network(in_team, R.phi, static_cast<float>(4u * R.j) * C.dN);
                __builtin_amdgcn_s_setprio(0);
#pragma unroll
                for (int q = 0; q < NQ; ++q) (void)group4<POT, BIAS>(C, j_cap, zz[q], r_mlp, R, running, F, far);
            };
            // E = 1: an evaluation before every step
            auto pass1 = [&](auto in_team) {
                F4 z;
                if constexpr (decltype(in_team)::value == 8) z = team_fetch8(team, batch, batch_at);
                else if constexpr (decltype(in_team)::value) z = team_next(0);
                else z = normals4(R.j, noise, a.key0, a.key1, odd_mask);
                const float ns[4] = {z.a, z.b, z.c, z.d};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t k0 = 4u * R.j + s;
                    const float r_mlp = network(in_team, R.phi, static_cast<float>(k0) * C.dN);
                    float dlw, sxi;
                    (void)em_step<POT, BIAS>(C, R.phi, ns[s], r_mlp, dlw, sxi);
                    R.lw += static_cast<double>(dlw);
                    const uint64_t m = __ballot(stops(C, R.phi, k0 + 1)) & running;
                    if ((m >> lane) & 1u) *F = Stopped{R.phi, k0 + 1, R.lw};
                    running &= ~m;
                }
                R.j += 1;
            };
            // the passes until a run stops; a team's until its last one has, or half its slots are idle
            auto passes = [&](auto one) {
                if (teamed) {
                    while (running) {
                        team_form(team, running, lt_mask, lane, noise, 8);
                        batch_at = 0;
                        g_mask = team.groups() - 1;
                        if (g_mask == 7) {
                            // a batch of normals serves 8 / NQ passes of NQ groups (E = 1: one each)
                            while (running) {
                                batch = team_draw(team, lane, R.j, a.key0, a.key1, odd_mask);
#pragma unroll 1
                                for (batch_at = 0; batch_at < 8 && running; batch_at += n_q) one(std::integral_constant<int, 8>{});
                            }
                        } else {
                            do one(std::integral_constant<int, 1>{});
                            while (running && !team_halves(team.shift, __popcll(running), 8));
                        }
                    }
                } else {
                    const uint64_t before = running;
                    do one(std::integral_constant<int, 0>{});
                    while (running == before);
                }
            };
            using std::integral_constant;
            if (E == 16) passes([&](auto in_team) { pass(in_team, integral_constant<int, 4>{}); });
            else if (E == 8) passes([&](auto in_team) { pass(in_team, integral_constant<int, 2>{}); });
            else if (E == 4) passes([&](auto in_team) { pass(in_team, integral_constant<int, 1>{}); });
            else passes(pass1);
        }

        // ---- retire finished runs into the workgroup table: at once while their lanes can take new
        // ones, else all together when the wave's last run has stopped (a retirement is a chain of
        // dependent loads and atomics, as long as some tens of passes)
        const uint64_t fin = (!drained || running == 0) ? active & ~running : 0ull;
        if ((fin >> lane) & 1u) {
            const InstDev &I = a.inst[cur_inst];
            const uint32_t n_bins = I.n_bins, row_base = I.row_base, thr_base = I.thr_base, k_center = I.k_center;
            const uint64_t t0 = I.t_first;
            const float phi = F->phi;
            const double lw = F->lw;
            const uint32_t k = F->k;
            const int st = final_status(C, phi, k);
            uint32_t rl;
            if (st == ST_ENDED) {
                const uint32_t *K = a.thr + thr_base;
                uint32_t lo = 0, hi = n_bins + 1;   // first index with K >= k
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (K[mid] < k) lo = mid + 1; else hi = mid;
                }
                rl = (lo == 0) ? n_bins : ((lo == n_bins + 1) ? n_bins + 1 : lo - 1);
            } else {
                rl = (st == ST_CENSORED) ? n_bins + 2 : n_bins + 3;
            }
            const uint32_t row = row_base + rl;
            const uint32_t sub = static_cast<uint32_t>(t % J);
            atomicAdd(&T.cnt[sub * RT + row], 1u);
            atomic_lse(&T.jk_lse[sub * RT + row], lw);
            atomic_lse(&T.lse_w2[row], 2.0 * lw);
            unsigned long long *sp = reinterpret_cast<unsigned long long *>(&T.shift[row]);
            unsigned long long cb = __hip_atomic_load(sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const unsigned long long lwb = static_cast<unsigned long long>(__double_as_longlong(lw));
            if (cb == FPT_NAN_BITS) {
                const unsigned long long prev = atomicCAS(sp, FPT_NAN_BITS, lwb);
                cb = (prev == FPT_NAN_BITS) ? lwb : prev;
            }
            const double d = lw - __longlong_as_double(static_cast<long long>(cb));
            const double d2 = d * d;
            atomic_add_f64(&T.s1[row], d);
            atomic_add_f64(&T.s2[row], d2);
            atomic_add_f64(&T.s3[row], d2 * d);
            atomic_add_f64(&T.s4[row], d2 * d2);
            if (st == ST_ENDED) {
                // correlation of ln w with N over the ended runs (Sec. 3.4)
                double *sc = T.scal + static_cast<size_t>(cur_inst) * 16;
                const double y = static_cast<double>(static_cast<int64_t>(k) - static_cast<int64_t>(k_center));
                atomic_add_f64(sc + 6, 1.0);
                atomic_add_f64(sc + 7, lw);
                atomic_add_f64(sc + 8, lw * lw);
                atomic_add_f64(sc + 9, y);
                atomic_add_f64(sc + 10, y * y);
                atomic_add_f64(sc + 11, lw * y);
            }
            // instance-wide sums: of k in the table (exact: integers below 2^53), of k^2 as the integer
            // sums of its two 32-bit words (exact up to 2^32 runs a workgroup; one binary64 sum of the
            // workgroup's runs in turn rounds once a run beyond 2^53), the log-sums in lane registers
            const double kd = static_cast<double>(k);
            const uint64_t k2 = static_cast<uint64_t>(k) * k;
            unsigned long long *sk = reinterpret_cast<unsigned long long *>(T.scal + static_cast<size_t>(cur_inst) * 16);
            atomicAdd(sk + 0, static_cast<unsigned long long>(k2 & 0xFFFFFFFFu));
            atomicAdd(sk + 1, static_cast<unsigned long long>(k2 >> 32));
            atomic_add_f64(T.scal + static_cast<size_t>(cur_inst) * 16 + 5, kd);
            const double lk = log(kd);
            acc.wk = lse2(acc.wk, lw + lk);
            acc.wk2 = lse2(acc.wk2, lw + 2.0 * lk);
            if (a.dump.n != 0 && ((t - t0) % a.dump.stride) == 0) {
                const uint64_t idx = (t - t0) / a.dump.stride;
                if (idx < a.dump.n) {
                    const uint64_t pos = static_cast<uint64_t>(I.dump_slot) * a.dump.n + idx;
                    a.dump.k[pos] = k;
                    a.dump.lw[pos] = lw;
                    a.dump.phi[pos] = phi;
                    a.dump.status[pos] = st;
                }
            }
        }
        active &= ~fin;
        need = fin;
    }

    // ---- flush lane accumulators: one wave reduction per distinct instance
    bool pending = acc.inst >= 0;
    while (true) {
        const uint64_t pm = __ballot(pending);
        if (!pm) break;
        const int leader = __ffsll(static_cast<unsigned long long>(pm)) - 1;
        const int inst_l = __shfl(acc.inst, leader, 64);
        const bool mine = pending && acc.inst == inst_l;
        const double wk = wave_lse(mine ? acc.wk : -INFINITY);
        const double wk2 = wave_lse(mine ? acc.wk2 : -INFINITY);
        if (static_cast<int>(lane) == leader) {
            LaneAcc r;
            r.inst = inst_l;
            r.wk = wk;
            r.wk2 = wk2;
            acc_commit_direct(T, r);
        }
        if (mine) pending = false;
    }
    __syncthreads();
    if constexpr (LDS) {
        const unsigned long long *src = reinterpret_cast<const unsigned long long *>(lds);
        unsigned long long *dst = reinterpret_cast<unsigned long long *>(gslice);
        const uint32_t n_words = a.lay.slice_bytes / 8;
        for (uint32_t i = threadIdx.x; i < n_words; i += blockDim.x) dst[i] = src[i];
    }
}

// Workgroups of up to 1024 threads for the closed-form biases; up to 256 for the learned bias, whose
// several-instance kernel fits two waves per SIMD.
template <int POT, int BIAS, bool LDS>
__global__ __launch_bounds__(1024) void fpt_step_kernel(StepArgs a) {
    fpt_step_body<POT, BIAS, LDS>(a);
}

template <int POT, bool LDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void fpt_step_mlp_kernel(StepArgs a) {
    fpt_step_body<POT, BIAS_MLP, LDS>(a);
}

// One instance: uniform constants in scalar registers and the network's operand tiles in LDS,
// fitted to three waves per SIMD so that one wave's matrix-core work and latency overlap the
// others' vector work.
template <int POT, bool LDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void fpt_step_mlp1_kernel(StepArgs a) {
    fpt_step_body<POT, BIAS_MLP, LDS, true>(a);
}

__global__ void fpt_init_queue_kernel(unsigned long long *q) {
    if (threadIdx.x == 0) q[0] = 0ull;
}

// Instance owning global row r (rows are assigned in instance order).
__device__ __forceinline__ int inst_of_row(const MergeInst *mi, int n_inst, uint32_t r) {
    int lo = 0, hi = n_inst;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (mi[mid].row_base <= r) lo = mid; else hi = mid;
    }
    return lo;
}

// Running log-sum-exp as (m, s) = (max, sum of e^(x - m)): one exponential per term and one
// logarithm at the end.  -inf terms add nothing; +inf and NaN carry through as in lse2.
struct LseAcc {
    double m = -INFINITY, s = 0.0;
    __device__ __forceinline__ void add(double x) { fold(x, 1.0); }
    __device__ __forceinline__ void fold(double xm, double xs) {
        if (__builtin_isinf(xm) && xm < 0) return;
        if (xm <= m) {
            s += xs * exp(xm - m);
        } else {
            s = s * exp(m - xm) + xs;
            m = xm;
        }
    }
    __device__ __forceinline__ double value() const {
        return (__builtin_isinf(m) && m < 0) ? m : m + log(s);
    }
};

// Merge: MERGE_CELLS table cells by MERGE_SPLIT slice ranges per workgroup.  Bound by the reads of
// the slices where tables are large, by the chain of exponentials over the slices where they are
// small: with one thread per cell that chain was n_wg log-sum-exp updates long and took 0.5 ms
// (512 workgroups, 104 rows) to 6.3 ms (1024 workgroups, 164 rows, all cells in use).  Split over
// MERGE_SPLIT threads per cell, each folding slices w, w + MERGE_SPLIT, ... with one exponential
// apiece, and a tree over the threads in LDS.  32 neighbouring cells read 256 consecutive bytes of
// a slice.  The order of the sums is fixed by the launch shape.
//
// The power sums of ln w are one chain over the slices in order: the lognormal estimate's upper error
// is exp(u) - 1 with u up to some hundreds in bins of a few widely spread runs, u times the rounding of
// the second moment, and folding partial sums into one another would round more often than adding the
// slices' terms one by one.  Only the additions are in turn; the terms are formed by all threads, from
// loads of which all but the counts are in flight together (with a tree for them the kernel took 120 us
// at 1000 workgroups of 104 rows and 875 us at 13 056 rows, now 117 and 917).
constexpr int MERGE_CELLS = 32, MERGE_SPLIT = 16, MERGE_BLOCK = MERGE_CELLS * MERGE_SPLIT;
constexpr int MERGE_CHUNK = 2 * MERGE_SPLIT;        // slices whose terms are in LDS at a time

__device__ __forceinline__ uint32_t merge_blocks(uint32_t cells) { return (cells + MERGE_CELLS - 1) / MERGE_CELLS; }

static_assert(4 * MERGE_CHUNK * MERGE_CELLS == 8 * MERGE_BLOCK, "the terms fill the LDS array");

__global__ __launch_bounds__(MERGE_BLOCK) void fpt_merge_kernel(MergeArgs a) {
    __shared__ double red[8][MERGE_BLOCK];
    const TableLayout &L = a.lay;
    const uint32_t RT = L.n_rows, J = L.n_sub;
    const uint32_t n_cell_blocks = merge_blocks(J * RT), n_row_blocks = merge_blocks(RT);
    const int tid = threadIdx.x;
    const uint32_t lc = tid % MERGE_CELLS;
    const int part = tid / MERGE_CELLS;
    if (blockIdx.x < n_cell_blocks) {
        // counts and log-sums of w per (subset, row)
        const uint32_t cell = blockIdx.x * MERGE_CELLS + lc;
        const bool have = cell < J * RT;
        LseAcc l;
        unsigned long long cnt = 0;
        if (have)
            for (int w = part; w < a.n_wg; w += MERGE_SPLIT) {
                const unsigned char *sl = a.slices + static_cast<size_t>(w) * L.slice_bytes;
                cnt += reinterpret_cast<const uint32_t *>(sl + L.off_cnt)[cell];
                l.add(reinterpret_cast<const double *>(sl + L.off_jk_lse)[cell]);
            }
        for (int half = MERGE_SPLIT / 2; half >= 1; half >>= 1) {
            red[0][tid] = l.m;
            red[1][tid] = l.s;
            red[2][tid] = __longlong_as_double(static_cast<long long>(cnt));
            __syncthreads();
            if (part < half) {
                const int o = tid + half * MERGE_CELLS;
                l.fold(red[0][o], red[1][o]);
                cnt += static_cast<unsigned long long>(__double_as_longlong(red[2][o]));
            }
            __syncthreads();
        }
        if (have && part == 0) {
            const uint32_t s = cell / RT, r = cell % RT;
            const MergeInst m = a.mi[inst_of_row(a.mi, a.n_inst, r)];
            const ResultLayout RL = result_layout(m.n_bins, J);
            const uint64_t at = static_cast<uint64_t>(s) * m.n_rows + (r - m.row_base);
            a.counts[m.counts_off + RL.jk_count + at] = cnt;
            a.values[m.values_off + RL.jk_lse_w + at] = l.value();
        }
    } else if (blockIdx.x < n_cell_blocks + n_row_blocks) {
        // log-sum of w^2 and the moments of ln w per row
        const uint32_t r = (blockIdx.x - n_cell_blocks) * MERGE_CELLS + lc;
        const bool have = r < RT;
        double c = NAN;             // shift of the first slice that has one
        int first = a.n_wg;
        if (have) {
#pragma unroll 8
            for (int w = part; w < a.n_wg; w += MERGE_SPLIT) {
                const double cw = reinterpret_cast<const double *>(a.slices + static_cast<size_t>(w) * L.slice_bytes + L.off_shift)[r];
                const bool take = first == a.n_wg && !isnan(cw);
                first = take ? w : first;
                c = take ? cw : c;
            }
        }
        red[0][tid] = static_cast<double>(first);
        red[1][tid] = c;
        __syncthreads();
        for (int q = 0; q < MERGE_SPLIT; ++q)
            if (red[0][q * MERGE_CELLS + lc] < static_cast<double>(first)) {
                first = static_cast<int>(red[0][q * MERGE_CELLS + lc]);
                c = red[1][q * MERGE_CELLS + lc];
            }
        __syncthreads();
        LseAcc l2;
        // n values and their power sums about c, sum (x - c)^j = sum ((x - cw) + d)^j: the slices' terms
        // by all threads, MERGE_CHUNK slices at a time, then their sums in slice order, S_j by part j - 1
        double n = 0.0, S = 0.0;
        double *const term = &red[0][0];        // [4][MERGE_CHUNK][MERGE_CELLS]
        for (int w0 = 0; w0 < a.n_wg; w0 += MERGE_CHUNK) {
#pragma unroll
            for (int u = 0; u < MERGE_CHUNK / MERGE_SPLIT; ++u) {
                const int at = u * MERGE_SPLIT + part, w = w0 + at;
                double t1 = 0.0, t2 = 0.0, t3 = 0.0, t4 = 0.0;
                if (have && w < a.n_wg) {
                    // (all loads before the first test, so that they are in flight together)
                    const unsigned char *sl = a.slices + static_cast<size_t>(w) * L.slice_bytes;
                    const double xw2 = reinterpret_cast<const double *>(sl + L.off_lse_w2)[r];
                    const double cw = reinterpret_cast<const double *>(sl + L.off_shift)[r];
                    const double s1 = reinterpret_cast<const double *>(sl + L.off_s1)[r];
                    const double s2 = reinterpret_cast<const double *>(sl + L.off_s2)[r];
                    const double s3 = reinterpret_cast<const double *>(sl + L.off_s3)[r];
                    const double s4 = reinterpret_cast<const double *>(sl + L.off_s4)[r];
                    l2.add(xw2);
                    if (!isnan(cw)) {
                        double nw = 0.0;
                        for (uint32_t s = 0; s < J; ++s)
                            nw += static_cast<double>(reinterpret_cast<const uint32_t *>(sl + L.off_cnt)[s * RT + r]);
                        const double d = cw - c;
                        t4 = s4 + 4.0 * d * s3 + 6.0 * d * d * s2 + 4.0 * d * d * d * s1 + nw * d * d * d * d;
                        t3 = s3 + 3.0 * d * s2 + 3.0 * d * d * s1 + nw * d * d * d;
                        t2 = s2 + 2.0 * d * s1 + nw * d * d;
                        t1 = s1 + nw * d;
                        n += nw;
                    }
                }
                term[(0 * MERGE_CHUNK + at) * MERGE_CELLS + lc] = t1;
                term[(1 * MERGE_CHUNK + at) * MERGE_CELLS + lc] = t2;
                term[(2 * MERGE_CHUNK + at) * MERGE_CELLS + lc] = t3;
                term[(3 * MERGE_CHUNK + at) * MERGE_CELLS + lc] = t4;
            }
            __syncthreads();
            if (part < 4) {
#pragma unroll
                for (int at = 0; at < MERGE_CHUNK; ++at) S += term[(part * MERGE_CHUNK + at) * MERGE_CELLS + lc];
            }
            __syncthreads();
        }
        for (int half = MERGE_SPLIT / 2; half >= 1; half >>= 1) {
            red[0][tid] = l2.m;
            red[1][tid] = l2.s;
            red[2][tid] = n;
            __syncthreads();
            if (part < half) {
                const int o = tid + half * MERGE_CELLS;
                l2.fold(red[0][o], red[1][o]);
                n += red[2][o];
            }
            __syncthreads();
        }
        red[0][tid] = S;
        __syncthreads();
        if (have && part == 0) {
            const MergeInst m = a.mi[inst_of_row(a.mi, a.n_inst, r)];
            const uint32_t lr = r - m.row_base;
            const ResultLayout RL = result_layout(m.n_bins, J);
            double *V = a.values + m.values_off;
            V[RL.lse_w2 + lr] = l2.value();
            if (n > 0.0) {
                const double mu = S / n;
                const double e2 = red[0][MERGE_CELLS + lc] / n, e3 = red[0][2 * MERGE_CELLS + lc] / n,
                             e4 = red[0][3 * MERGE_CELLS + lc] / n;
                V[RL.mean_lnw + lr] = c + mu;
                V[RL.m2_lnw + lr] = e2 - mu * mu;
                V[RL.m3_lnw + lr] = e3 - 3.0 * mu * e2 + 2.0 * mu * mu * mu;
                V[RL.m4_lnw + lr] = e4 - 4.0 * mu * e3 + 6.0 * mu * mu * e2 - 3.0 * mu * mu * mu * mu;
            } else {
                V[RL.mean_lnw + lr] = NAN;
                V[RL.m2_lnw + lr] = NAN;
                V[RL.m3_lnw + lr] = NAN;
                V[RL.m4_lnw + lr] = NAN;
            }
        }
    } else {
        // one instance's whole-run sums
        const int i = static_cast<int>(blockIdx.x - n_cell_blocks - n_row_blocks);
        LseAcc f[2];
        unsigned long long k2[2] = {0, 0};          // sum of k^2: low and high words of the runs' k^2
        double acc[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int w = tid; w < a.n_wg; w += MERGE_BLOCK) {
            const double *sc = reinterpret_cast<const double *>(a.slices + static_cast<size_t>(w) * L.slice_bytes + L.off_scal) +
                               static_cast<size_t>(i) * 16;
            // (each workgroup's low sum carried, so that the sums over all stay in range)
            const unsigned long long lo = static_cast<unsigned long long>(__double_as_longlong(sc[0]));
            k2[0] += lo & 0xFFFFFFFFull;
            k2[1] += static_cast<unsigned long long>(__double_as_longlong(sc[1])) + (lo >> 32);
#pragma unroll
            for (int q = 0; q < 2; ++q) f[q].add(sc[2 + q]);
#pragma unroll
            for (int q = 0; q < 7; ++q) acc[q] += sc[5 + q];
        }
        // fold each wave, then the waves in order
        for (int h = 32; h >= 1; h >>= 1) {
#pragma unroll
            for (int q = 0; q < 2; ++q) k2[q] += __shfl_down(k2[q], h, 64);
#pragma unroll
            for (int q = 0; q < 2; ++q) f[q].fold(__shfl_down(f[q].m, h, 64), __shfl_down(f[q].s, h, 64));
#pragma unroll
            for (int q = 0; q < 7; ++q) acc[q] += __shfl_down(acc[q], h, 64);
        }
        if (tid % 64 == 0) {
            double *o = &red[0][0] + (tid / 64) * 16;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                o[2 * q] = f[q].m;
                o[2 * q + 1] = f[q].s;
                o[4 + q] = __longlong_as_double(static_cast<long long>(k2[q]));
            }
#pragma unroll
            for (int q = 0; q < 7; ++q) o[8 + q] = acc[q];
        }
        __syncthreads();
        if (tid == 0) {
            for (int wave = 1; wave < MERGE_BLOCK / 64; ++wave) {
                const double *o = &red[0][0] + wave * 16;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    f[q].fold(o[2 * q], o[2 * q + 1]);
                    k2[q] += static_cast<unsigned long long>(__double_as_longlong(o[4 + q]));
                }
#pragma unroll
                for (int q = 0; q < 7; ++q) acc[q] += o[8 + q];
            }
            const MergeInst m = a.mi[i];
            const ResultLayout RL = result_layout(m.n_bins, J);
            double *V = a.values + m.values_off;
            V[RL.lse_wk] = f[0].value();
            V[RL.lse_wk2] = f[1].value();
            // one rounding while the high sum is below 2^53
            V[RL.sum_k2] = static_cast<double>(k2[1] + (k2[0] >> 32)) * 4294967296.0 + static_cast<double>(k2[0] & 0xFFFFFFFFull);
            // Pearson's r of ln w with N over the ended runs (equal to that of log10 w with N)
            const double n = acc[1];
            const double mx = acc[2] / n, my = acc[4] / n;
            const double cxy = acc[6] / n - mx * my;
            const double vx = acc[3] / n - mx * mx, vy = acc[5] / n - my * my;
            V[RL.pearson_r] = (n >= 2.0 && vx > 0.0 && vy > 0.0) ? cxy / sqrt(vx * vy) : NAN;
            a.counts[m.counts_off + RL.n_traj] = m.n_traj;
            a.counts[m.counts_off + RL.total_steps] = static_cast<uint64_t>(acc[0]);
            V[RL.lognormal_gate] = 1.0;     // cleared by the finalize kernel where a bin fails
        }
    }
}

// D'Agostino and Pearson's omnibus K^2 test of normality from the sample skewness g1 = m3/m2^1.5
// and kurtosis b2 = m4/m2^2 (population central moments) of n values: the skewness is mapped to a
// standard normal by D'Agostino's (1970) Johnson S_U transformation, the kurtosis by Anscombe and
// Glynn's (1983) Wilson-Hilferty-type transformation, and K^2 = Z1^2 + Z2^2 is chi^2 with two
// degrees of freedom, so p = exp(-K^2/2).
__device__ double dagostino_pearson_p(double n, double g1, double b2) {
    // skewness
    const double y = g1 * sqrt((n + 1.0) * (n + 3.0) / (6.0 * (n - 2.0)));
    const double beta2 = 3.0 * (n * n + 27.0 * n - 70.0) * (n + 1.0) * (n + 3.0) /
                         ((n - 2.0) * (n + 5.0) * (n + 7.0) * (n + 9.0));
    const double w2 = -1.0 + sqrt(2.0 * (beta2 - 1.0));
    const double delta = 1.0 / sqrt(0.5 * log(w2));
    const double alpha = sqrt(2.0 / (w2 - 1.0));
    const double z1 = delta * asinh(y / alpha);
    // kurtosis
    const double e = 3.0 * (n - 1.0) / (n + 1.0);
    const double var = 24.0 * n * (n - 2.0) * (n - 3.0) / ((n + 1.0) * (n + 1.0) * (n + 3.0) * (n + 5.0));
    const double x = (b2 - e) / sqrt(var);
    const double sb1 = 6.0 * (n * n - 5.0 * n + 2.0) / ((n + 7.0) * (n + 9.0)) *
                       sqrt(6.0 * (n + 3.0) * (n + 5.0) / (n * (n - 2.0) * (n - 3.0)));
    const double A = 6.0 + 8.0 / sb1 * (2.0 / sb1 + sqrt(1.0 + 4.0 / (sb1 * sb1)));
    const double den = 1.0 + x * sqrt(2.0 / (A - 4.0));
    if (den == 0.0) return NAN;
    const double z2 = ((1.0 - 2.0 / (9.0 * A)) - cbrt((1.0 - 2.0 / A) / den)) / sqrt(2.0 / (9.0 * A));
    return exp(-0.5 * (z1 * z1 + z2 * z2));
}

// Lognormal estimator of one bin (Sec. 2.4): <w> = exp(<ln w> + s^2/2) with s^2 the unbiased
// sample variance of ln w; P_hat = n_j <w> / (n_traj width); its Cox interval
// P_hat exp(+-u), u = sqrt(s^2/n + s^4/(2n - 2)); and the normality p-value of ln w.
// log_norm = log(width) + log(n_traj).
__device__ void lognormal_bin(double *V, const ResultLayout &RL, uint32_t lr, uint64_t cnt, double log_norm) {
    double lp = NAN, lo = NAN, hi = NAN, pv = NAN;
    if (cnt >= 2) {
        const double n = static_cast<double>(cnt);
        const double c2 = V[RL.m2_lnw + lr];
        const double s2 = c2 * n / (n - 1.0);
        lp = log(n) + V[RL.mean_lnw + lr] + 0.5 * s2 - log_norm;
        const double u = sqrt(s2 / n + s2 * s2 / (2.0 * n - 2.0));
        hi = expm1(u);
        lo = -expm1(-u);
        if (cnt >= 8 && c2 > 0.0) {
            const double g1 = V[RL.m3_lnw + lr] / (c2 * sqrt(c2));
            const double b2 = V[RL.m4_lnw + lr] / (c2 * c2);
            pv = dagostino_pearson_p(n, g1, b2);
        }
    }
    V[RL.log_p_ln + lr] = lp;
    V[RL.rel_err_ln_lo + lr] = lo;
    V[RL.rel_err_ln_hi + lr] = hi;
    V[RL.normal_p + lr] = pv;
}

// Finalize: FIN_LANES lanes per row, each taking every FIN_LANES-th jackknife subset (with one
// thread per row the chain of 2 J exponentials took 17 to 22 us).
constexpr int FIN_LANES = 16, FIN_ROWS = 4;

// One wave per instance: the log-sums of w and w^2 over all its runs, from the merged cells.
__device__ void whole_run_sums(const MergeArgs &a, int i) {
    const MergeInst m = a.mi[i];
    const uint32_t J = a.lay.n_sub;
    const ResultLayout RL = result_layout(m.n_bins, J);
    double *V = a.values + m.values_off;
    LseAcc w, w2;
    for (uint64_t c = threadIdx.x; c < static_cast<uint64_t>(J) * m.n_rows; c += 64) w.add(V[RL.jk_lse_w + c]);
    for (uint32_t r = threadIdx.x; r < m.n_rows; r += 64) w2.add(V[RL.lse_w2 + r]);
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) {
        w.fold(__shfl_down(w.m, h, 64), __shfl_down(w.s, h, 64));
        w2.fold(__shfl_down(w2.m, h, 64), __shfl_down(w2.s, h, 64));
    }
    if (threadIdx.x == 0) {
        V[RL.lse_w_all] = w.value();
        V[RL.lse_w2_all] = w2.value();
    }
}

static_assert(FIN_LANES * FIN_ROWS == 64, "finalize workgroups are one wave");

__global__ __launch_bounds__(FIN_LANES * FIN_ROWS) void fpt_finalize_kernel(MergeArgs a) {
    const uint32_t row_blocks = (a.lay.n_rows + FIN_ROWS - 1) / FIN_ROWS;
    if (blockIdx.x >= row_blocks) {
        whole_run_sums(a, static_cast<int>(blockIdx.x - row_blocks));
        return;
    }
    const uint32_t r0 = blockIdx.x * FIN_ROWS + threadIdx.x / FIN_LANES;
    const uint32_t q = threadIdx.x % FIN_LANES;
    const uint32_t RT = a.lay.n_rows, J = a.lay.n_sub;
    const uint32_t r = r0 < RT ? r0 : RT - 1;      // lanes past the last row repeat it and do not write
    const int i = inst_of_row(a.mi, a.n_inst, r);
    const MergeInst m = a.mi[i];
    const uint32_t lr = r - m.row_base;
    const ResultLayout RL = result_layout(m.n_bins, J);
    uint64_t *Cn = a.counts + m.counts_off;
    double *V = a.values + m.values_off;
    unsigned long long cnt = 0;
    LseAcc la;
    for (uint32_t s = q; s < J; s += FIN_LANES) {
        cnt += Cn[RL.jk_count + static_cast<uint64_t>(s) * m.n_rows + lr];
        la.add(V[RL.jk_lse_w + static_cast<uint64_t>(s) * m.n_rows + lr]);
    }
#pragma unroll
    for (int h = FIN_LANES / 2; h >= 1; h >>= 1) {
        cnt += __shfl_down(cnt, h, FIN_LANES);
        la.fold(__shfl_down(la.m, h, FIN_LANES), __shfl_down(la.s, h, FIN_LANES));
    }
    const bool owner = q == 0 && r0 < RT;
    cnt = __shfl(cnt, 0, FIN_LANES);
    const double l = __shfl(la.value(), 0, FIN_LANES);
    if (owner) {
        Cn[RL.count + lr] = cnt;
        V[RL.lse_w + lr] = l;
    }
    if (lr < m.n_bins) {
        const double width = a.edges[m.edge_base + lr + 1] - a.edges[m.edge_base + lr];
        const double nt = static_cast<double>(m.n_traj);
        // jackknife: P_s / P = exp(lse_s - lse) * n_traj / n_s; spread over subsets / sqrt(J)
        double rel[64 / FIN_LANES], sum = 0.0, m2 = 0.0;
#pragma unroll
        for (int k = 0; k < 64 / FIN_LANES; ++k) {
            const uint32_t s = q + k * FIN_LANES;
            rel[k] = 0.0;
            if (s < J) {
                // runs of subset s: ids t = s mod J in [t_first, t_first + n_traj), as the number below
                // the end minus the number below the start (ids below x in subset s: x/J + (x mod J > s))
                const uint64_t x1 = m.t_first + m.n_traj, x0 = m.t_first;
                const double ns = static_cast<double>((x1 / J + ((x1 % J) > s ? 1 : 0)) - (x0 / J + ((x0 % J) > s ? 1 : 0)));
                rel[k] = exp(V[RL.jk_lse_w + static_cast<uint64_t>(s) * m.n_rows + lr] - l) * (nt / ns);
                sum += rel[k];
            }
        }
#pragma unroll
        for (int h = FIN_LANES / 2; h >= 1; h >>= 1) sum += __shfl_xor(sum, h, FIN_LANES);
        const double mean = sum / static_cast<double>(J);
#pragma unroll
        for (int k = 0; k < 64 / FIN_LANES; ++k)
            if (q + k * FIN_LANES < J) m2 += (rel[k] - mean) * (rel[k] - mean);
#pragma unroll
        for (int h = FIN_LANES / 2; h >= 1; h >>= 1) m2 += __shfl_xor(m2, h, FIN_LANES);
        if (owner) {
            V[RL.log_p + lr] = l - log(width) - log(nt);
            V[RL.rel_err_jk + lr] = (cnt == 0) ? NAN : sqrt(m2 / static_cast<double>(J - 1)) / sqrt(static_cast<double>(J));
            const double k2 = exp(V[RL.lse_w2 + lr] - 2.0 * l) - 1.0 / nt;
            V[RL.rel_err_kish + lr] = (cnt == 0) ? NAN : sqrt(fmax(k2, 0.0));
            // Kish's effective sample size of the bin, (sum w)^2 / sum w^2
            V[RL.ess + lr] = (cnt == 0) ? 0.0 : exp(2.0 * l - V[RL.lse_w2 + lr]);
            lognormal_bin(V, RL, lr, cnt, log(width) + log(nt));
            // the paper's gate (Sec. 2.4): the lognormal estimator holds for the result when no bin
            // with a normality p-value (n_j >= 8) falls below 0.5 %; every failing bin writes 0
            const double pv = V[RL.normal_p + lr];
            if (cnt >= 8 && pv == pv && pv < 0.005) V[RL.lognormal_gate] = 0.0;
        }
    }
}

// The learned bias on its own: r_theta at n given (phi, N) points (waves run full; lanes past
// n compute on a copy of the last point and do not write).
__global__ __launch_bounds__(256) void fpt_mlp_forward_kernel(const uint16_t *params, MlpConsts c, const float *phi,
                                                             const float *N, float *r, uint64_t n) {
    MlpTiles tiles;
    mlp_load_tiles(params, tiles);
    const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    const uint64_t j = i < n ? i : n - 1;
    const float out = mlp_forward(tiles, c, phi[j], N[j]);
    if (i < n) r[i] = out;
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
template <int POT, int BIAS, bool LDS>
static hipError_t launch_step_t(int n_wg, int block, size_t lds_bytes, const StepArgs &args, hipStream_t stream) {
    void (*kern)(StepArgs);
    if constexpr (BIAS == BIAS_MLP) {
        if (block > 256) return hipErrorInvalidConfiguration;
        kern = args.n_inst == 1 ? fpt_step_mlp1_kernel<POT, LDS> : fpt_step_mlp_kernel<POT, LDS>;
    } else {
        kern = fpt_step_kernel<POT, BIAS, LDS>;
    }
    if (lds_bytes > 0) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds_bytes));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(n_wg), dim3(block), lds_bytes, stream, args);
    return hipGetLastError();
}

template <int POT, bool LDS>
static hipError_t launch_step_b(int bias, int n_wg, int block, size_t lds, const StepArgs &a, hipStream_t s) {
    switch (bias) {
    case BIAS_NONE: return launch_step_t<POT, BIAS_NONE, LDS>(n_wg, block, lds, a, s);
    case BIAS_NOISE_SCALED: return launch_step_t<POT, BIAS_NOISE_SCALED, LDS>(n_wg, block, lds, a, s);
    case BIAS_POWER: return launch_step_t<POT, BIAS_POWER, LDS>(n_wg, block, lds, a, s);
    case BIAS_MLP: return launch_step_t<POT, BIAS_MLP, LDS>(n_wg, block, lds, a, s);
    default: return hipErrorInvalidValue;
    }
}

template <bool LDS>
static hipError_t launch_step_p(int pot, int bias, int n_wg, int block, size_t lds, const StepArgs &a, hipStream_t s) {
    switch (pot) {
    case POT_QUADRATIC: return launch_step_b<POT_QUADRATIC, LDS>(bias, n_wg, block, lds, a, s);
    case POT_QUADRATIC_BUMP: return launch_step_b<POT_QUADRATIC_BUMP, LDS>(bias, n_wg, block, lds, a, s);
    case POT_FLAT: return launch_step_b<POT_FLAT, LDS>(bias, n_wg, block, lds, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_step(int pot, int bias, bool tables_in_lds, int n_wg, int block, size_t lds_bytes,
                       const StepArgs &args, hipStream_t stream) {
    if (tables_in_lds) return launch_step_p<true>(pot, bias, n_wg, block, lds_bytes, args, stream);
    return launch_step_p<false>(pot, bias, n_wg, block, lds_bytes, args, stream);
}

hipError_t launch_init_queue(unsigned long long *queue, hipStream_t stream) {
    hipLaunchKernelGGL(fpt_init_queue_kernel, dim3(1), dim3(64), 0, stream, queue);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const uint16_t *params, MlpConsts c, const float *phi, const float *N, float *r,
                              uint64_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    const uint64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(fpt_mlp_forward_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, params, c,
                       phi, N, r, n);
    return hipGetLastError();
}

hipError_t launch_merge(const MergeArgs &args, int total_rows, int n_sub, hipStream_t stream) {
    const int64_t cells = static_cast<int64_t>(n_sub) * total_rows;
    const int64_t blocks = (cells + MERGE_CELLS - 1) / MERGE_CELLS + (total_rows + MERGE_CELLS - 1) / MERGE_CELLS + args.n_inst;
    hipLaunchKernelGGL(fpt_merge_kernel, dim3(static_cast<unsigned>(blocks)), dim3(MERGE_BLOCK), 0, stream, args);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fpt_finalize_kernel, dim3((total_rows + FIN_ROWS - 1) / FIN_ROWS + args.n_inst), dim3(FIN_LANES * FIN_ROWS), 0, stream, args);
    return hipGetLastError();
}

}  // namespace fpt

// fpt_train.hip -- training kernels of the learned proposal.
//
// The paper leaves the choice of the best bias open (Sec. 3.4); the learned proposal is trained
// to minimise the second moment of the importance weights of runs that end in a target window
// B*:  M2(theta) = E_0[w_0 w_theta 1_B*], estimated on paths drawn once from the current
// proposal theta_0 (Sec. 2.2: the weight is the ratio of the target and sample path densities).
// On a fixed path, step k's target-measure noise increment is eta_k = r_0,k dN + sqrt(dN) xi_k,
// and the weight the same path would have under a candidate bias held over groups of E steps
// is  ln w_theta = sum_e [ -r_theta(x_e) H_e + r_theta(x_e)^2 n_e dN/2 ],  H_e = sum of eta over
// group e, n_e its length.  So a path reduces to records (phi_e, k_e, H_e, n_e):
//
//   fpt_record_kernel    replays paths under theta_0 (the sampler's own step and network code,
//                        so the replay reproduces the sampled runs) and writes their records
//                        (every group's, or every stride-th group's, each then standing for
//                        stride groups: an unbiased estimate of the sums over a path);
//   fpt_train_eval_kernel  r_theta per record (binary32 network on the master weights);
//   fpt_train_path_kernel  per-path sum of ln w_theta in binary64 (one workgroup per path, fixed
//                        order);
//   fpt_train_softmax_kernel  c_i = w_0,i w_theta,i / sum_j w_0,j w_theta,j and log M2, or for
//                        the cross-entropy objective c_i = w_0,i / sum_j w_0,j and
//                        sum_i c_i ln w_theta,i (the KL divergence of the proposal from the
//                        target restricted to the window, up to a constant); w_0 may be
//                        tempered to w_0^beta;
//   fpt_train_bwd_kernel gradient of the objective: per record (forward recomputed in place) the
//                        coefficient
//                        c_i (r n dN - H) out_scale multiplies d(w3.h2 + b3)/d theta; each lane
//                        back-propagates one record, and the weight gradient of the 64x64 layer,
//                        a contraction over the 64 records of a wave, runs on
//                        v_mfma_f32_32x32x2f32 from LDS tiles;
//   fpt_train_reduce_kernel  per-workgroup partial gradients summed in a fixed order (binary64);
//   fpt_adam_kernel      Adam (Kingma & Ba) on the binary32 master weights, then the bfloat16
//                        copy that the sampler reads.
#include <hip/hip_runtime.h>
#include <math.h>

#include "fpt_kernels.h"
#include "fpt_team.h"
#include "fpt_train.h"

namespace fpt {

// ---------------------------------------------------------------------------
// replay into records
// ---------------------------------------------------------------------------
// One wave replays up to `slots` paths: with fewer paths than the chip has lanes a replay lasts as
// long as its longest path's steps at a lone wave's rate, so a wave takes 8 to 32 paths, its other lanes
// draw normals ahead for them (Team), and the network's unused columns are left out.
template <int POT, int BIAS>
__global__ __launch_bounds__(256) void fpt_record_kernel(RecordArgs a) {
    const uint32_t lane = __lane_id();
    const uint32_t wave = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
    const uint32_t i = wave * a.slots + lane;
    const bool have = lane < a.slots && i < a.n_paths;
    const StepConsts C = a.inst.c;
    const uint32_t j_cap = cap_groups(C.k_max);
    __shared__ bf16x8 tile_lds[BIAS == BIAS_MLP ? MLP_N_FRAG * 64 : 1];
    if constexpr (BIAS == BIAS_MLP) {
        if (threadIdx.x < 64) {
            MlpTiles tiles;
            mlp_load_tiles(a.mlp_params, tiles);
            mlp_store_tiles_lds(tiles, tile_lds);
        }
        __syncthreads();
    }
    const MlpConsts mc = a.inst.mlp;
    const uint64_t t = have ? a.t_ids[i] : 0;
    const uint64_t base = have ? a.rec_off[i] : 0;
    const uint64_t cap = have ? a.rec_off[i + 1] - base : 0;
    const uint32_t group = static_cast<uint32_t>(a.group), stride = static_cast<uint32_t>(a.stride);
    const PhiloxRun noise = philox_run(t, a.inst.stream, a.key0, a.key1);
    RunState R{C.phi_in, 0u, 0.0};
    Stopped F{0.0f, 0u, 0.0};
    uint64_t running = __ballot(have);
    float H = 0.0f, phi_e = R.phi;
    uint32_t k_e = 0;           // first step of the record's group
    uint32_t skip = 0;          // groups until the next that is kept
    uint64_t n_rec = 0;
    auto record = [&](uint32_t k_end) __attribute__((always_inline)) {      // the group k_e .. k_end - 1 is complete
        if (skip == 0) {
            skip = stride;
            if (n_rec < cap) {
                TrainRec rec;
                rec.phi = phi_e;
                rec.k = k_e;
                rec.H = H;
                rec.pn = (i << 5) | (k_end - k_e);
                a.rec[base + n_rec] = rec;
            }
            n_rec += 1;
        }
        skip -= 1;
        k_e = k_end;
        phi_e = R.phi;
        H = 0.0f;
    };
    // the sampling network (if any) is evaluated every E steps, wave-wide: a pass covers
    // max(4, E) steps, so every lane is at a multiple of the pass length at its start
    const int E = (BIAS == BIAS_MLP) ? a.mlp_every : 4;
    const int n_q = E > 4 ? E >> 2 : 1;
    const bool teamed = a.slots <= 32;
    Team team;
    if (teamed) {
        team_form(team, running, (lane == 0) ? 0ull : (~0ull >> (64 - lane)), lane, noise, 8);
    }
    auto network = [&](float phi_, float N_) __attribute__((always_inline)) {
        const MlpIn x = mlp_input(mc, phi_, N_);
        if (!teamed) return mc.out_scale * mlp_forward_lds(tile_lds, x);
        const MlpIn xs{lane_read(team.slot_lane, x.lo), lane_read(team.slot_lane, x.hi)};
        const float o = mlp_team_lds(tile_lds, xs, team.shift);
        return mc.out_scale * lane_read(team.fetch0, o);
    };
    const uint32_t odd_mask = normals_mask();
    BumpFar far{a.bump_far};    // bump potential: see group4
    F4 batch{};
    float r_mlp = 0.0f;
    const int batch_mask = team.groups() - 1;
    // the running lanes are all in group q; a record is due for all of them or for those that stopped
    auto step_group = [&](const F4 &z, uint32_t q) __attribute__((always_inline)) {
        const uint64_t before = running;
        const uint64_t m = group4<POT, BIAS>(C, j_cap, z, r_mlp, R, running, &F, far, &H);
        if (m || ((4u * q + 4u) & (group - 1)) == 0) {
            const bool stopped = (m >> lane) & 1u;
            const uint32_t k_end = stopped ? F.k : 4u * R.j;
            if (((before >> lane) & 1u) && ((k_end & (group - 1)) == 0 || stopped)) record(k_end);
        }
    };
    // With 8 paths or fewer a wave, a batch of normals is drawn for the passes that use it and a pass's
    // normals are fetched before its evaluation: a wave is alone on its SIMD here, and asking before
    // each group whether a batch, an evaluation or a fetch is due and waiting for the latter took a
    // fifth of its time (600 paths of 6e4 steps, evaluated every 16: 12.8 ms, now 10.5).
    if (teamed && batch_mask == 7 && E != 1 && group >= 4) {
        uint32_t q = 0;
        auto passes = [&](auto n_groups) {
            constexpr int NQ = decltype(n_groups)::value;
            while (running) {
                batch = team_draw(team, lane, R.j, a.key0, a.key1, odd_mask);
#pragma unroll 1
                for (int at = 0; at < 8 && running; at += NQ) {
                    F4 zz[NQ];
#pragma unroll
                    for (int i = 0; i < NQ; ++i) zz[i] = team_fetch8(team, batch, at + i);
                    if constexpr (BIAS == BIAS_MLP) r_mlp = network(R.phi, static_cast<float>(4u * R.j) * C.dN);
#pragma unroll
                    for (int i = 0; i < NQ; ++i) step_group(zz[i], q + i);
                    q += NQ;
                }
            }
        };
        using std::integral_constant;
        if (BIAS != BIAS_MLP || n_q == 4) passes(integral_constant<int, 4>{});
        else if (n_q == 2) passes(integral_constant<int, 2>{});
        else passes(integral_constant<int, 1>{});
    }
    for (int q = 0; running; ++q) {
        // q-th group of four steps; the lanes still running are all in their group q
        if constexpr (BIAS == BIAS_MLP) {
            if ((q & (n_q - 1)) == 0) r_mlp = network(R.phi, static_cast<float>(4u * R.j) * C.dN);
        }
        F4 z;
        if (teamed) {
            if ((q & batch_mask) == 0) batch = team_draw(team, lane, R.j, a.key0, a.key1, odd_mask);
            z = team_fetch(team, batch, q & batch_mask);
        } else {
            z = normals4(R.j, noise, a.key0, a.key1, odd_mask);
        }
        if (E == 1 || group < 4) {
            // the network before every step, or a record of every step
            const float ns[4] = {z.a, z.b, z.c, z.d};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const uint32_t ks = 4u * R.j + s;
                if constexpr (BIAS == BIAS_MLP) {
                    if (s > 0 && E == 1) r_mlp = network(R.phi, static_cast<float>(ks) * C.dN);
                }
                float dlw, sxi;
                const float r = em_step<POT, BIAS>(C, R.phi, ns[s], r_mlp, dlw, sxi);
                R.lw += static_cast<double>(dlw);
                H = H + __builtin_fmaf(r, C.dN, sxi);
                const uint64_t m = __ballot(stops(C, R.phi, ks + 1)) & running;
                const bool stopped = (m >> lane) & 1u;
                if (stopped) F = Stopped{R.phi, ks + 1, R.lw};
                if (((running >> lane) & 1u) && (((ks + 1) & (group - 1)) == 0 || stopped)) record(ks + 1);
                running &= ~m;
            }
            R.j += 1;
        } else {
            step_group(z, q);
        }
    }
    if (have) {
        a.k_out[i] = F.k;
        a.lw_out[i] = F.lw;
        a.st_out[i] = final_status(C, F.phi, F.k);
        a.n_rec_out[i] = n_rec;
    }
}

// ---------------------------------------------------------------------------
// the network being trained (binary32, master weights, no roundings)
// ---------------------------------------------------------------------------
// The weights are loop-invariant in the record loops; reading them through a pointer offset
// by a zero the compiler cannot see through keeps it from hoisting thousands of them out of
// the loop into registers (they stay uniform, scalar loads).
__device__ __forceinline__ int opaque_zero() {
    int z = 0;
    asm volatile("" : "+s"(z));
    return z;
}

__device__ __forceinline__ void net_inputs(const MlpConsts &M, float phi, uint32_t k, float dN, float x[3]) {
    const float N = static_cast<float>(k) * dN;
    x[0] = (phi - M.in_mean[0]) * M.in_inv[0];
    x[1] = (N - M.in_mean[1]) * M.in_inv[1];
    x[2] = (M.target_N - M.in_mean[2]) * M.in_inv[2];
}

__device__ __forceinline__ float net_unit1(const float *__restrict__ th, int u, const float x[3]) {
    float s = th[NET_B1 + u];
    s = __builtin_fmaf(th[NET_W1 + 3 * u + 0], x[0], s);
    s = __builtin_fmaf(th[NET_W1 + 3 * u + 1], x[1], s);
    s = __builtin_fmaf(th[NET_W1 + 3 * u + 2], x[2], s);
    return tanh_hw(s);
}

__device__ __forceinline__ void net_layer1(const float *__restrict__ th, const float x[3], float h1[64]) {
#pragma unroll
    for (int u = 0; u < 64; ++u) h1[u] = net_unit1(th, u, x);
}

// ---------------------------------------------------------------------------
// forward: r per record, ln w_theta per path
// ---------------------------------------------------------------------------
// Bound by arithmetic: 4500 fused multiply-adds and 128 activations per record.  A wave takes 64 records
// in order, whatever their paths, and keeps h2 = W2 h1 on the matrix cores (M = unit, N = record,
// K = input), W2 in registers for the whole kernel: one lane computes both units of a k pair for its
// record, and a swap of half waves turns them into the operands of records 0 .. 31 and 32 .. 63; the
// same swap of the two results gives each lane its record's units back, so nothing goes through LDS.
// The binary32 product adds k in ascending order with one rounding each, as a chain of fma does, so r
// is the same bit for bit.  7.4e5 records of 700 paths: one workgroup per path 190 us; two records per
// lane with W2 (more than the scalar cache) read by scalar loads 126 us; now 87 us.
typedef float f32x16v __attribute__((ext_vector_type(16)));

struct Half2 {
    float lo, hi;
};
// lo = the low half waves of x and y, hi = their high halves
__device__ __forceinline__ Half2 swap_halves(float x, float y) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return {__uint_as_float(p[0]), __uint_as_float(p[1])};
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(EVAL_WG_PER_CU, EVAL_WG_PER_CU))) void
fpt_train_eval_kernel(TrainArgs a, const float *__restrict__ th0) {
    const int lane = threadIdx.x & 63;
    const int col = lane & 31, kh = lane >> 5;
    // A fragments of W2: row = unit 32 ub + col, k = 2 ks + kh
    float W[2][32];
#pragma unroll
    for (int ub = 0; ub < 2; ++ub)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float4 v = *reinterpret_cast<const float4 *>(th0 + NET_W2 + 64 * (32 * ub + col) + 8 * j + 4 * kh);
            const Half2 p = swap_halves(v.x, v.y), q = swap_halves(v.z, v.w);
            W[ub][4 * j + 0] = p.lo;
            W[ub][4 * j + 1] = q.lo;
            W[ub][4 * j + 2] = p.hi;
            W[ub][4 * j + 3] = q.hi;
        }
    const uint64_t n_tiles = (a.n_rec + 63) / 64;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    for (uint64_t tile = wave; tile < n_tiles; tile += 4 * gridDim.x) {
        const float *th = th0 + opaque_zero();
        const uint64_t e = tile * 64 + lane;
        const TrainRec R = a.rec[e < a.n_rec ? e : a.n_rec - 1];
        float x[3];
        net_inputs(a.mc, R.phi, R.k, a.dN, x);
        f32x16v z[2][2];
#pragma unroll
        for (int ub = 0; ub < 2; ++ub)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 b = *reinterpret_cast<const float4 *>(th + NET_B2 + 32 * ub + 8 * g + 4 * kh);
                z[ub][0][4 * g + 0] = z[ub][1][4 * g + 0] = b.x;
                z[ub][0][4 * g + 1] = z[ub][1][4 * g + 1] = b.y;
                z[ub][0][4 * g + 2] = z[ub][1][4 * g + 2] = b.z;
                z[ub][0][4 * g + 3] = z[ub][1][4 * g + 3] = b.w;
            }
#pragma unroll
        for (int ks = 0; ks < 32; ++ks) {
            const Half2 h = swap_halves(net_unit1(th, 2 * ks, x), net_unit1(th, 2 * ks + 1, x));
#pragma unroll
            for (int ub = 0; ub < 2; ++ub) {
                z[ub][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(W[ub][ks], h.lo, z[ub][0], 0, 0, 0);
                z[ub][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(W[ub][ks], h.hi, z[ub][1], 0, 0, 0);
            }
        }
        float o = 0.0f;
#pragma unroll
        for (int ub = 0; ub < 2; ++ub)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                Half2 h[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) h[q] = swap_halves(z[ub][0][4 * g + q], z[ub][1][4 * g + q]);
#pragma unroll
                for (int q = 0; q < 4; ++q) o = __builtin_fmaf(th[NET_W3 + 32 * ub + 8 * g + q], tanh_hw(h[q].lo), o);
#pragma unroll
                for (int q = 0; q < 4; ++q) o = __builtin_fmaf(th[NET_W3 + 32 * ub + 8 * g + 4 + q], tanh_hw(h[q].hi), o);
            }
        if (e < a.n_rec) a.r[e] = a.mc.out_scale * (o + th[NET_B3]);
    }
}

// ln w_theta of a path: its records' terms in binary64, one workgroup per path, in a fixed order.
__global__ __launch_bounds__(256) void fpt_train_path_kernel(TrainArgs a) {
    __shared__ double red[256];
    const int i = a.path0 + blockIdx.x;
    const uint64_t e0 = a.rec_off[i], e1 = a.rec_off[i + 1];
    const double hdN = 0.5 * static_cast<double>(a.dN);
    double s = 0.0;
    for (uint64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
        const TrainRec R = a.rec[e];
        const double rd = static_cast<double>(a.r[e - a.rec0]);
        const double n = static_cast<double>(R.pn & 31u);
        s += (-rd * static_cast<double>(R.H) + rd * rd * n * hdN) * static_cast<double>(a.rec_weight);
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.lw_theta[i] = red[0];
}

// The lowest index of a record whose path index or step count is out of range (a host loop over 7.4e5
// records took longer than the kernels that use them).
__global__ __launch_bounds__(256) void fpt_train_check_kernel(const TrainRec *rec, uint64_t n_rec, uint32_t n_paths,
                                                              unsigned long long *first_bad) {
    for (uint64_t e = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < n_rec;
         e += static_cast<uint64_t>(gridDim.x) * blockDim.x)
        if (!train_record_ok(rec[e].pn, n_paths)) atomicMin(first_bad, static_cast<unsigned long long>(e));
}

// ---------------------------------------------------------------------------
// softmax over paths and log M2
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void fpt_train_softmax_kernel(TrainArgs a) {
    __shared__ double red[1024];
    const int tid = threadIdx.x;
    const double use_t = a.objective == 0 ? 1.0 : 0.0;
    double m = -INFINITY;
    const double beta = static_cast<double>(a.temper);
    for (int i = tid; i < a.n_paths; i += 1024) m = fmax(m, beta * a.lw0[i] + use_t * a.lw_theta[i]);
    red[tid] = m;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) red[tid] = fmax(red[tid], red[tid + w]);
        __syncthreads();
    }
    const double M = red[0];
    __syncthreads();
    double s = 0.0;
    for (int i = tid; i < a.n_paths; i += 1024) s += exp(beta * a.lw0[i] + use_t * a.lw_theta[i] - M);
    red[tid] = s;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    const double S = red[0];
    __syncthreads();
    double ce = 0.0;
    for (int i = tid; i < a.n_paths; i += 1024) {
        const double c = exp(beta * a.lw0[i] + use_t * a.lw_theta[i] - M) / S;
        a.c[i] = c;
        ce += c * a.lw_theta[i];
    }
    red[tid] = ce;
    __syncthreads();
    for (int w = 512; w > 0; w >>= 1) {
        if (tid < w) red[tid] += red[tid + w];
        __syncthreads();
    }
    if (tid == 0) a.loss[0] = a.objective == 0 ? M + log(S) - log(a.n_total) : red[0];
}

// ---------------------------------------------------------------------------
// backward: four waves per workgroup, 64 records per tile
// ---------------------------------------------------------------------------
constexpr int TS = 65;  // padded row stride of the [sample][unit] LDS tiles

// The three 64x64x64 contractions of a tile run on v_mfma_f32_32x32x2f32 (binary32 products and
// sums, like the rest of the training network).  Operand layout of that instruction, per lane l
// and k-step: A[m = l & 31][k = l >> 5], B[k = l >> 5][n = l & 31]; accumulator element q of lane l
// is D[m = (q & 3) + 8 (q >> 2) + 4 (l >> 5)][n = l & 31] of its 32x32 block.
//
// Bound by the phases of a tile that wait for one another beside the matrix work (384 instructions of
// 72 cycles on a SIMD, measured: 27 600 cycles a tile).  The four waves of a workgroup, one per SIMD,
// take a 32x32 block each of the contractions, 16 of the 64 units each of layer 1, and a different one
// of the per-record and per-unit sums; four workgroups share a CU, so that on each SIMD one tile's
// matrix work runs beside the others' vector work and waits.  With one wave per tile and SIMD, every
// phase of a tile after the other, a tile took 61 000 cycles; now 50 000 (7.4e5 records in 286 and
// 243 us, 1.4e6 in 487 and 422 us).
// Every sum keeps its order, so that the gradient is the same bit for bit.
__device__ __forceinline__ int acc_row(int q, int lane) { return (q & 3) + 8 * (q >> 2) + 4 * (lane >> 5); }

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void fpt_train_bwd_kernel(TrainArgs a,
                                                                                          const float *__restrict__ th0) {
    // two [sample][unit] tiles: HA holds h1, then delta1; HB holds h2, then delta2 (35 KB with the
    // inputs and coefficients, so four workgroups share a CU)
    __shared__ float HA[64 * TS];
    __shared__ float HB[64 * TS];
    __shared__ float XS[64 * 4];
    __shared__ float GS[64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mb = wave >> 1, nb = wave & 1;        // this wave's block of the contractions
    const int u0 = 16 * wave;                       // and its units of layer 1 and delta2
    const int col = lane & 31, kh = lane >> 5;
    const double dNd = static_cast<double>(a.dN);
    // this lane's B fragments of W2 for the whole kernel: WT for h1 W2^T (k = input v, n = unit u),
    // WN for delta2 W2 (k = unit u, n = input v); and its unit's b2
    float WT[32], WN[32];
#pragma unroll
    for (int ks = 0; ks < 32; ++ks) {
        WT[ks] = th0[NET_W2 + 64 * (32 * nb + col) + 2 * ks + kh];
        WN[ks] = th0[NET_W2 + 64 * (2 * ks + kh) + 32 * nb + col];
    }
    const float b2v = th0[NET_B2 + 32 * nb + col];
    f32x16v acc;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
    // per-unit sums: w3 and b3 (wave 0), b2 (wave 1), W1 and b1 (wave 2)
    float g0 = 0.0f, g1 = 0.0f, g2 = 0.0f, g3 = 0.0f;
    const uint64_t n_tiles = (a.n_rec + 63) / 64;
    for (uint64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const float *th = th0 + opaque_zero();
        const uint64_t e = tile * 64 + lane;
        const bool valid = e < a.n_rec;
        TrainRec R{};
        if (valid) R = a.rec[e];
        else R.phi = a.mc.in_mean[0];
        // forward: h1 into HA (this lane's record, this wave's units), h2 = tanh(W2 h1 + b2) into HB
        // on the matrix cores (M = record, N = unit, K = input), then r from a record's row of HB
        {
            float x[3];
            net_inputs(a.mc, R.phi, R.k, a.dN, x);
#pragma unroll
            for (int u = 0; u < 16; ++u) HA[lane * TS + u0 + u] = net_unit1(th, u0 + u, x);
            if (wave == 0) {
                XS[lane * 4 + 0] = x[0];
                XS[lane * 4 + 1] = x[1];
                XS[lane * 4 + 2] = x[2];
                XS[lane * 4 + 3] = 1.0f;
            }
        }
        __syncthreads();
        {
            f32x16v z;
#pragma unroll
            for (int q = 0; q < 16; ++q) z[q] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < 32; ++ks)
                z = __builtin_amdgcn_mfma_f32_32x32x2f32(HA[(32 * mb + col) * TS + 2 * ks + kh], WT[ks], z, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 16; ++q) HB[(32 * mb + acc_row(q, lane)) * TS + 32 * nb + col] = tanh_hw(z[q] + b2v);
        }
        __syncthreads();
        if (wave == 0) {
            float o = 0.0f, g = 0.0f;
#pragma unroll 16
            for (int u = 0; u < 64; ++u) o = __builtin_fmaf(th[NET_W3 + u], HB[lane * TS + u], o);
            if (valid) {
                const double r = static_cast<double>(a.mc.out_scale * (o + th[NET_B3]));
                // (a path index out of range is reported once the call's work is done)
                const uint32_t path = min(R.pn >> 5, static_cast<uint32_t>(a.n_paths - 1));
                const double n = static_cast<double>(R.pn & 31u);
                g = static_cast<float>(a.c[path] * (r * n * dNd - static_cast<double>(R.H)) *
                                       static_cast<double>(a.mc.out_scale) * static_cast<double>(a.rec_weight));
            }
            GS[lane] = g;
            // lane = unit: w3 and b3 from h2 (GS is this wave's own: no barrier)
            float sw3 = 0.0f, sb3 = 0.0f;
#pragma unroll 16
            for (int s = 0; s < 64; ++s) {
                const float gs = GS[s];
                sw3 = __builtin_fmaf(gs, HB[s * TS + lane], sw3);
                sb3 += gs;
            }
            g0 += sw3;
            g1 += sb3;
        }
        __syncthreads();
        // delta2 = g w3 (1 - h2^2), in place over h2 (this lane's record, this wave's units)
        {
            const float g = GS[lane];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const float h = HB[lane * TS + u0 + u];
                HB[lane * TS + u0 + u] = (g * th[NET_W3 + u0 + u]) * __builtin_fmaf(-h, h, 1.0f);
            }
        }
        __syncthreads();
        // lane = unit: b2 from delta2
        if (wave == 1) {
            float sb2 = 0.0f;
#pragma unroll 16
            for (int s = 0; s < 64; ++s) sb2 += HB[s * TS + lane];
            g0 += sb2;
        }
        // dW2[u][v] += sum_s delta2[s][u] h1[s][v]: M = u, N = v, K = the tile's samples; and
        // delta1 = (delta2 W2) (1 - h1^2) (M = record, N = input, K = unit), whose elements overwrite
        // the h1 that they are scaled by (one lane owns each) once every wave has read its h1 for dW2
        {
#pragma unroll 8
            for (int ks = 0; ks < 32; ++ks) {
                const int s = 2 * ks + kh;
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(HB[s * TS + 32 * mb + col], HA[s * TS + 32 * nb + col], acc, 0, 0, 0);
            }
            f32x16v z;
#pragma unroll
            for (int q = 0; q < 16; ++q) z[q] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < 32; ++ks)
                z = __builtin_amdgcn_mfma_f32_32x32x2f32(HB[(32 * mb + col) * TS + 2 * ks + kh], WN[ks], z, 0, 0, 0);
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int idx = (32 * mb + acc_row(q, lane)) * TS + 32 * nb + col;
                const float h = HA[idx];
                HA[idx] = z[q] * __builtin_fmaf(-h, h, 1.0f);
            }
        }
        __syncthreads();
        // lane = unit: W1, b1 from delta1
        if (wave == 2) {
            float sb1 = 0.0f, s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll 8
            for (int s = 0; s < 64; ++s) {
                const float d = HA[s * TS + lane];
                sb1 += d;
                s0 = __builtin_fmaf(d, XS[s * 4 + 0], s0);
                s1 = __builtin_fmaf(d, XS[s * 4 + 1], s1);
                s2 = __builtin_fmaf(d, XS[s * 4 + 2], s2);
            }
            g0 += sb1;
            g1 += s0;
            g2 += s1;
            g3 += s2;
        }
        __syncthreads();
    }
    // partial gradient of this workgroup
    float *P = a.part + static_cast<size_t>(blockIdx.x) * NET_N_PARAMS;
#pragma unroll
    for (int q = 0; q < 16; ++q) P[NET_W2 + 64 * (32 * mb + acc_row(q, lane)) + 32 * nb + col] = acc[q];
    if (wave == 0) {
        P[NET_W3 + lane] = g0;
        if (lane == 0) P[NET_B3] = g1;
    } else if (wave == 1) {
        P[NET_B2 + lane] = g0;
    } else if (wave == 2) {
        P[NET_B1 + lane] = g0;
        P[NET_W1 + 3 * lane + 0] = g1;
        P[NET_W1 + 3 * lane + 1] = g2;
        P[NET_W1 + 3 * lane + 2] = g3;
    }
}

// Partial gradients summed in binary64 in a fixed order: RED_COLS parameters by RED_SPLIT ranges of
// workgroups, then the ranges in order.  One thread per parameter waited for 1024 loads in turn
// (260 us for 18 MB); RED_SPLIT threads per parameter, with eight loads in flight each, share them.
constexpr int RED_COLS = 32, RED_SPLIT = 32;

__global__ __launch_bounds__(RED_COLS * RED_SPLIT) void fpt_train_reduce_kernel(const float *part, int n_part, double *grad) {
    __shared__ double red[RED_SPLIT][RED_COLS];
    const int col = threadIdx.x % RED_COLS, q = threadIdx.x / RED_COLS;
    const int j = blockIdx.x * RED_COLS + col;
    double s = 0.0;
    if (j < NET_N_PARAMS) {
#pragma unroll 8
        for (int w = q; w < n_part; w += RED_SPLIT) s += static_cast<double>(part[static_cast<size_t>(w) * NET_N_PARAMS + j]);
    }
    red[q][col] = s;
    __syncthreads();
    if (q == 0 && j < NET_N_PARAMS) {
        for (int k = 1; k < RED_SPLIT; ++k) s += red[k][col];
        grad[j] = s;
    }
}

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    uint32_t b = __float_as_uint(x);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return static_cast<uint16_t>(b >> 16);
}

__global__ __launch_bounds__(256) void fpt_adam_kernel(AdamArgs a) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= NET_N_PARAMS) return;
    const float g = static_cast<float>(a.grad[j]);
    const float m = a.beta1 * a.m[j] + (1.0f - a.beta1) * g;
    const float v = a.beta2 * a.v[j] + (1.0f - a.beta2) * g * g;
    a.m[j] = m;
    a.v[j] = v;
    const float mh = m / a.bc1;
    const float vh = v / a.bc2;
    const float th = a.theta[j] - a.lr * mh / (sqrtf(vh) + a.eps);
    a.theta[j] = th;
    a.bf16[j] = bf16_bits(th);
}

__global__ __launch_bounds__(256) void fpt_to_bf16_kernel(const float *theta, uint16_t *bf) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < NET_N_PARAMS) bf[j] = bf16_bits(theta[j]);
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
template <int POT, int BIAS>
static hipError_t launch_record_t(const RecordArgs &a, hipStream_t s) {
    const unsigned waves = (a.n_paths + a.slots - 1) / a.slots;
    const unsigned per_wg = record_waves_per_group(waves, a.cus);
    hipLaunchKernelGGL((fpt_record_kernel<POT, BIAS>), dim3((waves + per_wg - 1) / per_wg), dim3(64 * per_wg), 0, s, a);
    return hipGetLastError();
}

template <int POT>
static hipError_t launch_record_b(int bias, const RecordArgs &a, hipStream_t s) {
    switch (bias) {
    case BIAS_NONE: return launch_record_t<POT, BIAS_NONE>(a, s);
    case BIAS_NOISE_SCALED: return launch_record_t<POT, BIAS_NOISE_SCALED>(a, s);
    case BIAS_POWER: return launch_record_t<POT, BIAS_POWER>(a, s);
    case BIAS_MLP: return launch_record_t<POT, BIAS_MLP>(a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_records(int pot, int bias, const RecordArgs &a, hipStream_t s) {
    if (a.n_paths == 0) return hipSuccess;
    switch (pot) {
    case POT_QUADRATIC: return launch_record_b<POT_QUADRATIC>(bias, a, s);
    case POT_QUADRATIC_BUMP: return launch_record_b<POT_QUADRATIC_BUMP>(bias, a, s);
    case POT_FLAT: return launch_record_b<POT_FLAT>(bias, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_train_check(const TrainArgs &a, unsigned long long *first_bad, hipStream_t s) {
    if (a.n_rec == 0) return hipSuccess;
    hipLaunchKernelGGL(fpt_train_check_kernel, dim3(check_groups(a.n_rec, a.cus)), dim3(256), 0, s, a.rec, a.n_rec,
                       static_cast<uint32_t>(a.n_paths), first_bad);
    return hipGetLastError();
}

hipError_t launch_train_loss(const TrainArgs &a, const uint64_t *h_off, hipStream_t s) {
    if (a.n_paths <= 0) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    for (int64_t i = 0, j; i < a.n_paths; i = j) {
        j = eval_piece_end(h_off, a.n_paths, i);
        TrainArgs p = a;
        p.path0 = static_cast<int32_t>(i);
        p.rec0 = h_off[i];
        if (h_off[j] > h_off[i]) {
            p.rec = a.rec + h_off[i];
            p.n_rec = h_off[j] - h_off[i];
            hipLaunchKernelGGL(fpt_train_eval_kernel, dim3(eval_groups(p.n_rec, a.cus)), dim3(256), 0, s, p, a.theta);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
            p.rec = a.rec;
        }
        hipLaunchKernelGGL(fpt_train_path_kernel, dim3(static_cast<unsigned>(j - i)), dim3(256), 0, s, p);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fpt_train_softmax_kernel, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_train_grad(const TrainArgs &a, hipStream_t s) {
    if (a.n_part <= 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(fpt_train_bwd_kernel, dim3(a.n_part), dim3(256), 0, s, a, a.theta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fpt_train_reduce_kernel, dim3((NET_N_PARAMS + RED_COLS - 1) / RED_COLS), dim3(RED_COLS * RED_SPLIT), 0, s,
                       a.part, a.n_part, a.grad);
    return hipGetLastError();
}

hipError_t launch_adam(const AdamArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(fpt_adam_kernel, dim3((NET_N_PARAMS + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float *theta, uint16_t *bf, hipStream_t s) {
    hipLaunchKernelGGL(fpt_to_bf16_kernel, dim3((NET_N_PARAMS + 255) / 256), dim3(256), 0, s, theta, bf);
    return hipGetLastError();
}

}  // namespace fpt

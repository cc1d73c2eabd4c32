// fpt_team.h -- a wave's lanes working together on fewer runs than lanes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fpt_device.h"

namespace fpt {

// A wave's lanes shared out over the few runs it has left.  With n <= 32 runs the wave works
// G = 2, 4 or 8 groups of steps ahead: lane l draws the normals of group j + l / S of the run in
// slot l % S (S = 64 / G slots, the n runs in the first n of them), and in each of the next G groups
// a run's own lane reads its four normals from the lane that drew them; they are the values it would
// draw itself.  A step costs a wave about 38 instructions of normals and 22 of stepping whatever its
// number of runs, and a wave issues at most one per 5 cycles (two waves on a SIMD one per 2.4), so a
// lone wave's step falls from 60 x 5 cycles towards the 130 of its chain of dependent operations
// (measured with 8 runs or fewer: 137 with a wall, 151 without one).
struct Team {
    int shift = 6;                // S = 1 << shift slots
    int slot_lane = 0;            // byte address (4 x lane) of the lane that owns this lane's slot's run
    int fetch0 = 0;               // byte address of the lane that draws this lane's run's first group
    PhiloxRun noise{};            // noise of the slot's run
    __device__ __forceinline__ int groups() const { return 64 >> shift; }
};

__device__ __forceinline__ uint32_t lane_read(int addr, uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_ds_bpermute(addr, static_cast<int>(v)));
}
__device__ __forceinline__ float lane_read(int addr, float v) { return __uint_as_float(lane_read(addr, __float_as_uint(v))); }

// Whether a wave with n runs left, on S = 1 << shift slots, can share its lanes out further.
__device__ __forceinline__ bool team_halves(int shift, int n, int most) {
    return 2 * n <= (1 << shift) && (64 >> shift) < most;
}

// Share the wave's lanes out over the runs of the lanes in `act` (at most 32; wave-uniform).  Runs
// that end later leave their slots idle until the team is formed anew.
__device__ __forceinline__ void team_form(Team &T, uint64_t act, uint64_t lt_mask, uint32_t lane, const PhiloxRun &own, int most) {
    const int n = __popcll(act);
    const int before = __popcll(act & lt_mask);
    int shift = 6;
    while (team_halves(shift, n, most)) --shift;
    T.shift = shift;
    const bool mine = (act >> lane) & 1u;
    // a permutation that sends the owners to lanes 0 .. n-1 in order and the others after them
    const int to = mine ? before : n + (static_cast<int>(lane) - before);
    const int owner = __builtin_amdgcn_ds_permute(4 * to, static_cast<int>(lane));
    T.slot_lane = 4 * __builtin_amdgcn_ds_bpermute(4 * (static_cast<int>(lane) & ((1 << shift) - 1)), owner);
    T.fetch0 = 4 * before;
    T.noise = PhiloxRun{lane_read(T.slot_lane, own.a), lane_read(T.slot_lane, own.b), lane_read(T.slot_lane, own.c),
                        lane_read(T.slot_lane, own.d)};
}

// The normals of this lane's slot's run, lane / S groups after the group j of that run (own_j:
// every lane's own run's group).
__device__ __forceinline__ F4 team_draw(const Team &T, uint32_t lane, uint32_t own_j, uint32_t key0, uint32_t key1,
                                        uint32_t odd_mask) {
    return normals4(lane_read(T.slot_lane, own_j) + (lane >> T.shift), T.noise, key0, key1, odd_mask);
}

// This lane's run's normals of the g-th group of the batch z.
__device__ __forceinline__ F4 team_fetch(const Team &T, const F4 &z, int g) {
    const int from = T.fetch0 + ((4 * g) << T.shift);
    return F4{lane_read(from, z.a), lane_read(from, z.b), lane_read(from, z.c), lane_read(from, z.d)};
}

// The same for G = 8, where the place in the batch is an offset of the exchange.
__device__ __forceinline__ F4 team_fetch8(const Team &T, const F4 &z, int g) {
    const int from = T.fetch0 + 32 * g;
    return F4{lane_read(from, z.a), lane_read(from, z.b), lane_read(from, z.c), lane_read(from, z.d)};
}

}  // namespace fpt

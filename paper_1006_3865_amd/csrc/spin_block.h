// spin_block.h -- several sweeps of a tile per launch (k_block): plan, host
// rule and launch.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spin_internal.h"

namespace spin {

// Shape of a k_block launch: k sweeps; tiles of TX 8-site groups (2D, L % 8 == 0;
// 0: full rows) by TY rows (by TZ planes in 3D), threads per workgroup.
struct BlockPlan {
  uint32_t k, TX, TY, TZ, threads;
};

// Tiles (workgroups) and LDS bytes of a plan.
uint32_t block_tiles(const Lat& lat, const BlockPlan& p);
size_t block_lds_bytes(const Lat& lat, const BlockPlan& p);
// Whether k_block can run this lattice and bounds at all, and this plan.
bool block_lattice_ok(const Lat& lat, const Accept& acc);
bool block_plan_ok(const Lat& lat, const BlockPlan& p);

// Plan for launches of k sweeps (1 .. kBlockMaxK) and its estimated time in microseconds; k == 0 in
// the plan: none fits.  Host only.
constexpr uint32_t kBlockMaxK = 8;
BlockPlan block_plan(const Lat& lat, uint32_t k, double* us);

// p.k sweeps t .. t+k-1 from src into dst.  Bit j of rec_mask: count (E, M)
// after sweep t+j into part[(r * tiles + tile) * 2 ...], r = the number of
// lower set bits.
hipError_t launch_block(const Lat& lat, const int8_t* src, int8_t* dst, uint32_t t, const Accept& acc,
                        const BlockPlan& p, uint32_t rec_mask, int64_t* part, hipStream_t stream);

// n sweeps of a whole small lattice by one workgroup, in place (k_whole): its estimated time in
// microseconds (< 0: it cannot run this lattice), and the launch; E, M: device arrays of n / every.
double whole_us(const Lat& lat, const Accept& acc, uint32_t n);
hipError_t launch_whole(const Lat& lat, uint32_t t, uint32_t n, const Accept& acc, uint32_t every, int64_t* E, int64_t* M,
                        hipStream_t stream);

}  // namespace spin

// spin_block_kernels.hip -- k sweeps of a tile per launch (k_block): the
// lattices between the smallest and the register-column sizes, where one
// launch per sweep is bound by its own latency (loads, two dependent colour
// phases, stores) and not by arithmetic or memory.  Microseconds a sweep, one
// launch per sweep (or two) before and k_block now: 2D Ising L = 1024 5.6 ->
// 1.5, L = 1000 14.5 -> 1.5; 3D Ising
// L = 64 7.3 -> 2.4, L = 100 30 -> 5.1, L = 256 24 -> 17.8; 3D +-J L = 128 13.5 -> 5.7.
//
// A workgroup owns a tile and loads it with a halo of 2k sites on every open
// side into LDS, then runs the 2k colour phases of k sweeps there: phase p
// (1 .. 2k) updates the rows at least p away from the edge of the loaded
// region, so after the last one the tile itself is exact and goes to dst (the
// other buffer of the ping-pong pair; neighbouring tiles recompute the shared
// halo from the same data and draws, so all agree bit for bit).
//   2D, L % 8 == 0: tiles of TX groups x TY rows, with hx = ceil(2k / 8) halo
//     groups left and right (what is wrong at the outer edge moves inwards by
//     one site a phase and never reaches the tile), 2k rows above and below;
//   3D, and 2D with L % 8 != 0: full rows (periodic in x), TY rows (x TZ planes).
//
// LDS keeps one byte per site, 0x00 (+1) or 0x02 (-1), in two planes by
// colour: plane c holds the four colour-c sites of an 8-site group as one
// dword (byte x / 2 of the row).  The active sites of a phase are then a dword
// as they stand and their neighbours are dwords of the other plane at the same
// place (the row neighbour on one side: moved by a byte), so with n = negative
// neighbours and a = the site is negative one byte per site holds
//   v = 2 n + 16 a = sum of the neighbour bytes + 8 * the site's own byte
// with one add per neighbour and no masks.  v_dot4 turns two such bytes into
// the offset of an 8-byte entry with both sites' accept bounds (15 x 15
// entries).  For the glass a coupling byte (0x02 for -1) joins each neighbour
// by an XOR.
//
// The rows of the region are listed in LDS from the innermost outwards (LDS
// offset, parity, Philox counter base), so that the rows of phase p are the
// first so many entries and no coordinate is wrapped or divided in the loop.
//
// L % 8 != 0 (RAG): the 8-site groups of the Philox counter run across row
// ends, so row r begins o = (r L) mod 8 sites into its first group and keeps
// that place in LDS: its own dwords are aligned, a neighbour row's are cut from
// two aligned dwords by the difference of the rows' o / 2 bytes (reading LDS at
// odd bytes instead took four times as long), sites outside the row are masked
// and the periodic neighbour of its ends is inserted.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "spin_block.h"
#include "spin_device.h"
#include "spin_launch.h"
#include "spin_lds.h"
#include "spin_tile.h"

namespace spin {

struct BlockArgs {
  RoundKeys keys;
  uint32_t bound[8];
  uint32_t L, GPR;           // edge; full groups per row (L / 8)
  uint32_t t, k, replica;
  uint32_t TX, TY, TZ, hx;   // tile (TX in groups; full rows: all) and halo groups
  uint32_t nbx;              // tiles along x (2D) / y (3D)
  uint32_t plane, jplane;    // LDS bytes of one spin plane (all rows); offset of the coupling planes
  uint32_t first;            // LDS offset of spin plane 0
  uint32_t rec_mask;
  uint32_t nbytes;           // L^d rounded up to 8
  uint32_t jstride;          // bytes between the coupling directions (L^d)
};

typedef uint32_t blk_u2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kNeg = 0x02020202u;
constexpr uint32_t kBlkTable = 15u * 15u * 8u;                           // accept-bound pairs
constexpr uint32_t kBlkRec = kBlkTable;                                  // record counts, 2 uint32 each
constexpr uint32_t kBlkList = (kBlkTable + 8u * kBlockMaxK + 15u) & ~15u;  // row list

// A listed row.  x: bit 0 the parity of y + z, bits 2-17 the LDS offset of its first dword in a
// plane; RAG also bits 18-19 o / 2, and from bit 20 for the rows y-1, y+1, z-1, z+1 three bits
// each: their o / 2 minus this row's (signed), the byte shift of a dword read there.
// y: the Philox counter of its first group.
__device__ __forceinline__ uint32_t row_at(uint32_t e) { return e & 0x3FFFCu; }
__device__ __forceinline__ uint32_t row_o2(uint32_t e) { return (e >> 18) & 3u; }
template <int I>
__device__ __forceinline__ int row_shift(uint32_t e) { return (int)(e << (9 - 3 * I)) >> 29; }

// Negative-site bytes of an 8-site group of int8 values (0x01 / 0xFF): x = even sites, y = odd sites.
__device__ __forceinline__ uint2 blk_split(uint32_t lo, uint32_t hi) {
  return make_uint2(__builtin_amdgcn_perm(hi, lo, 0x06040200u), __builtin_amdgcn_perm(hi, lo, 0x07050301u));
}
// The reverse: v_perm as a table of two bytes (0x00 -> 0x01, 0x02 -> 0xFF), then joined.
__device__ __forceinline__ uint2 blk_join(uint32_t even, uint32_t odd) {
  const uint32_t e = __builtin_amdgcn_perm(0u, 0x00FF0001u, even), o = __builtin_amdgcn_perm(0u, 0x00FF0001u, odd);
  return make_uint2(__builtin_amdgcn_perm(o, e, 0x05010400u), __builtin_amdgcn_perm(o, e, 0x07030602u));
}

// The entry of lattice row (gy, gz) whose LDS row begins at byte `at` of plane 0 (RAG: after a pad dword).
template <int D, bool RAG>
__device__ __forceinline__ uint2 blk_row(uint32_t at, uint32_t gy, uint32_t gz, uint32_t L, uint32_t GPR) {
  const uint32_t row = gz * L + gy;
  uint2 e;
  e.x = (at + (RAG ? 4u : 0u)) | ((gy + gz) & 1u);
  if (RAG) {
    const uint32_t o2 = ((row * L) >> 1) & 3u;  // low bits of a product: no overflow matters
    e.x |= o2 << 18;
    const uint32_t nb[4] = {gz * L + (gy ? gy - 1u : L - 1u), gz * L + (gy + 1u < L ? gy + 1u : 0u),
                            (gz ? gz - 1u : L - 1u) * L + gy, (gz + 1u < L ? gz + 1u : 0u) * L + gy};
#pragma unroll
    for (int i = 0; i < 2 * D - 2; ++i) e.x |= (((((nb[i] * L) >> 1) & 3u) - o2) & 7u) << (20 + 3 * i);
    e.y = (uint32_t)(((uint64_t)row * L) >> 3);
  } else {
    e.y = row * GPR;
  }
  return e;
}

// The accept-bound pairs by v / 2 = n + 8 a of two sites, at LDS address base.
template <int D>
__device__ __forceinline__ void blk_fill_table(uint32_t base, const uint32_t (&bound)[8]) {
  for (uint32_t i = threadIdx.x; i < 225u; i += blockDim.x) {
    constexpr uint32_t z2 = 2u * (uint32_t)D;
    const uint32_t i0 = i % 15u, i1 = i / 15u;
    const uint32_t u0 = (i0 & 7u) > z2 ? 0u : ((i0 & 8u) ? z2 - (i0 & 7u) : (i0 & 7u));
    const uint32_t u1 = (i1 & 7u) > z2 ? 0u : ((i1 & 8u) ? z2 - (i1 & 7u) : (i1 & 7u));
    lds_store64(base + 8u * i, make_uint2(bound[u0], bound[u1]));
  }
}

// What a thread keeps for the whole launch.
struct BlockGeo {
  uint32_t base;        // LDS address of the workgroup's memory
  uint32_t g4;          // LDS byte of the thread's group in a row
  uint32_t gx;          // its group column in the lattice row
  uint32_t rl, rpt;     // first listed row, rows per pass
  uint32_t adjm, adjp;  // byte distance to the dword left / right of the group (periodic in full rows)
  uint32_t sy, sz;      // LDS bytes to the row y + 1 / z + 1
  uint32_t half;        // RAG: L / 2
};

// RAG: bytes of the thread's dword that are sites of the row (0xFF each).
__device__ __forceinline__ uint32_t rag_mask(const BlockGeo& G, uint32_t o2) {
  const int lo = (int)o2 - (int)G.g4, hi = (int)(G.half + o2) - (int)G.g4;  // valid bytes [lo, hi) of 0..3
  uint32_t m = 0xFFFFFFFFu;
  if (lo > 0) m <<= 8 * lo;  // only the first group: lo <= 3
  if (hi < 4) m &= hi > 0 ? 0xFFFFFFFFu >> (8 * (4 - hi)) : 0u;
  return m;
}

// The dword of a neighbour row at the same x as the dword at `at` here: RAG rows begin at another
// byte (shift sh in -3 .. 3), so it is cut from two dwords.
template <bool RAG>
__device__ __forceinline__ uint32_t lds_nb(uint32_t at, int sh) {
  if (!RAG) return lds_load32(at);
  const uint32_t lo = at + (uint32_t)(sh & ~3);  // one dword down where sh < 0
  return __builtin_amdgcn_alignbyte(lds_load32(lo + 4u), lds_load32(lo), (uint32_t)sh & 3u);
}

// An 8-site group as loaded (w[0]; with couplings w[1..D], a word per direction) into the planes.
template <int D, bool EA, bool RAG>
__device__ __forceinline__ void blk_put(const BlockArgs& a, const BlockGeo& G, uint32_t at, uint32_t ex,
                                        const blk_u2 (&w)[EA ? D + 1 : 1]) {
  const uint32_t vm = RAG ? rag_mask(G, row_o2(ex)) : 0xFFFFFFFFu;
  const bool odd = (ex & 1u) != 0;  // colour-0 sites of the row are its odd x
  const uint2 h = blk_split(w[0].x & kNeg, w[0].y & kNeg);
  lds_store32(at, (odd ? h.y : h.x) & vm);
  lds_store32(at + a.plane, (odd ? h.x : h.y) & vm);
  if (EA) {
    uint32_t lo = (w[1].x & kNeg) | (w[EA ? 2 : 0].x & (kNeg << 1)), hi = (w[1].y & kNeg) | (w[EA ? 2 : 0].y & (kNeg << 1));
    if (D == 3) {
      lo |= w[EA ? D : 0].x & (kNeg << 2);
      hi |= w[EA ? D : 0].y & (kNeg << 2);
    }
    const uint2 j = blk_split(lo, hi);
    lds_store32(at + a.jplane, (odd ? j.y : j.x) & vm);
    lds_store32(at + a.jplane + a.plane, (odd ? j.x : j.y) & vm);
  }
}

// A unit: the group of a listed row that a thread updates.
struct BlockUnit {
  uint32_t at;   // LDS address of its dword in plane 0
  uint32_t ex;   // the row's list word (parity and RAG fields)
  uint32_t ctr;  // its Philox counter
  uint32_t ym, yp, zm, zp;  // LDS bytes to the neighbour rows (the same for all units of a tile with halos)
};

__device__ __forceinline__ BlockUnit blk_unit(const BlockGeo& G, uint32_t idx) {
  const uint2 e = lds_load64(G.base + kBlkList + 8u * idx);
  return BlockUnit{G.base + row_at(e.x) + G.g4, e.x, e.y + G.gx, 0u - G.sy, G.sy, 0u - G.sz, G.sz};
}

// A unit's group from the planes to the lattice.
template <bool RAG>
__device__ __forceinline__ void blk_get(const BlockArgs& a, const BlockGeo& G, const BlockUnit& u, int8_t* dst) {
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)dst, 0, (int)a.nbytes, 0x00020000);
  const uint32_t c0 = lds_load32(u.at), c1 = lds_load32(u.at + a.plane);
  const bool odd = (u.ex & 1u) != 0;
  const uint2 w = blk_join(odd ? c1 : c0, odd ? c0 : c1);
  const uint32_t off = 8u * u.ctr;
  const uint32_t vm = RAG ? rag_mask(G, row_o2(u.ex)) : 0xFFFFFFFFu;
  if (vm == 0xFFFFFFFFu) {
    const blk_u2 o = {w.x, w.y};
    __builtin_amdgcn_raw_buffer_store_b64(o, rd, off, 0, 0);
  } else {
    // a group shared with the row before or after: only this row's site pairs
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
      if ((vm >> (8u * i)) & 1u)
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)((i < 2 ? w.x : w.y) >> (16u * (i & 1u))), rd, off + 2u * i, 0, 0);
  }
}

// The colour-c update of a unit in steps, so that a caller can put the draws' rounds of arithmetic
// between the LDS reads and their use.
template <int D, bool EA, bool RAG>
struct BlockStep {
  uint32_t A, I, W, ym, yp, zm, zp;     // own dword, the other colour's, its neighbour, the neighbour rows'
  uint32_t own_j, oth, left, jym, jzm;  // couplings
  uint32_t wrap, jwrap;                 // RAG: the byte at the row's other end
  uint32_t nn, v;
  uint2 b01, b23;

  // LDS reads
  __device__ __forceinline__ void read(const BlockArgs& a, const BlockGeo& G, const BlockUnit& u, uint32_t c) {
    const uint32_t po = c ? 0u : a.plane, pm = c ? a.plane : 0u;  // the other colour's plane, this one's
    const bool P = ((u.ex ^ c) & 1u) != 0;                        // active sites: odd x
    const uint32_t ao = u.at + po, am = u.at + pm;
    I = lds_load32(ao);
    W = lds_load32(ao + (P ? G.adjp : G.adjm));
    ym = lds_nb<RAG>(ao + u.ym, row_shift<0>(u.ex));
    yp = lds_nb<RAG>(ao + u.yp, row_shift<1>(u.ex));
    if (D == 3) {
      zm = lds_nb<RAG>(ao + u.zm, row_shift<2>(u.ex));
      zp = lds_nb<RAG>(ao + u.zp, row_shift<3>(u.ex));
    }
    if (RAG) wrap = lds_load8(ao - G.g4 + row_o2(u.ex) + (P ? 0u : G.half - 1u));
    if (EA) {
      const uint32_t jm = a.jplane + am, jo = a.jplane + ao;
      own_j = lds_load32(jm);
      oth = lds_load32(jo);
      left = lds_load32(jo + G.adjm);
      jym = lds_nb<RAG>(jo + u.ym, row_shift<0>(u.ex));
      if (D == 3) jzm = lds_nb<RAG>(jo + u.zm, row_shift<2>(u.ex));
      if (RAG) jwrap = lds_load8(jo - G.g4 + G.half - 1u + row_o2(u.ex));
    }
    A = lds_load32(am);
  }

  // the neighbour sums, and the reads of the bounds
  __device__ __forceinline__ void sums(const BlockGeo& G, const BlockUnit& u, uint32_t c) {
    const bool P = ((u.ex ^ c) & 1u) != 0;
    // N: the row neighbours on the other side, the other plane moved by a byte
    uint32_t N = __builtin_amdgcn_perm(I, W, P ? 0x00070605u : 0x06050403u);
    uint32_t wmask = 0, wsh = 0;
    if (RAG) {
      // the row's first (P = 0) or last (P = 1) site takes the site at the other end
      const uint32_t b = (P ? G.half - 1u : 0u) + row_o2(u.ex);
      wsh = 8u * (b & 3u);
      wmask = (b & ~3u) == G.g4 ? 0xFFu << wsh : 0u;
      N = (N & ~wmask) | ((wrap << wsh) & wmask);
    }
    if (EA) {
      // coupling bytes: bit 1 the bond to x+1, bit 2 to y+1, bit 3 to z+1.  The bond to I is the
      // site's own when I is to its right (P = 0), else I's; the bond to N the other one
      uint32_t lj = __builtin_amdgcn_perm(oth, left, 0x06050403u);  // of the sites to the left
      if (RAG) lj = (lj & ~wmask) | ((jwrap << wsh) & wmask);       // used where P = 0 only
      const uint32_t jI = P ? oth : own_j, jN = P ? own_j : lj;
      nn = ((I ^ jI) & kNeg) + ((N ^ jN) & kNeg);
      nn += ((yp ^ (own_j >> 1)) & kNeg) + ((ym ^ (jym >> 1)) & kNeg);
      if (D == 3) nn += ((zp ^ (own_j >> 2)) & kNeg) + ((zm ^ (jzm >> 2)) & kNeg);
    } else {
      nn = I + N + ym + yp;
      if (D == 3) nn += zm + zp;
    }
    v = (A << 3) + nn;
    b01 = lds_load64(__builtin_amdgcn_udot4(v, 0x00003C04u, G.base, false));
    b23 = lds_load64(__builtin_amdgcn_udot4(v, 0x3C040000u, G.base, false));
  }

  // the decisions with draws r; MEAS: where own (the tile), adds twice the unsatisfied bonds of the
  // colour-c sites after the update to unsat2 and the negative sites of both colours to neg
  template <bool NEVER, bool MEAS>
  __device__ __forceinline__ void decide(const BlockArgs& a, const BlockGeo& G, const BlockUnit& u, uint32_t c,
                                         uint32_t (&r)[4], bool own, uint32_t& unsat2, uint32_t& neg) {
    if (NEVER) {
      // T = 0 classes hold bound 0 and no class has T = 1 (bound 0 as well), so a draw of 0, the only
      // one those would accept, may count as 1 everywhere
#pragma unroll
      for (int i = 0; i < 4; ++i) r[i] = __builtin_elementwise_max(r[i], 1u);
    }
    uint32_t F = xor3(r[0] <= b01.x ? 0x02u : 0u, r[1] <= b01.y ? 0x0200u : 0u, r[2] <= b23.x ? 0x020000u : 0u) ^
                 (r[3] <= b23.y ? 0x02000000u : 0u);
    uint32_t vm = 0xFFFFFFFFu;
    if (RAG) {
      vm = rag_mask(G, row_o2(u.ex));
      F &= vm;
    }
    const uint32_t An = A ^ F;
    lds_store32(u.at + (c ? a.plane : 0u), An);
    if (MEAS) {
      if (own) {
        constexpr uint32_t kZ = 0x01010101u * (4u * (uint32_t)D);   // 2 * (2D) per byte
        const uint32_t h = An >> 1, full = (h << 8) - h;            // 0xFF where the site is negative
        const uint32_t u2 = (nn ^ ((nn ^ (kZ - nn)) & full)) & vm;  // negative: 2 (2D - n), else 2 n
        unsat2 = __builtin_amdgcn_sad_u8(u2, 0u, unsat2);
        neg += __popc(An & vm) + __popc(I & vm);
      }
    }
  }
};

// One unit.  ORDERED: its LDS reads, half the rounds of its draws, the sums and bound reads, the other
// rounds, the decisions, held in this order, so that the rounds cover both latencies (left to itself
// the compiler puts the reads late and waits for each table entry by itself; 2D L = 64 whole 0.75 ->
// 0.61 us a sweep, L = 1024 in launches of 8 sweeps 1.59 -> 1.48).  Not in the loop over many units,
// where other wavefronts cover them (3D L = 100 2 % slower).
template <int D, bool EA, bool NEVER, bool RAG, bool MEAS, bool ORDERED>
__device__ __forceinline__ void blk_update(const BlockArgs& a, const BlockGeo& G, const BlockUnit& u, uint32_t c,
                                           const PhiloxUniform& U, bool own, uint32_t& unsat2, uint32_t& neg) {
  BlockStep<D, EA, RAG> s;
  uint32_t r[4];
  if (ORDERED) {
    s.read(a, G, u, c);
    __builtin_amdgcn_sched_barrier(0);
    philox_head((uint64_t)kPhiloxM0 * u.ctr, U, a.keys, r);
    philox_rounds<3, 6>(r, a.keys);
    __builtin_amdgcn_sched_barrier(0);
    s.sums(G, u, c);
    __builtin_amdgcn_sched_barrier(0);
    philox_rounds<6, 10>(r, a.keys);
    __builtin_amdgcn_sched_barrier(0);
  } else {
    philox_lane(u.ctr, U, a.keys, r);
    s.read(a, G, u, c);
    s.sums(G, u, c);
  }
  s.template decide<NEVER, MEAS>(a, G, u, c, r, own, unsat2, neg);
}

// One colour phase over the first `count` listed rows.  M > 0: a thread has at most M units, whose
// rows it keeps in registers (they are the same in every phase); M == 0: any number.
template <int D, bool EA, bool NEVER, bool RAG, bool MEAS, int M>
__device__ __forceinline__ void blk_phase(const BlockArgs& a, const BlockGeo& G, const BlockUnit (&un)[M ? M : 1],
                                          uint32_t c, uint32_t count, const PhiloxUniform& U, uint32_t own_rows,
                                          bool own_g, uint32_t& unsat2, uint32_t& neg) {
  if (M) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const uint32_t idx = G.rl + m * G.rpt;
      if (idx < count)
        blk_update<D, EA, NEVER, RAG, MEAS, true>(a, G, un[m], c, U, idx < own_rows && own_g, unsat2, neg);
    }
  } else {
    for (uint32_t idx = G.rl; idx < count; idx += G.rpt)
      blk_update<D, EA, NEVER, RAG, MEAS, false>(a, G, blk_unit(G, idx), c, U, idx < own_rows && own_g, unsat2, neg);
  }
}

template <int D, bool EA, bool NEVER, bool RAG, int M>
__global__ __launch_bounds__(1024) void k_block(const int8_t* __restrict__ src, int8_t* __restrict__ dst,
                                                const int8_t* __restrict__ J, BlockArgs a,
                                                int64_t* __restrict__ part) {
  extern __shared__ __align__(16) char lds[];
  const uint32_t base = lds_addr(lds);
  const uint32_t L = a.L, NT = blockDim.x, tid = threadIdx.x;
  const uint32_t nt = gridDim.x, tile = xcd_tile();
  const uint32_t bx = tile % a.nbx, by = tile / a.nbx;
  const uint32_t H = 2u * a.k;
  uint32_t x0 = 0, y0, z0 = 0, tx = a.TX, ty, tz = 1;
  if (D == 3) {
    y0 = bx * a.TY;
    z0 = by * a.TZ;
    tz = L - z0 < a.TZ ? L - z0 : a.TZ;
  } else {
    x0 = bx * a.TX;
    y0 = by * a.TY;
    if (!RAG) tx = a.GPR - x0 < a.TX ? a.GPR - x0 : a.TX;
  }
  ty = L - y0 < a.TY ? L - y0 : a.TY;
  const uint32_t GW = tx + 2u * a.hx;  // groups of a row in LDS
  const uint32_t Y = ty + 2u * H, Z = D == 3 ? tz + 2u * H : 1u;
  const uint32_t RS = 4u * GW + (RAG ? 8u : 0u);  // RAG: a dword before and after each row
  const uint32_t rows = Y * Z, own_rows = ty * tz;
  blk_fill_table<D>(base, a.bound);
  if (tid < 2u * kBlockMaxK) lds_store32(base + kBlkRec + 4u * tid, 0u);
  if (RAG)  // bytes around the rows are read (and masked later): keep them in the table's range
    for (uint32_t i = 4u * tid; i < a.plane * (EA ? 4u : 2u); i += 4u * NT) lds_store32(base + a.first + i, 0u);
  // the row list (tile_row_rank)
  for (uint32_t lr = tid; lr < rows; lr += NT) {
    const uint32_t y = lr % Y, z = D == 3 ? lr / Y : 0u;
    const uint32_t rank = tile_row_rank<D>(y, z, Y, Z);
    // lattice coordinates (the halo may be wider than the lattice)
    const uint32_t gy = (y0 + y + L * (H / L + 1u) - H) % L;
    const uint32_t gz = D == 3 ? (z0 + z + L * (H / L + 1u) - H) % L : 0u;
    lds_store64(base + kBlkList + 8u * rank, blk_row<D, RAG>(a.first + lr * RS, gy, gz, L, a.GPR));
  }
  keys_resident(a.keys);
  BlockGeo G;
  G.base = base;
  G.rpt = NT / GW;
  const uint32_t g = tid % GW;
  G.rl = tid / GW;
  const bool active = G.rl < G.rpt;
  if (!active) G.rl = 0x7FFFFFFFu;
  G.g4 = 4u * g;
  G.gx = g;
  if (D == 2 && !RAG) {
    uint32_t x = x0 + g + a.GPR * (a.hx / a.GPR + 1u) - a.hx;
    while (x >= a.GPR) x -= a.GPR;
    G.gx = x;
  }
  if (RAG) {
    G.adjm = 0u - 4u;
    G.adjp = 4u;
  } else {
    // periodic neighbours in full rows; at the ends of a halo row any dword will do
    const bool full = D == 3 || a.hx == 0;
    G.adjm = g ? 0u - 4u : (full ? 4u * (GW - 1u) : 0u);
    G.adjp = g + 1u < GW ? 4u : (full ? 0u - 4u * (GW - 1u) : 0u);
  }
  G.sy = RS;
  G.sz = RS * Y;
  G.half = L / 2u;
  const bool own_g = active && g >= a.hx && g < a.hx + tx;
  __syncthreads();
  // load the region: several rows' groups of a thread in flight at a time
  {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, (int)a.nbytes, 0x00020000);
    const uint32_t jbytes = (D - 1) * a.jstride + a.nbytes;
    const __amdgpu_buffer_rsrc_t rj = __builtin_amdgcn_make_buffer_rsrc((void*)J, 0, EA ? (int)jbytes : 0, 0x00020000);
    constexpr int UN = EA ? 2 : 4;
    constexpr int W = EA ? D + 1 : 1;
    for (uint32_t i0 = G.rl; i0 < rows; i0 += UN * G.rpt) {
      uint2 e[UN];
      blk_u2 w[UN][W];
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const uint32_t idx = i0 + u * G.rpt;
        e[u] = lds_load64(base + kBlkList + 8u * (idx < rows ? idx : i0));
        const uint32_t off = 8u * (e[u].y + G.gx);
        w[u][0] = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
#pragma unroll
        for (int dir = 0; dir < W - 1; ++dir)
          w[u][dir + 1] = __builtin_amdgcn_raw_buffer_load_b64(rj, off, dir * a.jstride, 0);
      }
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        if (i0 + u * G.rpt < rows) {
          blk_put<D, EA, RAG>(a, G, G.base + row_at(e[u].x) + G.g4, e[u].x, w[u]);
        }
      }
    }
  }
  __syncthreads();
  BlockUnit un[M ? M : 1];
  if (M) {
    const uint32_t most = tile_rows<D>(Y, Z, 1u);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const uint32_t idx = G.rl + m * G.rpt;
      un[m] = blk_unit(G, idx < most ? idx : 0u);
    }
  }
  uint32_t rec = 0;
  for (uint32_t sweep = 0; sweep < a.k; ++sweep) {
    const uint32_t p = 2u * sweep + 1u;
    const uint32_t n0 = tile_rows<D>(Y, Z, p), n1 = tile_rows<D>(Y, Z, p + 1u);
    uint32_t unsat2 = 0, neg = 0;
    blk_phase<D, EA, NEVER, RAG, false, M>(a, G, un, 0u, n0, philox_uniform(a.t + sweep, a.replica, 0u, a.keys), own_rows,
                                           own_g, unsat2, neg);
    __syncthreads();
    const PhiloxUniform U1 = philox_uniform(a.t + sweep, a.replica, 1u, a.keys);
    if ((a.rec_mask >> sweep) & 1u) {
      blk_phase<D, EA, NEVER, RAG, true, M>(a, G, un, 1u, n1, U1, own_rows, own_g, unsat2, neg);
      const int64_t su = wave_count_dpp(unsat2), sn = wave_count_dpp(neg);
      if ((tid & 63u) == 0) {
        atomicAdd(reinterpret_cast<uint32_t*>(lds + kBlkRec) + 2u * rec, (uint32_t)su);
        atomicAdd(reinterpret_cast<uint32_t*>(lds + kBlkRec) + 2u * rec + 1u, (uint32_t)sn);
      }
      ++rec;
    } else {
      blk_phase<D, EA, NEVER, RAG, false, M>(a, G, un, 1u, n1, U1, own_rows, own_g, unsat2, neg);
    }
    __syncthreads();
  }
  // the tile's rows to dst
  if (own_g)
    for (uint32_t idx = G.rl; idx < own_rows; idx += G.rpt) blk_get<RAG>(a, G, blk_unit(G, idx), dst);
  if (tid < 2u * rec) {
    const uint32_t r = tid >> 1, s = tid & 1u;
    const uint32_t v = lds_load32(base + kBlkRec + 4u * tid);
    part[((uint64_t)r * nt + tile) * 2u + s] = (int64_t)(s ? v : v >> 1);
  }
}

// ---------------------------------------------------------------------------
// n sweeps of a whole small lattice by one workgroup (k_whole), in place: the
// planes of k_block without a halo (neighbour rows wrap), every thread with
// at most M units whose places it keeps in registers, (E, M) written after
// every every-th sweep.  A sweep is two phases of LDS and Philox latency and a
// barrier each, with nothing else a launch would add, so it is the
// fastest form while one compute unit's issue is not the bound: 2D L = 64 0.61 us
// a sweep (k_block 0.87 in launches of 8 sweeps, the pool's nibble kernel 1.09).
template <int D, bool EA, bool NEVER, bool RAG, int M>
__global__ __launch_bounds__(1024) void k_whole(int8_t* __restrict__ spins, const int8_t* __restrict__ J, BlockArgs a,
                                                uint32_t n, uint32_t every, int64_t* __restrict__ E,
                                                int64_t* __restrict__ Mg) {
  extern __shared__ __align__(16) char lds[];
  const uint32_t base = lds_addr(lds), tid = threadIdx.x, L = a.L, GW = a.TX;
  const uint32_t rows = D == 3 ? L * L : L, RS = 4u * GW + (RAG ? 8u : 0u);
  blk_fill_table<D>(base, a.bound);
  if (tid < 4u) lds_store32(base + kBlkRec + 4u * tid, 0u);
  if (RAG)
    for (uint32_t i = 4u * tid; i < a.plane * (EA ? 4u : 2u); i += 4u * blockDim.x) lds_store32(base + a.first + i, 0u);
  keys_resident(a.keys);
  BlockGeo G;
  G.base = base;
  G.rpt = blockDim.x / GW;
  G.rl = tid / GW;
  G.gx = tid - G.rl * GW;
  G.g4 = 4u * G.gx;
  if (G.rl >= G.rpt) G.rl = 0x7FFFFFFFu;
  G.adjm = RAG || G.gx ? 0u - 4u : 4u * (GW - 1u);
  G.adjp = RAG || G.gx + 1u < GW ? 4u : 0u - 4u * (GW - 1u);
  G.sy = RS;
  G.sz = RS * L;
  G.half = L / 2u;
  __syncthreads();
  BlockUnit un[M];
  {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)spins, 0, (int)a.nbytes, 0x00020000);
    const uint32_t jbytes = (D - 1) * a.jstride + a.nbytes;
    const __amdgpu_buffer_rsrc_t rj = __builtin_amdgcn_make_buffer_rsrc((void*)J, 0, EA ? (int)jbytes : 0, 0x00020000);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const uint32_t mine = G.rl + m * G.rpt, row = mine < rows ? mine : 0u;  // no row: any valid place
      const uint32_t z = D == 3 ? row / L : 0u, y = row - z * L;
      const uint2 e = blk_row<D, RAG>(a.first + row * RS, y, z, L, a.GPR);
      un[m] = BlockUnit{base + row_at(e.x) + G.g4,
                        e.x,
                        e.y + G.gx,
                        y ? 0u - G.sy : G.sy * (L - 1u),
                        y + 1u < L ? G.sy : 0u - G.sy * (L - 1u),
                        z ? 0u - G.sz : G.sz * (L - 1u),
                        z + 1u < L ? G.sz : 0u - G.sz * (L - 1u)};
      if (mine < rows) {
        blk_u2 w[EA ? D + 1 : 1];
        w[0] = __builtin_amdgcn_raw_buffer_load_b64(rs, 8u * un[m].ctr, 0, 0);
#pragma unroll
        for (int dir = 0; dir < (EA ? D : 0); ++dir)
          w[EA ? dir + 1 : 0] = __builtin_amdgcn_raw_buffer_load_b64(rj, 8u * un[m].ctr, dir * a.jstride, 0);
        blk_put<D, EA, RAG>(a, G, un[m].at, e.x, w);
      }
    }
  }
  __syncthreads();
  const int64_t N = D == 3 ? (int64_t)L * L * L : (int64_t)L * L;
  uint32_t due = every, rec = 0;
  for (uint32_t i = 0; i < n; ++i) {
    uint32_t unsat2 = 0, neg = 0;
    blk_phase<D, EA, NEVER, RAG, false, M>(a, G, un, 0u, rows, philox_uniform(a.t + i, a.replica, 0u, a.keys), rows, true,
                                           unsat2, neg);
    __syncthreads();
    const PhiloxUniform U1 = philox_uniform(a.t + i, a.replica, 1u, a.keys);
    if (every && --due == 0) {
      due = every;
      blk_phase<D, EA, NEVER, RAG, true, M>(a, G, un, 1u, rows, U1, rows, true, unsat2, neg);
      // both counts in one reduction: of a wavefront's M <= 4 units a lane, 2 u sums to at most
      // 64 * 4 * 48 and the negative sites to 64 * 4 * 8, below 2^16 each
      const uint32_t both = (uint32_t)wave_count_dpp(unsat2 << 16 | neg);
      // two slots in turn: one is added to while thread 0 takes and clears the other
      uint32_t* slot = reinterpret_cast<uint32_t*>(lds + kBlkRec) + 2u * (rec & 1u);
      if ((tid & 63u) == 0) {
        atomicAdd(slot, both >> 16);
        atomicAdd(slot + 1, both & 0xFFFFu);
      }
      __syncthreads();
      if (tid == 0) {
        E[rec] = -(int64_t)D * N + (int64_t)slot[0];
        Mg[rec] = N - 2 * (int64_t)slot[1];
        slot[0] = 0;
        slot[1] = 0;
      }
      ++rec;
    } else {
      blk_phase<D, EA, NEVER, RAG, false, M>(a, G, un, 1u, rows, U1, rows, true, unsat2, neg);
      __syncthreads();
    }
  }
#pragma unroll
  for (int m = 0; m < M; ++m)
    if (G.rl + m * G.rpt < rows) blk_get<RAG>(a, G, un[m], spins);
}

// ------------------------------------------------------------------ host

static bool is_rag(const Lat& lat) { return lat.L % 8 != 0; }

static BlockArgs block_args(const Lat& lat, const BlockPlan& p) {
  BlockArgs a;
  const uint32_t L = lat.L, H = 2u * p.k;
  a.keys = lat.keys;
  a.L = L;
  a.GPR = L / 8u;
  a.k = p.k;
  a.replica = lat.replica;
  const bool rag = is_rag(lat), tiled = lat.d == 2 && !rag && p.TX && p.TX < a.GPR;
  a.hx = tiled ? (H + 7u) / 8u : 0u;
  a.TX = tiled ? p.TX : (rag ? (L + 13u) / 8u : a.GPR);
  a.TY = p.TY;
  a.TZ = lat.d == 3 ? p.TZ : 1u;
  a.nbx = lat.d == 3 ? (L + p.TY - 1u) / p.TY : (tiled ? (a.GPR + p.TX - 1u) / p.TX : 1u);
  const uint32_t GW = a.TX + 2u * a.hx;
  const uint32_t RS = 4u * GW + (rag ? 8u : 0u);
  const uint32_t rows = (a.TY + 2u * H) * (lat.d == 3 ? a.TZ + 2u * H : 1u);
  a.first = (kBlkList + 8u * rows + 15u) & ~15u;
  a.plane = (rows * RS + 15u) & ~15u;
  a.jplane = 2u * a.plane;  // the couplings' planes (three bits a byte) follow the spins'
  a.nbytes = (uint32_t)((lat.N + 7u) & ~(uint64_t)7u);
  a.jstride = (uint32_t)lat.N;
  return a;
}

uint32_t block_tiles(const Lat& lat, const BlockPlan& p) {
  const BlockArgs a = block_args(lat, p);
  const uint32_t nby = lat.d == 3 ? (lat.L + p.TZ - 1u) / p.TZ : (lat.L + p.TY - 1u) / p.TY;
  return a.nbx * nby;
}

size_t block_lds_bytes(const Lat& lat, const BlockPlan& p) {
  const BlockArgs a = block_args(lat, p);
  return (size_t)a.first + (size_t)a.plane * (lat.J ? 4u : 2u);
}

// 32-bit byte offsets, and no class with T = 1 next to one with T = 0 (their bounds coincide).
bool block_lattice_ok(const Lat& lat, const Accept& acc) {
  if (lat.L < 8u) return false;
  const uint64_t bytes = (lat.N + 8u) * (lat.J ? lat.d : 1u);
  if (bytes >= ((uint64_t)1 << 31)) return false;
  if (acc.never_level > 0)
    for (uint32_t u = 0; u <= 2u * lat.d; ++u)
      if (acc.T[2u * lat.d - u] == 1) return false;
  return true;
}

bool block_plan_ok(const Lat& lat, const BlockPlan& p) {
  if (p.k < 1 || p.k > kBlockMaxK || p.TY < 1 || p.TY > lat.L) return false;
  if (lat.d == 3 && (p.TZ < 1 || p.TZ > lat.L)) return false;
  if (p.threads < 64 || p.threads > 1024 || p.threads % 64 != 0) return false;
  const BlockArgs a = block_args(lat, p);
  if (a.TX + 2u * a.hx > p.threads) return false;  // a pass holds at least one row
  // a tiled row's halo may not reach round the lattice onto itself (distinct LDS copies are fine)
  if ((uint64_t)(p.TY + 4u * p.k) * (lat.d == 3 ? p.TZ + 4u * p.k : 1u) > 65536u) return false;
  return block_lds_bytes(lat, p) <= 160u * 1024u;
}

// Estimated microseconds of one launch: a fixed part (launch, loads, stores), the loaded dwords, and
// per phase the larger of the issue time of its wavefronts on a compute unit's SIMDs and the
// latency of a thread's passes.  The constants are a fit to 25 000 timed launches (2D L = 50 .. 4104,
// 3D L = 16 .. 256, both models, every candidate shape below; rms 7 %).  Over those lattices the shape
// it picks takes on average 1.02 times as long as the best one timed, and at most 1.14.
static double block_us(const Lat& lat, const BlockPlan& p) {
  const bool rag = is_rag(lat), ea = lat.J != nullptr;
  const BlockArgs a = block_args(lat, p);
  const uint32_t H = 2u * p.k, GW = a.TX + 2u * a.hx, rpt = p.threads / GW, waves = p.threads / 64u;
  const uint32_t TZ = lat.d == 3 ? a.TZ : 0u;
  const uint64_t tiles = block_tiles(lat, p);
  const uint64_t by_lds = 160u * 1024u / block_lds_bytes(lat, p), by_threads = 2048u / p.threads;
  const uint64_t per_cu = std::min<uint64_t>(8, std::min(by_lds, by_threads)), slots = 256u * per_cu;
  const double issue = (lat.d == 2 ? 0.1071 : 0.1336) * (ea ? 1.13 : 1.0) * (rag ? 1.66 : 1.0);
  auto rows_at = [&](uint32_t m) { return (a.TY + 2u * m) * (lat.d == 3 ? TZ + 2u * m : 1u); };
  const uint32_t most = (rows_at(H - 1u) + rpt - 1u) / rpt;
  const double pass = most <= (rag ? 2u : 4u) ? 0.114 : 0.254;  // units in registers, or listed per pass
  auto round_us = [&](uint64_t n) {
    const double q = (double)((n + 255u) / 256u);  // workgroups a compute unit holds
    double us = 0.000238 * rows_at(H) * GW * q * (ea ? 1.0 + lat.d : 1.0);
    for (uint32_t m = 0; m < H; ++m) {
      const uint32_t rows = rows_at(m), passes = (rows + rpt - 1u) / rpt;
      const uint32_t wu = (passes - 1u) * waves + ((rows - (passes - 1u) * rpt) * GW + 63u) / 64u;
      us += 0.120 + std::max(issue * wu * q / 4.0, pass * passes);
    }
    return us;
  };
  double us = 3.47 + (double)(tiles / slots) * round_us(slots);
  if (tiles % slots) us += round_us(tiles % slots);
  return us;
}

BlockPlan block_plan(const Lat& lat, uint32_t k, double* us) {
  BlockPlan best{0, 0, 0, 0, 0};
  double best_us = 1e30;
  auto consider = [&](const BlockPlan& p) {
    if (!block_plan_ok(lat, p)) return;
    const double t = block_us(lat, p);
    if (t < best_us) {
      best_us = t;
      best = p;
    }
  };
  if (lat.d == 3) {
    const uint32_t side[7] = {2, 4, 6, 8, 12, 16, 20};
    for (uint32_t ty : side)
      for (uint32_t tz : side)
        if ((ty > tz ? ty - tz : tz - ty) <= 8u) consider(BlockPlan{k, 0, ty, tz, 1024});
  } else if (is_rag(lat)) {
    for (uint32_t ty : {1u, 2u, 4u, 6u, 8u, 16u}) consider(BlockPlan{k, 0, ty, 1, 1024});
  } else if (lat.N >= 1u << 24) {
    // several rounds of workgroups a compute unit, where the estimate takes shapes whose registers
    // (89 a lane with up to four units kept there) halve what a compute unit holds: the listed form
    // (31 registers) with this tile was the fastest of the shapes below at L = 4608 .. 15360 for k <= 3 and
    // within 4 % of it for k <= 5.  us a sweep, the estimate's choice and now: L = 5120 k = 1 35.6 -> 24.9, L =
    // 6144 k = 1 49.5 -> 30.8, k = 2 35.5 -> 25.2, k = 4 27.7 -> 23.0
    consider(BlockPlan{k, 32, 64, 1, 512});
  } else {
    for (uint32_t tx : {4u, 8u, 16u, 32u})
      for (uint32_t ty : {4u, 8u, 16u, 32u, 64u})
        for (uint32_t nt : {512u, 768u, 1024u}) consider(BlockPlan{k, tx, ty, 1, nt});
  }
  *us = best_us;
  return best;
}

// Most units of a thread in a phase (all tiles).
static uint32_t block_passes(const Lat& lat, const BlockPlan& p, const BlockArgs& a) {
  const uint32_t H = 2u * p.k, GW = a.TX + 2u * a.hx, rpt = p.threads / GW;
  const uint32_t rows = (a.TY + 2u * H - 2u) * (lat.d == 3 ? a.TZ + 2u * H - 2u : 1u);
  return (rows + rpt - 1u) / rpt;  // narrower last tiles have more rows a pass, shorter ones fewer rows
}

template <int D, bool EA, bool NEVER, bool RAG, int M>
static hipError_t go_block(const int8_t* src, int8_t* dst, const int8_t* J, const BlockArgs& a, uint32_t tiles,
                           uint32_t threads, size_t lds, int64_t* part, hipStream_t stream) {
  static OncePerDevice once;
  const hipError_t e = allow_lds(once, {(const void*)k_block<D, EA, NEVER, RAG, M>}, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_block<D, EA, NEVER, RAG, M>), dim3(tiles), dim3(threads), lds, stream, src, dst, J, a, part);
  return hipGetLastError();
}

template <int D, bool EA, bool NEVER, bool RAG>
static hipError_t go_block_m(uint32_t passes, const int8_t* src, int8_t* dst, const int8_t* J, const BlockArgs& a,
                             uint32_t tiles, uint32_t threads, size_t lds, int64_t* part, hipStream_t stream) {
  if (passes <= 1) return go_block<D, EA, NEVER, RAG, 1>(src, dst, J, a, tiles, threads, lds, part, stream);
  if (passes <= 2) return go_block<D, EA, NEVER, RAG, 2>(src, dst, J, a, tiles, threads, lds, part, stream);
  if (!RAG && passes <= 4) return go_block<D, EA, NEVER, false, RAG ? 0 : 4>(src, dst, J, a, tiles, threads, lds, part, stream);
  return go_block<D, EA, NEVER, RAG, 0>(src, dst, J, a, tiles, threads, lds, part, stream);
}

// k_whole: threads (whole rows of groups) and units a thread has; 0 where the lattice is too large.
static uint32_t whole_passes(const Lat& lat, uint32_t* threads) {
  const uint32_t GW = is_rag(lat) ? (lat.L + 13u) / 8u : lat.L / 8u;
  const uint64_t rows = lat.N / lat.L;
  if (lat.N > 65536 || GW > 1024) return 0;
  const uint64_t units = rows * GW;
  *threads = units <= 256 ? 256u : (units <= 512 ? 512u : 1024u);
  const uint64_t m = (rows + *threads / GW - 1) / (*threads / GW);
  if (m > (is_rag(lat) ? 2u : 4u)) {
    *threads = 1024;
    return 0;
  }
  return (uint32_t)m;
}

static BlockArgs whole_args(const Lat& lat, size_t* lds) {
  BlockArgs a;
  const bool rag = is_rag(lat);
  a.keys = lat.keys;
  a.L = lat.L;
  a.GPR = lat.L / 8u;
  a.k = 1;
  a.replica = lat.replica;
  a.TX = rag ? (lat.L + 13u) / 8u : a.GPR;
  a.TY = a.TZ = a.nbx = a.hx = 0;
  const uint32_t RS = 4u * a.TX + (rag ? 8u : 0u);
  a.first = kBlkList;
  a.plane = ((uint32_t)(lat.N / lat.L) * RS + 15u) & ~15u;
  a.jplane = 2u * a.plane;
  a.rec_mask = 0;
  a.nbytes = (uint32_t)((lat.N + 7u) & ~(uint64_t)7u);
  a.jstride = (uint32_t)lat.N;
  *lds = (size_t)a.first + (size_t)a.plane * (lat.J ? 4u : 2u);
  return a;
}

// Estimated microseconds of n sweeps, by the constants of block_us; < 0: k_whole cannot run it.
double whole_us(const Lat& lat, const Accept& acc, uint32_t n) {
  uint32_t threads = 0;
  size_t lds = 0;
  const uint32_t m = whole_passes(lat, &threads);
  if (m == 0 || !block_lattice_ok(lat, acc)) return -1.0;
  const BlockArgs a = whole_args(lat, &lds);
  if (lds > 160u * 1024u) return -1.0;
  const bool rag = is_rag(lat);
  const double issue = (lat.d == 2 ? 0.1071 : 0.1336) * (lat.J ? 1.13 : 1.0) * (rag ? 1.66 : 1.0);
  const double waves = (double)(lat.N / lat.L) * a.TX / 64.0;
  return 3.47 + n * 2.0 * (0.120 + std::max(issue * waves / 4.0, 0.114 * m));
}

template <int D, bool EA, bool NEVER, bool RAG, int M>
static hipError_t go_whole_m(int8_t* spins, const int8_t* J, const BlockArgs& a, uint32_t threads, size_t lds, uint32_t n,
                             uint32_t every, int64_t* E, int64_t* Mg, hipStream_t stream) {
  static OncePerDevice once;
  const hipError_t e = allow_lds(once, {(const void*)k_whole<D, EA, NEVER, RAG, M>}, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_whole<D, EA, NEVER, RAG, M>), dim3(1), dim3(threads), lds, stream, spins, J, a, n, every, E, Mg);
  return hipGetLastError();
}

template <int D, bool EA, bool NEVER, bool RAG>
static hipError_t go_whole(uint32_t m, int8_t* spins, const int8_t* J, const BlockArgs& a, uint32_t threads, size_t lds,
                           uint32_t n, uint32_t every, int64_t* E, int64_t* Mg, hipStream_t stream) {
  if (m <= 1) return go_whole_m<D, EA, NEVER, RAG, 1>(spins, J, a, threads, lds, n, every, E, Mg, stream);
  if (m <= 2) return go_whole_m<D, EA, NEVER, RAG, 2>(spins, J, a, threads, lds, n, every, E, Mg, stream);
  return go_whole_m<D, EA, NEVER, RAG, RAG ? 2 : 4>(spins, J, a, threads, lds, n, every, E, Mg, stream);
}

// n sweeps t .. t+n-1 in place, (E, M) after every every-th (0: none) into E, M.
hipError_t launch_whole(const Lat& lat, uint32_t t, uint32_t n, const Accept& acc, uint32_t every, int64_t* E, int64_t* Mg,
                        hipStream_t stream) {
  uint32_t threads = 0;
  size_t lds = 0;
  const uint32_t m = whole_passes(lat, &threads);
  if (m == 0 || !block_lattice_ok(lat, acc)) return hipErrorInvalidValue;
  BlockArgs a = whole_args(lat, &lds);
  if (lds > 160u * 1024u) return hipErrorInvalidValue;
  for (int i = 0; i < 8; ++i) a.bound[i] = acc.bound[i];
  a.t = t;
  const bool never = acc.never_level > 0, rag = is_rag(lat), ea = lat.J != nullptr;
  auto go = [&](auto d, auto j, auto v, auto r) {
    return go_whole<decltype(d)::value, decltype(j)::value, decltype(v)::value, decltype(r)::value>(
        m, lat.spins, lat.J, a, threads, lds, n, every, E, Mg, stream);
  };
  using std::false_type;
  using std::true_type;
  auto go_r = [&](auto d, auto j, auto v) { return rag ? go(d, j, v, true_type{}) : go(d, j, v, false_type{}); };
  auto go_v = [&](auto d, auto j) { return never ? go_r(d, j, true_type{}) : go_r(d, j, false_type{}); };
  auto go_j = [&](auto d) { return ea ? go_v(d, true_type{}) : go_v(d, false_type{}); };
  return lat.d == 2 ? go_j(std::integral_constant<int, 2>{}) : go_j(std::integral_constant<int, 3>{});
}

template <int D, bool EA>
static hipError_t go_block_de(uint32_t m, const int8_t* src, int8_t* dst, const int8_t* J, const BlockArgs& a, bool never,
                              bool rag, uint32_t tiles, uint32_t threads, size_t lds, int64_t* part, hipStream_t stream) {
  if (rag)
    return never ? go_block_m<D, EA, true, true>(m, src, dst, J, a, tiles, threads, lds, part, stream)
                 : go_block_m<D, EA, false, true>(m, src, dst, J, a, tiles, threads, lds, part, stream);
  return never ? go_block_m<D, EA, true, false>(m, src, dst, J, a, tiles, threads, lds, part, stream)
               : go_block_m<D, EA, false, false>(m, src, dst, J, a, tiles, threads, lds, part, stream);
}

hipError_t launch_block(const Lat& lat, const int8_t* src, int8_t* dst, uint32_t t, const Accept& acc,
                        const BlockPlan& p, uint32_t rec_mask, int64_t* part, hipStream_t stream) {
  if (!block_lattice_ok(lat, acc) || !block_plan_ok(lat, p)) return hipErrorInvalidValue;
  BlockArgs a = block_args(lat, p);
  for (int i = 0; i < 8; ++i) a.bound[i] = acc.bound[i];
  a.t = t;
  a.rec_mask = rec_mask;
  const uint32_t tiles = block_tiles(lat, p), m = block_passes(lat, p, a);
  const size_t lds = block_lds_bytes(lat, p);
  const bool never = acc.never_level > 0, rag = is_rag(lat), ea = lat.J != nullptr;
  if (lat.d == 2)
    return ea ? go_block_de<2, true>(m, src, dst, lat.J, a, never, rag, tiles, p.threads, lds, part, stream)
              : go_block_de<2, false>(m, src, dst, lat.J, a, never, rag, tiles, p.threads, lds, part, stream);
  return ea ? go_block_de<3, true>(m, src, dst, lat.J, a, never, rag, tiles, p.threads, lds, part, stream)
            : go_block_de<3, false>(m, src, dst, lat.J, a, never, rag, tiles, p.threads, lds, part, stream);
}

}  // namespace spin

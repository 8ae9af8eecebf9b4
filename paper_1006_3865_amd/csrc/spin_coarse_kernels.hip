// spin_coarse_kernels.hip -- the paper's own schedule (Sec. 3, steps 1-7,
// with the generalized multi-hit of the paragraph after them), a mode with
// its own chain: tiles of edge T on a coarse checkerboard; one launch
// updates every tile of one parity, each workgroup one tile: it loads the
// tile and a one-site boundary layer into LDS, updates the tile's colour-0
// sites, then its colour-1 sites, k times, and writes the tile back.  Tiles
// of one parity are never neighbours and the boundary layer belongs to
// tiles of the other parity, which this launch does not write, so the
// update is in place and race-free.
//
// A workgroup holds T^d / 8 units a tile, a unit being an 8-site group, and as many tiles
// as make at least one wavefront (8 of edge 8, 2 of edge 16 in 2D), so that every lane has one unit
// in either colour; with a wavefront to itself an edge-16 tile left half its lanes idle, an edge-8
// one seven eighths.
//
// A launch is as long as its chain: load, then 2 k colour phases of an LDS read, the
// neighbour sums, the decision and an LDS write, then the store; 2D L = 1024 has one or two wavefronts
// a SIMD to hide any of it.  So the draws leave the chain: those of up to 4 hits
// are made while the tile's loads are in flight and kept as thresholds, one byte a site (0x80 -
// 2 u*, u* the smallest count of unsatisfied bonds that accepts), and a phase adds to them twice the
// unsatisfied bonds and flips where bit 7 comes up.  LDS keeps a byte per site, 0x00 (+1) or 0x02
// (-1), in two planes by colour: plane c holds the four colour-c sites of a group as one dword, so the
// active sites and the row and plane neighbours of a phase are dwords as they stand.  For the +-J
// glass two more planes hold the couplings (bit 1 the bond to x+1, bit 2 to y+1, bit 3 to z+1 of
// each site), read once per launch into registers and reused by all k hits.  Hit h of sweep t draws from Philox
// counter (s>>3, t*k + h, replica, colour), as the oracle's coarse mode does.
// Hits after the fourth look their bounds up in 3D, where the three thresholds of a draw cost more than a lookup: 3D L =
// 384, T = 8, 64 hits two sweeps 3007 us with nibble words, 3250 with thresholds, 2440 so (+-J 3280, 3775, 2600).
// us a launch of 4 hits, before (nibble words, bounds looked up in each phase) and now, 2D Ising L = 1024: T = 8
// 11.1 -> 4.7, 16 5.6 -> 4.3, 32 5.8 -> 4.8, 64 6.9 -> 5.2; L = 4096, T = 8 120 -> 26, T = 32, where issue
// bounds it, 21.2 -> 20.1; 3D L = 256, T = 16 25.8 -> 24.4.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spin_internal.h"
#include "spin_device.h"
#include "spin_lds.h"
#include "spin_nibble.h"
#include "spin_packed.h"
#include "spin_tile.h"

namespace spin {

struct CoarseArgs {
  RoundKeys keys;
  uint32_t bound[8];
  uint32_t never;    // never_level
  uint32_t L;
  uint32_t tiles;    // tiles of one parity
  uint32_t t;        // sweep index
  uint32_t k;        // hits per tile load
  uint32_t replica;
  uint32_t q;        // tile parity of this launch
};

constexpr uint32_t kCoarseNeg = 0x02020202u;
constexpr uint32_t kCoarseAhead = 4;  // hits drawn at a time

__device__ __forceinline__ uint32_t wrap_m1(uint32_t v, uint32_t n) {  // (v - 1) mod n for v < 2n
  uint32_t w = v + n - 1u;
  return w >= n ? (w >= 2u * n ? w - 2u * n : w - n) : w;
}

// Thresholds of a unit's four sites: byte i is 0x80 - 2 u*, u* = the classes u < D that draw i does
// not accept (the bounds grow with u, and u >= D always accepts).
template <int D, bool NEVER>
__device__ __forceinline__ uint32_t coarse_draw(const CoarseArgs& a, uint32_t w, uint32_t hit, uint32_t c) {
  const PhiloxUniform U = philox_uniform(hit, a.replica, c, a.keys);
  uint32_t r[4], k = 0;
  philox_lane(w, U, a.keys, r);
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    if (i < 3) k <<= 8;
#pragma unroll
    for (uint32_t u = 0; u < (uint32_t)D; ++u) k += (r[i] > a.bound[u]) | (NEVER && u < a.never) ? 1u : 0u;
  }
  return 0x80808080u - (k << 1);
}

// Tile `first + slot` of the launch's parity (bx + by (+ bz) = q mod 2): word column, row and plane of its first
// site.  first is uniform: the divisions are done once for the workgroup.
template <int D, int T>
__device__ __forceinline__ void coarse_tile(const CoarseArgs& a, uint32_t first, uint32_t slot, uint32_t& x0w,
                                            uint32_t& y0, uint32_t& z0) {
  const uint32_t B = a.L / T, nbx = B / 2u;
  uint32_t bxh = first % nbx + slot, byz = first / nbx;
  if (slot) {  // (always 0 where a tile fills the workgroup)
    const uint32_t last = a.tiles - 1u - first;  // a slot past the last tile repeats that
    if (slot > last) bxh += last - slot;
    while (bxh >= nbx) {
      bxh -= nbx;
      ++byz;
    }
  }
  const uint32_t by = D == 3 ? byz % B : byz, bz = D == 3 ? byz / B : 0u;
  x0w = (2u * bxh + ((by + bz + a.q) & 1u)) * (T / 8u);
  y0 = by * T;
  z0 = bz * T;
}

template <int D, int T, bool EA, bool NEVER>
struct CoarseShape {
  static constexpr uint32_t TW = T / 8;                       // groups per tile row
  static constexpr uint32_t U = (D == 3 ? T : 1) * T * TW;    // units of a tile
  static constexpr uint32_t NT = U < 64 ? 64 : U;             // threads: a unit each
  static constexpr uint32_t TPW = NT / U;                     // tiles of a workgroup
  static constexpr uint32_t RW = TW + 2;                      // groups per LDS row: one more on either side
  static constexpr uint32_t RR = T + 2;                       // rows per LDS plane
  static constexpr uint32_t NG = (D == 3 ? T + 2 : 1) * RR * RW;  // groups of a tile's region
  static constexpr uint32_t PB = 4 * NG;                      // bytes of a colour plane
  static constexpr uint32_t TB = PB * (EA ? 4 : 2);           // bytes of a tile
  // Groups read, NL a thread.  2D: its own and those left and right of the tile's rows; 3D, where a tile's
  // row is one or two groups, whole rows with both (a wavefront's loads of the sides alone touch as many
  // lines again: +-J L = 256, T = 8, k = 1 47.8 us a launch so, 34.7 by rows).  Both: the rows
  // around the tile's.  Edges and corners are not read.
  static constexpr bool OWN = D == 2;
  static constexpr uint32_t CX = OWN ? 2 : RW;                // of a tile's row
  static constexpr uint32_t RX = CX * (D == 3 ? T * T : T);
  static constexpr uint32_t RG = RX + (D == 3 ? 4 * T : 2) * TW;
  static constexpr uint32_t NL = (TPW * RG + NT - 1) / NT;
  // group number e of a tile: LDS plane p, row r and column wi, counted from the boundary
  __device__ static __forceinline__ void place(uint32_t e, uint32_t& p, uint32_t& r, uint32_t& wi) {
    if (e < RX) {
      const uint32_t row = e / CX;
      wi = e - row * CX;
      if (OWN) wi = wi ? TW + 1u : 0u;
      r = row % T + 1u;
      p = D == 3 ? row / T + 1u : 0u;
    } else {
      const uint32_t f = e - RX, row = f / TW, side = D == 3 ? row / T : row, i = row % T + 1u;
      wi = f % TW + 1u;
      const uint32_t out = (side & 1u) ? T + 1u : 0u;
      r = side < 2u ? out : i;
      p = D == 2 ? 0u : (side < 2u ? i : out);
    }
  }
};

// LOOK (3D, more hits than kCoarseAhead): the later hits take their accept bounds from a table, two sites by their u
// (phase_look); drawn under the loads, thresholds are off the chain, after that they are 27 operations a unit where a lookup
// is 12.  A kernel of its own: with the table and its code in every launch, 3D L = 32, T = 8, 1 hit took 3.6 us a
// launch, 3.3 without.
template <int D, int T, bool EA, bool NEVER, bool LOOK>
__global__ __launch_bounds__((CoarseShape<D, T, EA, NEVER>::NT)) void k_coarse(int8_t* __restrict__ spins,
                                                                              const uint32_t* __restrict__ Jraw,
                                                                              CoarseArgs a) {
  using S = CoarseShape<D, T, EA, NEVER>;
  constexpr uint32_t RS = 4 * S::RW, PS = RS * S::RR;  // LDS bytes of a row, of a z plane
  constexpr uint32_t kPairs = LOOK ? 7 * 7 * 8 : 0;
  __shared__ __align__(16) char lds[S::TPW * S::TB + kPairs];
  const uint32_t base = lds_addr(lds), tid = threadIdx.x, pairs = base + S::TPW * S::TB;
  const uint32_t L = a.L, GPR = L / 8;
  const uint32_t first = xcd_tile() * S::TPW;  // neighbouring tiles share the lines of their rows: one L2
  gu32* Jn = as_global(Jraw);
  // this thread's unit: group cw of row ry, plane rz of tile `slot` (a tile past the last one repeats
  // that: loaded, updated, not stored)
  const uint32_t slot = S::TPW > 1 ? tid / S::U : 0u, u = tid - slot * S::U;
  const uint32_t cw = u % S::TW, rows = u / S::TW;
  const uint32_t ry = rows % T, rz = (D == 3) ? rows / T : 0u;
  uint32_t x0w, y0, z0;
  coarse_tile<D, T>(a, first, slot, x0w, y0, z0);
  const uint32_t w = ((z0 + rz) * L + y0 + ry) * GPR + x0w + cw;
  const uint32_t at = base + slot * S::TB + (D == 3 ? (rz + 1u) * PS : 0u) + (ry + 1u) * RS + 4u * (cw + 1u);
  const bool odd = ((ry + rz) & 1u) != 0;  // colour-0 sites of the row are its odd x (tile edges are even)
  if (LOOK && tid < 49u) lds_store64(pairs + 8u * tid, make_uint2(a.bound[tid % 7u], a.bound[tid / 7u]));
  uint2 sp[S::NL + 1];
  uint32_t jw[S::NL + 1];
  auto load = [&](uint32_t n, uint32_t g) {
    sp[n] = reinterpret_cast<const uint2*>(spins)[g];
    if (EA) jw[n] = Jn[g];
  };
  if (S::OWN) load(S::NL, w);
#pragma unroll
  for (uint32_t n = 0; n < S::NL; ++n) {
    const uint32_t i = tid + n * S::NT;
    if (S::TPW * S::RG % S::NT == 0 || i < S::TPW * S::RG) {
      const uint32_t sl = S::TPW > 1 ? i / S::RG : 0u;
      uint32_t p, r, wi, xw, y, z;
      S::place(i - sl * S::RG, p, r, wi);
      coarse_tile<D, T>(a, first, sl, xw, y, z);
      y = wrap_m1(y + r, L);
      xw = wrap_m1(xw + wi, GPR);
      z = (D == 3) ? wrap_m1(z + p, L) : 0u;
      load(n, (z * L + y) * GPR + xw);
    }
  }
  uint32_t th[kCoarseAhead][2];
#pragma unroll
  for (uint32_t j = 0; j < kCoarseAhead; ++j)
    if (j < a.k) {
      th[j][0] = coarse_draw<D, NEVER>(a, w, a.t * a.k + j, 0u);
      th[j][1] = coarse_draw<D, NEVER>(a, w, a.t * a.k + j, 1u);
    }
  __builtin_amdgcn_sched_barrier(0);
  auto put = [&](uint32_t n, uint32_t o, bool po) {
    const uint2 h = split_group(sp[n].x & kCoarseNeg, sp[n].y & kCoarseNeg);
    lds_store32(o, po ? h.y : h.x);
    lds_store32(o + S::PB, po ? h.x : h.y);
    if (EA) {
      // nibble j of a word has site j's couplings: its even and its odd nibbles are the two planes' bytes
      const uint32_t je = jw[n] & (7u * kCoarseNeg), jo = (jw[n] >> 4) & (7u * kCoarseNeg);
      lds_store32(o + 2u * S::PB, po ? jo : je);
      lds_store32(o + 3u * S::PB, po ? je : jo);
    }
  };
  if (S::OWN) put(S::NL, at, odd);
#pragma unroll
  for (uint32_t n = 0; n < S::NL; ++n) {
    const uint32_t i = tid + n * S::NT;
    if (S::TPW * S::RG % S::NT == 0 || i < S::TPW * S::RG) {
      const uint32_t sl = S::TPW > 1 ? i / S::RG : 0u;
      uint32_t p, r, wi;
      S::place(i - sl * S::RG, p, r, wi);
      // rows count from the boundary row, planes from its plane
      put(n, base + sl * S::TB + p * PS + r * RS + 4u * wi, ((r + (D == 3 ? p : 1u)) & 1u) != 0);
    }
  }
  __syncthreads();
  // The couplings of the unit's bonds by colour, one bit (0x02) a site: to I, to N, to the rows y+1 and y-1, the planes
  // z+1 and z-1.  They are the same in all hits: read once (five reads a phase and their masks
  // otherwise: 3D +-J L = 256, T = 16, 100 hits 2035 us for two sweeps, 1631 so).
  uint32_t js[2][EA ? 2 * D : 1];
  if (EA) {
#pragma unroll
    for (uint32_t c = 0; c < 2; ++c) {
      const uint32_t jm = at + (2u + c) * S::PB, jo = at + (3u - c) * S::PB;
      const bool P = odd == (c != 0);
      const uint32_t own = lds_load32(jm), oth = lds_load32(jo), left = lds_load32(jo - 4u), jym = lds_load32(jo - RS);
      const uint32_t lj = __builtin_amdgcn_perm(oth, left, 0x06050403u);  // x bonds of the sites to the left
      js[c][0] = (P ? own : oth) & kCoarseNeg;
      js[c][EA ? 1 : 0] = (P ? lj : own) & kCoarseNeg;
      js[c][EA ? 2 : 0] = (own >> 1) & kCoarseNeg;
      js[c][EA ? 3 : 0] = (jym >> 1) & kCoarseNeg;
      if (D == 3) {
        js[c][EA ? 2 * D - 2 : 0] = (own >> 2) & kCoarseNeg;
        js[c][EA ? 2 * D - 1 : 0] = (lds_load32(jo - PS) >> 2) & kCoarseNeg;
      }
    }
  }
  // t plus twice the unsatisfied bonds, a byte a site, of the colour-c sites A
  auto unsat2 = [&](uint32_t c, uint32_t t, uint32_t& A) {
    const uint32_t am = at + (c ? S::PB : 0u), ao = at + (c ? 0u : S::PB);
    const bool P = odd == (c != 0);  // active sites: even x (row parity and colour the same)
    A = lds_load32(am);
    const uint32_t I = lds_load32(ao), W = lds_load32(P ? ao - 4u : ao + 4u);
    const uint32_t ym = lds_load32(ao - RS), yp = lds_load32(ao + RS);
    const uint32_t zm = D == 3 ? lds_load32(ao - PS) : 0u, zp = D == 3 ? lds_load32(ao + PS) : 0u;
    // the row neighbours on the other side: the other plane moved by a byte
    const uint32_t N = __builtin_amdgcn_perm(I, W, P ? 0x06050403u : 0x00070605u);
    uint32_t X = t;
    if (EA) {
      X += xor3(I, js[c][0], A);
      X += xor3(N, js[c][EA ? 1 : 0], A);
      X += xor3(yp, js[c][EA ? 2 : 0], A);
      X += xor3(ym, js[c][EA ? 3 : 0], A);
      if (D == 3) {
        X += xor3(zp, js[c][EA ? 2 * D - 2 : 0], A);
        X += xor3(zm, js[c][EA ? 2 * D - 1 : 0], A);
      }
    } else {
      X += I ^ A;
      X += N ^ A;
      X += ym ^ A;
      X += yp ^ A;
      if (D == 3) {
        X += zm ^ A;
        X += zp ^ A;
      }
    }
    return X;
  };
  // colour c of a hit with thresholds t
  auto phase = [&](uint32_t c, uint32_t t) {
    uint32_t A;
    const uint32_t X = unsat2(c, t, A);
    lds_store32(at + (c ? S::PB : 0u), A ^ ((X >> 6) & kCoarseNeg));
    __syncthreads();
  };
  // colour c of hit `hit` with its draws' bounds looked up, those of two sites at a time
  auto phase_look = [&](uint32_t c, uint32_t hit) {
    constexpr uint32_t kW = 4u + 256u * 4u * (2u * (uint32_t)D + 1u);  // byte 2u of two sites -> 8 (u0 + (2D + 1) u1)
    uint32_t A, r[4];
    philox_lane(w, philox_uniform(hit, a.replica, c, a.keys), a.keys, r);
    // T = 0 classes hold bound 0 and (LOOK) no class has T = 1: the draw 0, the only one those would accept, may count as 1
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = NEVER ? __builtin_elementwise_max(r[i], 1u) : r[i];
    const uint32_t X = unsat2(c, 0u, A);
    const uint2 b01 = lds_load64(__builtin_amdgcn_udot4(X, kW, pairs, false));
    const uint2 b23 = lds_load64(__builtin_amdgcn_udot4(X, kW << 16, pairs, false));
    const uint32_t F = xor3(r[0] <= b01.x ? 0x02u : 0u, r[1] <= b01.y ? 0x0200u : 0u, r[2] <= b23.x ? 0x020000u : 0u) ^
                       (r[3] <= b23.y ? 0x02000000u : 0u);
    lds_store32(at + (c ? S::PB : 0u), A ^ F);
    __syncthreads();
  };
  for (uint32_t h = 0;;) {
#pragma unroll
    for (uint32_t j = 0; j < kCoarseAhead; ++j)
      if (h + j < a.k) {
        phase(0u, th[j][0]);
        phase(1u, th[j][1]);
      }
    h += kCoarseAhead;
    if (h >= a.k) break;
    if (LOOK) {
      for (; h < a.k; ++h) {
        phase_look(0u, a.t * a.k + h);
        phase_look(1u, a.t * a.k + h);
      }
      break;
    }
#pragma unroll
    for (uint32_t j = 0; j < kCoarseAhead; ++j)
      if (h + j < a.k) {
        th[j][0] = coarse_draw<D, NEVER>(a, w, a.t * a.k + h + j, 0u);
        th[j][1] = coarse_draw<D, NEVER>(a, w, a.t * a.k + h + j, 1u);
      }
  }
  // write the tile back: 0x00 -> 0x01, 0x02 -> 0xFF by v_perm as a table of two bytes
  if (first + slot < a.tiles) {
    const uint32_t c0 = __builtin_amdgcn_perm(0u, 0x00FF0001u, lds_load32(at));
    const uint32_t c1 = __builtin_amdgcn_perm(0u, 0x00FF0001u, lds_load32(at + S::PB));
    reinterpret_cast<uint2*>(spins)[w] = join_group(odd ? make_uint2(c1, c0) : make_uint2(c0, c1));
  }
}

bool coarse_supported(const Lat& lat, int T) {
  if (lat.L % (uint32_t)T != 0 || (lat.L / (uint32_t)T) % 2 != 0) return false;
  if (lat.J != nullptr && (uint64_t)lat.d * lat.N / 8 >= ((uint64_t)1 << 32)) return false;
  if (lat.d == 2) return T == 8 || T == 16 || T == 32 || T == 64;
  return T == 8 || T == 16;
}

template <int D, int T, bool EA, bool NEVER>
static hipError_t run_coarse(const Lat& lat, const uint32_t* Jn, const CoarseArgs& a, bool look, hipStream_t stream) {
  using S = CoarseShape<D, T, EA, NEVER>;
  const dim3 grid((a.tiles + S::TPW - 1) / S::TPW), block(S::NT);
  if (look)
    hipLaunchKernelGGL((k_coarse<D, T, EA, NEVER, D == 3>), grid, block, 0, stream, lat.spins, Jn, a);
  else
    hipLaunchKernelGGL((k_coarse<D, T, EA, NEVER, false>), grid, block, 0, stream, lat.spins, Jn, a);
  return hipGetLastError();
}

template <int D, int T>
static hipError_t go_coarse(const Lat& lat, const uint32_t* Jn, CoarseArgs a, bool never, bool look, hipStream_t stream) {
  const uint32_t B = lat.L / T;
  a.tiles = B / 2 * B * (D == 3 ? B : 1);
  if (lat.J != nullptr)
    return never ? run_coarse<D, T, true, true>(lat, Jn, a, look, stream)
                 : run_coarse<D, T, true, false>(lat, Jn, a, look, stream);
  return never ? run_coarse<D, T, false, true>(lat, Jn, a, look, stream)
               : run_coarse<D, T, false, false>(lat, Jn, a, look, stream);
}

hipError_t launch_coarse_phase(const Lat& lat, const uint32_t* Jn, uint32_t t, uint32_t k, uint32_t q,
                               const Accept& acc, int T, hipStream_t stream) {
  if (!coarse_supported(lat, T) || k < 1) return hipErrorInvalidValue;
  if (lat.J != nullptr && !Jn) return hipErrorInvalidValue;
  CoarseArgs a;
  a.keys = lat.keys;
  for (int i = 0; i < 8; ++i) a.bound[i] = acc.bound[i];
  a.never = acc.never_level;
  a.L = lat.L;
  a.t = t;
  a.k = k;
  a.replica = lat.replica;
  a.q = q;
  const bool never = acc.never_level > 0;
  // not where a class with T = 1 is next to one with T = 0: their bounds coincide
  bool look = lat.d == 3 && k > kCoarseAhead;
  if (never)
    for (uint32_t u = 0; u <= 2u * lat.d; ++u)
      if (acc.T[u] == 1) look = false;
  if (lat.d == 2) {
    if (T == 8) return go_coarse<2, 8>(lat, Jn, a, never, look, stream);
    if (T == 16) return go_coarse<2, 16>(lat, Jn, a, never, look, stream);
    if (T == 32) return go_coarse<2, 32>(lat, Jn, a, never, look, stream);
    return go_coarse<2, 64>(lat, Jn, a, never, look, stream);
  }
  if (T == 8) return go_coarse<3, 8>(lat, Jn, a, never, look, stream);
  return go_coarse<3, 16>(lat, Jn, a, never, look, stream);
}

}  // namespace spin

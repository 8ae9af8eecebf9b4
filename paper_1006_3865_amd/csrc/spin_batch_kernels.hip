// spin_batch_kernels.hip -- many lattices per launch (disorder realisations x
// temperatures, Sec. 4, last paragraph).
//
// A persistent kernel takes tasks (one lattice, n sweeps) from a queue; the
// workgroup holding a task keeps the whole lattice in LDS for all n sweeps and
// writes it back at the end.  In LDS the spins are packed 8 per 32-bit word:
// site 8w+j is nibble j of word w, +1 = 0x1, -1 = 0xF (the low nibble of the
// int8 value), so bits 1..3 of a nibble carry the sign.  (a ^ b) & 0x2 per
// nibble marks an unsatisfied bond (with a coupling nibble in the XOR for the
// +-J glass), the sum over the 2d neighbours is 2u per nibble (u <= 6), and
// a flip XORs the nibble with 0xE.  The Metropolis decision is the same
// bound lookup as in the single-lattice kernels.  The chain is unchanged:
// same Philox counters (group s>>3 = word index), same tables, same order.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "spin_batch.h"
#include "spin_device.h"
#include "spin_launch.h"
#include "spin_lds.h"

namespace spin {

// ---------------------------------------------------------------- couplings

// Generate couplings (Philox rule of spin.h) directly as coupling words.
__global__ void k_couplings_nibble(uint32_t* __restrict__ Jn, uint32_t nwords, uint32_t d,
                                   RoundKeys K, uint32_t realisation) {
  for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < nwords; w += gridDim.x * blockDim.x) {
    uint32_t v = 0;
    for (uint32_t dir = 0; dir < d; ++dir)
#pragma unroll
      for (uint32_t h = 0; h < 2; ++h) {
        uint32_t r[4];
        philox(2 * w + h, dir, realisation, 3u, K, r);
#pragma unroll
        for (int j = 0; j < 4; ++j) v |= (r[j] >> 31) << (4 * (4 * h + j) + 1 + dir);
      }
    Jn[w] = v;
  }
}

// Pack int8 couplings [dir][site] (N sites, a multiple of 8) into coupling words.
__global__ void k_pack_nibbles(const int8_t* __restrict__ src, uint32_t* __restrict__ dst, uint32_t nwords, uint32_t d) {
  for (uint32_t w = blockIdx.x * blockDim.x + threadIdx.x; w < nwords; w += gridDim.x * blockDim.x) {
    uint32_t v = 0;
    for (uint32_t dir = 0; dir < d; ++dir) {
      const uint2 b = reinterpret_cast<const uint2*>(src)[(size_t)dir * nwords + w];
      v |= coupling_bits(b.x, b.y, (int)dir);
    }
    dst[w] = v;
  }
}

hipError_t launch_couplings_nibble(uint32_t* Jn, uint64_t N, uint32_t d, uint64_t cseed,
                                   uint32_t realisation, hipStream_t stream) {
  const uint32_t nwords = (uint32_t)(N / 8);
  const uint32_t blocks = (nwords + 255) / 256 < 4096 ? (nwords + 255) / 256 : 4096;
  hipLaunchKernelGGL(k_couplings_nibble, dim3(blocks ? blocks : 1), dim3(256), 0, stream, Jn, nwords, d,
                     make_round_keys(cseed), realisation);
  return hipGetLastError();
}

hipError_t launch_pack_nibbles(const int8_t* src, uint32_t* dst, uint64_t N, uint32_t d, hipStream_t stream) {
  const uint32_t nwords = (uint32_t)(N / 8);
  const uint32_t blocks = (nwords + 255) / 256 < 4096 ? (nwords + 255) / 256 : 4096;
  hipLaunchKernelGGL(k_pack_nibbles, dim3(blocks ? blocks : 1), dim3(256), 0, stream, src, dst, nwords, d);
  return hipGetLastError();
}

// --------------------------------------------------------- batch kernel

__global__ void k_zero_u32(uint32_t* p, uint32_t n) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// E = -d N + 2 (unsatisfied bonds), M = N - 2 (negative spins) of the LDS
// lattice into Cl.E[rec], Cl.M[rec].
template <int D, bool EA, int NT>
__device__ void batch_record(const BatchLattice& B, const BatchCall& Cl, const uint32_t* sp, int64_t* red,
                             uint32_t rec) {
  const uint32_t L = B.L, LG = L / 8, R = (D == 3) ? L * L : L, NW = R * LG, PS = L * LG;
  int64_t unsat = 0, neg = 0;
  for (uint32_t w = threadIdx.x; w < NW; w += NT) {
    const uint32_t c = sp[w];
    const uint32_t x = w % LG, row = w / LG, y = row % L, z = row / L;
    neg += __popc(c & 0x88888888u);
    const uint32_t rwd = sp[(x + 1 < LG) ? w + 1 : w - (LG - 1)];
    const uint32_t Rx = __builtin_amdgcn_alignbit(rwd, c, 4);
    const uint32_t yp = sp[(y + 1 < L) ? w + LG : w - (L - 1) * LG];
    const uint32_t j = EA ? B.Jn[w] : 0u;
    unsat += __popc(xor3(c, Rx, j) & 0x22222222u);
    unsat += __popc(xor3(c, yp, j) & 0x44444444u);
    if (D == 3) {
      const uint32_t zp = sp[(z + 1 < L) ? w + PS : w - (L - 1) * PS];
      unsat += __popc(xor3(c, zp, j) & 0x88888888u);
    }
  }
  const int64_t su = block_sum<NT>(unsat, red);
  const int64_t sn = block_sum<NT>(neg, red);
  if (threadIdx.x == 0) {
    const int64_t N = (int64_t)NW * 8;
    Cl.E[rec] = -(int64_t)D * N + 2 * su;
    Cl.M[rec] = N - 2 * sn;
  }
}

// Wavefront-uniform copies of a task's parameters.  The descriptors are read
// from global memory by every lane; readfirstlane tells the compiler the
// values are the same in all lanes, so they live in scalar registers and the
// coupling loads below take a scalar base with 32-bit lane offsets.
__device__ __forceinline__ uint32_t uni(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

template <class T>
__device__ __forceinline__ T* uni_ptr(T* p) {
  const uint64_t v = (uint64_t)p;
  return (T*)(((uint64_t)uni((uint32_t)(v >> 32)) << 32) | uni((uint32_t)v));
}

__device__ __forceinline__ BatchLattice uniform_lattice(const BatchLattice& B) {
  BatchLattice u;
  u.spins = uni_ptr(B.spins);
  u.Jn = uni_ptr(B.Jn);
  u.L = uni(B.L);
  u.d = uni(B.d);
  u.replica = uni(B.replica);
  u.t = uni(B.t);
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    u.keys.k0[i] = uni(B.keys.k0[i]);
    u.keys.k1[i] = uni(B.keys.k1[i]);
  }
  return u;
}

__device__ __forceinline__ BatchCall uniform_call(const BatchCall& C) {
  BatchCall u;
  u.n = uni(C.n);
  u.every = uni(C.every);
  u.never4 = uni(C.never4);
#pragma unroll
  for (int i = 0; i < 8; ++i) u.bound[i] = uni(C.bound[i]);
  u.E = uni_ptr(C.E);
  u.M = uni_ptr(C.M);
  return u;
}

// Per-thread geometry of a task: thread -> (column xg of words or pairs of words, first row); rows
// advance by RI per iteration.  Places and distances are in bytes, of the LDS words and of the coupling
// words alike, so that one sum per neighbour addresses both.
struct BatchGeo {
  uint32_t L, LG, R, NB, PB, RI, xg, r_first, dy, dz, wl, wr, ym_wrap;
};

// Flip mask (nib_flips) with the bounds of two sites from one 8-byte entry of the pair table at LDS address
// table: v_dot4 turns two bytes 2u into its offset 8 (u0 + (2D + 1) u1).
template <int D, bool NEVER>
__device__ __forceinline__ uint32_t batch_flips(uint32_t S, uint32_t p, const uint32_t r[4], uint32_t table,
                                                uint32_t nev) {
  constexpr uint32_t W = 4u + 256u * 4u * (2u * D + 1u);
  const uint32_t T = (S >> (4u * p)) & 0x0F0F0F0Fu;  // byte i: 2u of active nibble i
  const uint2 b01 = lds_load64(__builtin_amdgcn_udot4(T, W, table, false));
  const uint2 b23 = lds_load64(__builtin_amdgcn_udot4(T, W << 16, table, false));
  bool a0 = r[0] <= b01.x, a1 = r[1] <= b01.y, a2 = r[2] <= b23.x, a3 = r[3] <= b23.y;
  if (NEVER) {
    a0 = a0 && (T & 0xFFu) >= nev;
    a1 = a1 && __builtin_amdgcn_perm(0u, T, 0x0C0C0C01u) >= nev;
    a2 = a2 && __builtin_amdgcn_ubfe(T, 16u, 8u) >= nev;
    a3 = a3 && (T >> 24) >= nev;
  }
  return (xor3(a0 ? 0xEu : 0u, a1 ? 0xE00u : 0u, a2 ? 0xE0000u : 0u) ^ (a3 ? 0xE000000u : 0u)) << (4u * p);
}

// One colour phase over the thread's rows, a word (PAIR: two adjacent words, rows of an even number of
// words) at a time.  YFIX: RI is a multiple of L, so every row the thread visits has the same y: its
// y-neighbour offsets are fixed, and the parity of the active sites steps by dz per row.
//
// Bound by VALU issue (92 % of the cycles of a busy compute unit): a pair is 172 operations for 8 attempts, 84 of
// them the two draws, 181 with word indices and four single bounds a word.  Lattices L = 16 .. 64, 410 of
// each, 50 sweeps: 6.52 -> 6.19 ms, and 6.16 with round 3 of the draws folded as elsewhere (slower while this
// kernel waited for its coupling loads).
// A pair is one 8-byte LDS access and one 8-byte coupling load per neighbour row; the x neighbours and the x
// bond between its words come from itself.  g describes the columns: wl / wr the distances to the words
// left of the first and right of the last word.
template <int D, bool EA, bool NEVER, bool YFIX, bool PAIR>
__device__ __forceinline__ void batch_colour(uint32_t base, uint32_t table, __amdgpu_buffer_rsrc_t rj, const BatchGeo& g,
                                             const PhiloxUniform& U, const RoundKeys& K, uint32_t colour, uint32_t nev) {
  typedef uint32_t u2v __attribute__((ext_vector_type(2)));
  const uint32_t L = g.L, RB = 4u * g.LG;
  uint32_t y = g.r_first % L, z = g.r_first / L;
  const uint32_t ymo = y ? 0u - RB : g.ym_wrap;               // used when YFIX
  const uint32_t ypo = (y + 1 < L) ? RB : 0u - g.ym_wrap;
  uint32_t p = (colour + y + z) & 1u;
  const uint32_t pstep = g.dz & 1u;
  const uint32_t wstep = g.RI * RB;
  uint32_t w = g.r_first * RB + (PAIR ? 8u : 4u) * g.xg;
  auto get = [&](uint32_t at) {
    return PAIR ? lds_load64(base + at) : make_uint2(lds_load32(base + at), 0u);
  };
  auto bonds = [&](uint32_t at) {
    if (PAIR) {
      const u2v v = __builtin_amdgcn_raw_buffer_load_b64(rj, at, 0, 0);
      return make_uint2(v.x, v.y);
    }
    return make_uint2(__builtin_amdgcn_raw_buffer_load_b32(rj, at, 0, 0), 0u);
  };
  for (uint32_t row = g.r_first; row < g.R; row += g.RI, w += wstep) {
    // keeps the compiler from giving each neighbour's address a register of its own to step (26
    // additions a row where these sums are 9)
    asm("" : "+v"(w));
    const uint2 c = get(w);
    const uint32_t wl = w + g.wl;
    const uint32_t lw = lds_load32(base + wl), rw = lds_load32(base + w + g.wr);
    const uint32_t wym = w + (YFIX ? ymo : (y ? 0u - RB : g.ym_wrap));
    const uint32_t wyp = w + (YFIX ? ypo : ((y + 1 < L) ? RB : 0u - g.ym_wrap));
    uint2 nb[2 * D - 2];
    nb[0] = get(wym);
    nb[1] = get(wyp);
    uint32_t wzm = 0;
    if (D == 3) {
      // planes z-1 and z+1, periodic: w -/+ PB wrapped into [0, NB) by an unsigned minimum (the
      // out-of-range candidate has wrapped past 2^32 or is at least NB), no per-lane select
      const uint32_t m = w - g.PB, q = w + g.PB;
      wzm = __builtin_elementwise_min(m, m + g.NB);
      const uint32_t wzp = __builtin_elementwise_min(q, q - g.NB);
      nb[2 * D - 4] = get(wzm);
      nb[2 * D - 3] = get(wzp);
    }
    uint32_t nb0[2 * D - 2], nb1[2 * D - 2], j0[D + 1], j1[D + 1];
#pragma unroll
    for (int k = 0; k < 2 * D - 2; ++k) {
      nb0[k] = nb[k].x;
      nb1[k] = nb[k].y;
    }
    if (EA) {
      j0[0] = __builtin_amdgcn_raw_buffer_load_b32(rj, wl, 0, 0);
      const uint2 j = bonds(w), jym = bonds(wym);
      j0[1] = j1[0] = j.x;
      j1[1] = j.y;
      j0[2] = jym.x;
      j1[2] = jym.y;
      if (D == 3) {
        const uint2 jzm = bonds(wzm);
        j0[D] = jzm.x;
        j1[D] = jzm.y;
      }
    }
    uint32_t r0[4], r1[4];
    const uint32_t S0 = nib_unsat<D, EA>(c.x, lw, PAIR ? c.y : rw, nb0, j0);
    philox_lane(w >> 2, U, K, r0);
    if (PAIR) {
      const uint32_t S1 = nib_unsat<D, EA>(c.y, c.x, rw, nb1, j1);
      philox_lane((w >> 2) + 1u, U, K, r1);
      lds_store64(base + w, make_uint2(c.x ^ batch_flips<D, NEVER>(S0, p, r0, table, nev),
                                       c.y ^ batch_flips<D, NEVER>(S1, p, r1, table, nev)));
    } else {
      lds_store32(base + w, c.x ^ batch_flips<D, NEVER>(S0, p, r0, table, nev));
    }
    if (YFIX) {
      z += g.dz;
      p ^= pstep;
    } else {
      y += g.dy;
      z += g.dz;
      if (y >= L) {
        y -= L;
        z += 1;
      }
      p = (colour + y + z) & 1u;
    }
  }
}

// n sweeps of lattice B (uniform parameters) in LDS, NEVER: the table has
// classes with T == 0.
template <int D, bool EA, int NT, bool NEVER>
__device__ __forceinline__ void batch_sweeps(const BatchLattice& B, const BatchCall& Cl, uint32_t* sp,
                                             const uint32_t* pair_table, int64_t* red) {
  const uint32_t base = lds_addr(sp), table = lds_addr(pair_table);
  BatchGeo g;
  g.L = B.L;
  g.LG = g.L / 8;                                  // words per row
  g.R = (D == 3) ? g.L * g.L : g.L;                // rows
  g.NB = 4u * g.R * g.LG;
  g.PB = 4u * g.L * g.LG;                          // a plane (3D)
  const uint32_t tid = threadIdx.x;
  g.RI = NT / g.LG;                                // rows per iteration (>= 1: L <= 8192)
  // rows of a fixed y per thread (a multiple of L rows per iteration) when that keeps at least 4/5
  // of the threads busy (L = 48 at 1024 threads: 144 of 170 rows, L = 24 at 256: 72 of 85)
  if (g.RI > g.L && g.RI % g.L != 0 && 5u * (g.RI - g.RI % g.L) >= 4u * g.RI) g.RI -= g.RI % g.L;
  const bool active = tid < g.RI * g.LG;           // active threads
  g.xg = tid % g.LG;
  g.r_first = tid / g.LG;
  g.dz = g.RI / g.L;                               // row step in (y, z)
  g.dy = g.RI % g.L;
  g.wl = g.xg ? 0u - 4u : 4u * (g.LG - 1u);        // to the word on the left
  g.wr = (g.xg + 1 < g.LG) ? 4u : 0u - 4u * (g.LG - 1u);
  g.ym_wrap = 4u * (g.L - 1) * g.LG;
  const bool yfix = g.dy == 0;
  // rows of an even number of words: pairs of words per thread
  const bool pair = (g.LG & 1u) == 0;
  BatchGeo g2 = g;
  if (pair) {
    const uint32_t PG = g.LG / 2;                  // pairs per row
    g2.RI = NT / PG;
    if (g2.RI > g.L && g2.RI % g.L != 0 && 5u * (g2.RI - g2.RI % g.L) >= 4u * g2.RI) g2.RI -= g2.RI % g.L;
    g2.xg = tid % PG;
    g2.r_first = tid / PG;
    g2.dz = g2.RI / g.L;
    g2.dy = g2.RI % g.L;
    g2.wl = g2.xg ? 0u - 4u : 4u * (g.LG - 1u);     // word left of the pair's first word
    g2.wr = (g2.xg + 1 < PG) ? 8u : 8u - 4u * g.LG; // word right of its second word
  }
  const bool active2 = pair && tid < g2.RI * (g.LG / 2);
  const bool yfix2 = g2.dy == 0;
  // couplings by buffer loads: one descriptor over the words, byte offsets per lane
  const __amdgpu_buffer_rsrc_t rj =
      __builtin_amdgcn_make_buffer_rsrc((void*)B.Jn, 0, (int)g.NB, 0x00020000);
  const uint32_t nev = NEVER ? Cl.never4 / 2u : 0u;
  uint32_t rec = 0;
  for (uint32_t i = 0; i < Cl.n; ++i) {
    const uint32_t t = B.t + i;
#pragma unroll 1
    for (uint32_t colour = 0; colour < 2; ++colour) {
      const PhiloxUniform U = philox_uniform(t, B.replica, colour, B.keys);
      if (pair) {
        if (active2) {
          if (yfix2)
            batch_colour<D, EA, NEVER, true, true>(base, table, rj, g2, U, B.keys, colour, nev);
          else
            batch_colour<D, EA, NEVER, false, true>(base, table, rj, g2, U, B.keys, colour, nev);
        }
      } else if (active) {
        if (yfix)
          batch_colour<D, EA, NEVER, true, false>(base, table, rj, g, U, B.keys, colour, nev);
        else
          batch_colour<D, EA, NEVER, false, false>(base, table, rj, g, U, B.keys, colour, nev);
      }
      __syncthreads();
    }
    if (Cl.every && (i + 1) % Cl.every == 0) {
      batch_record<D, EA, NT>(B, Cl, sp, red, rec);
      ++rec;
    }
  }
}

// One task: lattice B, sweeps B.t .. B.t+n-1, all in LDS.  n == 0 with
// every > 0 records the current state once.
template <int D, bool EA, int NT>
__device__ void batch_task(const BatchLattice& Bg, const BatchCall& Cg, uint32_t* sp, uint32_t* bound,
                           int64_t* red) {
  const BatchLattice B = uniform_lattice(Bg);
  const BatchCall Cl = uniform_call(Cg);
  const uint32_t L = B.L;
  const uint32_t R = (D == 3) ? L * L : L;
  const uint32_t NW = R * (L / 8);
  const uint32_t tid = threadIdx.x;
  // pack the lattice into LDS
  for (uint32_t w = tid; w < NW; w += NT) {
    const uint2 b = reinterpret_cast<const uint2*>(B.spins)[w];
    sp[w] = pack_nibbles(b.x, b.y);
  }
  // accept bounds of two sites by their u
  constexpr uint32_t Z1 = 2u * D + 1u;
  if (tid < Z1 * Z1) {
    uint32_t b0 = 0, b1 = 0;
#pragma unroll
    for (uint32_t u = 0; u < Z1; ++u) {  // (no indexed access to the uniform registers)
      b0 = tid % Z1 == u ? Cl.bound[u] : b0;
      b1 = tid / Z1 == u ? Cl.bound[u] : b1;
    }
    bound[2u * tid] = b0;
    bound[2u * tid + 1u] = b1;
  }
  __syncthreads();
  if (Cl.never4)
    batch_sweeps<D, EA, NT, true>(B, Cl, sp, bound, red);
  else
    batch_sweeps<D, EA, NT, false>(B, Cl, sp, bound, red);
  if (Cl.n == 0 && Cl.every) batch_record<D, EA, NT>(B, Cl, sp, red, 0);
  for (uint32_t w = tid; w < NW; w += NT) {
    uint2 b;
    unpack_nibbles(sp[w], b.x, b.y);
    reinterpret_cast<uint2*>(B.spins)[w] = b;
  }
}

static_assert(kBatchRed >= 7 * 7 * 8 && kBatchTask >= kBatchRed + 16 * 8 && kBatchCtl >= kBatchTask + 4, "");

template <int D, bool EA, int NT>
__global__ __launch_bounds__(NT) void k_batch(BatchLattice* lats, const BatchCall* calls,
                                              const uint32_t* order, uint32_t ntasks, uint32_t* next,
                                              uint32_t ctl) {
  // all LDS in one block, the lattice at its start: a word's LDS address is its byte offset, which also
  // addresses its couplings; behind it (at ctl) the pair table, sums and the task index
  extern __shared__ __align__(16) uint32_t lds[];
  uint32_t* sp = lds;
  char* const end = reinterpret_cast<char*>(lds) + ctl;
  uint32_t* bound = reinterpret_cast<uint32_t*>(end);
  int64_t* red = reinterpret_cast<int64_t*>(end + kBatchRed);
  uint32_t& task = *reinterpret_cast<uint32_t*>(end + kBatchTask);
  // Termination: the queue fetch, both barriers, the readfirstlane of the
  // task index and the exit test sit at this one loop level, and no branch
  // at this level depends on per-lane data: the fetch and the counter store
  // are made by all of wave 0 (a wave-uniform condition; lane 0 adds 1, the
  // other lanes 0, and every lane stores lane 0's result), the task body ends
  // with a barrier.  So every wave reads the same k and leaves on the same
  // iteration.  A lane-dependent branch here (thread 0 alone fetching) let
  // the compiler move the fetch into an outer loop and the barriers into a
  // nested one whose exit is per lane, so that lanes re-read a stale index
  // and the loop never ended.
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane = threadIdx.x & 63u;
  for (;;) {
    if (wave == 0) {
      const uint32_t got = atomicAdd(next, lane == 0 ? 1u : 0u);
      task = __builtin_amdgcn_readlane(got, 0);
    }
    __syncthreads();
    const uint32_t k = __builtin_amdgcn_readfirstlane(task);  // uniform: scalar loads below
    __syncthreads();
    if (k >= ntasks) break;
    const uint32_t li = __builtin_amdgcn_readfirstlane(order[k]);
    const BatchCall Cl = calls[li];
    const BatchLattice B = lats[li];
    batch_task<D, EA, NT>(B, Cl, sp, bound, red);
    if (wave == 0) lats[li].t = __builtin_amdgcn_readfirstlane(B.t + Cl.n);
    __syncthreads();
  }
}

size_t batch_lds_bytes(uint32_t L, uint32_t d) {
  const uint64_t N = (d == 3) ? (uint64_t)L * L * L : (uint64_t)L * L;
  return N / 2;
}

template <int NT>
static hipError_t set_batch_attrs() {
  static OncePerDevice once;
  return allow_lds(once, {(const void*)k_batch<2, false, NT>, (const void*)k_batch<2, true, NT>,
                          (const void*)k_batch<3, false, NT>, (const void*)k_batch<3, true, NT>},
                   (int)(kBatchMaxLds + kBatchCtl));
}

template <int NT>
static void go_batch(uint32_t d, bool ea, dim3 grid, size_t lds, hipStream_t stream, BatchLattice* lats,
                     const BatchCall* calls, const uint32_t* order, uint32_t ntasks, uint32_t* counter) {
  if (d == 2 && !ea) hipLaunchKernelGGL((k_batch<2, false, NT>), grid, dim3(NT), lds + kBatchCtl, stream, lats, calls, order, ntasks, counter, (uint32_t)lds);
  if (d == 2 && ea) hipLaunchKernelGGL((k_batch<2, true, NT>), grid, dim3(NT), lds + kBatchCtl, stream, lats, calls, order, ntasks, counter, (uint32_t)lds);
  if (d == 3 && !ea) hipLaunchKernelGGL((k_batch<3, false, NT>), grid, dim3(NT), lds + kBatchCtl, stream, lats, calls, order, ntasks, counter, (uint32_t)lds);
  if (d == 3 && ea) hipLaunchKernelGGL((k_batch<3, true, NT>), grid, dim3(NT), lds + kBatchCtl, stream, lats, calls, order, ntasks, counter, (uint32_t)lds);
}

hipError_t launch_batch(uint32_t d, bool ea, uint32_t nt, BatchLattice* lats, const BatchCall* calls,
                        const uint32_t* order, uint32_t ntasks, uint32_t* counter, size_t lds_bytes,
                        uint32_t grid, hipStream_t stream) {
  hipError_t e = nt == 256    ? set_batch_attrs<256>()
                 : nt == 512  ? set_batch_attrs<512>()
                 : nt == 576  ? set_batch_attrs<576>()
                 : nt == 1024 ? set_batch_attrs<1024>()
                              : hipErrorInvalidValue;
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, stream, counter, 1u);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nt == 256) go_batch<256>(d, ea, dim3(grid), lds_bytes, stream, lats, calls, order, ntasks, counter);
  else if (nt == 512) go_batch<512>(d, ea, dim3(grid), lds_bytes, stream, lats, calls, order, ntasks, counter);
  else if (nt == 576) go_batch<576>(d, ea, dim3(grid), lds_bytes, stream, lats, calls, order, ntasks, counter);
  else go_batch<1024>(d, ea, dim3(grid), lds_bytes, stream, lats, calls, order, ntasks, counter);
  return hipGetLastError();
}

__global__ void k_store_single(BatchSingle* blk, BatchLattice lat, BatchCall call) {
  if (threadIdx.x == 0) {
    blk->lat = lat;
    blk->call = call;
    blk->order = 0;
  }
}

hipError_t launch_batch_single(BatchSingle* blk, const BatchLattice& lat, const BatchCall& call, uint32_t nt,
                               hipStream_t stream) {
  hipLaunchKernelGGL(k_store_single, dim3(1), dim3(64), 0, stream, blk, lat, call);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_batch(lat.d, lat.Jn != nullptr, nt, &blk->lat, &blk->call, &blk->order, 1, &blk->counter,
                      batch_lds_bytes(lat.L, lat.d), 1, stream);
}

}  // namespace spin

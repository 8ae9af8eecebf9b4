// spin_heis_kernels.hip -- the classical Heisenberg ferromagnet (continuous
// spins in single precision), the generalisation the paper points to at the
// close of Sec. 4.  Spins are unit vectors stored as float4 (x, y, z, 0) in
// site order.  One launch per colour: a thread updates one site of that
// colour from its 2d neighbours (all of the other colour, untouched by the
// launch), so the update is in place and race-free.
//   draws of site s: hot start Philox (s, 0, replica, 9), update in sweep t,
//   colour c Philox (s, t, replica, 10 + c); u_i = (w_i >> 8) 2^-24;
//   direction (u0, u1): z = 2 u0 - 1, phi = 2 pi u1, rho = sqrt(fma(-z, z, 1)),
//   (rho cos phi, rho sin phi, z);
//   h = neighbour vectors added in the order -x, +x, -y, +y, -z, +z;
//   dE = S.h - S'.h, a.h = fma(a.x, h.x, fma(a.y, h.y, a.z h.z));
//   accept iff dE <= 0 (the Metropolis rule of Sec. 3, Eq. 2, also at beta =
//   inf) or u2 < exp(-(beta dE)).
// cos, sin and exp are evaluated by one stated method (octant reduction of
// u1 and Taylor polynomials; Cody-Waite reduction by ln 2 and a Taylor
// polynomial, scaled by 2^k), every step a single IEEE float operation with
// fused multiply-adds written out and contraction switched off, so each
// result is a definite float.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spin_device.h"
#include "spin_heis.h"
#include "spin_launch.h"
#include "spin_lds.h"
#include "spin_tile.h"

#pragma clang fp contract(off)

namespace spin {

__device__ __forceinline__ float heis_uniform(uint32_t w) { return (float)(w >> 8) * 0x1p-24f; }

// cos and sin of x in [0, pi/4]: Taylor polynomials to x^10 and x^9, Horner steps in x^2.
__device__ __forceinline__ void heis_cos_sin(float x, float& c, float& sn) {
  const float x2 = x * x;
  float pc = -1.0f / 3628800.0f;
  pc = __builtin_fmaf(pc, x2, 1.0f / 40320.0f);
  pc = __builtin_fmaf(pc, x2, -1.0f / 720.0f);
  pc = __builtin_fmaf(pc, x2, 1.0f / 24.0f);
  pc = __builtin_fmaf(pc, x2, -0.5f);
  c = __builtin_fmaf(pc, x2, 1.0f);
  float ps = 1.0f / 362880.0f;
  ps = __builtin_fmaf(ps, x2, -1.0f / 5040.0f);
  ps = __builtin_fmaf(ps, x2, 1.0f / 120.0f);
  ps = __builtin_fmaf(ps, x2, -1.0f / 6.0f);
  sn = __builtin_fmaf(ps * x2, x, x);
}

// sqrt(v), correctly rounded, for v = 0 or 2^-23 <= v <= 1: the hardware's root is within one unit in
// the last place, and s is the nearest float iff s s' < v <= s s'' for its neighbours s' < s < s'' (Tuckerman's
// test: P. Markstein, IBM J. Res. Dev. 34 (1990) 111), told here by the signs of the exactly rounded residuals
// v - s' s and v - s'' s.  The AMDGPU back end of LLVM expands a correctly rounded root by the same test, with a
// scaling and special cases that this range does not need; at v = 0 both tests fail and the root stays 0.
__device__ __forceinline__ float heis_sqrt(float v) {
  const float s = __builtin_amdgcn_sqrtf(v);
  const float dn = __uint_as_float(__float_as_uint(s) - 1u), up = __uint_as_float(__float_as_uint(s) + 1u);
  const float rd = __builtin_fmaf(-dn, s, v), ru = __builtin_fmaf(-up, s, v);
  const float t = rd <= 0.0f ? dn : s;
  return ru > 0.0f ? up : t;
}

// Direction from (u0, u1): z = 2 u0 - 1; the angle 2 pi u1 reduced to its octant o = floor(8 u1) and
// the offset r = 8 u1 - o (exact), the polynomial taken at r pi/4 (even o) or (1 - r) pi/4 (odd o,
// cos and sin swapped), then rotated by the quadrant o >> 1.  All of it up to the polynomials is
// exact, so it is done on the words: z = (w0 / 2^8 - 2^23) 2^-23, o = w1 >> 29, r or 1 - r = v 2^-21 with
// v of 21 bits (the power of two goes into pi/4); the rotation is a swap and two sign bits.
__device__ __forceinline__ float4 heis_direction(uint32_t w0, uint32_t w1) {
  const float z = (float)((int)(w0 ^ 0x80000000u) >> 8) * 0x1p-23f;
  const float rho = heis_sqrt(__builtin_fmaf(-z, z, 1.0f));
  const uint32_t o = w1 >> 29, v = (w1 >> 8) & 0x1FFFFFu;
  float c, sn;
  heis_cos_sin((float)((o & 1u) ? 0x200000u - v : v) * (0.785398163397448309616f * 0x1p-21f), c, sn);
  // cos and sin change places when exactly one of the octant's and the quadrant's parity is odd
  const bool swap = ((o ^ (o >> 1)) & 1u) != 0;
  const uint32_t a = __float_as_uint(swap ? sn : c), b = __float_as_uint(swap ? c : sn);
  // quadrants 1 and 2: cos negative; 2 and 3: sin negative
  const float cx = __uint_as_float(a ^ (((o << 29) ^ (o << 30)) & 0x80000000u));
  const float sy = __uint_as_float(b ^ ((o << 29) & 0x80000000u));
  return make_float4(rho * cx, rho * sy, z, 0.0f);
}

// u < exp(y): true for y >= 0, false for y <= -87 (exp(y) < 2^-125), else against 2^k e^r with
// k = floor(y log2(e) + 1/2), r = y - k ln 2 (ln 2 split into a high part exact in float and the
// rest) and e^r by its Taylor polynomial to r^7.  Evaluated for every y (k held to the range that
// counts), so that no branch splits the wavefront.
__device__ __forceinline__ bool heis_accept(float u, float y) {
  const float yc = y > -87.0f ? y : -87.0f;
  const float k = __builtin_floorf(__builtin_fmaf(yc, 1.44269504088896340736f, 0.5f));
  float r = __builtin_fmaf(-k, 0.693145751953125f, yc);
  r = __builtin_fmaf(-k, 1.428606765330187045e-06f, r);
  float p = 1.0f / 5040.0f;
  p = __builtin_fmaf(p, r, 1.0f / 720.0f);
  p = __builtin_fmaf(p, r, 1.0f / 120.0f);
  p = __builtin_fmaf(p, r, 1.0f / 24.0f);
  p = __builtin_fmaf(p, r, 1.0f / 6.0f);
  p = __builtin_fmaf(p, r, 0.5f);
  p = __builtin_fmaf(p, r, 1.0f);
  p = __builtin_fmaf(p, r, 1.0f);
  return y >= 0.0f || (y > -87.0f && u < __builtin_ldexpf(p, (int)k));
}

__device__ __forceinline__ float heis_dot(const float4& a, const float4& h) {
  return __builtin_fmaf(a.x, h.x, __builtin_fmaf(a.y, h.y, a.z * h.z));
}

__device__ __forceinline__ void heis_add(float4& h, const float4& v) {
  h.x = h.x + v.x;
  h.y = h.y + v.y;
  h.z = h.z + v.z;
}

__global__ void k_heis_init(float4* __restrict__ S, uint64_t N, RoundKeys K, uint32_t replica) {
  for (uint64_t s = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; s < N; s += (uint64_t)gridDim.x * blockDim.x) {
    uint32_t w[4];
    philox((uint32_t)s, 0u, replica, 9u, K, w);
    S[s] = heis_direction(w[0], w[1]);
  }
}

// The Metropolis decision of one site.
__device__ __forceinline__ bool heis_decide(const float4& cur, const float4& trial, const float4& h, float u, float beta) {
  const float dE = heis_dot(cur, h) - heis_dot(trial, h);
  return (dE <= 0.0f) | heis_accept(u, -(beta * dE));
}

// Order of a colour's workgroups.  XCD x (workgroups are dealt to the eight in turn) takes runs of `chunk`
// consecutive ones, `groups` such runs, so that neighbouring rows and planes come from one L2; the rest
// follow as numbered.  Colour 1 goes through them from the last to the first: it begins where colour 0 ended, with what the
// memory-side cache still holds.
struct HeisOrder {
  uint32_t groups, chunk;
};
__device__ __forceinline__ uint32_t heis_order(const HeisOrder& o, bool reverse) {
  const uint32_t b = blockIdx.x, span = 8u * o.chunk;
  if (b >= o.groups * span) return b;
  uint32_t g = o.groups > 1u ? b / span : 0u, i = (b - g * span) >> 3;
  if (reverse) {
    g = o.groups - 1u - g;
    i = o.chunk - 1u - i;
  }
  return g * span + (b & 7u) * o.chunk + i;
}

// One colour in place, a thread per site of the colour: a workgroup of xw sites (segment `seg`, of nseg, of a
// row's) by rpt rows.  Coordinates come without a division a lane (the 64-bit divisions by L that stood here
// at first were most of the kernel: 2D L = 1024 16 us a colour), and all loads are under way
// before the draws (the site's own vector, left to the compiler, was asked for after the neighbours had come).
template <int D>
__global__ __launch_bounds__(512) void k_heis_phase(float4* __restrict__ S, HeisArgs a, HeisOrder o, uint32_t nrows,
                                                    uint32_t nseg, uint32_t xw, uint32_t rpt) {
  const uint32_t L = a.L, half = L / 2, b = heis_order(o, a.colour != 0);
  uint32_t rb = b, seg = 0;
  if (nseg > 1) {
    rb = b / nseg;
    seg = b - rb * nseg;
  }
  const uint32_t row0 = rb * rpt, row = row0 + threadIdx.y, j = threadIdx.x + xw * seg;
  if (row >= nrows || j >= half) return;
  uint32_t z = D == 3 ? row0 / L : 0u, y = row0 - z * L + threadIdx.y;  // the workgroup's first row, then this one
  if (D == 3)
    while (y >= L) {
      y -= L;
      ++z;
    }
  const uint64_t plane = (uint64_t)L * L;
  const PhiloxUniform U = philox_uniform(a.t, a.replica, 10u + a.colour, a.keys);
  keys_resident(a.keys);
  const uint64_t base = (uint64_t)row * L;
  const uint32_t x = 2 * j + ((a.colour + y + z) & 1u);
  float4* const P = S + base + x;
  float4 n[2 * D];
  n[0] = x ? P[-1] : P[L - 1];
  n[1] = x + 1 < L ? P[1] : P[1 - (int64_t)L];
  n[2] = y ? P[-(int64_t)L] : P[plane - L];
  n[3] = y + 1 < L ? P[L] : P[(int64_t)L - (int64_t)plane];
  if (D == 3) {
    n[2 * D - 2] = z ? P[-(int64_t)plane] : P[plane * (L - 1u)];
    n[2 * D - 1] = z + 1 < L ? P[plane] : P[-(int64_t)(plane * (L - 1u))];
  }
  const float4 cur = *P;
  __builtin_amdgcn_sched_barrier(0);
  uint32_t w[4];
  philox_lane((uint32_t)(base + x), U, a.keys, w);
  const float4 trial = heis_direction(w[0], w[1]);
  __builtin_amdgcn_sched_barrier(0);
  float4 h = n[0];
#pragma unroll
  for (int k = 1; k < 2 * D; ++k) heis_add(h, n[k]);
  if (heis_decide(cur, trial, h, heis_uniform(w[2]), a.beta)) *P = trial;
}

// ---------------------------------------------------------------------------
// k sweeps of a tile per launch (k_heis_block), from src into dst.
//
// With one launch per colour every attempt moves 48 bytes (its own vector read
// and written, and read once more as a neighbour) and every launch waits for
// its first loads.  Here a workgroup loads a tile and a halo of 2k sites on
// every side into LDS (16 bytes a site, a plane per colour, so that lanes read
// consecutive vectors), runs the 2k colour phases there -- phase p
// on the rows at least p away from the edge of the loaded region -- and
// writes the tile: 32 bytes a site and launch, and the halo.  Neighbouring
// tiles recompute the shared halo from the same vectors and draws with the
// same float operations, so all agree bit for bit.  In x all columns are
// computed in every phase; what is wrong at the region's ends moves inwards
// one site a phase and never reaches the tile.  What bounds it is the issue of
// about 165 vector operations an attempt.
struct HeisBlockArgs {
  RoundKeys keys;
  float beta;
  uint32_t L, t, k, replica;
  uint32_t TX, TY, TZ;   // tile (TX even)
  uint32_t nbx, nby;     // tiles along x and y
  uint32_t plane;        // vectors of one colour's plane (all rows)
};

template <int D>
__global__ __launch_bounds__(1024) void k_heis_block(const float4* __restrict__ src, float4* __restrict__ dst,
                                                     HeisBlockArgs a) {
  extern __shared__ __align__(16) char lds[];
  const uint32_t L = a.L, NT = blockDim.x, tid = threadIdx.x, H = 2u * a.k;
  const uint32_t tile = xcd_tile();
  const uint32_t bx = tile % a.nbx, byz = tile / a.nbx, by = byz % a.nby, bz = byz / a.nby;
  const uint32_t x0 = bx * a.TX, y0 = by * a.TY, z0 = bz * a.TZ;
  const uint32_t tx = L - x0 < a.TX ? L - x0 : a.TX, ty = L - y0 < a.TY ? L - y0 : a.TY;
  const uint32_t tz = D == 3 ? (L - z0 < a.TZ ? L - z0 : a.TZ) : 1u;
  const uint32_t W = tx + 2u * H, W2 = W / 2u;                      // sites / columns of a region row
  const uint32_t Y = ty + 2u * H, Z = D == 3 ? tz + 2u * H : 1u;
  const uint32_t rows = Y * Z, own_rows = ty * tz;
  const uint32_t list = lds_addr(lds), first = (list + 8u * rows + 15u) & ~15u;  // row list, planes
  const uint32_t colour = 16u * a.plane;                           // bytes between the colours' planes
  // the rows of the region (tile_row_rank): x = LDS byte offset of column 0 in a plane | parity of y + z, y = first
  // site of the lattice row
  for (uint32_t lr = tid; lr < rows; lr += NT) {
    const uint32_t y = lr % Y, z = D == 3 ? lr / Y : 0u;
    const uint32_t rank = tile_row_rank<D>(y, z, Y, Z);
    const uint32_t gy = (y0 + y + L * (H / L + 1u) - H) % L;
    const uint32_t gz = D == 3 ? (z0 + z + L * (H / L + 1u) - H) % L : 0u;
    lds_store64(list + 8u * rank, make_uint2(16u * lr * W2 | ((gy + gz) & 1u), (gz * L + gy) * L));
  }
  __syncthreads();
  // load: threads over (listed row, site)
  {
    const uint32_t rpt = NT / W, lx = tid % W;
    uint32_t gx = x0 + lx + L * (H / L + 1u) - H;
    gx %= L;
    const uint32_t rl = tid / W;
    if (rl < rpt)
      for (uint32_t i0 = rl; i0 < rows; i0 += 4u * rpt) {
        uint2 e[4];
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t i = i0 + u * rpt;
          e[u] = lds_load64(list + 8u * (i < rows ? i : i0));
          v[u] = src[(uint64_t)e[u].y + gx];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (i0 + u * rpt < rows) {
            lds_store128(first + (e[u].x & ~15u) + 16u * (lx >> 1) + (((e[u].x ^ lx) & 1u) ? colour : 0u), v[u]);
          }
      }
  }
  const uint32_t rpt = NT / W2, j = tid % W2, rl0 = tid / W2, rl = rl0 < rpt ? rl0 : 0x7FFFFFFFu;
  // lattice x of the thread's even site (column j holds local x 2j and 2j + 1; H is even)
  const uint32_t gx0 = (x0 + 2u * j + L * (H / L + 1u) - H) % L;
  const uint32_t sy = 16u * W2, sz = sy * Y;
  const uint32_t left = j ? 16u : 0u, right = j + 1u < W2 ? 16u : 0u;
  __syncthreads();
  for (uint32_t p = 1; p <= H; ++p) {
    const uint32_t c = (p - 1u) & 1u, t = a.t + ((p - 1u) >> 1);
    const uint32_t count = tile_rows<D>(Y, Z, p);
    const PhiloxUniform U = philox_uniform(t, a.replica, 10u + c, a.keys);
    const uint32_t mine = first + (c ? colour : 0u), other = first + (c ? 0u : colour);
    for (uint32_t i = rl; i < count; i += rpt) {
      const uint2 e = lds_load64(list + 8u * i);
      const uint32_t par = (e.x ^ c) & 1u;  // active site: local x = 2 j + par
      const uint32_t at = (e.x & ~15u) + 16u * j, ao = other + at, am = mine + at;
      uint32_t w[4];
      philox_lane(e.y + gx0 + par, U, a.keys, w);
      // neighbours in the stated order; at the region's ends the column itself stands in
      float4 h = lds_load128(par ? ao : ao - left);
      heis_add(h, lds_load128(par ? ao + right : ao));
      heis_add(h, lds_load128(ao - sy));
      heis_add(h, lds_load128(ao + sy));
      if (D == 3) {
        heis_add(h, lds_load128(ao - sz));
        heis_add(h, lds_load128(ao + sz));
      }
      const float4 trial = heis_direction(w[0], w[1]);
      if (heis_decide(lds_load128(am), trial, h, heis_uniform(w[2]), a.beta)) lds_store128(am, trial);
    }
    __syncthreads();
  }
  // the tile's sites to dst: threads over (listed row, site)
  {
    const uint32_t rs = NT / tx, ox = tid % tx, rl1 = tid / tx, lx = ox + H;
    if (rl1 < rs)
      for (uint32_t i = rl1; i < own_rows; i += rs) {
        const uint2 e = lds_load64(list + 8u * i);
        dst[(uint64_t)e.y + x0 + ox] =
            lds_load128(first + (e.x & ~15u) + 16u * (lx >> 1) + (((e.x ^ lx) & 1u) ? colour : 0u));
      }
  }
}

// Per-workgroup sums (E, Mx, My, Mz) in double: E = -sum of the d forward bonds of each site.
template <int D>
__global__ __launch_bounds__(256) void k_heis_measure(const float4* __restrict__ S, uint32_t L, uint64_t N,
                                                      double* __restrict__ part) {
  __shared__ double red[4][256];
  const uint64_t row = L, plane = (uint64_t)L * L;
  double e = 0, mx = 0, my = 0, mz = 0;
  for (uint64_t s = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; s < N; s += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t x = (uint32_t)(s % L), y = (uint32_t)((s / L) % L), z = (D == 3) ? (uint32_t)(s / plane) : 0u;
    const float4 v = S[s];
    mx += v.x;
    my += v.y;
    mz += v.z;
    const float4 bx = S[x + 1 < L ? s + 1 : s + 1 - L];
    const float4 by = S[y + 1 < L ? s + row : s - (L - 1) * row];
    double b = (double)v.x * bx.x + (double)v.y * bx.y + (double)v.z * bx.z;
    b += (double)v.x * by.x + (double)v.y * by.y + (double)v.z * by.z;
    if (D == 3) {
      const float4 bz = S[z + 1 < L ? s + plane : s - (L - 1) * plane];
      b += (double)v.x * bz.x + (double)v.y * bz.y + (double)v.z * bz.z;
    }
    e -= b;
  }
  red[0][threadIdx.x] = e;
  red[1][threadIdx.x] = mx;
  red[2][threadIdx.x] = my;
  red[3][threadIdx.x] = mz;
  __syncthreads();
  for (uint32_t off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off)
      for (int k = 0; k < 4; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[(uint64_t)blockIdx.x * 4 + threadIdx.x] = red[threadIdx.x][0];
}

static unsigned heis_blocks(uint64_t work, unsigned cap) {
  const uint64_t b = (work + 255) / 256;
  return (unsigned)(b < cap ? (b ? b : 1) : cap);
}

uint32_t heis_measure_blocks(uint64_t N) { return heis_blocks(N, 1024); }

hipError_t launch_heis_init(float4* S, uint64_t N, uint64_t seed, uint32_t replica, hipStream_t stream) {
  hipLaunchKernelGGL(k_heis_init, dim3(heis_blocks(N, 8192)), dim3(256), 0, stream, S, N, make_round_keys(seed),
                     replica);
  return hipGetLastError();
}

// Rows are cut into equal segments of at most NT sites of the colour, and as many whole ones as NT threads hold go
// into a workgroup (with one row each the lanes of 128 < L / 2 < 256 were up to half idle).  NT = 512 pays
// from about 48 MiB in 3D, where rows above and below in one workgroup share more loads (us a sweep, 256 threads and
// 512: L = 144 22.8 / 22.9, 160 31.4 / 30.7, 200 62.5 / 59.5, 320 444 / 404); below, and in 2D, the smaller one spreads the
// lattice over more CUs (3D L = 66 6.9 / 7.9, 80 8.3 / 9.2, 128 15.8 / 16.4).  Each
// XCD takes an eighth of the lattice; beyond the 256 MB memory-side cache all eight go through it together, four
// planes each at a time, and the planes that are read again stay cached.  us a sweep 3D, the flat order of one thread a
// site and the kernel before this rule, then now: L = 256 218, 149, 141; 258 389, 244, 194; 300 407, 462, 355;
// 320 489, 556, 463; 400 1072, 1120, 1066; 520 3571, 4040, 2489.
hipError_t launch_heis_phase(float4* S, uint32_t d, const HeisArgs& a, hipStream_t stream) {
  const uint32_t NT = d == 3 && a.N * sizeof(float4) >= (uint64_t)48 << 20 ? 512 : 256;
  const uint32_t half = a.L / 2u, nseg = (half + NT - 1u) / NT, xw = (half + nseg - 1u) / nseg;
  const uint32_t nrows = (uint32_t)(a.N / a.L), rpt = std::min(NT / xw, nrows), blocks = (nrows + rpt - 1u) / rpt * nseg;
  HeisOrder o{1u, blocks / 8u};
  if (d == 3 && a.N * sizeof(float4) > (uint64_t)300 << 20) {
    o.chunk = 4u * a.L / rpt * nseg;
    o.groups = blocks / (8u * o.chunk);
  }
  if (d == 3)
    hipLaunchKernelGGL(k_heis_phase<3>, dim3(blocks), dim3(xw, rpt), 0, stream, S, a, o, nrows, nseg, xw, rpt);
  else
    hipLaunchKernelGGL(k_heis_phase<2>, dim3(blocks), dim3(xw, rpt), 0, stream, S, a, o, nrows, nseg, xw, rpt);
  return hipGetLastError();
}

static uint32_t heis_block_rows(uint32_t d, const HeisPlan& p) {
  return (p.TY + 4u * p.k) * (d == 3 ? p.TZ + 4u * p.k : 1u);
}

size_t heis_block_lds(uint32_t d, const HeisPlan& p) {
  const size_t rows = heis_block_rows(d, p);
  return ((8u * rows + 15u) & ~(size_t)15u) + 32u * rows * ((p.TX + 4u * p.k) / 2u);
}

uint32_t heis_block_tiles(uint32_t L, uint32_t d, const HeisPlan& p) {
  const uint32_t nx = (L + p.TX - 1u) / p.TX, ny = (L + p.TY - 1u) / p.TY;
  return nx * ny * (d == 3 ? (L + p.TZ - 1u) / p.TZ : 1u);
}

// A region row fits the workgroup, the region fits LDS, site indexes fit 32 bits.
bool heis_block_ok(uint32_t L, uint32_t d, uint64_t N, const HeisPlan& p) {
  if (p.k < 1 || p.k > 8 || p.TX < 2 || p.TX % 2 != 0 || p.TX > L || p.TY < 1 || p.TY > L || p.TZ < 1 || p.TZ > L) return false;
  if (p.threads < 64 || p.threads > 1024 || p.threads % 64 != 0 || p.TX + 4u * p.k > p.threads) return false;
  return N <= ((uint64_t)1 << 32) && L >= 4 && heis_block_lds(d, p) <= 160u * 1024u;
}

template <int D>
static hipError_t go_heis_block(const float4* src, float4* dst, const HeisBlockArgs& a, uint32_t tiles, uint32_t threads,
                                size_t lds, hipStream_t stream) {
  static OncePerDevice once;
  const hipError_t e = allow_lds(once, {(const void*)k_heis_block<D>}, 160 * 1024);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_heis_block<D>, dim3(tiles), dim3(threads), lds, stream, src, dst, a);
  return hipGetLastError();
}

hipError_t launch_heis_block(const float4* src, float4* dst, uint32_t d, const HeisArgs& h, const HeisPlan& p,
                             hipStream_t stream) {
  if (!heis_block_ok(h.L, d, h.N, p)) return hipErrorInvalidValue;
  HeisBlockArgs a;
  a.keys = h.keys;
  a.beta = h.beta;
  a.L = h.L;
  a.t = h.t;
  a.k = p.k;
  a.replica = h.replica;
  a.TX = p.TX;
  a.TY = p.TY;
  a.TZ = d == 3 ? p.TZ : 1u;
  a.nbx = (h.L + p.TX - 1u) / p.TX;
  a.nby = (h.L + p.TY - 1u) / p.TY;
  a.plane = heis_block_rows(d, p) * ((p.TX + 4u * p.k) / 2u);
  const uint32_t tiles = heis_block_tiles(h.L, d, p);
  const size_t lds = heis_block_lds(d, p);
  return d == 3 ? go_heis_block<3>(src, dst, a, tiles, p.threads, lds, stream)
                : go_heis_block<2>(src, dst, a, tiles, p.threads, lds, stream);
}

hipError_t launch_heis_measure(const float4* S, uint32_t L, uint32_t d, uint64_t N, double* part, hipStream_t stream) {
  const unsigned blocks = heis_measure_blocks(N);
  if (d == 3)
    hipLaunchKernelGGL(k_heis_measure<3>, dim3(blocks), dim3(256), 0, stream, S, L, N, part);
  else
    hipLaunchKernelGGL(k_heis_measure<2>, dim3(blocks), dim3(256), 0, stream, S, L, N, part);
  return hipGetLastError();
}

}  // namespace spin

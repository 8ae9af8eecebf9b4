// spin_msc_kernels.hip -- multi-spin-coded +-J glass (Sec. 4, last paragraph:
// many disorder realisations at once, combined with multi-spin coding): 32
// systems share the lattice, bit b of every word belongs to system b.
//
// spins: one uint32 per site, bit set = spin -1.  couplings: one uint32 per
// direction and site ([dir][site]), bit set = J -1 for the bond (s, s+e_dir).
// A bond is unsatisfied in system b iff bit b of s_i ^ s_j ^ J is set.  An
// update of site s counts its unsatisfied bonds u (0..2d) in every bit at
// once with a bit-sliced adder (full adders: sum = xor3, carry = majority,
// one v_bitop3 each), then accepts system b iff r < T at k_b = 2d - 2u_b,
// i.e. iff u_b >= u*(r), where u*(r) = #{u < d : r >= T at k = 2d - 2u} is
// one scalar per site (T grows as u grows, and is 2^32 for u >= d).  r is
// the site's shared draw: word
// (s>>1)&3 of Philox counter (s>>3, t, p0, 4 + colour), the chain of the
// oracle's multi-spin-coded mode.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "spin_device.h"
#include "spin_internal.h"
#include "spin_launch.h"
#include "spin_msc.h"
#include "spin_tile.h"

namespace spin {

// A register vector: copies of uint4 structs are lowered to memcpy and left in scratch.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}

// Hot start: bit b of word s is set iff system b's spin is -1, i.e. iff
// bit 31 of word s&3 of Philox(seed, (s>>2, 0, p0 + b, 2)) is clear.
__global__ void k_msc_init(uint32_t* __restrict__ S, uint64_t nquads, RoundKeys K, uint32_t p0) {
  for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < nquads; q += (uint64_t)gridDim.x * blockDim.x) {
    uint32_t w[4] = {0, 0, 0, 0};
    for (uint32_t b = 0; b < 32; ++b) {
      uint32_t r[4];
      philox((uint32_t)q, 0u, p0 + b, 2u, K, r);
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] |= ((r[j] >> 31) ^ 1u) << b;
    }
    reinterpret_cast<uint4*>(S)[q] = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// Device layout of the couplings: J[dir * N + jidx(dir, s)].  The x bonds
// (dir 0) are in site order; the y and z bonds (dir 1, 2) keep each row of L
// words split by x parity, the L/2 even-x words first, then the odd-x ones,
// so that the four same-colour sites of an 8-site group find their y and z
// bonds in 16 contiguous bytes.
__device__ __forceinline__ uint64_t msc_split(uint64_t s, uint32_t L) {
  const uint32_t x = (uint32_t)(s % L);
  return s - x + (x & 1u) * (L / 2) + (x >> 1);
}

// Couplings: bit b of the word of bond (dir, s) is set iff bit 31 of word
// s&3 of Philox(cseed, (s>>2, dir, r0 + b, 3)) is set (J = -1).
__global__ void k_msc_couplings(uint32_t* __restrict__ J, uint64_t nquads, uint32_t L, uint32_t d, RoundKeys K,
                                uint32_t r0) {
  const uint64_t N = nquads * 4;
  for (uint32_t dir = 0; dir < d; ++dir)
    for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < nquads;
         q += (uint64_t)gridDim.x * blockDim.x) {
      uint32_t w[4] = {0, 0, 0, 0};
      for (uint32_t b = 0; b < 32; ++b) {
        uint32_t r[4];
        philox((uint32_t)q, dir, r0 + b, 3u, K, r);
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] |= (r[j] >> 31) << b;
      }
      if (dir == 0) {
        reinterpret_cast<uint4*>(J)[q] = make_uint4(w[0], w[1], w[2], w[3]);
      } else {  // sites 4q .. 4q+3 start at an even x of one row (L % 8 == 0)
        const uint64_t e = (uint64_t)dir * N + msc_split(4 * q, L);
        reinterpret_cast<uint2*>(J + e)[0] = make_uint2(w[0], w[2]);
        reinterpret_cast<uint2*>(J + e + L / 2)[0] = make_uint2(w[1], w[3]);
      }
    }
}

__device__ __forceinline__ void load4(const uint32_t* p, uint32_t (&v)[4]) {
  const uint4 a = reinterpret_cast<const uint4*>(p)[0];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
}

__device__ __forceinline__ void load8(const uint32_t* p, uint32_t (&v)[8]) {
  const uint4 a = reinterpret_cast<const uint4*>(p)[0];
  const uint4 b = reinterpret_cast<const uint4*>(p)[1];
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Flips of a site's 32 systems: those whose unsatisfied count u (bit-sliced u2
// u1 u0) is at least u*(r).  The thresholds grow with u, so r reaches them in
// order and each one reached replaces the mask by the next narrower one: a
// compare and a select each (counting u* first and comparing it cost three more
// operations a threshold).  A threshold of 2^32 is reached by no r.
// SPLIT: that is asked once, of the high word, and the low words are compared.  The phase kernel takes it
// (2D L = 2048 24.8 us a sweep, 26.9 with 64-bit compares); in the marching ones the scalar masks that it
// keeps do not fit the registers next to the rest (2D L = 2944 43.6 us, 40.5 with 64-bit compares; 3D L = 400 457 and 447).
template <int D, bool SPLIT>
__device__ __forceinline__ uint32_t msc_flips(uint32_t u0, uint32_t u1, uint32_t u2, uint32_t r,
                                              const uint64_t (&thr)[3]) {
  auto reached = [&](int k) {
    return SPLIT ? (r >= (uint32_t)thr[k]) & ((uint32_t)(thr[k] >> 32) == 0u) : r >= thr[k];
  };
  uint32_t m = 0xFFFFFFFFu;
  m = reached(0) ? (u0 | u1 | u2) : m;
  m = reached(1) ? (u1 | u2) : m;
  if (D == 3) m = reached(2) ? (u2 | (u1 & u0)) : m;
  return m;
}

// The four colour-P sites of an 8-site group (words c[]; neighbours: lw, rw
// the sites left and right of the group, ym/yp rows y-1/y+1 and zm/zp planes
// z-1/z+1 at the same x); jb[i]: the couplings of active site i = 0..3
// (site 2i + P) in the order -x, +x, -y, +y (, -z, +z); r: the shared draws.
template <int D, int P>
__device__ __forceinline__ void msc_update8(uint32_t (&c)[8], uint32_t lw, uint32_t rw, const uint32_t (&ym)[8],
                                            const uint32_t (&yp)[8], const uint32_t (&zm)[8], const uint32_t (&zp)[8],
                                            const uint32_t (&jb)[4][2 * D], const uint32_t (&r)[4],
                                            const MscArgs& a) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = 2 * i + P;
    const uint32_t left = j ? c[j - 1] : lw;
    const uint32_t right = j < 7 ? c[j + 1] : rw;
    const uint32_t s = c[j];
    // unsatisfied bits of the 2d bonds
    const uint32_t b0 = xor3(s, left, jb[i][0]), b1 = xor3(s, right, jb[i][1]);
    const uint32_t b2 = xor3(s, ym[j], jb[i][2]), b3 = xor3(s, yp[j], jb[i][3]);
    uint32_t u0, u1, u2;
    if (D == 3) {
      const uint32_t b4 = xor3(s, zm[j], jb[i][4]), b5 = xor3(s, zp[j], jb[i][5]);
      const uint32_t s1 = xor3(b0, b1, b2), c1 = maj3(b0, b1, b2);
      const uint32_t s2 = xor3(b3, b4, b5), c2 = maj3(b3, b4, b5);
      u0 = s1 ^ s2;
      const uint32_t t = s1 & s2;
      u1 = xor3(c1, c2, t);
      u2 = maj3(c1, c2, t);
    } else {
      const uint32_t s1 = xor3(b0, b1, b2), c1 = maj3(b0, b1, b2);
      u0 = s1 ^ b3;
      const uint32_t t = s1 & b3;
      // u1 | u2 in one word, as only their or is asked for (in two, the compiler keeps both: 32 vector operations
      // more a plane step)
      u1 = c1 | t;
      u2 = 0u;
    }
    c[j] = s ^ msc_flips<D, false>(u0, u1, u2, r[i], a.thr);
  }
}

// The couplings of the four active sites of a group in the order of
// msc_update8: x bonds from the group's x-bond words jx (jl: the word left of
// the group), y and z bonds from the parity-P halves jy/jym (rows y, y-1) and
// jz/jzm (planes z, z-1), word i for site 2i + P.
template <int D, int P>
__device__ __forceinline__ void bonds_split(const uint32_t (&jx)[8], uint32_t jl, const uint32_t (&jy)[4],
                                            const uint32_t (&jym)[4], const uint32_t (&jz)[4],
                                            const uint32_t (&jzm)[4], uint32_t (&jb)[4][2 * D]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = 2 * i + P;
    jb[i][0] = j ? jx[j - 1] : jl;
    jb[i][1] = jx[j];
    jb[i][2] = jym[i];
    jb[i][3] = jy[i];
    if (D == 3) {
      jb[i][4] = jzm[i];
      jb[i][5] = jz[i];
    }
  }
}

// The four active sites A of a group after their update: o the other colour's sites of the group, of which
// each is a neighbour on one side, and N the neighbours on the other; ym, yp, zm, zp those in the
// neighbouring rows and planes; jo, jn, jym, jy, jzm, jz the bonds to them; r the shared draws.
template <int D>
__device__ __forceinline__ u32x4 msc_update4(u32x4 A, u32x4 o, u32x4 N, u32x4 ym, u32x4 yp, u32x4 zm, u32x4 zp, u32x4 jo,
                                             u32x4 jn, u32x4 jym, u32x4 jy, u32x4 jzm, u32x4 jz, const uint32_t (&r)[4],
                                             const uint64_t (&thr)[3]) {
  u32x4 out;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t s = A[i];
    const uint32_t b0 = xor3(s, o[i], jo[i]), b1 = xor3(s, N[i], jn[i]);
    const uint32_t b2 = xor3(s, ym[i], jym[i]), b3 = xor3(s, yp[i], jy[i]);
    const uint32_t s1 = xor3(b0, b1, b2), c1 = maj3(b0, b1, b2);
    uint32_t u0, u1, u2;
    if (D == 3) {
      const uint32_t b4 = xor3(s, zm[i], jzm[i]), b5 = xor3(s, zp[i], jz[i]);
      const uint32_t s2 = xor3(b3, b4, b5), c2 = maj3(b3, b4, b5);
      u0 = s1 ^ s2;
      const uint32_t t = s1 & s2;
      u1 = xor3(c1, c2, t);
      u2 = maj3(c1, c2, t);
    } else {
      u0 = s1 ^ b3;
      const uint32_t t = s1 & b3;
      u1 = c1 | t;  // u1 | u2, as in msc_update8
      u2 = 0u;
    }
    out[i] = s ^ msc_flips<D, true>(u0, u1, u2, r[i], thr);
  }
  return out;
}

__device__ __forceinline__ u32x4 sel4(bool c, u32x4 x, u32x4 y) {
  return u32x4{c ? x.x : y.x, c ? x.y : y.y, c ? x.z : y.z, c ? x.w : y.w};
}

// One colour phase, in place: thread = 8-site group, its four sites of colour c (offset P = (c + y +
// z) & 1 inside the group).  Bound by its own latency (one round of loads) while the lattice is small, by
// memory above: the row and plane neighbours come from cache, so a phase reads the spins and the
// couplings once and writes the spins.  Consecutive workgroups of an XCD take consecutive groups, whose
// neighbour rows are then in its L2.  P differs between the rows of a wavefront: halves are selected, the
// arithmetic is not branched over.  us a sweep (two phases), with a copy of the couplings by colour, twice
// their size, and a branch on P before: 2D L = 64 8.6 -> 7.3, 1024 16.0 -> 9.1, 2048 54 -> 25; 3D L = 64 13.2 ->
// 8.1, 160 61 -> 32, 256 251 -> 100.
template <int D>
__global__ __launch_bounds__(256) void k_msc_phase(uint32_t* __restrict__ S, const uint32_t* __restrict__ J,
                                                   MscArgs a) {
  const uint32_t L = a.L, GPR = L / 8;
  const PhiloxUniform U = philox_uniform(a.t, a.p0, 4u + a.colour, a.keys);
  const uint64_t row = L, plane = (uint64_t)L * L, N = a.N;
  for (uint64_t g = xcd_tile() * (uint64_t)256 + threadIdx.x; g < N / 8; g += (uint64_t)gridDim.x * 256) {
    const uint32_t rowi = (uint32_t)g / GPR, gx = (uint32_t)g - rowi * GPR;  // N / 8 < 2^32
    const uint32_t z = D == 3 ? rowi / L : 0u, y = rowi - z * L;
    const uint64_t r0 = (uint64_t)rowi * L, s0 = r0 + 8u * gx;
    const uint64_t dym = y ? 0 - row : (L - 1) * row, dyp = y + 1 < L ? row : 0 - (L - 1) * row;
    const uint64_t dzm = z ? 0 - plane : (L - 1) * plane, dzp = z + 1 < L ? plane : 0 - (L - 1) * plane;
    const bool P = ((a.colour + y + z) & 1u) != 0;
    const uint64_t sl = gx ? s0 - 1 : r0 + L - 1, sr = gx + 1 < GPR ? s0 + 8 : r0;  // left and right of the group
    auto ld = [&](const uint32_t* p) { return *reinterpret_cast<const u32x4*>(p); };
    const u32x4 c0 = ld(S + s0), c1 = ld(S + s0 + 4), m0 = ld(S + s0 + dym), m1 = ld(S + s0 + dym + 4),
                p0 = ld(S + s0 + dyp), p1 = ld(S + s0 + dyp + 4);
    const uint32_t w = S[P ? sr : sl];
    u32x4 q0{}, q1{}, t0{}, t1{};
    if (D == 3) {
      q0 = ld(S + s0 + dzm);
      q1 = ld(S + s0 + dzm + 4);
      t0 = ld(S + s0 + dzp);
      t1 = ld(S + s0 + dzp + 4);
    }
    const u32x4 x0 = ld(J + s0), x1 = ld(J + s0 + 4);
    const uint32_t xl = J[sl];
    const uint64_t h = N + r0 + (P ? L / 2 : 0) + 4u * gx;  // the active sites' y bonds
    const u32x4 jy = ld(J + h), jym = ld(J + h + dym);
    u32x4 jz{}, jzm{};
    if (D == 3) {
      jz = ld(J + N + h);
      jzm = ld(J + N + h + dzm);
    }
    uint32_t r[4];
    philox_lane((uint32_t)g, U, a.keys, r);
    auto even = [](u32x4 v0, u32x4 v1) { return u32x4{v0.x, v0.z, v1.x, v1.z}; };
    auto oddw = [](u32x4 v0, u32x4 v1) { return u32x4{v0.y, v0.w, v1.y, v1.w}; };
    auto half = [&](u32x4 v0, u32x4 v1) { return sel4(P, oddw(v0, v1), even(v0, v1)); };
    const u32x4 ev = even(c0, c1), od = oddw(c0, c1), jo = oddw(x0, x1);
    // the bond to the other site of a pair is the even site's either way; the one on the other side its
    // own (P = 1) or that of the site to its left
    const u32x4 Nb = sel4(P, u32x4{ev.y, ev.z, ev.w, w}, u32x4{w, od.x, od.y, od.z});
    const u32x4 jn = sel4(P, jo, u32x4{xl, jo.x, jo.y, jo.z});
    const u32x4 n = msc_update4<D>(sel4(P, od, ev), sel4(P, ev, od), Nb, half(m0, m1), half(p0, p1), half(q0, q1),
                                   half(t0, t1), even(x0, x1), jn, jym, jy, jzm, jz, r, a.thr);
    const u32x4 e1 = sel4(P, ev, n), o1 = sel4(P, n, od);
    *reinterpret_cast<u32x4*>(S + s0) = u32x4{e1.x, o1.x, e1.y, o1.y};
    *reinterpret_cast<u32x4*>(S + s0 + 4) = u32x4{e1.z, o1.z, e1.w, o1.w};
  }
}

// ------------------------------------------------------------ streaming
// One whole sweep per launch, streamed over planes (z in 3D, rows in 2D)
// like the general streaming kernel: a workgroup owns planes [z0, z0+H), in
// 3D rows [y0, y0+TY), and sites [x0, x0+XW) of each row, and keeps a ring
// of 6 plane slices of site words in LDS.  A slice row holds the 8-site
// groups x0/8-2 .. x0/8+XW/8+1 (two neighbouring groups on each side,
// periodic); 3D slices hold rows y0-2 .. y0+TY+1.  A slice row keeps words
// 0-3 of its groups in its first half and words 4-7 in its second, so that
// neighbouring lanes touch neighbouring 16 bytes.  Step i, plane a =
// z0-1+i: fetch plane a+2 into registers; colour 0 on plane a over slice
// rows 1..TY+2 and groups 1..XW/8+2 (the owned part and a one-group /
// one-row ring that colour 1 needs), written back into the ring; colour 1
// on plane a-2 over the owned rows and groups, written to dst with both
// colours; store the fetched plane; barrier.  Couplings come from HBM.
constexpr int kMscFetch = 4;  // slice groups per thread
__device__ __forceinline__ uint32_t msc_wrap2(uint32_t v, uint32_t L) {  // (v - 2) mod L, v < 2L + 2
  uint32_t w = v + L - 2u;
  if (w >= L) w -= L;
  if (w >= L) w -= L;
  return w;
}

struct MscGeom {
  uint32_t L, GPR;   // edge, groups per row
  uint32_t SG;       // groups per slice row (XW/8 + 4)
  uint32_t RW;       // words per slice row (8 * SG)
  uint32_t HW;       // offset of the second half of a slice row (4 * SG)
  uint32_t gx0;      // first owned group column (x0 / 8)
};

template <int D, int NT>
__device__ __forceinline__ void msc_fetch(const uint32_t* __restrict__ src, uint32_t z, uint32_t y0, const MscGeom& G,
                                          uint32_t tot, u32x4 (&v)[2 * kMscFetch]) {
#pragma unroll
  for (int q = 0; q < kMscFetch; ++q) {
    const uint32_t u = threadIdx.x + NT * q;
    if (u < tot) {
      const uint32_t r = u / G.SG, k = u - r * G.SG;
      const uint32_t y = (D == 3) ? msc_wrap2(y0 + r, G.L) : 0u;
      const uint32_t gx = msc_wrap2(G.gx0 + k, G.GPR);
      const uint64_t s0 = ((D == 3) ? ((uint64_t)z * G.L + y) * G.L : (uint64_t)z * G.L) + 8u * gx;
      v[2 * q] = reinterpret_cast<const u32x4*>(src + s0)[0];
      v[2 * q + 1] = reinterpret_cast<const u32x4*>(src + s0)[1];
    }
  }
}

template <int NT>
__device__ __forceinline__ void msc_put(uint32_t* slot, const MscGeom& G, uint32_t tot,
                                        const u32x4 (&v)[2 * kMscFetch]) {
#pragma unroll
  for (int q = 0; q < kMscFetch; ++q) {
    const uint32_t u = threadIdx.x + NT * q;
    if (u < tot) {
      const uint32_t r = u / G.SG, k = u - r * G.SG;
      uint32_t* p = slot + r * G.RW + 4 * k;
      *reinterpret_cast<u32x4*>(p) = v[2 * q];
      *reinterpret_cast<u32x4*>(p + G.HW) = v[2 * q + 1];
    }
  }
}

// The 8 words of a slice group: words 0-3 at p, words 4-7 at p + hw.
__device__ __forceinline__ void lds8(const uint32_t* p, uint32_t hw, uint32_t (&v)[8]) {
  const u32x4 a = *reinterpret_cast<const u32x4*>(p);
  const u32x4 b = *reinterpret_cast<const u32x4*>(p + hw);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// Colour-C groups of one step: slice rows RB0 + u / NG, slice groups KB0 + u % NG.
template <int D, int NT, uint32_t C>
__device__ __forceinline__ void msc_units(const uint32_t* pm, uint32_t* pc, const uint32_t* pp, uint32_t n,
                                          uint32_t NG, uint32_t y0, uint32_t z, const MscGeom& G, const MscArgs& a,
                                          const PhiloxUniform& U, const uint32_t* __restrict__ J,
                                          uint32_t* __restrict__ dst) {
  const uint32_t L = G.L, RW = G.RW, HW = G.HW;
  constexpr uint32_t RB0 = (D == 3) ? (C == 0 ? 1u : 2u) : 0u;
  constexpr uint32_t KB0 = C == 0 ? 1u : 2u;
  for (uint32_t u = threadIdx.x; u < n; u += NT) {
    const uint32_t rr = u / NG, kk = u - rr * NG;
    const uint32_t r = rr + RB0, k = kk + KB0;
    const uint32_t y = (D == 3) ? (C == 0 ? msc_wrap2(y0 + r, L) : y0 + r - 2u) : z;
    const uint32_t zz = (D == 3) ? z : 0u;
    const uint32_t gx = msc_wrap2(G.gx0 + k, G.GPR);
    const uint64_t rowbase = (D == 3) ? ((uint64_t)zz * L + y) * L : (uint64_t)y * L;
    const uint64_t s0 = rowbase + 8u * gx;
    const uint32_t o = r * RW + 4 * k;
    uint32_t c[8], ym[8], yp[8], zm[8], zp[8];
    lds8(pc + o, HW, c);
    if (D == 3) {
      lds8(pc + o - RW, HW, ym);
      lds8(pc + o + RW, HW, yp);
      lds8(pm + o, HW, zm);
      lds8(pp + o, HW, zp);
    } else {
      lds8(pm + o, HW, ym);
      lds8(pp + o, HW, yp);
    }
    const uint32_t lw = pc[o + HW - 1], rw = pc[o + 4];  // word 7 of group k-1, word 0 of group k+1
    // couplings from HBM: the group's 8 x-bond words and the one left of it; the y and z bonds of
    // the four active sites (x parity P) from the parity-P halves of rows y and y-1 (planes z, z-1)
    const uint64_t N = a.N, plane = (uint64_t)L * L;
    const uint64_t sl = gx ? s0 - 1 : s0 + L - 1;
    const uint32_t P = (C + y + zz) & 1u;
    const uint64_t hoff = (uint64_t)P * (L / 2) + 4u * gx;
    const uint64_t rym = y ? rowbase - L : rowbase + (uint64_t)(L - 1) * L;  // start of row y-1
    uint32_t jx[8], jy[4], jym[4], jz[4], jzm[4];
    load8(J + s0, jx);
    load4(J + N + rowbase + hoff, jy);
    load4(J + N + rym + hoff, jym);
    if (D == 3) {
      const uint64_t rzm = zz ? rowbase - plane : rowbase + (uint64_t)(L - 1) * plane;  // row y of plane z-1
      load4(J + 2 * N + rowbase + hoff, jz);
      load4(J + 2 * N + rzm + hoff, jzm);
    }
    const uint32_t jl = J[sl];
    uint32_t rnd[4];
    philox_lane((uint32_t)(s0 >> 3), U, a.keys, rnd);
    uint32_t jb[4][2 * D];
    if (P == 0) {
      bonds_split<D, 0>(jx, jl, jy, jym, jz, jzm, jb);
      msc_update8<D, 0>(c, lw, rw, ym, yp, zm, zp, jb, rnd, a);
    } else {
      bonds_split<D, 1>(jx, jl, jy, jym, jz, jzm, jb);
      msc_update8<D, 1>(c, lw, rw, ym, yp, zm, zp, jb, rnd, a);
    }
    const u32x4 lo = {c[0], c[1], c[2], c[3]}, hi = {c[4], c[5], c[6], c[7]};
    if (C == 0) {
      *reinterpret_cast<u32x4*>(pc + o) = lo;
      *reinterpret_cast<u32x4*>(pc + o + HW) = hi;
    } else {
      reinterpret_cast<u32x4*>(dst + s0)[0] = lo;
      reinterpret_cast<u32x4*>(dst + s0)[1] = hi;
    }
  }
}

template <int D, int NT>
__global__ __launch_bounds__(NT) void k_msc_stream(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst,
                                                   const uint32_t* __restrict__ J, MscArgs a, uint32_t TYa,
                                                   uint32_t Ha, uint32_t XW) {
  extern __shared__ __align__(16) uint32_t ring[];
  MscGeom G;
  G.L = a.L;
  G.GPR = a.L / 8;
  G.SG = XW / 8 + 4;
  G.RW = 8 * G.SG;
  G.HW = 4 * G.SG;
  const uint32_t L = a.L;
  const uint32_t TY = (D == 3) ? TYa : 1u;
  const uint32_t RP = (D == 3) ? TY + 4 : 1u;
  const uint32_t SB = RP * G.RW;
  const uint32_t nseg = L / XW;
  const uint32_t gx = (D == 3) ? (L / TY) * nseg : nseg;
  uint32_t blk = blockIdx.x;
  if ((gridDim.x & 7u) == 0) blk = (blk & 7u) * (gridDim.x >> 3) + (blk >> 3);
  const uint32_t bx = blk % gx, by = blk / gx;
  const uint32_t seg = bx % nseg;
  G.gx0 = seg * (XW / 8);
  const uint32_t y0 = (D == 3) ? (bx / nseg) * TY : 0u;
  const uint32_t z0 = by * Ha;
  const uint32_t H = (L - z0 < Ha) ? L - z0 : Ha;
  const PhiloxUniform U0 = philox_uniform(a.t, a.p0, 4u, a.keys);
  const PhiloxUniform U1 = philox_uniform(a.t, a.p0, 5u, a.keys);
  const uint32_t tot = RP * G.SG;
  u32x4 nxt[2 * kMscFetch];
  for (uint32_t k = 0; k < 3; ++k) {
    msc_fetch<D, NT>(src, msc_wrap2(z0 + k, L), y0, G, tot, nxt);
    msc_put<NT>(ring + k * SB, G, tot, nxt);
  }
  __syncthreads();
  const uint32_t NG0 = XW / 8 + 2, NG1 = XW / 8;            // groups per row of colour 0 / colour 1 units
  const uint32_t U0n = ((D == 3) ? TY + 2 : 1u) * NG0;
  const uint32_t U1n = ((D == 3) ? TY : 1u) * NG1;
  uint32_t sa = 1;
  for (uint32_t i = 0; i < H + 3; ++i) {
    const uint32_t s_m3 = sa >= 3 ? sa - 3 : sa + 3;
    const uint32_t s_m2 = sa >= 2 ? sa - 2 : sa + 4;
    const uint32_t s_m1 = sa >= 1 ? sa - 1 : 5;
    const uint32_t s_p1 = sa <= 4 ? sa + 1 : 0;
    const uint32_t s_p2 = sa <= 3 ? sa + 2 : sa - 4;
    if (i <= H) msc_fetch<D, NT>(src, msc_wrap2(z0 + i + 3, L), y0, G, tot, nxt);
    if (i <= H + 1)
      msc_units<D, NT, 0>(ring + s_m1 * SB, ring + sa * SB, ring + s_p1 * SB, U0n, NG0, y0, msc_wrap2(z0 + i + 1, L),
                          G, a, U0, J, dst);
    if (i >= 3)
      msc_units<D, NT, 1>(ring + s_m3 * SB, ring + s_m2 * SB, ring + s_m1 * SB, U1n, NG1, y0, z0 + i - 3u, G, a, U1, J,
                          dst);
    if (i <= H) msc_put<NT>(ring + s_p2 * SB, G, tot, nxt);
    __syncthreads();
    sa = sa == 5 ? 0 : sa + 1;
  }
}

constexpr size_t kMscMaxLds = 160 * 1024;  // all of a CU's LDS

size_t msc_stream_lds(uint32_t L, uint32_t d, uint32_t TY, uint32_t XW) {
  (void)L;
  const size_t RP = d == 3 ? TY + 4 : 1;
  return 6 * RP * (XW + 32) * 4;
}

bool msc_stream_supported(uint32_t L, uint32_t d, uint32_t TY, uint32_t H, uint32_t NT, uint32_t XW) {
  if (L % 8 != 0 || L < 16 || H < 1 || H > L) return false;
  if (NT != 256 && NT != 512) return false;
  if (XW < 8 || XW % 8 != 0 || L % XW != 0) return false;
  if (d == 3 && (TY == 0 || L % TY != 0 || TY > 32)) return false;
  const uint32_t RP = d == 3 ? TY + 4 : 1;
  if (RP * (XW / 8 + 4) > (uint32_t)kMscFetch * NT) return false;
  return msc_stream_lds(L, d, TY, XW) <= kMscMaxLds;
}

template <int D, int NT>
static hipError_t go_msc_stream(const uint32_t* src, uint32_t* dst, const uint32_t* J, const MscArgs& a,
                                uint32_t TY, uint32_t H, uint32_t XW, hipStream_t stream) {
  static OncePerDevice once;
  const hipError_t e = allow_lds(once, {(const void*)k_msc_stream<D, NT>}, (int)kMscMaxLds);
  if (e != hipSuccess) return e;
  const uint32_t nseg = a.L / XW;
  const dim3 grid((D == 3 ? (a.L / TY) * nseg : nseg) * ((a.L + H - 1) / H));
  hipLaunchKernelGGL((k_msc_stream<D, NT>), grid, dim3(NT), msc_stream_lds(a.L, D, TY, XW), stream, src, dst, J, a,
                     TY, H, XW);
  return hipGetLastError();
}

hipError_t launch_msc_stream(const uint32_t* src, uint32_t* dst, const uint32_t* J, const MscArgs& a, uint32_t d,
                             uint32_t TY, uint32_t H, uint32_t NT, uint32_t XW, hipStream_t stream) {
  if (!msc_stream_supported(a.L, d, TY, H, NT, XW)) return hipErrorInvalidValue;
  if (d == 3) return NT == 256 ? go_msc_stream<3, 256>(src, dst, J, a, TY, H, XW, stream)
                               : go_msc_stream<3, 512>(src, dst, J, a, TY, H, XW, stream);
  return NT == 256 ? go_msc_stream<2, 256>(src, dst, J, a, TY, H, XW, stream)
                   : go_msc_stream<2, 512>(src, dst, J, a, TY, H, XW, stream);
}

// ------------------------------------------------------------ register columns
// 3D, L = 512, 256 or 128: one whole sweep per launch with each row's z column
// in registers, and every coupling word read from HBM once per sweep (the plane
// streaming kernel above reads the couplings of a site once per colour).
//
// Bound by memory at 20 B a site (3 coupling words, the site's word read and
// written): 500 us a sweep at L = 512 (5.4 TB/s) and 65 at L = 256 (5.2 TB/s, as
// a large copy reaches).  A row of L = 256 or 128 fills half or a quarter of a
// wavefront's lanes; the others take the same row of other strips, 79 -> 69 us
// at L = 256 and 22 -> 14.7 at L = 128 against repeating the row in them.  Sweeps
// march up and down in turn, so that a sweep begins where the last one ended,
// in the planes the memory-side cache still holds: 69 -> 65 us at L = 256 (320
// MB a sweep against a 256 MB cache), L = 512 and 128 as before.
//
// A workgroup owns the TY rows [y0, y0+TY) of the planes [z0, z0+H) and has
// TY + 2 waves; wave w keeps slab row r = w + 1 (y = y0 - 2 + r) for the
// whole launch: rows 2..TY+1 are owned, 1 and TY+2 a ring whose colour 0 is
// recomputed here (colour 1 of the owned edge rows needs it), and 0 and TY+3
// a halo that the ring's colour 0 reads.  Lane l holds the group of sites
// x = 8l .. 8l+7 of its row (a 512-site row is one wavefront; struct Planes
// has the smaller ones).  Planes are counted along the march here; with REV it
// goes down from z0 + H - 1 and "above" is below.
// Step i = 0..H+1 with a = z0-1+i, b = a-1.  Both colour units of a step
// have active sites of x parity P = (y + a) & 1 (colour 0 on plane a,
// colour 1 on plane b):
//   write plane a+1's spins as loaded (the parity-P words: colour-1 sites,
//     which the neighbouring rows' colour 0 reads in step i+1) and y bonds
//     (all words) into LDS slot N;
//   issue the loads of plane a+2's spins and y bonds and plane a+1's x and z
//     bonds (registers; used in step i+1);
//   colour 0 on plane a: z neighbours plane b after its colour 0 (its
//     colour-1 words still the old ones) and plane a+1 as loaded, from
//     registers; y neighbours and y bonds from slot A; x neighbours and the
//     x bond left of the group by a wavefront rotate; the new parity-P words
//     go into slot A (the other rows read the other half of it in this step);
//   colour 1 on plane b (owned rows, i >= 2): z neighbours plane b-1 and
//     plane a after colour 0 (registers), y neighbours and bonds from slot B
//     (plane b after colour 0, written in step i-1); the group goes to dst;
//   barrier.
// Register lifetimes: an x-bond word serves colour 0 of its plane in one
// step and colour 1 of the same plane in the next; a z-bond word (bond to the
// plane above) serves its plane's colour-0 unit and the next plane's
// colour-1 unit for one parity half, and the next plane's colour-0 and its
// own plane's colour-1 unit for the other, over three steps.  LDS rows keep
// the parity split of the y and z bonds in HBM (even-x words, then odd-x
// words), so the four active words of a group are 16 contiguous bytes.
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

namespace col {

struct G8 {  // one group, natural site order: words 0-3 in lo, 4-7 in hi
  v4u lo, hi;
};
struct H8 {  // one group's y or z bonds, split by parity: h[0] even x, h[1] odd x
  v4u h[2];
};

template <uint32_t P>
__device__ __forceinline__ v4u half(const G8& g) {
  return v4u{g.lo[P], g.lo[2 + P], g.hi[P], g.hi[2 + P]};
}

// Where a plane's rows lie for the lanes.  A row has GPR = L/8 groups: with
// GPR < 64 the wavefront's 64/GPR parts each hold the row of another plane, the
// same row y of planes zc = L/C apart (C parts; with C < 64/GPR the further
// parts repeat the first ones and store what those store).  The scalar part of
// an address takes the plane modulo zc, the lanes' part the rest, modulo C.
template <uint32_t L>
struct Planes {
  static constexpr uint32_t GPR = L / 8;
  static constexpr bool kParts = GPR < 64;
  uint32_t zc, tz;      // planes of a part, log2 of it
  uint32_t unit, mask;  // groups of a part's planes, (C - 1) times that
  uint32_t part, lane;  // this lane's part times unit; its group of the row
  __device__ __forceinline__ uint32_t row(uint32_t z, uint32_t y) const {  // first group of the row, scalar part
    return ((kParts ? (z & (zc - 1u)) : z) * L + y) * GPR;
  }
  __device__ __forceinline__ uint32_t rest(uint32_t z) const {  // groups to add to it in this lane
    return kParts ? ((part + (z >> tz) * unit) & mask) : 0u;
  }
};

template <uint32_t L>
__device__ __forceinline__ G8 ld_group(__amdgpu_buffer_rsrc_t r, const Planes<L>& p, uint32_t z, uint32_t y) {
  const uint32_t v = 32u * (p.rest(z) | p.lane), row = 32u * p.row(z, y);
  G8 g;
  g.lo = __builtin_amdgcn_raw_buffer_load_b128(r, v, row, 0);
  g.hi = __builtin_amdgcn_raw_buffer_load_b128(r, v + 16u, row, 0);
  return g;
}

template <uint32_t L>
__device__ __forceinline__ H8 ld_split(__amdgpu_buffer_rsrc_t r, const Planes<L>& p, uint32_t z, uint32_t y) {
  const uint32_t v = 32u * p.rest(z) | 16u * p.lane, row = 32u * p.row(z, y);
  H8 g;
  g.h[0] = __builtin_amdgcn_raw_buffer_load_b128(r, v, row, 0);
  g.h[1] = __builtin_amdgcn_raw_buffer_load_b128(r, v + 2u * L, row, 0);  // the odd-x half
  return g;
}

// Lane l gets the value of the lane of the group left (ror1) or right (rol1) of its own in the
// periodic row of GPR lanes: a rotate of the wavefront, with two rows in it the two ends exchanged, with
// four a rotate of each 16 lanes.
template <uint32_t GPR>
__device__ __forceinline__ uint32_t ror1(uint32_t v) {
  if (GPR == 16) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xF, 0xF, false);
  const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x13C, 0xF, 0xF, false);
  if (GPR == 64) return t;
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 31), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
  const uint32_t l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  return l == 0u ? a : (l == 32u ? b : t);
}
template <uint32_t GPR>
__device__ __forceinline__ uint32_t rol1(uint32_t v) {
  if (GPR == 16) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x12F, 0xF, 0xF, false);
  const uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x134, 0xF, 0xF, false);
  if (GPR == 64) return t;
  const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, 0), b = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
  const uint32_t l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  return l == 31u ? a : (l == 63u ? b : t);
}

// One colour unit on the active sites j = 2i + P of group g: nb is the x
// neighbour outside the group (P = 0: word 7 of the group to the left; P = 1:
// word 0 of the group to the right), jx the group's x bonds and jl the x
// bond left of the group (P = 0 only); ym, yp, zm, zp the active sites'
// neighbours and jym, jy, jzm, jz their y and z bonds, word i for site 2i+P;
// r the shared draws.  Same bit-sliced count and acceptance as msc_update8.
template <uint32_t P>
__device__ __forceinline__ void unit(G8& g, uint32_t nb, const G8& jx, uint32_t jl, v4u ym, v4u yp, v4u zm, v4u zp,
                                     v4u jym, v4u jy, v4u jzm, v4u jz, const uint32_t (&r)[4],
                                     const uint64_t (&thr)[3]) {
  uint32_t w[8] = {g.lo.x, g.lo.y, g.lo.z, g.lo.w, g.hi.x, g.hi.y, g.hi.z, g.hi.w};
  const uint32_t x[8] = {jx.lo.x, jx.lo.y, jx.lo.z, jx.lo.w, jx.hi.x, jx.hi.y, jx.hi.z, jx.hi.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = 2 * i + (int)P;
    const uint32_t s = w[j];
    const uint32_t left = j ? w[j - 1] : nb;
    const uint32_t right = j < 7 ? w[j + 1] : nb;
    const uint32_t b0 = xor3(s, left, j ? x[j - 1] : jl), b1 = xor3(s, right, x[j]);
    const uint32_t b2 = xor3(s, ym[i], jym[i]), b3 = xor3(s, yp[i], jy[i]);
    const uint32_t b4 = xor3(s, zm[i], jzm[i]), b5 = xor3(s, zp[i], jz[i]);
    const uint32_t s1 = xor3(b0, b1, b2), c1 = maj3(b0, b1, b2);
    const uint32_t s2 = xor3(b3, b4, b5), c2 = maj3(b3, b4, b5);
    const uint32_t u0 = s1 ^ s2, t = s1 & s2;
    const uint32_t u1 = xor3(c1, c2, t), u2 = maj3(c1, c2, t);
    w[j] = s ^ msc_flips<3, false>(u0, u1, u2, r[i], thr);
  }
  g.lo = v4u{w[0], w[1], w[2], w[3]};
  g.hi = v4u{w[4], w[5], w[6], w[7]};
}

// Roles of the waves: row r, its parity, whether it is owned, and which halo
// row it loads (TOP: spins of row 0; JH: y bonds of row 0; BOT: spins of row TY+3).
enum { TOP = 0, JH = 1, BOT = 2, ODD = 3, EVEN = 4 };

template <int ROLE>
struct Role {
  static constexpr uint32_t RP = (ROLE == TOP || ROLE == ODD) ? 1u : 0u;
  static constexpr bool OWN = ROLE != TOP && ROLE != BOT;
};

template <uint32_t L>
struct Ctx {
  __amdgpu_buffer_rsrc_t src, dst, jx, jy, jz;
  Planes<L> pl;
  uint32_t* ls;  // spin slices: 3 x (TY+4) rows
  uint32_t* lj;  // y-bond slices: 3 x (TY+3) rows
  const RoundKeys* keys;
  PhiloxUniform U0, U1;
  uint64_t thr[3];
  // m-th plane of the strip's march (m = -2 ..): upwards from z0, or with REV downwards from z0 + H - 1
  template <bool REV>
  __device__ __forceinline__ uint32_t plane(uint32_t m) const {
    return (REV ? z0 + H - 1u - m : z0 + m) & (L - 1u);
  }
  uint32_t z0, H, lane, r, y, yh;  // yh: the halo row this wave loads (TOP, JH: row 0; BOT: row TY+3)
};

struct Regs {
  G8 s2, s1, sa, sb;  // spins: plane a+2 (in flight), a+1 as loaded, a as loaded, b after colour 0
  v4u sbb;            // plane b-1 after colour 0, this step's active half
  H8 jy1;             // y bonds of plane a+1 (written to LDS at the start of the step), then of a+2
  G8 jxn, jxa, jxb;   // x bonds of planes a+1 (in flight), a, b
  H8 jzn, jza, jzb;   // z bonds of planes a+1 (in flight), a, b
  v4u jzbb;           // z bonds of plane b-1, this step's active half
  G8 hs;              // halo spins (TOP, BOT): plane a+1, then a+2
  H8 hj;              // halo y bonds (JH): plane a+1, then a+2
  uint32_t sA, sB, sN;  // LDS slots of planes a, b, a+1
};

// An LDS row is a wavefront's: 64 groups, their even-x words (the 4 of lane l at 4 l), then the odd-x ones.
constexpr uint32_t RW = 512, HW = 256;

template <uint32_t L, int TY, int ROLE, bool REV, uint32_t Q, bool C1>
__device__ __forceinline__ void step(const Ctx<L>& c, Regs& R, uint32_t i) {
  using RL = Role<ROLE>;
  constexpr uint32_t GPR = L / 8;
  constexpr uint32_t SS = (TY + 4) * RW, JS = (TY + 3) * RW;  // words per spin / y-bond slice
  constexpr uint32_t F = Q + 1u + (REV ? 1u : 0u);  // parity of plane a
  constexpr uint32_t P = (RL::RP + F) & 1u;
  const uint32_t lane = c.lane, r = c.r, y = c.y;
  const uint32_t a = c.template plane<REV>(i - 1u), b = c.template plane<REV>(i - 2u);
  const uint32_t ic = i <= c.H ? i : c.H;  // loads past the strip's needs reload a plane already read
  const uint32_t zs = c.template plane<REV>(ic + 1u), zx = c.template plane<REV>(ic);
  // plane a+1 into slot N (free since the last barrier: it held plane b-1)
  {
    uint32_t* sN = c.ls + R.sN * SS;
    uint32_t* jN = c.lj + R.sN * JS;
    *reinterpret_cast<v4u*>(sN + r * RW + P * HW + 4u * lane) = half<P>(R.s1);
    *reinterpret_cast<v4u*>(jN + r * RW + 4u * lane) = R.jy1.h[0];
    *reinterpret_cast<v4u*>(jN + r * RW + HW + 4u * lane) = R.jy1.h[1];
    if (ROLE == TOP) {
      constexpr uint32_t PH = F & 1u;
      *reinterpret_cast<v4u*>(sN + PH * HW + 4u * lane) = half<PH>(R.hs);
    }
    if (ROLE == BOT) {
      constexpr uint32_t PH = ((uint32_t)TY + 3u + F) & 1u;
      *reinterpret_cast<v4u*>(sN + (TY + 3) * RW + PH * HW + 4u * lane) = half<PH>(R.hs);
    }
    if (ROLE == JH) {
      *reinterpret_cast<v4u*>(jN + 4u * lane) = R.hj.h[0];
      *reinterpret_cast<v4u*>(jN + HW + 4u * lane) = R.hj.h[1];
    }
  }
  // loads for the next step
  R.s2 = ld_group(c.src, c.pl, zs, y);
  R.jy1 = ld_split(c.jy, c.pl, zs, y);
  R.jxn = ld_group(c.jx, c.pl, zx, y);
  R.jzn = ld_split(c.jz, c.pl, REV ? (zx + L - 1u) & (L - 1u) : zx, y);
  if (ROLE == TOP || ROLE == BOT) R.hs = ld_group(c.src, c.pl, zs, c.yh);
  if (ROLE == JH) R.hj = ld_split(c.jy, c.pl, zs, c.yh);
  // colour 0 on plane a
  const uint32_t* sA = c.ls + R.sA * SS;
  const uint32_t* jA = c.lj + R.sA * JS;
  const uint32_t o = P * HW + 4u * lane;
  uint32_t rnd[4];
  philox_lane(c.pl.row(a, y) + (c.pl.rest(a) | c.pl.lane), c.U0, *c.keys, rnd);
  G8 na = R.sa;
  {
    const v4u ym = *reinterpret_cast<const v4u*>(sA + (r - 1) * RW + o);
    const v4u yp = *reinterpret_cast<const v4u*>(sA + (r + 1) * RW + o);
    const v4u jy = *reinterpret_cast<const v4u*>(jA + r * RW + o);
    const v4u jym = *reinterpret_cast<const v4u*>(jA + (r - 1) * RW + o);
    const uint32_t nb = P == 0 ? ror1<GPR>(R.sa.hi.w) : rol1<GPR>(R.sa.lo.x);
    const uint32_t jl = P == 0 ? ror1<GPR>(R.jxa.hi.w) : 0u;
    unit<P>(na, nb, R.jxa, jl, ym, yp, half<P>(R.sb), half<P>(R.s1), jym, jy, R.jzb.h[P], R.jza.h[P], rnd, c.thr);
    *reinterpret_cast<v4u*>(c.ls + R.sA * SS + r * RW + o) = half<P>(na);
  }
  // colour 1 on plane b
  if (C1 && RL::OWN) {
    const uint32_t* sB = c.ls + R.sB * SS;
    const uint32_t* jB = c.lj + R.sB * JS;
    const uint32_t gb = c.pl.rest(b) | c.pl.lane, rb = c.pl.row(b, y);
    philox_lane(rb + gb, c.U1, *c.keys, rnd);
    const v4u ym = *reinterpret_cast<const v4u*>(sB + (r - 1) * RW + o);
    const v4u yp = *reinterpret_cast<const v4u*>(sB + (r + 1) * RW + o);
    const v4u jy = *reinterpret_cast<const v4u*>(jB + r * RW + o);
    const v4u jym = *reinterpret_cast<const v4u*>(jB + (r - 1) * RW + o);
    const uint32_t nb = P == 0 ? ror1<GPR>(R.sb.hi.w) : rol1<GPR>(R.sb.lo.x);
    const uint32_t jl = P == 0 ? ror1<GPR>(R.jxb.hi.w) : 0u;
    G8 nbk = R.sb;
    unit<P>(nbk, nb, R.jxb, jl, ym, yp, R.sbb, half<P>(na), jym, jy, R.jzbb, R.jzb.h[P], rnd, c.thr);
    __builtin_amdgcn_raw_buffer_store_b128(nbk.lo, c.dst, 32u * gb, 32u * rb, 0);
    __builtin_amdgcn_raw_buffer_store_b128(nbk.hi, c.dst, 32u * gb + 16u, 32u * rb, 0);
  }
  // the next step's registers (its active half is 1 - P)
  R.sbb = half<P ^ 1u>(R.sb);
  R.sb = na;
  R.sa = R.s1;
  R.s1 = R.s2;
  R.jxb = R.jxa;
  R.jxa = R.jxn;
  R.jzbb = R.jzb.h[P ^ 1u];
  R.jzb = R.jza;
  R.jza = R.jzn;
  const uint32_t t = R.sB;
  R.sB = R.sA;
  R.sA = R.sN;
  R.sN = t;
  __syncthreads();
}

template <uint32_t L, int TY, int ROLE, bool REV>
__device__ __forceinline__ void run(const Ctx<L>& c) {
  using RL = Role<ROLE>;
  constexpr uint32_t SS = (TY + 4) * RW, JS = (TY + 3) * RW;
  const uint32_t lane = c.lane, r = c.r, y = c.y;
  const uint32_t zm2 = c.template plane<REV>(0u - 2u), zm1 = c.template plane<REV>(0u - 1u);
  const uint32_t zf = c.template plane<REV>(0u);
  constexpr uint32_t F = REV ? 1u : 0u;  // half of an even row that step 0 reads of its neighbours
  Regs R;
  // prologue: plane z0-1 into slot 0 (spins half P(r, step -1) = r & 1, all y bonds); registers for step 0
  R.sb = ld_group(c.src, c.pl, zm2, y);
  R.sa = ld_group(c.src, c.pl, zm1, y);
  R.s1 = ld_group(c.src, c.pl, zf, y);
  R.jxa = ld_group(c.jx, c.pl, zm1, y);
  R.jza = ld_split(c.jz, c.pl, REV ? zf : zm1, y);
  R.jzb = ld_split(c.jz, c.pl, REV ? zm1 : zm2, y);
  const H8 jy0 = ld_split(c.jy, c.pl, zm1, y);
  R.jy1 = ld_split(c.jy, c.pl, zf, y);
  R.jxb = R.jxa;
  R.sbb = v4u{0u, 0u, 0u, 0u};
  R.jzbb = v4u{0u, 0u, 0u, 0u};
  R.hs.lo = R.hs.hi = v4u{0u, 0u, 0u, 0u};
  R.hj.h[0] = R.hj.h[1] = v4u{0u, 0u, 0u, 0u};
  *reinterpret_cast<v4u*>(c.ls + r * RW + ((RL::RP + F) & 1u) * HW + 4u * lane) = half<(RL::RP + F) & 1u>(R.sa);
  *reinterpret_cast<v4u*>(c.lj + r * RW + 4u * lane) = jy0.h[0];
  *reinterpret_cast<v4u*>(c.lj + r * RW + HW + 4u * lane) = jy0.h[1];
  if (ROLE == TOP) {  // row 0: half F
    const G8 h = ld_group(c.src, c.pl, zm1, c.yh);
    *reinterpret_cast<v4u*>(c.ls + F * HW + 4u * lane) = half<F>(h);
    R.hs = ld_group(c.src, c.pl, zf, c.yh);
  }
  if (ROLE == BOT) {  // row TY+3: half (TY + 3 + F) & 1
    const G8 h = ld_group(c.src, c.pl, zm1, c.yh);
    *reinterpret_cast<v4u*>(c.ls + (TY + 3) * RW + (1u - F) * HW + 4u * lane) = half<1u - F>(h);
    R.hs = ld_group(c.src, c.pl, zf, c.yh);
  }
  if (ROLE == JH) {
    const H8 h = ld_split(c.jy, c.pl, zm1, c.yh);
    *reinterpret_cast<v4u*>(c.lj + 4u * lane) = h.h[0];
    *reinterpret_cast<v4u*>(c.lj + HW + 4u * lane) = h.h[1];
    R.hj = ld_split(c.jy, c.pl, zf, c.yh);
  }
  (void)SS;
  (void)JS;
  R.sA = 0;
  R.sN = 1;
  R.sB = 2;
  __syncthreads();
  step<L, TY, ROLE, REV, 0, false>(c, R, 0u);
  step<L, TY, ROLE, REV, 1, false>(c, R, 1u);
  for (uint32_t i0 = 2; i0 < c.H + 2u; i0 += 2) {
    step<L, TY, ROLE, REV, 0, true>(c, R, i0);
    step<L, TY, ROLE, REV, 1, true>(c, R, i0 + 1u);
  }
}

}  // namespace col

template <uint32_t L, int TY, bool REV>
__global__ __launch_bounds__(64 * (TY + 2)) void k_msc_col(const uint32_t* __restrict__ src,
                                                           uint32_t* __restrict__ dst,
                                                           const uint32_t* __restrict__ J, MscArgs a,
                                                           uint32_t H, uint32_t parts) {
  using namespace col;
  extern __shared__ __align__(16) uint32_t lds[];
  constexpr uint32_t Nw = L * L * L;
  constexpr uint32_t GPR = L / 8;
  Ctx<L> c;
  c.src = __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, (int)(Nw * 4u), 0x00020000);
  c.dst = __builtin_amdgcn_make_buffer_rsrc((void*)dst, 0, (int)(Nw * 4u), 0x00020000);
  c.jx = __builtin_amdgcn_make_buffer_rsrc((void*)J, 0, (int)(Nw * 4u), 0x00020000);
  c.jy = __builtin_amdgcn_make_buffer_rsrc((void*)(J + Nw), 0, (int)(Nw * 4u), 0x00020000);
  c.jz = __builtin_amdgcn_make_buffer_rsrc((void*)(J + 2u * (size_t)Nw), 0, (int)(Nw * 4u), 0x00020000);
  c.ls = lds;
  c.lj = lds + 3u * (TY + 4) * RW;
  c.keys = &a.keys;
  c.U0 = philox_uniform(a.t, a.p0, 4u, a.keys);
  c.U1 = philox_uniform(a.t, a.p0, 5u, a.keys);
  c.thr[0] = a.thr[0];
  c.thr[1] = a.thr[1];
  c.thr[2] = a.thr[2];
  // workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of tiles (the slabs of
  // one strip side by side), so that the halo rows of neighbouring slabs are read through the same L2
  const uint32_t nslab = L / TY, nblk = gridDim.x, bk = blockIdx.x;
  const uint32_t tile = (nblk % 8u == 0u) ? (bk % 8u) * (nblk / 8u) + bk / 8u : bk;
  const uint32_t y0 = (tile % nslab) * TY;
  c.z0 = (tile / nslab) * H;  // of part 0; part q's strip begins q L / parts planes on
  c.H = H;
  c.lane = threadIdx.x & 63u;
  c.pl.zc = L / parts;
  c.pl.tz = 31u - (uint32_t)__builtin_clz(c.pl.zc);
  c.pl.unit = c.pl.zc * L * GPR;
  c.pl.mask = (parts - 1u) * c.pl.unit;
  c.pl.lane = c.lane & (GPR - 1u);
  c.pl.part = ((c.lane / GPR) & (parts - 1u)) * c.pl.unit;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  c.r = wave + 1u;
  c.y = (y0 + L - 2u + c.r) & (L - 1u);
  c.yh = (wave == (uint32_t)TY + 1u) ? (y0 + TY + 1u) & (L - 1u) : (y0 + L - 2u) & (L - 1u);
  if (wave == 0)
    run<L, TY, TOP, REV>(c);
  else if (wave == 1)
    run<L, TY, JH, REV>(c);
  else if (wave == (uint32_t)TY + 1u)
    run<L, TY, BOT, REV>(c);
  else if (c.r & 1u)
    run<L, TY, ODD, REV>(c);
  else
    run<L, TY, EVEN, REV>(c);
}

constexpr size_t msc_col_lds(uint32_t TY) { return (size_t)(3 * (TY + 4) + 3 * (TY + 3)) * col::RW * 4; }

bool msc_col_supported(uint32_t L, uint32_t d, uint32_t TY, uint32_t H) {
  return d == 3 && (L == 128 || L == 256 || L == 512) && (TY == 4 || TY == 8) && H >= 2 && H % 2 == 0 &&
         L % H == 0;
}

template <uint32_t L, int TY, bool REV>
static hipError_t go_msc_dir(const uint32_t* src, uint32_t* dst, const uint32_t* J, const MscArgs& a, uint32_t H,
                             hipStream_t stream) {
  static OncePerDevice once;
  const hipError_t e = allow_lds(once, {(const void*)k_msc_col<L, TY, REV>}, (int)msc_col_lds(TY));
  if (e != hipSuccess) return e;
  // strips side by side in a wavefront: as many as the row leaves lanes for, each L / parts planes
  // after the last, where that is a whole number of strips
  uint32_t parts = 512u / L;
  while (parts > 1 && (L / parts) % H != 0) parts >>= 1;
  const dim3 grid((L / TY) * (L / (H * parts)));
  hipLaunchKernelGGL((k_msc_col<L, TY, REV>), grid, dim3(64 * (TY + 2)), msc_col_lds(TY), stream, src, dst, J, a, H, parts);
  return hipGetLastError();
}

// Every other sweep marches down: it begins with the planes that the last one wrote and read last.
template <uint32_t L, int TY>
static hipError_t go_msc_col(const uint32_t* src, uint32_t* dst, const uint32_t* J, const MscArgs& a, uint32_t H,
                             hipStream_t stream) {
  return (a.t & 1u) ? go_msc_dir<L, TY, true>(src, dst, J, a, H, stream)
                    : go_msc_dir<L, TY, false>(src, dst, J, a, H, stream);
}

hipError_t launch_msc_col(const uint32_t* src, uint32_t* dst, const uint32_t* J, const MscArgs& a, uint32_t d,
                          uint32_t TY, uint32_t H, hipStream_t stream) {
  if (!msc_col_supported(a.L, d, TY, H)) return hipErrorInvalidValue;
  if (a.L == 512) return TY == 8 ? go_msc_col<512, 8>(src, dst, J, a, H, stream) : go_msc_col<512, 4>(src, dst, J, a, H, stream);
  if (a.L == 256) return TY == 8 ? go_msc_col<256, 8>(src, dst, J, a, H, stream) : go_msc_col<256, 4>(src, dst, J, a, H, stream);
  return TY == 8 ? go_msc_col<128, 8>(src, dst, J, a, H, stream) : go_msc_col<128, 4>(src, dst, J, a, H, stream);
}

// E and M of the 32 systems: per workgroup, counts of unsatisfied bonds and
// of negative spins for every bit into part[wg*64 + bit] (unsat) and
// part[wg*64 + 32 + bit] (negative); k_msc_finalize sums the workgroups.
//
// Bound by the words it reads, 16 B a site in 3D (the site's own word and its
// bonds; the neighbours' words come from cache), so the counting is kept below
// that: a lane adds the bonds of four sites at a time into bit-sliced
// counters (full adders, one sum and one carry operation for all 32 systems),
// about 12 operations a site where taking every bit of every word apart took
// 300, and after 64 sites a wavefront adds its lanes' counters, lane l of the
// result holding system l mod 32 (unsatisfied bonds below lane 32, negative spins
// from there).  Rows are walked by 32-bit coordinates, no division in the loop.
// 3D L = 256: 634 us with integer adds for every bit, 52 us now (5.1 TB/s).
struct MscSum {  // carry and sum of three bits of one weight
  uint32_t s, c;
};
__device__ __forceinline__ MscSum msc_fa(uint32_t a, uint32_t b, uint32_t c) {
  return MscSum{xor3(a, b, c), maj3(a, b, c)};
}

// Bit-sliced counters of P planes plus those of another lane (a DPP row
// permutation CTRL), into P + 1 planes.
template <int P, int CTRL>
__device__ __forceinline__ void msc_add_lane(uint32_t (&c)[12]) {
  uint32_t carry = 0;
#pragma unroll
  for (int p = 0; p < P; ++p) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)c[p], CTRL, 0xF, 0xF, true);
    const MscSum f = msc_fa(c[p], o, carry);
    c[p] = f.s;
    carry = f.c;
  }
  c[P] = carry;
}

// Counters of P planes of all 64 lanes: lane l gets the total of system l mod 32.
template <int P>
__device__ __forceinline__ uint32_t msc_wave_count(uint32_t (&c)[12]) {
  msc_add_lane<P, 0xB1>(c);       // quad_perm [1,0,3,2]
  msc_add_lane<P + 1, 0x4E>(c);   // quad_perm [2,3,0,1]
  msc_add_lane<P + 2, 0x141>(c);  // row_half_mirror: the other quad of eight lanes
  msc_add_lane<P + 3, 0x140>(c);  // row_mirror: the other half of sixteen
  const uint32_t bit = threadIdx.x & 31u;
  uint32_t n = 0;
#pragma unroll
  for (int p = 0; p < P + 4; ++p)
#pragma unroll
    for (int row = 0; row < 4; ++row)
      n += (((uint32_t)__builtin_amdgcn_readlane((int)c[p], 16 * row) >> bit) & 1u) << p;
  return n;
}

constexpr uint32_t kMscChunk = 64;  // sites a lane counts before its counters are taken up: 3 * 64 < 2^8

template <int D>
__global__ __launch_bounds__(256) void k_msc_count(const uint32_t* __restrict__ S, const uint32_t* __restrict__ J,
                                                   uint32_t L, uint64_t N, uint32_t nrows, uint32_t rpb,
                                                   int64_t* __restrict__ part) {
  __shared__ int64_t red[4][64];
  // threads over (row, x): whole rows side by side where they are shorter than the workgroup, else
  // segments of 256 sites; a workgroup's rows are rpb consecutive ones
  const uint32_t xw = L < 256u ? L : 256u, rpt = 256u / xw, nseg = (L + 255u) / 256u;
  const uint32_t rl = threadIdx.x / xw, x0 = threadIdx.x - rl * xw;
  const uint32_t r0 = blockIdx.x * rpb, r1 = nrows - r0 < rpb ? nrows : r0 + rpb;
  const uint32_t steps = ((r1 - r0 + rpt - 1u) / rpt) * nseg;
  const bool active = rl < rpt;
  uint32_t row = r0 + rl, seg = 0;
  uint32_t y = row % L, z = row / L;
  const uint64_t plane = (uint64_t)L * L;
  uint64_t total = 0;
  for (uint32_t i0 = 0; i0 < steps; i0 += kMscChunk) {
    uint32_t U[12] = {}, M[12] = {};
    const uint32_t i1 = steps - i0 < kMscChunk ? steps : i0 + kMscChunk;
    for (uint32_t i = i0; i < i1; i += 4) {
      uint32_t v[4], s[4], c[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t x = x0 + 256u * seg;
        const bool on = active && row < r1 && x < L && i + q < i1;
        // lanes with nothing to count read site 0 and add zeros
        const uint64_t base = on ? (uint64_t)row * L : 0u;
        const uint32_t xx = on ? x : 0u, yy = on ? y : 0u, zz = on ? z : 0u;
        const uint64_t at = base + xx, sj = base + (xx & 1u) * (L / 2u) + (xx >> 1);
        const uint32_t w = S[at];
        uint32_t bx = w ^ S[xx + 1u < L ? at + 1u : base] ^ J[at];
        uint32_t by = w ^ S[yy + 1u < L ? at + L : at - (uint64_t)(L - 1u) * L] ^ J[N + sj];
        uint32_t bz = 0;
        if (D == 3) bz = w ^ S[zz + 1u < L ? at + plane : at - (uint64_t)(L - 1u) * plane] ^ J[2u * N + sj];
        const uint32_t keep = on ? 0xFFFFFFFFu : 0u;
        v[q] = w & keep;
        const MscSum f = msc_fa(bx & keep, by & keep, bz & keep);
        s[q] = f.s;
        c[q] = f.c;
        if (++seg == nseg) {
          seg = 0;
          row += rpt;
          y += rpt;
          while (y >= L) {
            y -= L;
            ++z;
          }
        }
      }
      // unsatisfied bonds: four sums of weight 1 and four carries of weight 2 into U
      const MscSum a1 = msc_fa(s[0], s[1], s[2]), a2 = msc_fa(U[0], a1.s, s[3]);
      const MscSum b1 = msc_fa(c[0], c[1], c[2]), b2 = msc_fa(c[3], a1.c, a2.c), b3 = msc_fa(U[1], b1.s, b2.s);
      const MscSum d1 = msc_fa(b1.c, b2.c, b3.c);
      U[0] = a2.s;
      U[1] = b3.s;
      const uint32_t d2 = U[2] & d1.s;
      U[2] ^= d1.s;
      const MscSum e1 = msc_fa(U[3], d1.c, d2);
      U[3] = e1.s;
      uint32_t k = e1.c;
#pragma unroll
      for (int p = 4; p < 8; ++p) {
        const uint32_t t = U[p] & k;
        U[p] ^= k;
        k = t;
      }
      // negative spins: four of weight 1 into M
      const MscSum m1 = msc_fa(v[0], v[1], v[2]), m2 = msc_fa(M[0], m1.s, v[3]), m3 = msc_fa(M[1], m1.c, m2.c);
      M[0] = m2.s;
      M[1] = m3.s;
      k = m3.c;
#pragma unroll
      for (int p = 2; p < 7; ++p) {
        const uint32_t t = M[p] & k;
        M[p] ^= k;
        k = t;
      }
    }
    const uint32_t nu = msc_wave_count<8>(U), nm = msc_wave_count<7>(M);
    total += (threadIdx.x & 32u) ? nm : nu;
  }
  red[threadIdx.x >> 6][threadIdx.x & 63u] = (int64_t)total;
  __syncthreads();
  if (threadIdx.x < 64)
    part[(uint64_t)blockIdx.x * 64 + threadIdx.x] =
        red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// Sum over the workgroups: wave w of 16 adds every 16th row of 64 counts, then the waves are added
// (one wave alone, row after row, took 498 us at 2048 workgroups: a chain of dependent loads; now 18).
__global__ __launch_bounds__(1024) void k_msc_finalize(const int64_t* __restrict__ part, uint32_t nparts, int64_t nb,
                                                       int64_t N, int64_t* __restrict__ E, int64_t* __restrict__ M) {
  __shared__ int64_t red[16][64];
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  int64_t t = 0;
#pragma unroll 8
  for (uint32_t w = wave; w < nparts; w += 16) t += part[(uint64_t)w * 64 + lane];
  red[wave][lane] = t;
  __syncthreads();
  if (wave == 0) {
    t = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][lane];
    if (lane < 32)
      E[lane] = -nb + 2 * t;
    else
      M[lane - 32] = N - 2 * t;
  }
}

static unsigned blocks_for(uint64_t work, unsigned cap) {
  uint64_t b = (work + 255) / 256;
  return (unsigned)(b < cap ? (b ? b : 1) : cap);
}

hipError_t launch_msc_init(uint32_t* S, uint64_t N, uint64_t seed, uint32_t p0, hipStream_t stream) {
  hipLaunchKernelGGL(k_msc_init, dim3(blocks_for(N / 4, 8192)), dim3(256), 0, stream, S, N / 4, make_round_keys(seed),
                     p0);
  return hipGetLastError();
}

hipError_t launch_msc_couplings(uint32_t* J, uint64_t N, uint32_t L, uint32_t d, uint64_t cseed, uint32_t r0,
                                hipStream_t stream) {
  hipLaunchKernelGGL(k_msc_couplings, dim3(blocks_for(N / 4, 8192)), dim3(256), 0, stream, J, N / 4, L, d,
                     make_round_keys(cseed), r0);
  return hipGetLastError();
}

hipError_t launch_msc_phase(uint32_t* S, const uint32_t* J, const MscArgs& a, uint32_t d, hipStream_t stream) {
  const unsigned blocks = blocks_for(a.N / 8, 1u << 20);
  if (d == 3)
    hipLaunchKernelGGL(k_msc_phase<3>, dim3(blocks), dim3(256), 0, stream, S, J, a);
  else
    hipLaunchKernelGGL(k_msc_phase<2>, dim3(blocks), dim3(256), 0, stream, S, J, a);
  return hipGetLastError();
}

// Rows a counting workgroup takes: whole passes of its threads (rows side by side where they are
// short), as many as leave at most 2048 workgroups, and 32 sites a thread where there are enough.
static uint32_t msc_count_rows(uint32_t L, uint64_t nrows) {
  const uint32_t rpt = L < 256u ? 256u / L : 1u, nseg = (L + 255u) / 256u;
  const uint64_t want = rpt * std::max(1u, 32u / nseg);
  uint64_t rpb = std::max<uint64_t>((nrows + 2047u) / 2048u, std::min<uint64_t>(want, (nrows + 1023u) / 1024u));
  return (uint32_t)((rpb + rpt - 1u) / rpt * rpt);
}

uint32_t msc_count_parts(uint32_t L, uint64_t N) {
  const uint64_t nrows = N / L, rpb = msc_count_rows(L, nrows);
  return (uint32_t)((nrows + rpb - 1u) / rpb);
}

hipError_t launch_msc_measure(const uint32_t* S, const uint32_t* J, uint32_t L, uint32_t d, uint64_t N, int64_t* part,
                              int64_t* E, int64_t* M, hipStream_t stream) {
  const uint32_t nrows = (uint32_t)(N / L), rpb = msc_count_rows(L, nrows);
  const unsigned blocks = msc_count_parts(L, N);
  if (d == 3)
    hipLaunchKernelGGL(k_msc_count<3>, dim3(blocks), dim3(256), 0, stream, S, J, L, N, nrows, rpb, part);
  else
    hipLaunchKernelGGL(k_msc_count<2>, dim3(blocks), dim3(256), 0, stream, S, J, L, N, nrows, rpb, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_msc_finalize, dim3(1), dim3(1024), 0, stream, part, blocks, (int64_t)d * (int64_t)N, (int64_t)N,
                     E, M);
  return hipGetLastError();
}

}  // namespace spin

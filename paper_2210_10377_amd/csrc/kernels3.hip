// Kernels of the three-dimensional (D3Q27) path: the fused pull-stream + BGK step with
// the per-step forces (A, B, DRTT terms, SI), the control-volume momentum sweep, and the
// fixed-order reductions of the force partials into ring rows.
//
// One launch per step (two where the strips with force terms have their own).  A block of 256
// threads covers a tile of 256 nodes along x in one (y, z) row; each wave a 64-node strip whose
// class (strip table) picks its path:
//   plain / box-J: 27 loads at fixed offsets (no boundary within reach), collision,
//     27 non-temporal stores; box-J strips add the momentum of their pulled populations;
//   general: the node word and the coordinates select, per direction, plain streaming,
//     a periodic wrap, bounce-back (wall, body, outlet ghost of a solid node), the inlet
//     moving-wall rule or the outlet ghost copy; strips with force terms accumulate A, B,
//     J, Phi and SI in FP64 and reduce them over the wave into their slot.
// Large grids are bound by HBM (1280 x 128 x 64 in binary32: 5.8 TB/s), small ones by the
// latency of a strip with force terms: 64 x 32 x 32 took 30 us a step, 22 of them in that
// strip's launch, while it branched on every direction of the pull and of the link terms and
// summed over lanes through LDS; without branches (selects by bit masks, walls and wrapped
// rows scalar), with lane sums by register swaps and rotations, and in the step's own launch
// it takes 12.
// The first block of a launch reduces the previous step's slots, in a fixed order, into
// that step's ring row.  Blocks are mapped to tiles so that runs of kXcdRun (8)
// neighbouring tiles along x go to one XCD (their +-1-shifted pulls share cache lines in
// that L2).
#include <hip/hip_runtime.h>

#include "device.h"
#include "kernels.h"
#include "kernels3.h"
#include "lbm.h"
#include "plan3.h"

namespace lbm3 {
namespace {

constexpr int kThreads = kTileW;

template <int P>
struct St3;
// kDev: arithmetic in deviation form; kStoreF: the stored value is f_i itself (else a
// deviation storage stores h_i = f_i - w_i); kSR: stores round stochastically.
template <>
struct St3<LBM_FP64> {
  using T = double;
  using C = double;
  static constexpr bool kDev = false, kStoreF = true, kSR = false;
};
template <>
struct St3<LBM_FP32> {
  using T = float;
  using C = float;
  static constexpr bool kDev = false, kStoreF = true, kSR = false;
};
template <>
struct St3<LBM_FP32DEV> {
  using T = float;
  using C = float;
  static constexpr bool kDev = true, kStoreF = false, kSR = false;
};
template <>
struct St3<LBM_FP16DEV> {
  using T = _Float16;
  using C = float;
  static constexpr bool kDev = true, kStoreF = false, kSR = false;
};
// Binary32 populations, arithmetic in deviation form from the binary32 weights, stores
// rounded stochastically.
template <>
struct St3<LBM_FP32SR> {
  using T = float;
  using C = float;
  static constexpr bool kDev = true, kStoreF = true, kSR = true;
};

// Weights: (2/3, 1/6, 1/6) per axis.
template <class C>
__device__ __forceinline__ constexpr C w27(int i) {
  return (kCx[i] == 0 ? C(2) / C(3) : C(1) / C(6)) * (kCy[i] == 0 ? C(2) / C(3) : C(1) / C(6)) *
         (kCz[i] == 0 ? C(2) / C(3) : C(1) / C(6));
}

// w_i x with the weight carried beyond binary32 precision: the binary32 weights are not
// exact, and an equilibrium formed with them alone would hold slightly more (or less)
// mass and momentum than its node; every collision would add that bias (relative ~1e-8
// per step, ~1e-4 in the forces over 10^4 steps).  The product with the binary32
// remainder of the weight is added first, so one rounding remains and no bias.
template <class C>
__device__ __forceinline__ C wmul27(int i, C x) {
  if constexpr (sizeof(C) == 8) {
    return w27<C>(i) * x;
  } else {
    const float lo = float(w27<double>(i) - double(w27<float>(i)));
    return __builtin_fmaf(w27<float>(i), x, lo * x);
  }
}

// Stored value of direction i -> f_i in binary64.
template <int P>
__device__ __forceinline__ double f64(typename St3<P>::T v, int i) {
  return (St3<P>::kDev && !St3<P>::kStoreF) ? w27<double>(i) + double(v) : double(v);
}

// Stored value of direction i -> arithmetic value, and back (rounded to nearest).  With
// f_i stored in binary32 and deviation arithmetic, the deviation is taken from the
// binary32 weight, h_i = f_i - fl(w_i), exactly for f_i within a factor of two of
// fl(w_i).  The binary32 weights are fl(8/27) scaled by powers of 4, so each is
// (1 + eps) w_i with one eps; the equilibrium deviation w_i (sum h + rho poly_i) with the
// exact weights then equals f^eq_i - fl(w_i) but for terms of order eps poly_i.
template <int P>
__device__ __forceinline__ typename St3<P>::C unpack3(typename St3<P>::T v, int i) {
  using S = St3<P>;
  if constexpr (S::kDev && S::kStoreF)
    return v - w27<float>(i);
  else
    return typename S::C(v);
}
template <int P>
__device__ __forceinline__ typename St3<P>::T pack3(typename St3<P>::C v, int i) {
  using S = St3<P>;
  if constexpr (S::kDev && S::kStoreF)
    return w27<float>(i) + v;
  else
    return typename S::T(v);
}
// f_i in binary64 from an arithmetic value of direction i.
template <int P>
__device__ __forceinline__ double pre64(typename St3<P>::C v, int i) {
  using S = St3<P>;
  if constexpr (!S::kDev)
    return double(v);
  else if constexpr (S::kStoreF)
    return double(w27<float>(i)) + double(v);
  else
    return w27<double>(i) + double(v);
}

// Stochastic rounding of f_i = fl(w_i) + h_i to binary32 (as in two dimensions): the
// neighbour on the side of the exact TwoSum error is taken with probability |error| /
// spacing, from the top 24 bits of the node's word + i * 0x9e3779b9; the node's word is
// fmix32 of the step key and the node index.  Round to nearest when kSR is off.
template <int P>
__device__ __forceinline__ typename St3<P>::T pack3_sr(typename St3<P>::C v, int i,
                                                       uint32_t word) {
  using S = St3<P>;
  if constexpr (S::kSR) {
    const float a = w27<float>(i);
    const float y = a + v;
    const float bb = y - a;
    const float e = (a - (y - bb)) + (v - bb);
    const uint32_t yb = __builtin_bit_cast(uint32_t, y);
    const uint32_t nb = yb + 1u - (((__builtin_bit_cast(uint32_t, e) ^ yb) >> 30) & 2u);
    const float yn = __builtin_bit_cast(float, nb);
    const float gap = __builtin_fabsf(yn - y);
    const float u = float((word + uint32_t(i) * 0x9e3779b9u) >> 8) * 0x1p-24f;
    return (u * gap < __builtin_fabsf(e)) ? yn : y;
  } else {
    return pack3<P>(v, i);
  }
}
__device__ __forceinline__ uint32_t sr_word3(uint32_t step_key, int64_t node) {
  return lbm::fmix32(step_key ^ uint32_t(node));
}

template <class T>
__device__ __forceinline__ void st_nt(T* p, T v) {
  __builtin_nontemporal_store(v, p);
}

// Collision of one node, in place, f or deviations h = f - w: BGK (Eq. CollideAdv), or
// with COLL = LBM_COLL_REGULARIZED the non-equilibrium part replaced by its projection
// w_i / (2 theta0^2) Q_i : Pi^neq on the second-order Hermite polynomials
// (Q_i = c_i c_i - theta0 I) and relaxed: f~ = f^eq + (1 - omega) f^(1).
template <class C, bool DEV, int COLL>
__device__ __forceinline__ void collide27(C (&f)[kQ], C omega) {
  C r = C(0), jx = C(0), jy = C(0), jz = C(0);
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    r += f[i];
    if (kCx[i]) jx += kCx[i] > 0 ? f[i] : -f[i];
    if (kCy[i]) jy += kCy[i] > 0 ? f[i] : -f[i];
    if (kCz[i]) jz += kCz[i] > 0 ? f[i] : -f[i];
  }
  const C rho = DEV ? C(1) + r : r;
  const C inv = C(1) / rho;
  const C ux = jx * inv, uy = jy * inv, uz = jz * inv;
  const C usq = C(1.5) * (ux * ux + uy * uy + uz * uz);
  if (COLL == LBM_COLL_REGULARIZED) {
    C pxx = C(0), pyy = C(0), pzz = C(0), pxy = C(0), pxz = C(0), pyz = C(0);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const C cu = C(kCx[i]) * ux + C(kCy[i]) * uy + C(kCz[i]) * uz;
      const C poly = C(3) * cu + C(4.5) * cu * cu - usq;
      const C feq = DEV ? wmul27<C>(i, r + rho * poly) : wmul27<C>(i, rho * (C(1) + poly));
      const C d = f[i] - feq;
      if (kCx[i]) pxx += d;
      if (kCy[i]) pyy += d;
      if (kCz[i]) pzz += d;
      if (kCx[i] * kCy[i]) pxy += kCx[i] * kCy[i] > 0 ? d : -d;
      if (kCx[i] * kCz[i]) pxz += kCx[i] * kCz[i] > 0 ? d : -d;
      if (kCy[i] * kCz[i]) pyz += kCy[i] * kCz[i] > 0 ? d : -d;
      f[i] = feq;
    }
    const C tr = (pxx + pyy + pzz) / C(3);
    const C k1 = (C(1) - omega) * C(4.5);
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const C q = C(kCx[i] * kCx[i]) * pxx + C(kCy[i] * kCy[i]) * pyy +
                  C(kCz[i] * kCz[i]) * pzz +
                  C(2) * (C(kCx[i] * kCy[i]) * pxy + C(kCx[i] * kCz[i]) * pxz +
                          C(kCy[i] * kCz[i]) * pyz) - tr;
      f[i] += k1 * w27<C>(i) * q;
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < kQ; ++i) {
    const C cu = C(kCx[i]) * ux + C(kCy[i]) * uy + C(kCz[i]) * uz;
    const C poly = C(3) * cu + C(4.5) * cu * cu - usq;
    const C feq = DEV ? wmul27<C>(i, r + rho * poly) : wmul27<C>(i, rho * (C(1) + poly));
    f[i] += omega * (feq - f[i]);
  }
}

__device__ __forceinline__ int wrapc(int s, int n) { return s < 0 ? s + n : (s >= n ? s - n : s); }

__device__ __forceinline__ bool in_range(const Geom3& g, int axis, int at) {
  return g.whole[axis] || (at >= g.box[2 * axis] && at < g.box[2 * axis + 1]);
}
__device__ __forceinline__ bool in_box(const Geom3& g, int x, int y, int z) {
  return in_range(g, 0, x) && in_range(g, 1, y) && in_range(g, 2, z);
}

// Bits of the directions whose component in c is v.
constexpr uint32_t dirs(const int (&c)[kQ], int v) {
  uint32_t m = 0;
  for (int i = 1; i < kQ; ++i)
    if (c[i] == v) m |= 1u << i;
  return m;
}
constexpr uint32_t kAllDirs = ((1u << kQ) - 1u) & ~1u;
// The same set of directions, each replaced by its opposite.
__device__ __forceinline__ uint32_t opposite(uint32_t m) {
  constexpr uint32_t kOdd = 0x2aaaaaau & kAllDirs;
  return ((m & kOdd) << 1) | ((m >> 1) & kOdd);
}

// Moving-wall term of the population pulled in direction i across a body link at node
// (x, y, z): 2 rho_w w_i (c_i . u_w) / theta0 with u_w the rigid-body velocity at the
// half-way point x - c_i / 2.
__device__ __forceinline__ double body_wall_term3(const Geom3& g, int i, int x, int y, int z) {
  const double r0 = x - 0.5 * kCx[i] - g.mc[0], r1 = y - 0.5 * kCy[i] - g.mc[1],
               r2 = z - 0.5 * kCz[i] - g.mc[2];
  const double u0 = g.mu[0] + g.mw[1] * r2 - g.mw[2] * r1;
  const double u1 = g.mu[1] + g.mw[2] * r0 - g.mw[0] * r2;
  const double u2 = g.mu[2] + g.mw[0] * r1 - g.mw[1] * r0;
  return g.rho_w6 * w27<double>(i) * (kCx[i] * u0 + kCy[i] * u1 + kCz[i] * u2);
}

// Pull of all 27 populations of a fluid node through the boundary rules; *links: bit d
// set for a body link in direction d.  MOV: the body links carry the moving-wall term.
// The row (y, z) is the wave's, so walls and wrapped rows are scalar; what differs by lane
// are the directions (bit masks) that read direction opp(i) of the node itself: bounce-back
// (wall, body, outlet ghost of a solid node) and the inlet's moving-wall rule.
template <int P, bool MOV>
__device__ __forceinline__ void pull27(const Geom3& g, const typename St3<P>::T* __restrict__ src,
                                       int x, int y, int z, uint32_t w,
                                       typename St3<P>::C (&f)[kQ], uint32_t* links) {
  using C = typename St3<P>::C;
  using T = typename St3<P>::T;
  const bool px = g.bc_x == LBM_BCX_PERIODIC, py = g.bc_y == LBM_BCY_PERIODIC,
             pz = g.bc_z == LBM_BCY_PERIODIC;
  const uint32_t wall = (!py && y == 0 ? dirs(kCy, 1) : 0u) |
                        (!py && y == g.ny - 1 ? dirs(kCy, -1) : 0u) |
                        (!pz && z == 0 ? dirs(kCz, 1) : 0u) |
                        (!pz && z == g.nz - 1 ? dirs(kCz, -1) : 0u);
  const uint32_t left = !px && x == 0 ? dirs(kCx, 1) : 0u;
  const uint32_t right = !px && x == g.nx - 1 ? dirs(kCx, -1) : 0u;
  const uint32_t solid = w & kAllDirs & ~wall;
  const uint32_t back = wall | solid | left;
  const uint32_t inl = left & ~(wall | solid);
  const uint32_t body = solid & ~(left | right);
  // Columns and rows of the sources (the outlet ghost copies plane nx - 1; a row past a wall
  // is not read).
  const int xs[3] = {x + 1 < g.nx ? x + 1 : (px ? 0 : x), x, x > 0 ? x - 1 : (px ? g.nx - 1 : 0)};
  const int ys[3] = {y + 1 < g.ny ? y + 1 : (py ? 0 : y), y, y > 0 ? y - 1 : (py ? g.ny - 1 : 0)};
  const int zs[3] = {z + 1 < g.nz ? z + 1 : (pz ? 0 : z), z, z > 0 ? z - 1 : (pz ? g.nz - 1 : 0)};
  const T* own = src + int64_t(z * g.ny + y) * g.rstride;
  T v[kQ];
  v[0] = own[x];
#pragma unroll
  for (int i = 1; i < kQ; ++i) {
    // Either source by a bit mask over the address (a choice of pointers compiles to a branch).
    const T* from = src + int64_t(i) * g.dstride +
                    int64_t(zs[kCz[i] + 1] * g.ny + ys[kCy[i] + 1]) * g.rstride;
    const int64_t turn = own + int64_t(opp(i)) * g.dstride - from;
    const int32_t m = int32_t(back << (31 - i)) >> 31;
    const int xc = xs[kCx[i] + 1];
    v[i] = from[(turn & int64_t(m)) + (xc + ((x - xc) & m))];
  }
#pragma unroll
  for (int i = 0; i < kQ; ++i) f[i] = unpack3<P>(v[i], i);  // w_opp(i) = w_i
  if (MOV && body) {
#pragma unroll
    for (int i = 1; i < kQ; ++i)
      if ((body >> i) & 1u) f[i] += C(body_wall_term3(g, i, x, y, z));
  }
  if (inl) {
    const double u = g.rho_w6 * g.uin[z * g.ny + y];
#pragma unroll
    for (int i = 1; i < kQ; ++i)
      if (kCx[i] && ((inl >> i) & 1u)) f[i] += C(u * (w27<double>(i) * kCx[i]));
  }
  *links = opposite(body);
}

// Sums of four values over the wave (in the order of a butterfly over the lane distances 32,
// 16, .., 1), component sum4_at() of them in each lane.
__device__ __forceinline__ double sum4(double a, double b, double c, double d) {
  using namespace lbm::dev;
  return row_sum(fold16(fold32(a, b), fold32(c, d)));
}
__device__ __forceinline__ int sum4_at() {
  const int row = (int(threadIdx.x) >> 4) & 3;
  return (row & 1) << 1 | row >> 1;
}

// Sum N doubles over the block in a fixed order; thread k < N gets total k in out[k].
template <int N>
__device__ __forceinline__ void block_sum(double (&v)[N], double* out) {
  __shared__ double red[kThreads / 64][N];
#pragma unroll
  for (int k = 0; k < N; ++k)
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v[k] += __shfl_xor(v[k], off, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < N; ++k) red[wave][k] = v[k];
  __syncthreads();
  if (threadIdx.x < N) {
    double s = red[0][threadIdx.x];
#pragma unroll
    for (int wv = 1; wv < kThreads / 64; ++wv) s += red[wv][threadIdx.x];
    out[threadIdx.x] = s;
  }
  __syncthreads();
}

// Previous step's partials -> ring row (15 values), its J -> J(t+1) of the row before;
// with jpart, the J of the next pull -> this row's J(t+1).  Thread t sums component
// t % 16 of slots t / 16, t / 16 + 16, ... (coalesced, one accumulator), then the 16
// partial sums of each component are added in a fixed order.
__device__ void reduce_row(const double* __restrict__ in, int nslots, int njslots, double* row,
                           double* prev_jnext, const double* __restrict__ jpart, int njblocks) {
  __shared__ double red[16][16];
  const int t = threadIdx.x, c = t & 15, g = t >> 4;
  // Loads in flight together (their latency is what the reduction of a few hundred slots
  // costs), added in slot order.
  constexpr int kU = 24;
  auto slots = [&](const double* p, int n, int stride, int at, double acc) {
    for (int s0 = g; s0 < n; s0 += 16 * kU) {
      double v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int s = s0 + 16 * u;
        v[u] = s < n ? p[int64_t(s) * stride + at] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) acc += v[u];
    }
    return acc;
  };
  double acc = 0.0;
  if (c < kPart) acc = slots(in, nslots, kPart, c, acc);
  if (c >= 6 && c < 9) acc = slots(in + int64_t(nslots) * kPart, njslots, 3, c - 6, acc);
  red[g][c] = acc;
  __syncthreads();
  if (t < kPart) {
    double v = 0.0;
    for (int k = 0; k < 16; ++k) v += red[k][t];
    row[t] = v;
    if (prev_jnext && t >= 6 && t < 9) prev_jnext[t - 6] = v;
  }
  if (jpart) {
    __syncthreads();
    double j = 0.0;
    if (c < 3)
      for (int b = g; b < njblocks; b += 16) j += jpart[int64_t(b) * 3 + c];
    red[g][c] = j;
    __syncthreads();
    if (t < 3) {
      double v = 0.0;
      for (int k = 0; k < 16; ++k) v += red[k][t];
      row[kPart + t] = v;
    }
  }
}

// Tile of block b: runs of kXcdRun consecutive tiles per XCD (blocks go to the 8 XCDs
// round-robin).
#ifndef LBM3_XCD_RUN
#define LBM3_XCD_RUN 8
#endif
constexpr int64_t kXcdRun = LBM3_XCD_RUN;
__device__ __forceinline__ int64_t tile_of(int64_t b) {
  const int64_t xcd = b & 7, k = b >> 3;
  return ((k / kXcdRun) * 8 + xcd) * kXcdRun + (k % kXcdRun);
}

// General path of one strip: the boundary-aware pull of every node, collision, store,
// and with FTERMS the force terms reduced over the wave into the strip's slot.
template <int P, bool FTERMS, int COLL, bool MOV>
__device__ __forceinline__ void general_strip(const Step3Args& a, uint32_t e, int64_t row, int x,
                                              int y, int z, int lane) {
  using S = St3<P>;
  using T = typename S::T;
  using C = typename S::C;
  const Geom3& g = a.g;
  const int64_t self = row * g.rstride + x;
  const T* __restrict__ src = static_cast<const T*>(a.src);
  T* __restrict__ dst = static_cast<T*>(a.dst);
  const C omega = C(a.omega);
  C f[kQ];
  const bool valid = x < g.nx;
  const uint32_t w = valid ? g.word[row * g.nx + x] : kSolid;
  const bool fluid = !(w & kSolid);
  constexpr bool fterms = FTERMS;
  // Force terms go through two fixed-order wave reductions (before and after the
  // collision), so that few of them are live across it.  Pre: A's lost momentum (0-2),
  // J (3-5), SI (6-8).  Post: A's returned momentum (0-2), B (3-5), Phi (6-8).
  double pre[9], post[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) pre[k] = post[k] = 0.0;
  uint32_t lk = 0;
  bool inV = false;
  if (fluid) {
    pull27<P, MOV>(g, src, x, y, z, w, f, &lk);
    if (fterms) {
      inV = g.has_box && in_box(g, x, y, z);
      if (inV)
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          const double v = pre64<P>(f[i], i);
          if (kCx[i]) pre[3] += kCx[i] * v;
          if (kCy[i]) pre[4] += kCy[i] * v;
          if (kCz[i]) pre[5] += kCz[i] * v;
        }
      if (lk) {
#pragma unroll
        for (int d = 1; d < kQ; ++d) {
          const double v = (lk >> d) & 1u ? pre64<P>(f[d], d) : 0.0;
          if (kCx[d]) pre[0] += kCx[d] * v;
          if (kCy[d]) pre[1] += kCy[d] * v;
          if (kCz[d]) pre[2] += kCz[d] * v;
        }
        // SI over the axis links of this node: (sigma - p I) . sum n, n = -c_d.
        if (lk & 0x7eu) {
          double rho = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
          for (int i = 0; i < kQ; ++i) {
            const double v = pre64<P>(f[i], i);
            rho += v;
            jx += kCx[i] * v;
            jy += kCy[i] * v;
            jz += kCz[i] * v;
          }
          const double ux = jx / rho, uy = jy / rho, uz = jz / rho;
          const double usq = ux * ux + uy * uy + uz * uz;
          double pxx = 0, pyy = 0, pzz = 0, pxy = 0, pxz = 0, pyz = 0;
#pragma unroll
          for (int i = 0; i < kQ; ++i) {
            const double v = pre64<P>(f[i], i);
            const double cu = kCx[i] * ux + kCy[i] * uy + kCz[i] * uz;
            const double neq =
                v - w27<double>(i) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq);
            pxx += kCx[i] * kCx[i] * neq;
            pyy += kCy[i] * kCy[i] * neq;
            pzz += kCz[i] * kCz[i] * neq;
            pxy += kCx[i] * kCy[i] * neq;
            pxz += kCx[i] * kCz[i] * neq;
            pyz += kCy[i] * kCz[i] * neq;
          }
          const double k = -(1.0 - 0.5 * a.omega), p = rho / 3.0;
          double nx = 0.0, ny = 0.0, nz = 0.0;
#pragma unroll
          for (int d = 1; d <= 6; ++d)
            if ((lk >> d) & 1u) {
              nx -= kCx[d];
              ny -= kCy[d];
              nz -= kCz[d];
            }
          pre[6] += (k * pxx - p) * nx + k * pxy * ny + k * pxz * nz;
          pre[7] += k * pxy * nx + (k * pyy - p) * ny + k * pyz * nz;
          pre[8] += k * pxz * nx + k * pyz * ny + (k * pzz - p) * nz;
        }
      }
    }
  }
  // Total 4 k + sum4_at() of the pre-collision terms.
  double before[3] = {};
  if (fterms) {
    before[0] = sum4(pre[0], pre[1], pre[2], pre[3]);
    before[1] = sum4(pre[4], pre[5], pre[6], pre[7]);
    before[2] = sum4(pre[8], 0.0, 0.0, 0.0);
  }
  if (fluid) {
    collide27<C, S::kDev, COLL>(f, omega);
    const uint32_t word = S::kSR ? sr_word3(a.step_key, row * g.nx + x) : 0u;
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const T q = pack3_sr<P>(f[i], i, word);
      st_nt(dst + int64_t(i) * g.dstride + self, q);
      f[i] = unpack3<P>(q, i);  // forces read the populations as stored
    }
    if (fterms) {
      if (lk) {
        // The population returned along link d at t+1 is f~_d plus, for a moving body,
        // the moving-wall term of the pull of opp(d) (half-way point x + c_d / 2).
#pragma unroll
        for (int d = 1; d < kQ; ++d) {
          const bool on = (lk >> d) & 1u;
          const double v = on ? pre64<P>(f[d], d) : 0.0;
          double back = v;
          if (MOV) back = on ? v + body_wall_term3(g, opp(d), x, y, z) : 0.0;
          if (kCx[d]) {
            post[0] += kCx[d] * back;
            post[3] += kCx[d] * (v + back);
          }
          if (kCy[d]) {
            post[1] += kCy[d] * back;
            post[4] += kCy[d] * (v + back);
          }
          if (kCz[d]) {
            post[2] += kCz[d] * back;
            post[5] += kCz[d] * (v + back);
          }
        }
      }
      if (g.has_box) {
        // Surface flux: populations leaving V (node inside) or entering it (outside).
        bool near = true;
        if (!g.whole[0]) near = near && x >= g.box[0] - 1 && x <= g.box[1];
        if (!g.whole[1]) near = near && y >= g.box[2] - 1 && y <= g.box[3];
        if (!g.whole[2]) near = near && z >= g.box[4] - 1 && z <= g.box[5];
        if (near) {
          // Whether the neighbours' columns and rows lie in V.
          bool ix[3], iy[3], iz[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const int tx = x + c - 1, ty = y + c - 1, tz = z + c - 1;
            ix[c] = in_range(g, 0, g.bc_x == LBM_BCX_PERIODIC ? wrapc(tx, g.nx) : tx);
            iy[c] = in_range(g, 1, g.bc_y == LBM_BCY_PERIODIC ? wrapc(ty, g.ny) : ty);
            iz[c] = in_range(g, 2, g.bc_z == LBM_BCY_PERIODIC ? wrapc(tz, g.nz) : tz);
          }
          const double out = inV ? -1.0 : 1.0;
#pragma unroll
          for (int d = 1; d < kQ; ++d) {
            const bool in = ix[kCx[d] + 1] && (iy[kCy[d] + 1] && iz[kCz[d] + 1]);
            const double v = in != inV ? pre64<P>(f[d], d) * out : 0.0;
            if (kCx[d]) post[6] += kCx[d] * v;
            if (kCy[d]) post[7] += kCy[d] * v;
            if (kCz[d]) post[8] += kCz[d] * v;
          }
        }
      }
    }
  }
  if (fterms) {
    const double after[3] = {sum4(post[0], post[1], post[2], post[3]),
                             sum4(post[4], post[5], post[6], post[7]),
                             sum4(post[8], 0.0, 0.0, 0.0)};
    // Slot layout FA(3) FB(3) J(3) Phi(3) SI(3).  Columns 0-2 of each row of 16 lanes take the
    // terms before the collision (with A = lost + returned), columns 3-5 those after it.
    const int col = lane & 15, c = sum4_at();
    const bool first = col < 3;
    const int part = first ? col : col - 3, k = 4 * part + c;
    double v = first ? (part == 0 ? before[0] : (part == 1 ? before[1] : before[2]))
                     : (part == 0 ? after[0] : (part == 1 ? after[1] : after[2]));
    if (col == 0 && c < 3) v = before[0] + after[0];
    const int at = first ? (k < 3 ? k : (k < 6 ? k + 3 : k + 6)) : (k < 6 ? k : k + 3);
    if (col < 6 && k < 9 && (first || k >= 3))
      a.part_out[int64_t(strip_slot(e)) * kPart + at] = v;
  }
}

// Strip of a force slot (one wave per slot, in slot order): the general path with A, B, J, Phi
// and SI.
template <int P, int COLL, bool MOV>
__device__ __forceinline__ void force_strip(const Step3Args& a, int64_t slot, int lane) {
  if (slot >= a.nslots) return;
  const uint32_t si = a.fstrips[slot];
  const int64_t tile = si / kStrips, row = tile / a.ntx;
  const int x = int(tile % a.ntx) * kTileW + int(si % kStrips) * kStripW + lane;
  general_strip<P, true, COLL, MOV>(a, a.strip[si], row, x, int(row % a.g.ny), int(row / a.g.ny),
                                    lane);
}

template <int P, int COLL, bool MOV>
__global__ __launch_bounds__(kThreads) void force3_kernel(Step3Args a) {
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  force_strip<P, COLL, MOV>(a, int64_t(blockIdx.x) * kStrips + wave, threadIdx.x & 63);
}

// Where the strips with force terms run: nowhere apart (no forces), in a launch of their own,
// or in the step's, which gives it their registers (140 against 46 - 80).
enum Forces3 { kNoForces, kApart, kJoined };

template <int P, int FORCES, int COLL, bool MOV>
__global__ __launch_bounds__(kThreads) void step3_kernel(Step3Args a) {
  using S = St3<P>;
  using T = typename S::T;
  using C = typename S::C;
  // With a reducer, blocks 0-7 (one per XCD) come first: block 0 reduces while the
  // tiles stream, and the tile blocks keep their XCD alignment.
  int64_t b = blockIdx.x;
  if (a.red_in) {
    if (b == 0)
      reduce_row(a.red_in, a.nslots, a.njslots, a.red_row, a.red_prev_jnext, nullptr, 0);
    if (b < 8) return;
    b -= 8;
  }
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = threadIdx.x & 63;
  if (FORCES == kJoined) {
    // Then the strips with force terms, which take longest.
    if (b < a.force_blocks) {
      force_strip<P, COLL, MOV>(a, b * kStrips + wave, lane);
      return;
    }
    b -= a.force_blocks;
  }
  const int64_t tile = tile_of(b);
  if (tile >= a.ntiles) return;
  const uint32_t e = a.strip[tile * kStrips + wave];
  if (e == kStripEmpty) return;
  const Geom3& g = a.g;
  const int tx = int(tile % a.ntx);
  const int64_t row = tile / a.ntx;
  const int y = int(row % g.ny), z = int(row / g.ny);
  const int x = tx * kTileW + wave * kStripW + lane;
  const int64_t self = row * g.rstride + x;
  const T* __restrict__ src = static_cast<const T*>(a.src);
  T* __restrict__ dst = static_cast<T*>(a.dst);
  const uint32_t cls = strip_class(e);
  const C omega = C(a.omega);
  C f[kQ];

  if (cls == kPlain || cls == kBoxJ) {
    // No boundary within reach: every source is the neighbour itself.
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      f[i] = unpack3<P>(src[int64_t(i) * g.dstride + self -
                             (int64_t(kCz[i]) * g.ny + kCy[i]) * g.rstride - kCx[i]], i);
    if (FORCES && cls == kBoxJ) {
      double j[3] = {0.0, 0.0, 0.0};
      if (P == LBM_FP16DEV) {
        // sum c_i w_i = 0, so the node's momentum is that of its deviations; binary16
        // deviations are summed in binary32 (the rounding stays far below theirs),
        // and the nodes in FP64.
        float jf[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          if (kCx[i]) jf[0] += kCx[i] > 0 ? float(f[i]) : -float(f[i]);
          if (kCy[i]) jf[1] += kCy[i] > 0 ? float(f[i]) : -float(f[i]);
          if (kCz[i]) jf[2] += kCz[i] > 0 ? float(f[i]) : -float(f[i]);
        }
        j[0] = jf[0];
        j[1] = jf[1];
        j[2] = jf[2];
      } else {
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          const double v = pre64<P>(f[i], i);
          if (kCx[i]) j[0] += kCx[i] * v;
          if (kCy[i]) j[1] += kCy[i] * v;
          if (kCz[i]) j[2] += kCz[i] * v;
        }
      }
      const double v = sum4(j[0], j[1], j[2], 0.0);
      const int k = sum4_at();
      if ((lane & 15) == 0 && k < 3)
        a.part_out[int64_t(a.nslots) * kPart + int64_t(strip_slot(e)) * 3 + k] = v;
    }
    collide27<C, S::kDev, COLL>(f, omega);
    const uint32_t word = S::kSR ? sr_word3(a.step_key, row * g.nx + x) : 0u;
#pragma unroll
    for (int i = 0; i < kQ; ++i) st_nt(dst + int64_t(i) * g.dstride + self, pack3_sr<P>(f[i], i, word));
    return;
  }
  // With forces, the strips with force terms have blocks of their own; they hold every body
  // link, so the edge strips left here need no moving-wall term then.
  if (FORCES && cls == kForce) return;
  general_strip<P, false, COLL, FORCES ? false : MOV>(a, e, row, x, y, z, lane);
}

// J of the pull of the state src over V, per block of 256 nodes along x in a box row.
template <int P, bool MOV>
__global__ __launch_bounds__(kThreads) void box3_kernel(Box3Args a) {
  using S = St3<P>;
  using T = typename S::T;
  using C = typename S::C;
  const Geom3& g = a.g;
  const int bw = g.box[1] - g.box[0];
  const int nbx = (bw + kThreads - 1) / kThreads;
  const int64_t r = blockIdx.x / nbx;
  const int bx = int(blockIdx.x % nbx);
  const int by = g.box[3] - g.box[2];
  const int y = g.box[2] + int(r % by), z = g.box[4] + int(r / by);
  const int x = g.box[0] + bx * kThreads + threadIdx.x;
  double j[3] = {0.0, 0.0, 0.0};
  if (x < g.box[1]) {
    const int64_t row = int64_t(z) * g.ny + y;
    const uint32_t w = g.word[row * g.nx + x];
    if (!(w & kSolid)) {
      C f[kQ];
      uint32_t lk;
      pull27<P, MOV>(g, static_cast<const T*>(a.src), x, y, z, w, f, &lk);
#pragma unroll
      for (int i = 1; i < kQ; ++i) {
        const double v = pre64<P>(f[i], i);
        if (kCx[i]) j[0] += kCx[i] * v;
        if (kCy[i]) j[1] += kCy[i] * v;
        if (kCz[i]) j[2] += kCz[i] * v;
      }
    }
  }
  __shared__ double out[3];
  block_sum<3>(j, out);
  if (threadIdx.x < 3) a.jpart[int64_t(blockIdx.x) * 3 + threadIdx.x] = out[threadIdx.x];
}

__global__ __launch_bounds__(kThreads) void final3_kernel(Final3Args a) {
  reduce_row(a.red_in, a.nslots, a.njslots, a.row, a.prev_jnext, a.jpart, a.njblocks);
}

// Mask change: one thread per listed node.  A covered node contributes its momentum; an
// uncovered one is refilled with f^eq(rho, u_w) (rho the mean density of its lattice
// neighbours fluid in both masks, periodic axes wrapping, rho_w when none; u_w the
// rigid-body velocity at the node) and contributes minus what it now stores.  Refills
// read valid neighbours only, so no thread reads what another writes.
template <int P>
__global__ __launch_bounds__(kThreads) void remask3_kernel(Remask3Args a) {
  using S = St3<P>;
  using T = typename S::T;
  using C = typename S::C;
  const Geom3& g = a.g;
  T* st = static_cast<T*>(a.state);
  double v[3] = {0.0, 0.0, 0.0};
  for (int64_t k = int64_t(blockIdx.x) * kThreads + threadIdx.x; k < a.n;
       k += int64_t(gridDim.x) * kThreads) {
    const uint32_t e = uint32_t(a.list[k]);
    const int32_t node = int32_t(e & 0x7fffffffu);
    const int x = node % g.nx, y = (node / g.nx) % g.ny, z = node / (g.nx * g.ny);
    const int64_t at = (int64_t(z) * g.ny + y) * g.rstride + x;
    if (!(e >> 31)) {
      for (int i = 0; i < kQ; ++i) {
        const double f = f64<P>(st[i * g.dstride + at], i);
        v[0] += kCx[i] * f;
        v[1] += kCy[i] * f;
        v[2] += kCz[i] * f;
      }
      continue;
    }
    double rsum = 0.0;
    int cnt = 0;
    for (int i = 1; i < kQ; ++i) {
      int ax = x + kCx[i], ay = y + kCy[i], az = z + kCz[i];
      if (g.bc_x == LBM_BCX_PERIODIC) ax = wrapc(ax, g.nx);
      if (g.bc_y == LBM_BCY_PERIODIC) ay = wrapc(ay, g.ny);
      if (g.bc_z == LBM_BCY_PERIODIC) az = wrapc(az, g.nz);
      if (ax < 0 || ax >= g.nx || ay < 0 || ay >= g.ny || az < 0 || az >= g.nz) continue;
      if (!a.valid[(int64_t(az) * g.ny + ay) * g.nx + ax]) continue;
      const int64_t nb = (int64_t(az) * g.ny + ay) * g.rstride + ax;
      double r = 0.0;
      for (int j = 0; j < kQ; ++j) r += f64<P>(st[j * g.dstride + nb], j);
      rsum += r;
      ++cnt;
    }
    const double rho = cnt > 0 ? rsum / double(cnt) : a.rho_w;
    const double r0 = x - g.mc[0], r1 = y - g.mc[1], r2 = z - g.mc[2];
    const double u0 = g.mu[0] + g.mw[1] * r2 - g.mw[2] * r1;
    const double u1 = g.mu[1] + g.mw[2] * r0 - g.mw[0] * r2;
    const double u2 = g.mu[2] + g.mw[0] * r1 - g.mw[1] * r0;
    const double uu = u0 * u0 + u1 * u1 + u2 * u2;
    for (int i = 0; i < kQ; ++i) {
      const double cu = kCx[i] * u0 + kCy[i] * u1 + kCz[i] * u2;
      const double feq = w27<double>(i) * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * uu);
      const T q = S::kStoreF ? T(feq) : T(C(feq - w27<double>(i)));
      st[i * g.dstride + at] = q;
      const double f = f64<P>(q, i);
      v[0] -= kCx[i] * f;
      v[1] -= kCy[i] * f;
      v[2] -= kCz[i] * f;
    }
  }
  __shared__ double out[3];
  block_sum<3>(v, out);
  if (threadIdx.x < 3) a.block_out[3 * int64_t(blockIdx.x) + threadIdx.x] = out[threadIdx.x];
}

// Sum of the per-block momenta in a fixed order (one block).
__global__ __launch_bounds__(kThreads) void remask3_sum_kernel(const double* block_out, int nb,
                                                               double* res) {
  double v[3] = {0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nb; b += kThreads)
    for (int k = 0; k < 3; ++k) v[k] += block_out[3 * int64_t(b) + k];
  __shared__ double out[3];
  block_sum<3>(v, out);
  if (threadIdx.x < 3) res[threadIdx.x] = out[threadIdx.x];
}

template <int P>
__global__ __launch_bounds__(kThreads) void fill_rest3_kernel(void* buf, int64_t n,
                                                                int64_t dstride) {
  using S = St3<P>;
  using T = typename S::T;
  T* p = static_cast<T*>(buf);
  // Both layouts repeat the 27 directions every 27 * dstride elements.
  const int64_t period = dstride * kQ;
  for (int64_t k = int64_t(blockIdx.x) * kThreads + threadIdx.x; k < n;
       k += int64_t(gridDim.x) * kThreads) {
    const int i = int((k % period) / dstride);
    // The stochastically rounded storage's rest state is its reference weights.
    p[k] = (S::kDev && !S::kStoreF) ? T(0)
                                    : (S::kDev ? T(w27<float>(i)) : T(w27<double>(i)));
  }
}

template <int P, int COLL, bool MOV>
hipError_t step_pcm(bool forces, Step3Args a, hipStream_t s) {
  const int64_t tiles = (a.ntiles + 8 * kXcdRun - 1) / (8 * kXcdRun) * (8 * kXcdRun);
  // Whole rounds over the XCDs, so that the tile blocks keep their alignment.
  const int force_blocks = (a.nslots + kStrips * 8 - 1) / (kStrips * 8) * 8;
  const bool joined = forces && a.joined;
  a.force_blocks = joined ? force_blocks : 0;
  const dim3 grid(unsigned(tiles + a.force_blocks + (a.red_in ? 8 : 0)));
  if (joined) {
    hipLaunchKernelGGL((step3_kernel<P, kJoined, COLL, MOV>), grid, dim3(kThreads), 0, s, a);
  } else if (forces) {
    hipLaunchKernelGGL((step3_kernel<P, kApart, COLL, MOV>), grid, dim3(kThreads), 0, s, a);
    if (a.nslots > 0) {
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL((force3_kernel<P, COLL, MOV>), dim3(force_blocks), dim3(kThreads), 0, s, a);
    }
  } else {
    hipLaunchKernelGGL((step3_kernel<P, kNoForces, COLL, MOV>), grid, dim3(kThreads), 0, s, a);
  }
  return hipGetLastError();
}

// Bodies in motion take their own instantiation, so the resting case keeps its
// registers.
template <int P, int COLL>
hipError_t step_pc(bool forces, const Step3Args& a, hipStream_t s) {
  return a.g.moving ? step_pcm<P, COLL, true>(forces, a, s)
                    : step_pcm<P, COLL, false>(forces, a, s);
}

template <int P>
hipError_t step_p(bool forces, const Step3Args& a, hipStream_t s) {
  return a.collision == LBM_COLL_REGULARIZED ? step_pc<P, LBM_COLL_REGULARIZED>(forces, a, s)
                                             : step_pc<P, LBM_COLL_BGK>(forces, a, s);
}

}  // namespace

hipError_t launch_step3(int precision, bool forces, const Step3Args& a, hipStream_t s) {
  switch (precision) {
    case LBM_FP64: return step_p<LBM_FP64>(forces, a, s);
    case LBM_FP32: return step_p<LBM_FP32>(forces, a, s);
    case LBM_FP32DEV: return step_p<LBM_FP32DEV>(forces, a, s);
    case LBM_FP32SR: return step_p<LBM_FP32SR>(forces, a, s);
    case LBM_FP16DEV: return step_p<LBM_FP16DEV>(forces, a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int P>
void box_p(const Box3Args& a, int blocks, hipStream_t s) {
  if (a.g.moving)
    hipLaunchKernelGGL((box3_kernel<P, true>), dim3(blocks), dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((box3_kernel<P, false>), dim3(blocks), dim3(kThreads), 0, s, a);
}

hipError_t launch_box3(int precision, const Box3Args& a, int blocks, hipStream_t s) {
  switch (precision) {
    case LBM_FP64: box_p<LBM_FP64>(a, blocks, s); break;
    case LBM_FP32: box_p<LBM_FP32>(a, blocks, s); break;
    case LBM_FP32DEV: box_p<LBM_FP32DEV>(a, blocks, s); break;
    case LBM_FP32SR: box_p<LBM_FP32SR>(a, blocks, s); break;
    case LBM_FP16DEV: box_p<LBM_FP16DEV>(a, blocks, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_final3(const Final3Args& a, hipStream_t s) {
  hipLaunchKernelGGL(final3_kernel, dim3(1), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_remask3(int precision, const Remask3Args& a, int blocks, double* out,
                          hipStream_t s) {
  switch (precision) {
    case LBM_FP64:
      hipLaunchKernelGGL(remask3_kernel<LBM_FP64>, dim3(blocks), dim3(kThreads), 0, s, a);
      break;
    case LBM_FP32:
      hipLaunchKernelGGL(remask3_kernel<LBM_FP32>, dim3(blocks), dim3(kThreads), 0, s, a);
      break;
    case LBM_FP32DEV:
      hipLaunchKernelGGL(remask3_kernel<LBM_FP32DEV>, dim3(blocks), dim3(kThreads), 0, s, a);
      break;
    case LBM_FP32SR:
      hipLaunchKernelGGL(remask3_kernel<LBM_FP32SR>, dim3(blocks), dim3(kThreads), 0, s, a);
      break;
    case LBM_FP16DEV:
      hipLaunchKernelGGL(remask3_kernel<LBM_FP16DEV>, dim3(blocks), dim3(kThreads), 0, s, a);
      break;
    default:
      return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(remask3_sum_kernel, dim3(1), dim3(kThreads), 0, s,
                     static_cast<const double*>(a.block_out), blocks, out);
  return hipGetLastError();
}

hipError_t launch_fill_rest3(int precision, void* buf, int64_t n, int64_t dstride, hipStream_t s) {
  const int blocks = 2048;
  switch (precision) {
    case LBM_FP64:
      hipLaunchKernelGGL(fill_rest3_kernel<LBM_FP64>, dim3(blocks), dim3(kThreads), 0, s, buf, n,
                         dstride);
      break;
    case LBM_FP32:
      hipLaunchKernelGGL(fill_rest3_kernel<LBM_FP32>, dim3(blocks), dim3(kThreads), 0, s, buf, n,
                         dstride);
      break;
    case LBM_FP32DEV:
      hipLaunchKernelGGL(fill_rest3_kernel<LBM_FP32DEV>, dim3(blocks), dim3(kThreads), 0, s, buf, n,
                         dstride);
      break;
    case LBM_FP32SR:
      hipLaunchKernelGGL(fill_rest3_kernel<LBM_FP32SR>, dim3(blocks), dim3(kThreads), 0, s, buf, n,
                         dstride);
      break;
    case LBM_FP16DEV:
      hipLaunchKernelGGL(fill_rest3_kernel<LBM_FP16DEV>, dim3(blocks), dim3(kThreads), 0, s, buf, n,
                         dstride);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lbm3

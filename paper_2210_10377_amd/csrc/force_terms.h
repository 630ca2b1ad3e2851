// Device building blocks shared by the step kernels: collision and rounding of a node, the
// force terms of one node under each estimator, and the fixed-order reduction of a step's
// partials.
#pragma once

#include "device.h"

namespace lbm {
namespace dev {

// Collision of arithmetic values f; s: the values to store.
template <int P, int COLL>
__device__ __forceinline__ void collide_pack(const StepArgs& a,
                                             const typename Storage<P>::C (&f)[kQ], uint32_t key,
                                             int x, int y, typename Storage<P>::T (&s)[kQ]) {
  using S = Storage<P>;
  using C = typename S::C;
  C g[kQ];
  collide<C, S::kDev, COLL, S::kExactW, sizeof(typename S::T) == 2>(f, C(a.omega), g);
  const uint32_t word = S::kSR ? sr_node_word(key, a.nx, x, y) : 0u;
#pragma unroll
  for (int i = 0; i < kQ; ++i) s[i] = pack_sr<P>(g[i], i, word);
}

// Force slot of the strip of row y that starts at column x0 (negative: none).
__device__ __forceinline__ int slot_of(const StepArgs& a, int x0, int y) {
  const int at = a.tile_rows == 1
                     ? y * (a.ntx * kStrips) + x0 / kStripW
                     : ((y >> 2) * a.ntx + x0 / kStripW) * kStrips + (y & 3);
  return a.strip_slot[at];
}

// Barrier of the block that orders LDS accesses only: loads and stores of global memory that
// are under way are not waited for (no wave reads what another one of the launch stores).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// acc += c v for a lattice velocity component c.
__device__ __forceinline__ void add_signed(int c, double v, double& acc) {
  if (c > 0) acc += v;
  if (c < 0) acc -= v;
}

// Control-volume terms of fluid node (x, y) (second Eq. rtt7) added to acc: the
// momentum of its populations before collision (f) and as stored after it (s) when it
// lies in the control volume, and the stored populations crossing the box surface:
// entering V (+) from a node outside, leaving V (-) from a node inside.
template <int P>
__device__ __forceinline__ void box_terms(const StepArgs& a, int x, int y,
                                          const typename Storage<P>::C (&f)[kQ],
                                          const typename Storage<P>::T (&s)[kQ],
                                          double (&acc)[kPart]) {
  using S = Storage<P>;
  // Memberships of the three columns and rows around the node.
  const bool cx[3] = {x - 1 >= a.bx0 && x - 1 < a.bx1, x >= a.bx0 && x < a.bx1,
                      x + 1 >= a.bx0 && x + 1 < a.bx1};
  const bool cy[3] = {y - 1 >= a.by0 && y - 1 < a.by1, y >= a.by0 && y < a.by1,
                      y + 1 >= a.by0 && y + 1 < a.by1};
  const bool in = cx[1] && cy[1];
  if (in) {
    double jx = 0.0, jy = 0.0, px = 0.0, py = 0.0;
#pragma unroll
    for (int i = 1; i < kQ; ++i) {
      const double fi = pre_f64<P>(f[i], i), sv = to_f64<P>(s[i], i);
      add_signed(kCx[i], fi, jx);
      add_signed(kCy[i], fi, jy);
      add_signed(kCx[i], sv, px);
      add_signed(kCy[i], sv, py);
    }
    acc[4] += jx;
    acc[5] += jy;
    acc[kJpost] += px;
    acc[kJpost + 1] += py;
  }
  // Only nodes beside the surface have a link across it.
  const bool all = cx[0] && cx[1] && cx[2] && cy[0] && cy[1] && cy[2];
  const bool any = (cx[0] || cx[1] || cx[2]) && (cy[0] || cy[1] || cy[2]);
  if (any && !all) {
#pragma unroll
    for (int i = 1; i < kQ; ++i)
      if ((cx[1 + kCx[i]] && cy[1 + kCy[i]]) != in) {
        const double sv = to_f64<P>(s[i], i), out = in ? -sv : sv;
        add_signed(kCx[i], out, acc[6]);
        add_signed(kCy[i], out, acc[7]);
      }
  }
}

// Momentum exchange of fluid node (x, y) with pull codes w, from its populations before
// collision (f) and as stored (s), added to acc.
template <int P, bool MOV>
__device__ __forceinline__ void link_terms(const StepArgs& a, uint32_t w, int x, int y,
                                           const typename Storage<P>::C (&f)[kQ],
                                           const typename Storage<P>::T (&s)[kQ],
                                           double (&acc)[kPart]) {
  // Momentum exchange on the links of this node (Sec. III; Eq. rtt4): the
  // population leaving along c_i towards the body is f_i before collision (A) or
  // f~_i after it (B); the body returns f~_i (as stored) along -c_i, less the
  // moving-wall term of that return when the body moves.
  const uint32_t body = body_dirs(w);
  if (body == 0) return;
#pragma unroll
  for (int i = 1; i < kQ; ++i) {
    if (!has_dir(body, kOpp[i])) continue;
    const double sv = to_f64<P>(s[i], i);
    const double back =
        (MOV && a.motion) ? sv + body_wall_term(*a.motion, a.rho_w6, kOpp[i], x, y) : sv;
    const double fa = pre_f64<P>(f[i], i) + back;
    add_signed(kCx[i], fa, acc[0]);
    add_signed(kCy[i], fa, acc[1]);
    add_signed(kCx[i], sv + back, acc[2]);
    add_signed(kCy[i], sv + back, acc[3]);
  }
}

// Stress integral of a fluid node with pull codes w, from its populations before collision.
template <int P>
__device__ __forceinline__ void stress_terms(const StepArgs& a, uint32_t w,
                                             const typename Storage<P>::C (&f)[kQ],
                                             double (&acc)[kPart]) {
  // Stress integration (Sec. III, Eq. stress_int): each axis link of this node is a
  // unit face of the staircase surface with normal -c_i out of the body; the
  // traction (-p I + sigma) . n uses p = rho/3 and sigma = -(1 - omega/2) Pi^neq of
  // the pre-collision populations (Pi^neq = sum c c f - rho u u - rho I/3), in
  // binary64.  Faces are linear in n, so the node adds the traction of their sum.
  const uint32_t body = body_dirs(w);
  int nsx = 0, nsy = 0;
#pragma unroll
  for (int i = 1; i <= 4; ++i)
    if (has_dir(body, kOpp[i])) {
      nsx -= kCx[i];
      nsy -= kCy[i];
    }
  if (nsx != 0 || nsy != 0) {
    double fd[kQ];
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      fd[i] = pre_f64<P>(f[i], i);
    const double rho = ((fd[0] + fd[1]) + (fd[2] + fd[3])) + ((fd[4] + fd[5]) + (fd[6] + fd[7])) + fd[8];
    const double ux = ((fd[1] + fd[5] + fd[8]) - (fd[3] + fd[6] + fd[7])) / rho;
    const double uy = ((fd[2] + fd[5] + fd[6]) - (fd[4] + fd[7] + fd[8])) / rho;
    const double diag = (fd[5] + fd[6]) + (fd[7] + fd[8]);
    const double p = rho * (1.0 / 3.0);
    const double visc = -(1.0 - 0.5 * a.omega);
    const double sxx = visc * (((fd[1] + fd[3]) + diag) - rho * ux * ux - p);
    const double syy = visc * (((fd[2] + fd[4]) + diag) - rho * uy * uy - p);
    const double sxy = visc * (((fd[5] + fd[7]) - (fd[6] + fd[8])) - rho * ux * uy);
    acc[8] += (sxx - p) * nsx + sxy * nsy;
    acc[9] += sxy * nsx + (syy - p) * nsy;
  }
}

// Force row of the previous step from its partial slots (fixed order).
__device__ __forceinline__ void reduce_row(const double* red_in, int nslots, int njslots,
                                           double* row, double* prev_jnext) {
  // General strips, and the box momenta of the box-interior strips (J before and after
  // collision, added to the two J sums; two waves share the last sums).
  __shared__ Partials<kPart> general;
  __shared__ Partials<kBoxPart> interior;
  __shared__ double ji[kBoxPart];
  general.gather(red_in, nslots);
  if (njslots > 0) interior.gather(red_in + int64_t(nslots) * kPart, njslots);
  __syncthreads();
  const int tid = int(threadIdx.x);
  double t = 0.0;
  if (tid < kPart) t = general.sum(tid);
  if (tid >= 64 && tid < 64 + kBoxPart) ji[tid - 64] = njslots > 0 ? interior.sum(tid - 64) : 0.0;
  __syncthreads();
  if (tid < kPart) {
    const bool pre = tid == 4 || tid == 5, post = tid == kJpost || tid == kJpost + 1;
    if (pre) t += ji[tid - 4];
    if (post) t += ji[tid - kJpost + 2];
    row[tid] = t;
    if (prev_jnext && pre) prev_jnext[tid - 4] = t;
  }
}

}  // namespace dev
}  // namespace lbm

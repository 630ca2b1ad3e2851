// The fused kernel: kFuse (3) time steps of the two-dimensional lattice in one launch.
//
// A single step reads and writes every population once, and on large grids that bounds it (72 B
// per node and step in binary32 at 6.1 TB/s).  Here a wave marches a window of columns down the
// rows of a chunk and keeps the intermediate states of the window in registers: row r of
// step 1 is pulled from memory, row r - 1 of step 2 from the rows r - 2 .. r of step 1, row
// r - 2 of step 3 likewise, and only step 3 is stored.  A population that streams along y
// waits in a register for its row; one that streams along x comes from the neighbouring lane
// (a rotation of the wavefront by one lane).  In the plain rectangles nothing is exchanged
// between waves and no LDS is used.  A third of the bytes per step remains, and vector
// arithmetic (about 115 instructions per node and step in binary32, and a fifth more on margins)
// comes to bound it together with HBM.  Measured at 8192 x 4096 in binary32, all forces: 396 us a
// step by single steps, fused 173 in a run of 2000 steps (194 GLUPS), 191 in one of 12, and 222 in
// one of 20, of which two are single steps (each run ends with a sweep over the control volume);
// 2.92 GB counted per launch of 541 us, 5.4 TB/s, where three single steps move 7.25; 2048 x 1024
// in binary64 52 and 29 us.
//
// The windows of the plain rectangles own 56 of their 64 lanes, 8 bytes of columns a lane, so
// that every store covers whole 64-byte sectors.  That decides: windows of 60 binary32 columns
// (which waste less) left 32-byte pieces of sectors to two waves and took 197 - 260 us where
// whole sectors take 164 - 177.  Units of 8 to 64 rows measure alike on large grids (shorter ones
// spend more on margins, longer ones keep more rows of memory open).
//
// Every node's arithmetic is that of step_kernel on the same inputs, so states are bitwise
// those of kFuse single steps, and the state buffers change roles as often (kFuse is odd).  In
// the body rectangle a wave owns half a strip of step_kernel's, and the force terms of the two
// halves meet in LDS, from where they are summed in the order of wave_sum_store: forces are
// bitwise those of single steps, too.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.h"
#include "force_terms.h"
#include "kernels.h"
#include "plan.h"

namespace lbm {

namespace {

using namespace dev;

constexpr int kM = kFuseM;

// Value of the lane whose column is x - CX (the source of a direction with c_x = CX).
template <int CX, class T>
__device__ __forceinline__ T from_source(T v) {
  if constexpr (CX == 0) {
    return v;
  } else {
    // Wavefront rotation by one lane: right (lane l takes l - 1) or left.
    constexpr int kCtrl = CX > 0 ? 0x13c : 0x134;
    if constexpr (sizeof(T) == 8) {
      const u32x2 b = __builtin_bit_cast(u32x2, v);
      u32x2 r;
      r.x = unsigned(__builtin_amdgcn_update_dpp(0, int(b.x), kCtrl, 0xf, 0xf, true));
      r.y = unsigned(__builtin_amdgcn_update_dpp(0, int(b.y), kCtrl, 0xf, 0xf, true));
      return __builtin_bit_cast(T, r);
    } else if constexpr (sizeof(T) == 4) {
      return __builtin_bit_cast(
          T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kCtrl, 0xf, 0xf, true));
    } else {
      const int b = __builtin_bit_cast(unsigned short, v);
      const int r = __builtin_amdgcn_update_dpp(0, b, kCtrl, 0xf, 0xf, true);
      return __builtin_bit_cast(T, static_cast<unsigned short>(r));
    }
  }
}

// The stored populations of one step around the row that the next step pulls: that row, the
// directions with c_y = +1 (2, 5, 6) of the row before it; the directions with c_y = -1 come
// from the row after it, just computed.
template <class T>
struct Rows {
  T cur[kQ];
  T up[3];
  __device__ __forceinline__ void advance(const T (&next)[kQ]) {
    up[0] = cur[2];
    up[1] = cur[5];
    up[2] = cur[6];
#pragma unroll
    for (int i = 0; i < kQ; ++i) cur[i] = next[i];
  }
  // Population of direction i at its source row.
  __device__ __forceinline__ T at_source_row(int i, const T (&next)[kQ]) const {
    return kCy[i] == 0 ? cur[i] : (kCy[i] > 0 ? up[i == 2 ? 0 : i - 4] : next[i]);
  }
};

template <int I, class T>
__device__ __forceinline__ void pull_dirs(const Rows<T>& R, const T (&next)[kQ], T (&v)[kQ]) {
  if constexpr (I < kQ) {
    v[I] = from_source<kCx[I]>(R.at_source_row(I, next));
    pull_dirs<I + 1>(R, next, v);
  }
}

// Pull through the boundary rules of the code word w from the rows in registers (pull_all's
// rules: bounce-back takes the opposite direction of the node itself, the outlet ghost
// the node's own column).
template <class T>
__device__ __forceinline__ void pull_coded(const Rows<T>& R, const T (&next)[kQ], uint32_t w,
                                           T (&v)[kQ]) {
  pull_dirs<0>(R, next, v);
  const uint32_t bd = back_dirs(w), od = outlet_dirs(w);
#pragma unroll
  for (int i = 1; i < kQ; ++i) {
    if (kCx[i] < 0 && has_dir(od, i)) v[i] = R.at_source_row(i, next);
    if (has_dir(bd, i)) v[i] = R.cur[kOpp[i]];
  }
}

// What a lane of a plain window keeps of a stored population: the value itself, or for
// binary16 its binary32 equal, which the next step needs.
template <int P>
struct Kept {
  using T = typename Storage<P>::T;
  static constexpr bool kWide = sizeof(T) == 2;
  using K = std::conditional_t<kWide, float, T>;
  static constexpr int kN = 8 / int(sizeof(T));  // columns of a lane
  typedef K Lane[kN];
  static __device__ __forceinline__ typename Storage<P>::C open(K v, int i) {
    if constexpr (kWide)
      return v;
    else
      return unpack<P>(v, i);
  }
};

// The columns of a lane (of kN) moved by one: those that a direction with c_x = CX streams to
// this lane's columns.
template <int CX, class K, int N>
__device__ __forceinline__ void from_source(const K (&in)[N], K (&out)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if constexpr (CX == 0)
      out[k] = in[k];
    else if constexpr (CX > 0)
      out[k] = k > 0 ? in[k > 0 ? k - 1 : 0] : from_source<1>(in[N - 1]);
    else
      out[k] = k + 1 < N ? in[k + 1 < N ? k + 1 : 0] : from_source<-1>(in[0]);
  }
}

template <int I, class K, int N>
__device__ __forceinline__ void pull_row(const K (&in)[kQ][N], K (&v)[kQ][N]) {
  if constexpr (I < kQ) {
    from_source<kCx[I]>(in[I], v[I]);
    pull_row<I + 1>(in, v);
  }
}

// Rows of a plain window (as Rows, kN columns a lane).
template <int P>
struct LaneRows {
  typename Kept<P>::Lane cur[kQ], up[3];
  template <int I>
  __device__ __forceinline__ void pull(const typename Kept<P>::Lane (&next)[kQ],
                                       typename Kept<P>::Lane (&v)[kQ]) const {
    if constexpr (I < kQ) {
      if constexpr (kCy[I] == 0)
        from_source<kCx[I]>(cur[I], v[I]);
      else if constexpr (kCy[I] > 0)
        from_source<kCx[I]>(up[I == 2 ? 0 : I - 4], v[I]);
      else
        from_source<kCx[I]>(next[I], v[I]);
      pull<I + 1>(next, v);
    }
  }
  __device__ __forceinline__ void advance(const typename Kept<P>::Lane (&next)[kQ]) {
#pragma unroll
    for (int k = 0; k < Kept<P>::kN; ++k) {
      up[0][k] = cur[2][k];
      up[1][k] = cur[5][k];
      up[2][k] = cur[6][k];
#pragma unroll
      for (int i = 0; i < kQ; ++i) cur[i][k] = next[i][k];
    }
  }
};

// Window whose pulls, margins included, are all plain streaming: no codes are read.  Lane l
// holds 8 bytes of columns, X being the first of lane 4; lanes 4 .. 59 own theirs.  The loads
// of a row are issued one row ahead.
template <int P, int COLL>
__device__ __forceinline__ void march_plain(const StepArgs& a, const FuseStep& q, int X, int xe,
                                            int ya, int h) {
  using S = Storage<P>;
  using T = typename S::T;
  using C = typename S::C;
  using KP = Kept<P>;
  constexpr int kN = KP::kN;
  using Lane = typename KP::Lane;
  struct Raw {
    T t[kN];
  };
  constexpr int kLeft = (64 - kFuseLanes) / 2;
  const int lane = int(threadIdx.x) & 63;
  const int x = X + (lane - kLeft) * kN;
  const Planes<T, true> src(a.src, a.plane, a.buf_bytes);
  const Planes<T, true> dst(a.dst, a.plane, a.buf_bytes);
  const uint32_t row_bytes = uint32_t(a.pitch) * uint32_t(sizeof(T));
  const uint32_t plane_bytes = src.plane_bytes;
  const uint32_t at = uint32_t(x) * uint32_t(sizeof(T));
  // Lanes that own no column store past the buffer's end, where stores are dropped.
  const uint32_t to =
      lane >= kLeft && lane < kLeft + kFuseLanes && x < xe ? at : 0xffffff00u;
  const int last = ya + h + kM - 1;
  // The source columns are loaded where they lie; binary16 ones (which are not aligned to
  // four bytes there) as the lane's own columns, and moved between lanes.
  auto load = [&](int y, u32x2 (&v)[kQ]) {
#pragma unroll
    for (int i = 0; i < kQ; ++i)
      v[i] = __builtin_amdgcn_raw_buffer_load_b64(
          src.r, at - uint32_t(KP::kWide ? 0 : kCx[i] * int(sizeof(T))),
          uint32_t(y - kCy[i]) * row_bytes + uint32_t(i) * plane_bytes, 0);
  };
  // One step of the lane's columns of row y from raw populations v.
  auto step = [&](const Lane(&v)[kQ], uint32_t key, int y, T (&s)[kQ][kN]) {
#pragma unroll
    for (int k = 0; k < kN; ++k) {
      C f[kQ];
      T t[kQ];
#pragma unroll
      for (int i = 0; i < kQ; ++i) f[i] = KP::open(v[i][k], i);
      collide_pack<P, COLL>(a, f, key, x + k, y, t);
#pragma unroll
      for (int i = 0; i < kQ; ++i) s[i][k] = t[i];
    }
  };
  auto keep = [&](const T (&s)[kQ][kN], Lane (&v)[kQ]) {
#pragma unroll
    for (int i = 0; i < kQ; ++i)
#pragma unroll
      for (int k = 0; k < kN; ++k) v[i][k] = typename KP::K(s[i][k]);
  };
  LaneRows<P> r1{}, r2{};
  u32x2 ahead[kQ];
  // Steps 1, 2, .. N of rows y, y - 1, ..
  auto row = [&](auto N, int y) __attribute__((always_inline)) {
    Lane v[kQ], n1[kQ];
    T s[kQ][kN];
#pragma unroll
    for (int i = 0; i < kQ; ++i) {
      const Raw w = __builtin_bit_cast(Raw, ahead[i]);
#pragma unroll
      for (int k = 0; k < kN; ++k) n1[i][k] = typename KP::K(w.t[k]);
    }
    load(min(y + 1, last), ahead);
    if constexpr (KP::kWide)
      pull_row<0>(n1, v);
    else
#pragma unroll
      for (int i = 0; i < kQ; ++i)
#pragma unroll
        for (int k = 0; k < kN; ++k) v[i][k] = n1[i][k];
    step(v, q.step_key[0], y, s);
    keep(s, n1);
    if constexpr (N.value >= 2) {
      Lane n2[kQ];
      r1.template pull<0>(n1, v);
      step(v, q.step_key[1], y - 1, s);
      keep(s, n2);
      if constexpr (N.value >= 3) {
        r2.template pull<0>(n2, v);
        step(v, q.step_key[2], y - 2, s);
        const uint32_t row = uint32_t(y - 2) * row_bytes;
#pragma unroll
        for (int i = 0; i < kQ; ++i) {
          Raw w;
#pragma unroll
          for (int k = 0; k < kN; ++k) w.t[k] = s[i][k];
          __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, w), dst.r, to,
                                                row + uint32_t(i) * plane_bytes, 2);
        }
      }
      r2.advance(n2);
    }
    r1.advance(n1);
  };
  // The rows of the margin are peeled off, so that in the loop the wait for a row's loads
  // need not wait for the stores issued after them.
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 2> two{};
  constexpr std::integral_constant<int, 3> three{};
  load(ya - 2, ahead);
  row(one, ya - 2);
  row(one, ya - 1);
  row(two, ya);
  row(two, ya + 1);
  for (int y = ya + kM; y <= last; ++y) row(three, y);
}

// The strip of a pair of waves in the body rectangle, and its chunk.
struct Pair {
  int x0, ya, yb;  // strip's first column, rows [ya, yb) (empty for an idle pair)
};

// Force exchange of the two halves of a strip (turn, pair, sending half, component, lane): each
// half sends the other one half of its components.
constexpr int kSend = kPart / 2;
typedef double Exchange[2][kStrips / 2][2][kSend][kHalf];

// Sum N (even) components of a strip over its two halves and its lanes and store them (the
// order of wave_sum_store: lane l + 32 onto lane l first, then 16, 8, 4, 2, 1).
template <int N>
__device__ __forceinline__ void strip_sum_store(const double* mine, const double (*other)[kHalf],
                                                double* out) {
  const int lane = int(threadIdx.x) & 63, l = lane & (kHalf - 1), col = lane & 15;
  double t = 0.0;
#pragma unroll
  for (int k = 0; k < N; k += 2) {
    const double s = row_sum(fold16(mine[k] + other[k][l], mine[k + 1] + other[k + 1][l]));
    t = col == k / 2 ? s : t;
  }
  if (lane < kHalf && col < N / 2) out[2 * col + (lane >> 4)] = t;
}

// Window with boundary rules: the edges of the grid (codes from coordinates, no forces), or
// BODY: half a strip of the body rectangle (codes and force slots from the plan).  Every
// wave of a BODY block runs the same number of rows and meets at the same barriers.  What a
// row needs besides its populations is read two rows ahead, its populations one row ahead.
// Lane columns are xv, `owned` those that the window stores; its columns with margins are
// [X - kM, X + own + kM) where own > 0 (a window of both sides of the grid has own = 0: it has
// no row that streams plainly).
template <int P, bool FORCES, int COLL, bool MOV, bool BODY>
__device__ __forceinline__ void march_coded(const StepArgs& a, const FuseStep& q, int X, int own,
                                            int xv, bool owned, int ya, int yb, int rows,
                                            const Pair (&pairs)[kStrips / 2], int pair, int half,
                                            Exchange& ex) {
  using S = Storage<P>;
  using T = typename S::T;
  using C = typename S::C;
  constexpr bool kForces = FORCES && BODY;
  const int lane = int(threadIdx.x) & 63;
  const bool periodic_x = a.bc_x == LBM_BCX_PERIODIC, periodic_y = a.bc_y == LBM_BCY_PERIODIC;
  // Column of the lane (xv): wrapped, or clamped past a bounded edge (such a lane is never read).
  int x = periodic_x ? xv % a.nx : min(max(xv, 0), a.nx - 1);
  if (x < 0) x += a.nx;
  const bool at_inlet = !periodic_x && X - kM <= 0;
  const Planes<T, true> src(a.src, a.plane, a.buf_bytes);
  const Planes<T, true> dst(a.dst, a.plane, a.buf_bytes);
  int turn = 0;

  auto wrapped = [&](int yy) { return yy < 0 ? yy + a.ny : (yy >= a.ny ? yy - a.ny : yy); };
  // Rows that this window needs (its own and the margin's).
  auto needed = [&](int yy) {
    return yy >= ya - kM && yy < yb + kM && (periodic_y || (yy >= 0 && yy < a.ny)) &&
           !(BODY && own <= 0);
  };
  // Does every pull of row y that this window needs stream plainly?
  auto plain_row = [&](int y) {
    return own > 0 && y > 0 && y + 1 < a.ny && X - kM > 0 && X + own + kM < a.nx &&
           !(BODY && y >= a.gy0 && y <= a.gy1 && X - kM <= a.gx1 && X + own + kM - 1 >= a.gx0);
  };
  struct Row {
    uint32_t w;    // code words (0 in a plain row)
    double u;      // inlet velocity
    int slot[2];   // force slots of the block's two strips at this point of their marches
    bool box;      // this wave's strip is a box-interior one
  };
  auto fetch = [&](int yy) {
    Row r{0u, 0.0, {-1, -1}, false};
    if (needed(yy)) {
      const int y = wrapped(yy);
      if (!plain_row(y)) {
        if constexpr (BODY)
          r.w = a.node[int64_t(y) * a.nx + x];
        else
          r.w = edge_word_bits(a.nx, a.ny, a.bc_x, a.bc_y, x, y);
        if (at_inlet) r.u = a.uin[y];
      }
    }
    if constexpr (kForces)
#pragma unroll
      for (int p = 0; p < kStrips / 2; ++p) {
        const int py = pairs[p].ya + (yy - ya);
        if (py >= pairs[p].ya && py < pairs[p].yb) r.slot[p] = slot_of(a, pairs[p].x0, py);
        if (p == pair)
          r.box = strip_class(a.nx, a.ny, a.gx0, a.gx1, a.gy0, a.gy1, a.bx0, a.bx1, a.by0, a.by1,
                              X - half * kHalf, py) == kStripBoxInterior;
      }
    return r;
  };
  // The populations that row yy pulls from memory.
  auto load = [&](int yy, const Row& r, T (&v)[kQ]) {
    if (!needed(yy)) return;
    const int y = wrapped(yy);
    if (plain_row(y)) {
      const int32_t o = y * a.pitch + xv;
#pragma unroll
      for (int i = 0; i < kQ; ++i) v[i] = src.ld(i, o - kCy[i] * a.pitch - kCx[i]);
    } else {
      pull_raw<P>(src, a.pitch, a.nx, a.ny, r.w, x, y, v);
    }
  };
  // Step j + 1 of row yy from its pulled populations v: collision, the stores of the last
  // step, and the force terms.
  auto step = [&](int j, int yy, const Row& r, const T (&v)[kQ], T (&s)[kQ]) {
    C f[kQ] = {};
    bool mine = false;
    int y = 0;
    if (needed(yy)) {
      y = wrapped(yy);
      if (at_inlet || MOV) {
        finish_pull<P>(v, r.u, a.rho_w6, r.w, x, y, f, MOV ? a.motion : nullptr);
      } else {
#pragma unroll
        for (int i = 0; i < kQ; ++i) f[i] = unpack<P>(v[i], i);
      }
      collide_pack<P, COLL>(a, f, q.step_key[j], x, y, s);
      mine = owned && yy >= ya && yy < yb && !(r.w & kSolidBit);
      if (j == kM && mine) {
        const int32_t o = y * a.pitch + x;
#pragma unroll
        for (int i = 0; i < kQ; ++i) dst.st(i, o, s[i]);
      }
    }
    if constexpr (kForces) {
      if (r.slot[0] < 0 && r.slot[1] < 0) return;
      const int slot = pair == 0 ? r.slot[0] : r.slot[1];
      const bool box = slot >= 0 && r.box;
      double acc[kPart] = {};
      if (slot >= 0 && mine) {
        if (box) {
#pragma unroll
          for (int i = 1; i < kQ; ++i) {
            const double fi = to_f64<P>(v[i], i), si = to_f64<P>(s[i], i);
            add_signed(kCx[i], fi, acc[0]);
            add_signed(kCy[i], fi, acc[1]);
            add_signed(kCx[i], si, acc[kSend]);
            add_signed(kCy[i], si, acc[kSend + 1]);
          }
        } else {
          link_terms<P, MOV>(a, r.w, x, y, f, s, acc);
          box_terms<P>(a, x, y, f, s, acc);
          stress_terms<P>(a, r.w, f, acc);
        }
      }
      // Half 0 sums the first components (box-interior: J before collision), half 1 the rest.
      auto send = [&](auto H) {
        double(*out)[kHalf] = ex[turn][pair][H.value];
#pragma unroll
        for (int k = 0; k < kSend; ++k)
          if (k < kBoxPart / 2 || !box) out[k][lane] = acc[(1 - H.value) * kSend + k];
      };
      auto sum = [&](auto H) {
        const double(*in)[kHalf] = ex[turn][pair][1 - H.value];
        const double* mine = acc + H.value * kSend;
        double* part = q.part_out + j * q.part_stride;
        if (box)
          strip_sum_store<kBoxPart / 2>(mine, in, part + int64_t(a.nslots) * kPart +
                                                      int64_t(slot) * kBoxPart +
                                                      H.value * (kBoxPart / 2));
        else
          strip_sum_store<kSend>(mine, in, part + int64_t(slot) * kPart + H.value * kSend);
      };
      constexpr std::integral_constant<int, 0> lower{};
      constexpr std::integral_constant<int, 1> upper{};
      if (slot >= 0 && lane < kHalf) {
        if (half == 0)
          send(lower);
        else
          send(upper);
      }
      lds_barrier();
      if (slot >= 0) {
        if (half == 0)
          sum(lower);
        else
          sum(upper);
      }
      turn ^= 1;  // the other boxes next: these are read until the next barrier
    }
  };

  Rows<T> r1{}, r2{};
  const int first = ya - kM;
  Row now = fetch(first), next = fetch(first + 1), last1{}, last2{};
  last1.slot[0] = last1.slot[1] = last2.slot[0] = last2.slot[1] = -1;
  T v[kQ] = {}, ahead[kQ] = {};
  load(first, now, v);
  const int steps = rows + 2 * kM;
  for (int it = 0; it < steps; ++it) {
    const int yy = first + it;
    const Row after = fetch(yy + 2);
    load(yy + 1, next, ahead);
    T s1[kQ] = {}, s2[kQ] = {};
    step(0, yy, now, v, s1);
    if (it >= 2) {
      if (needed(yy - 1)) {
        if (plain_row(wrapped(yy - 1)))
          pull_dirs<0>(r1, s1, v);
        else
          pull_coded(r1, s1, last1.w, v);
      }
      step(1, yy - 1, last1, v, s2);
      if (it >= 4) {
        T s3[kQ];
        if (needed(yy - 2)) {
          if (plain_row(wrapped(yy - 2)))
            pull_dirs<0>(r2, s2, v);
          else
            pull_coded(r2, s2, last2.w, v);
        }
        step(2, yy - 2, last2, v, s3);
      }
      r2.advance(s2);
    }
    r1.advance(s1);
    last2 = last1;
    last1 = now;
    now = next;
    next = after;
#pragma unroll
    for (int i = 0; i < kQ; ++i) v[i] = ahead[i];
  }
}

// Neighbouring blocks on one XCD, which share the lines their windows overlap in (runs of 1, 4
// and 35 measured alike to 2 %).
constexpr int kFuseGroup = 4;

// Block b of a lattice's work map.
template <int P, bool FORCES, int COLL, bool MOV>
__device__ __forceinline__ void fused_block(const StepArgs& a, const FuseMap& m, const FuseStep& q,
                                            int b, Exchange& ex) {
  const int lane = int(threadIdx.x) & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  int k = m.nrects - 1;
  while (k > 0 && b < m.r[k].first) --k;
  const FuseRect r = m.r[k];
  Pair pairs[kStrips / 2] = {};
  if (r.kind == kFuseBody) {
    const int pair = wave >> 1, half = wave & 1;
#pragma unroll
    for (int p = 0; p < kStrips / 2; ++p) {
      const int unit = (b - r.first) * (kStrips / 2) + p, chunk = unit / r.nw;
      const int ya = min(r.y0 + chunk * r.rows, r.y1);
      pairs[p] = {r.x0 / kStripW * kStripW + (unit - chunk * r.nw) * kStripW, ya,
                  min(ya + r.rows, r.y1)};
    }
    const Pair me = pair == 0 ? pairs[0] : pairs[1];
    const int X = me.x0 + half * kHalf;
    const int own = X >= r.x0 ? min(max(r.x1 - X, 0), kHalf) : 0;
    march_coded<P, FORCES, COLL, MOV, true>(a, q, X, own,
                                            X + lane - (lane < 64 - kHalf / 2 ? 0 : 64), lane < own,
                                            me.ya, me.yb, r.rows, pairs, pair, half, ex);
    return;
  }
  const int unit = (b - r.first) * kStrips + wave, chunk = unit / r.nw;
  const int ya = r.y0 + chunk * r.rows, yb = min(ya + r.rows, r.y1);
  if (ya >= yb) return;
  const int w = unit - chunk * r.nw;
  if (r.kind == kFusePlain) {
    march_plain<P, COLL>(a, q, r.x0 + w * (kFuseLanes * Kept<P>::kN), r.x1, ya, yb - ya);
  } else {
    // One call serves both kinds (it is long).
    const bool sides = r.kind == kFuseSides;
    const int X = sides ? 0 : r.x0 + w * kFuseEdgeW;
    const int own = sides ? 0 : min(kFuseEdgeW, r.x1 - X);
    const int edge = X + lane - (lane < 64 - kM ? 0 : 64);
    const int side = lane < kSideRight || lane >= 64 - kM ? edge : r.x1 - kM + lane - kSideRight;
    const bool side_owned =
        lane < r.x0 || (lane >= kSideRight + kM && lane < 64 - kM && side < a.nx);
    march_coded<P, false, COLL, false, false>(a, q, X, own, sides ? side : edge,
                                              sides ? side_owned : lane < own, ya, yb, yb - ya,
                                              pairs, 0, 0, ex);
  }
}

// Registers for three waves a SIMD with 4-byte storage (the stochastic rounding takes 191
// otherwise: 4096 x 4096 160 against 147 us a step), two with the others.
template <int P, bool FORCES, int COLL, bool MOV>
__global__ __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(sizeof(typename Storage<P>::T) == 4 ? 3 : 2)))
void fused_kernel(StepArgs a, FuseArgs q) {
  __shared__ Exchange ex;
  int b = int(blockIdx.x);
  if (q.nred > 0) {
    // The first eight blocks (one per XCD) reduce the force rows of the launch before this one.
    if (b < 8) {
      if (b < q.nred)
        reduce_row(q.red_in + b * q.step.part_stride, a.nslots, a.njslots, q.red_row + b * kRingRow,
                   b > 0 || q.red_has_prev ? q.red_row + (b - 1) * kRingRow + kJnext : nullptr);
      return;
    }
    b -= 8;
  }
  fused_block<P, FORCES, COLL, MOV>(a, q.map, q.step, block_tile<kFuseGroup>(b, q.map.nblocks), ex);
}

// kFuse steps of every instance of a batch: the first blocks reduce the force rows of the
// launch before this one, the others take the instances' blocks in the order of the item list.
template <int P, bool FORCES, bool MOV>
__global__ __launch_bounds__(kThreads)
    __attribute__((amdgpu_waves_per_eu(sizeof(typename Storage<P>::T) == 4 ? 3 : 2)))
void batch_fused_kernel(BatchFuse b) {
  __shared__ Exchange ex;
  int t = int(blockIdx.x);
  if (t < b.nred_blocks) {
    const int i = t / b.nred, r = t - i * b.nred;
    if (i >= b.n_inst) return;
    const BatchInst& I = b.inst[i];
    const int64_t rs = int64_t(b.n_inst) * kRingRow;  // rows are step-major
    double* row = I.ring + (b.red_row + r) * rs;
    reduce_row(I.part[b.turn ^ 1] + r * I.part_stride, I.a.nslots, I.a.njslots, row,
               r > 0 || b.red_has_prev ? row - rs + kJnext : nullptr);
    return;
  }
  t -= b.nred_blocks;
  const int i = b.item_inst[t];
  const BatchInst& I = b.inst[i];
  StepArgs a = I.a;
  a.src = I.buf[b.parity];
  a.dst = I.buf[1 - b.parity];
  FuseStep q;
  q.part_out = I.part[b.turn];
  q.part_stride = I.part_stride;
#pragma unroll
  for (int j = 0; j < kFuse; ++j)
    q.step_key[j] = Storage<P>::kSR ? sr_step_key(b.step0 + I.step_off + j) : 0u;
  fused_block<P, FORCES, LBM_COLL_BGK, MOV>(a, b.map[i], q, b.item_local[t], ex);
}

template <int P, bool MOV>
hipError_t fused_go2(bool forces, const StepArgs& a, const FuseArgs& q, hipStream_t s) {
  const dim3 grid(unsigned(q.map.nblocks + (q.nred > 0 ? 8 : 0)));
  if (forces)
    hipLaunchKernelGGL((fused_kernel<P, true, LBM_COLL_BGK, MOV>), grid, dim3(kThreads), 0, s, a, q);
  else
    hipLaunchKernelGGL((fused_kernel<P, false, LBM_COLL_BGK, MOV>), grid, dim3(kThreads), 0, s, a, q);
  return hipGetLastError();
}

template <int P>
hipError_t fused_go(bool forces, const StepArgs& a, const FuseArgs& q, hipStream_t s) {
  if (a.collision != LBM_COLL_BGK) return hipErrorInvalidValue;
  return a.motion ? fused_go2<P, true>(forces, a, q, s) : fused_go2<P, false>(forces, a, q, s);
}

template <int P>
hipError_t batch_fused_go(bool forces, const BatchFuse& b, hipStream_t s) {
  const dim3 grid(unsigned(b.nred_blocks + b.nitems));
  if (forces) {
    if (b.moving)
      hipLaunchKernelGGL((batch_fused_kernel<P, true, true>), grid, dim3(kThreads), 0, s, b);
    else
      hipLaunchKernelGGL((batch_fused_kernel<P, true, false>), grid, dim3(kThreads), 0, s, b);
  } else {
    if (b.moving)
      hipLaunchKernelGGL((batch_fused_kernel<P, false, true>), grid, dim3(kThreads), 0, s, b);
    else
      hipLaunchKernelGGL((batch_fused_kernel<P, false, false>), grid, dim3(kThreads), 0, s, b);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_batch_fused(int precision, bool forces, const BatchFuse& b, hipStream_t s) {
  switch (precision) {
    case LBM_FP64: return batch_fused_go<LBM_FP64>(forces, b, s);
    case LBM_FP32: return batch_fused_go<LBM_FP32>(forces, b, s);
    case LBM_FP32DEV: return batch_fused_go<LBM_FP32DEV>(forces, b, s);
    case LBM_FP32SR: return batch_fused_go<LBM_FP32SR>(forces, b, s);
    case LBM_FP16DEV: return batch_fused_go<LBM_FP16DEV>(forces, b, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fused(int precision, bool forces, const StepArgs& a, const FuseArgs& q,
                        hipStream_t s) {
  switch (precision) {
    case LBM_FP64: return fused_go<LBM_FP64>(forces, a, q, s);
    case LBM_FP32: return fused_go<LBM_FP32>(forces, a, q, s);
    case LBM_FP32DEV: return fused_go<LBM_FP32DEV>(forces, a, q, s);
    case LBM_FP32SR: return fused_go<LBM_FP32SR>(forces, a, q, s);
    case LBM_FP16DEV: return fused_go<LBM_FP16DEV>(forces, a, q, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lbm

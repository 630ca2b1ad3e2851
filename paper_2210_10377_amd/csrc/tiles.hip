// kFuse time steps in tiles: each block takes some rows of one strip's columns with kFuseM nodes
// around them, one thread a node; the first step pulls from memory, the others from LDS, and only
// the block's own nodes are stored (after every step where each state is kept).  A node's codes,
// inlet velocity and force slot are read once for all steps, and a strip with force terms is one
// wave, which sums as in step_kernel: states and forces are bitwise those of single steps.
//
// Small lattices are bound by latency: a launch of one step takes 3.4 us whatever its size, and
// a strip of the body with all forces 1.7 us more.  A launch of three steps takes 6 us on 60 x 40
// nodes, 10 with forces (binary64 200 x 80: 5.2 -> 3.4 us a step with forces, 3.6 -> 2.8 without),
// of which the chain of 600 instructions of a strip's force terms and sums is 1.3 us a step.  Rows:
// 4 while that gives at most one block a CU, else 8, where the margins take half of the work
// instead of the same again.  Cached stores, blocks grouped by XCD and one block a CU measured
// alike to 2 %.
#include <hip/hip_runtime.h>

#include "device.h"
#include "force_terms.h"
#include "kernels.h"
#include "lbm.h"
#include "plan.h"

namespace lbm {
namespace {

using namespace dev;

constexpr int kM = kFuseM;
constexpr int kTileCols = kStripW + 2 * kM;

// Waves of a block: one for each row with its margins, and those of the margin columns (four a
// row).
constexpr int tile_waves(int rows) {
  return rows + 2 * kM + ((rows + 2 * kM) * 2 * kM + 63) / 64;
}

// Stored populations of the directions 1 .. 8 of a tile, after the first step and after the second.
template <int P, int ROWS>
using TileState = typename Storage<P>::T[kFuse - 1][kQ - 1][ROWS + 2 * kM][kTileCols];

// kFuse steps of rows [ya, min(ya + ROWS, y1)) of the strip from column x0; columns [c0, c1) of
// it are stored.
template <int P, bool FORCES, int COLL, bool MOV, int ROWS>
__device__ __forceinline__ void tile_block(const StepArgs& a, const FuseStep& q, int x0, int ya,
                                           int y1, int c0, int c1, TileState<P, ROWS>& st) {
  using S = Storage<P>;
  using T = typename S::T;
  using C = typename S::C;
  constexpr int kRows = ROWS + 2 * kM;
  const int width = min(kStripW, a.nx - x0), yb = min(ya + ROWS, y1);
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
  const int lane = int(threadIdx.x) & 63;
  const bool periodic_x = a.bc_x == LBM_BCX_PERIODIC, periodic_y = a.bc_y == LBM_BCY_PERIODIC;

  // Node of the thread: row e and column p of the tile, margins included.
  int e = wave, p = lane + kM;
  bool valid = lane < width;
  if (wave >= kRows) {
    const int k = (wave - kRows) * 64 + lane, c = k % (2 * kM);
    e = min(k / (2 * kM), kRows - 1);
    p = c < kM ? c : width + c;
    valid = k < kRows * 2 * kM;
  }
  int x = x0 - kM + p, y = ya - kM + e;
  valid = valid && y < yb + kM && (periodic_x || (x >= 0 && x < a.nx)) &&
          (periodic_y || (y >= 0 && y < a.ny));
  x = periodic_x ? ((x % a.nx) + a.nx) % a.nx : min(max(x, 0), a.nx - 1);
  y = periodic_y ? ((y % a.ny) + a.ny) % a.ny : min(max(y, 0), a.ny - 1);

  // Its codes: from the plan where a node differs from what its coordinates say.
  const bool coded = y >= a.gy0 && y <= a.gy1 && x >= a.gx0 && x <= a.gx1;
  uint32_t w = 0;
  if (coded)
    w = a.node[int64_t(y) * a.nx + x];
  else
    w = edge_word_bits(a.nx, a.ny, a.bc_x, a.bc_y, x, y);
  const double u = a.uin[y];
  const bool own_row = wave < kRows && e >= kM && e < kM + ROWS && ya - kM + e < yb;
  int slot = -1;
  bool box = false;
  if (FORCES && own_row) {
    slot = slot_of(a, x0, ya - kM + e);
    box = strip_class(a.nx, a.ny, a.gx0, a.gx1, a.gy0, a.gy1, a.bx0, a.bx1, a.by0, a.by1, x0,
                      ya - kM + e) == kStripBoxInterior;
  }
  const Planes<T, true> src(a.src, a.plane, a.buf_bytes);
  T v[kQ] = {}, s[kQ] = {};
  if (valid) pull_raw<P>(src, a.pitch, a.nx, a.ny, w, x, y, v);
  valid = valid && !(w & kSolidBit);

  auto step = [&](auto J) __attribute__((always_inline)) {
    constexpr int j = J.value;
    // Nodes that later steps still reach.
    const bool need = valid && e >= j && e < yb - ya + 2 * kM - j && p >= j && p < width + 2 * kM - j;
    const bool mine = own_row && need && wave < kRows;
    C f[kQ] = {};
    if (need) {
      if constexpr (j > 0) {
        const uint32_t bd = back_dirs(w), od = outlet_dirs(w);
        const T(&in)[kQ - 1][kRows][kTileCols] = st[j - 1];
        v[0] = s[0];
#pragma unroll
        for (int i = 1; i < kQ; ++i) {
          const int from = kCx[i] < 0 && has_dir(od, i) ? p : p - kCx[i];
          const T t = in[i - 1][e - kCy[i]][from];
          v[i] = has_dir(bd, i) ? s[kOpp[i]] : t;
        }
      }
      finish_pull<P>(v, u, a.rho_w6, w, x, y, f, MOV ? a.motion : nullptr);
      T n[kQ];
      collide_pack<P, COLL>(a, f, q.step_key[j], x, y, n);
      if constexpr (j < kFuse - 1) {
#pragma unroll
        for (int i = 1; i < kQ; ++i) st[j][i - 1][e][p] = n[i];
      }
      if (mine && x >= c0 && x < c1 && (j == kFuse - 1 || (!FORCES && q.mid[j % (kFuse - 1)]))) {
        const Planes<T, true> out(j == kFuse - 1 ? a.dst : q.mid[j % (kFuse - 1)], a.plane,
                                  a.buf_bytes);
        const int32_t o = y * a.pitch + x;
#pragma unroll
        for (int i = 0; i < kQ; ++i) out.st(i, o, n[i]);
      }
#pragma unroll
      for (int i = 0; i < kQ; ++i) s[i] = n[i];
    }
    if (FORCES && slot >= 0) {
      double* part = q.part_out + j * q.part_stride;
      double acc[kPart] = {};
      if (box) {
        double jb[kBoxPart] = {};
        if (mine) {
#pragma unroll
          for (int i = 1; i < kQ; ++i) {
            const double fi = to_f64<P>(v[i], i), si = to_f64<P>(s[i], i);
            add_signed(kCx[i], fi, jb[0]);
            add_signed(kCy[i], fi, jb[1]);
            add_signed(kCx[i], si, jb[2]);
            add_signed(kCy[i], si, jb[3]);
          }
        }
        wave_sum_store<kBoxPart>(jb, part + int64_t(a.nslots) * kPart + int64_t(slot) * kBoxPart);
      } else {
        if (mine) {
          link_terms<P, MOV>(a, w, x, y, f, s, acc);
          box_terms<P>(a, x, y, f, s, acc);
          stress_terms<P>(a, w, f, acc);
        }
        wave_sum_store<kPart>(acc, part + int64_t(slot) * kPart);
      }
    }
    if constexpr (j < kFuse - 1) __syncthreads();
  };
  step(std::integral_constant<int, 0>{});
  step(std::integral_constant<int, 1>{});
  step(std::integral_constant<int, 2>{});
}

template <int P, bool FORCES, int COLL, bool MOV, int ROWS>
__global__ __launch_bounds__(64 * tile_waves(ROWS)) void tile_kernel(StepArgs a, FuseArgs q) {
  __shared__ TileState<P, ROWS> st;
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
  const int ns = (a.nx + kStripW - 1) / kStripW, chunk = b / ns;
  tile_block<P, FORCES, COLL, MOV, ROWS>(a, q.step, (b - chunk * ns) * kStripW, chunk * ROWS, a.ny,
                                         0, a.nx, st);
}

// The body rectangles of a batch, with forces: kBatchTileRows rows of a strip a block, in the
// order of the item list.
template <int P, bool MOV>
__global__ __launch_bounds__(64 * tile_waves(kBatchTileRows)) void batch_tile_kernel(BatchFuse b) {
  __shared__ TileState<P, kBatchTileRows> st;
  const int t = int(blockIdx.x), i = b.item_inst[t];
  const BatchInst& I = b.inst[i];
  StepArgs a = I.a;
  a.src = I.buf[b.parity];
  a.dst = I.buf[1 - b.parity];
  FuseStep q{};
  q.part_out = I.part[b.turn];
  q.part_stride = I.part_stride;
#pragma unroll
  for (int j = 0; j < kFuse; ++j)
    q.step_key[j] = Storage<P>::kSR ? sr_step_key(b.step0 + I.step_off + j) : 0u;
  const FuseRect r = b.map[i].r[0];
  const int first = r.x0 / kStripW, ns = (r.x1 + kStripW - 1) / kStripW - first;
  const int local = b.item_local[t], chunk = local / ns;
  tile_block<P, true, LBM_COLL_BGK, MOV, kBatchTileRows>(
      a, q, (first + local - chunk * ns) * kStripW, r.y0 + chunk * kBatchTileRows, r.y1, r.x0, r.x1,
      st);
}

template <int P, bool FORCES, int COLL, bool MOV>
hipError_t tile_rows(const StepArgs& a, const FuseArgs& q, hipStream_t s) {
  const dim3 grid(unsigned(q.map.nblocks + (q.nred > 0 ? 8 : 0)));
  switch (q.map.tile_rows) {
    case 4:
      hipLaunchKernelGGL((tile_kernel<P, FORCES, COLL, MOV, 4>), grid, dim3(64 * tile_waves(4)), 0,
                         s, a, q);
      break;
    case 8:
      hipLaunchKernelGGL((tile_kernel<P, FORCES, COLL, MOV, 8>), grid, dim3(64 * tile_waves(8)), 0,
                         s, a, q);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int P, int COLL>
hipError_t tile_coll(bool forces, const StepArgs& a, const FuseArgs& q, hipStream_t s) {
  if (forces)
    return a.motion ? tile_rows<P, true, COLL, true>(a, q, s)
                    : tile_rows<P, true, COLL, false>(a, q, s);
  return a.motion ? tile_rows<P, false, COLL, true>(a, q, s)
                  : tile_rows<P, false, COLL, false>(a, q, s);
}

template <int P>
hipError_t tile_go(bool forces, const StepArgs& a, const FuseArgs& q, hipStream_t s) {
  switch (a.collision) {
    case LBM_COLL_BGK: return tile_coll<P, LBM_COLL_BGK>(forces, a, q, s);
    case LBM_COLL_KBC: return tile_coll<P, LBM_COLL_KBC>(forces, a, q, s);
    default: return hipErrorInvalidValue;
  }
}

template <int P>
hipError_t batch_tile_go(const BatchFuse& b, hipStream_t s) {
  const dim3 grid(unsigned(b.nitems)), block(64 * tile_waves(kBatchTileRows));
  if (b.moving)
    hipLaunchKernelGGL((batch_tile_kernel<P, true>), grid, block, 0, s, b);
  else
    hipLaunchKernelGGL((batch_tile_kernel<P, false>), grid, block, 0, s, b);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_batch_tiles(int precision, const BatchFuse& b, hipStream_t s) {
  switch (precision) {
    case LBM_FP64: return batch_tile_go<LBM_FP64>(b, s);
    case LBM_FP32: return batch_tile_go<LBM_FP32>(b, s);
    case LBM_FP32DEV: return batch_tile_go<LBM_FP32DEV>(b, s);
    case LBM_FP32SR: return batch_tile_go<LBM_FP32SR>(b, s);
    case LBM_FP16DEV: return batch_tile_go<LBM_FP16DEV>(b, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tiles(int precision, bool forces, const StepArgs& a, const FuseArgs& q,
                        hipStream_t s) {
  switch (precision) {
    case LBM_FP64: return tile_go<LBM_FP64>(forces, a, q, s);
    case LBM_FP32: return tile_go<LBM_FP32>(forces, a, q, s);
    case LBM_FP32DEV: return tile_go<LBM_FP32DEV>(forces, a, q, s);
    case LBM_FP32SR: return tile_go<LBM_FP32SR>(forces, a, q, s);
    case LBM_FP16DEV: return tile_go<LBM_FP16DEV>(forces, a, q, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace lbm

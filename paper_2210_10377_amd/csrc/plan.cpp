// Host-side classification of every node and direction (the pull rules), the canonical
// link list, and the interior/general tile split of the step kernel.
#include "plan.h"

#include <algorithm>
#include <cstdio>
#include <cstring>

namespace lbm {

namespace {

bool in_box(const Plan& p, int x, int y) {
  return p.has_box && x >= p.box[0] && x < p.box[1] && y >= p.box[2] && y < p.box[3];
}

// Code of the pull rule for fluid node (x, y), direction i (first match wins:
// periodic wrap > wall > inlet > outlet > body > stream).
uint32_t classify(const Plan& p, const uint8_t* mask, int x, int y, int i) {
  int sx = x - kCx[i], sy = y - kCy[i];
  bool wrapped = false;
  if (p.bc_x == LBM_BCX_PERIODIC && (sx < 0 || sx >= p.nx)) {
    sx = (sx + p.nx) % p.nx;
    wrapped = true;
  }
  if (p.bc_y == LBM_BCY_PERIODIC && (sy < 0 || sy >= p.ny)) {
    sy = (sy + p.ny) % p.ny;
    wrapped = true;
  }
  if (p.bc_y == LBM_BCY_WALL && (sy < 0 || sy >= p.ny)) return kWall;
  if (p.bc_x == LBM_BCX_INLET_OUTLET && sx < 0) return kInlet;
  if (p.bc_x == LBM_BCX_INLET_OUTLET && sx >= p.nx)
    return mask[size_t(sy) * p.nx + (p.nx - 1)] ? kWall : kOutlet;
  if (mask[size_t(sy) * p.nx + sx]) return kBody;
  return wrapped ? kWrap : kStream;
}

// Solid nodes of a mask: their number and bounding box (x0 > x1 when there is none).
struct Solids {
  int64_t count = 0;
  int x0 = 0, x1 = -1, y0 = 0, y1 = -1;
};

// Checks of a grid and mask that need no plan: codes, sizes, mask bytes, and the
// control volume (one node inside the domain, every solid node strictly inside it).
// Fills the solid nodes' count and bounding box.
int validate(const lbm_grid& g, const uint8_t* mask, Solids& sol, std::string& err) {
  char buf[256];
  if (g.nx < 3 || g.ny < 3) {
    err = "nx and ny must be >= 3";
    return LBM_EINVAL;
  }
  if (g.bc_x != LBM_BCX_INLET_OUTLET && g.bc_x != LBM_BCX_PERIODIC) {
    err = "unknown bc_x";
    return LBM_EINVAL;
  }
  if (g.bc_y != LBM_BCY_WALL && g.bc_y != LBM_BCY_PERIODIC) {
    err = "unknown bc_y";
    return LBM_EINVAL;
  }
  if (g.tile != LBM_TILE_AUTO && g.tile != LBM_TILE_WIDE && g.tile != LBM_TILE_NARROW) {
    err = "unknown tile shape";
    return LBM_EINVAL;
  }
  if (g.precision != LBM_FP64 && g.precision != LBM_FP32 && g.precision != LBM_FP16DEV &&
      g.precision != LBM_FP32DEV && g.precision != LBM_FP32SR) {
    err = "unknown precision";
    return LBM_EINVAL;
  }
  if (g.collision != LBM_COLL_BGK && g.collision != LBM_COLL_REGULARIZED &&
      g.collision != LBM_COLL_KBC) {
    err = "unknown collision";
    return LBM_EINVAL;
  }
  if (g.max_record < 1) {
    err = "max_record must be >= 1";
    return LBM_EINVAL;
  }
  // One population plane must stay below 2^31 elements (32-bit in-plane offsets).
  const int64_t pitch = (int64_t(g.nx) + 63) / 64 * 64 + 256;  // row padding margin
  if (pitch * int64_t(g.ny) + 4096 >= (int64_t(1) << 31)) {
    err = "grid too large";
    return LBM_ENOMEM;
  }
  // Mask bytes, and the bounding box of the solid nodes (the control volume holds every
  // solid node strictly inside it exactly when it holds their bounding box).
  int sx0 = g.nx, sx1 = -1, sy0 = g.ny, sy1 = -1, fx = 0, fy = 0;
  int64_t count = 0;
  for (int y = 0; y < g.ny; ++y) {
    const uint8_t* row = mask + size_t(y) * g.nx;
    for (int x = 0; x < g.nx; ++x) {
      if (x + 8 <= g.nx) {  // skip eight fluid nodes at a time
        uint64_t v;
        std::memcpy(&v, row + x, 8);
        if (v == 0) {
          x += 7;
          continue;
        }
      }
      if (row[x] == 0) continue;
      ++count;
      if (row[x] > 1) {
        std::snprintf(buf, sizeof buf, "mask byte %zu is %d (must be 0 or 1)",
                      size_t(y) * g.nx + x, int(row[x]));
        err = buf;
        return LBM_EINVAL;
      }
      if (sx1 < 0) {
        fx = x;
        fy = y;
      }
      sx0 = std::min(sx0, x);
      sx1 = std::max(sx1, x);
      sy0 = std::min(sy0, y);
      sy1 = std::max(sy1, y);
    }
  }
  sol.count = count;
  sol.x0 = sx0;
  sol.x1 = sx1;
  sol.y0 = sy0;
  sol.y1 = sy1;
  if (g.box[0] >= 0) {
    const int x0 = g.box[0], x1 = g.box[1], y0 = g.box[2], y1 = g.box[3];
    if (x0 < 1 || y0 < 1 || x1 > g.nx - 1 || y1 > g.ny - 1 || x1 - x0 < 3 || y1 - y0 < 3) {
      err = "control-volume box must lie one node inside the domain and span >= 3 nodes";
      return LBM_EINVAL;
    }
    if (sx1 >= 0 && !(sx0 >= x0 + 1 && sx1 < x1 - 1 && sy0 >= y0 + 1 && sy1 < y1 - 1)) {
      // Name one offending node.
      for (int y = sy0; y <= sy1; ++y)
        for (int x = sx0; x <= sx1; ++x)
          if (mask[size_t(y) * g.nx + x] &&
              !(x >= x0 + 1 && x < x1 - 1 && y >= y0 + 1 && y < y1 - 1)) {
            fx = x;
            fy = y;
            y = sy1 + 1;
            break;
          }
      std::snprintf(buf, sizeof buf,
                    "solid node (%d,%d) is not strictly inside the control-volume box", fx, fy);
      err = buf;
      return LBM_EINVAL;
    }
  }
  return LBM_OK;
}

void set_geometry(Plan& p, const lbm_grid& g) {
  p.nx = g.nx;
  p.ny = g.ny;
  p.bc_x = g.bc_x;
  p.bc_y = g.bc_y;
  p.has_box = g.box[0] >= 0;
  for (int k = 0; k < 4; ++k) p.box[k] = g.box[k];
  p.tile_rows = tile_rows_for(g.nx, g.tile);
}

uint32_t node_word(const Plan& p, const uint8_t* mask, int x, int y) {
  if (mask[size_t(y) * p.nx + x]) return kSolidBit;
  uint32_t w = 0;
  for (int i = 1; i < kQ; ++i) w |= classify(p, mask, x, y, i) << (3 * (i - 1));
  return w;
}

// Everything the plan derives from its node words and geometry: node counts, the
// general rectangle, the canonical link list, strip classes and slots, the box sweep.
void derive(Plan& p, const Solids& sol) {
  const int nx = p.nx, ny = p.ny;
  p.n_fluid = int64_t(nx) * ny - sol.count;
  p.n_box = 0;
  if (p.has_box)
    for (int y = p.box[2]; y < p.box[3]; ++y)
      for (int x = p.box[0]; x < p.box[1]; ++x)
        p.n_box += (p.node[size_t(y) * nx + x] & kSolidBit) ? 0 : 1;

  // Rectangle of every node whose codes need the general path.  `band`: the nodes with
  // a control-volume term (the box and the ring around it).
  auto band = [&](int x, int y) {
    return p.has_box && x >= p.box[0] - 1 && x <= p.box[1] && y >= p.box[2] - 1 &&
           y <= p.box[3];
  };
  p.gx0 = 0;
  p.gx1 = -1;
  p.gy0 = 0;
  p.gy1 = -1;
  // Every such node is a solid node or the neighbour of one (a pull from a solid node,
  // or the outlet rule reading a solid node of the last column), so only the solid
  // nodes' bounding box grown by one node (the whole axis when that crosses a periodic
  // edge) is scanned.
  int xa = sol.x0 - 1, xb = sol.x1 + 1, ya = sol.y0 - 1, yb = sol.y1 + 1;
  if (p.bc_x == LBM_BCX_PERIODIC && (xa < 0 || xb > nx - 1)) {
    xa = 0;
    xb = nx - 1;
  }
  if (p.bc_y == LBM_BCY_PERIODIC && (ya < 0 || yb > ny - 1)) {
    ya = 0;
    yb = ny - 1;
  }
  xa = std::max(xa, 0);
  xb = std::min(xb, nx - 1);
  ya = std::max(ya, 0);
  yb = std::min(yb, ny - 1);
  if (sol.count == 0) yb = ya - 1;
  for (int y = ya; y <= yb; ++y) {
    const uint32_t* row = p.node.data() + size_t(y) * nx;
    // Away from x = 0 and x = nx - 1 the edge word of a row is one value.
    const uint32_t emid = edge_word(nx, ny, p.bc_x, p.bc_y, nx / 2, y);
    int lo = -1, hi = -1;
    for (int x = xa; x <= xb; ++x)
      if (row[x] != ((x == 0 || x == nx - 1) ? edge_word(nx, ny, p.bc_x, p.bc_y, x, y) : emid)) {
        if (lo < 0) lo = x;
        hi = x;
      }
    if (lo < 0) continue;
    if (p.gx0 > p.gx1) {
      p.gx0 = lo;
      p.gx1 = hi;
      p.gy0 = p.gy1 = y;
    } else {
      p.gx0 = std::min(p.gx0, lo);
      p.gx1 = std::max(p.gx1, hi);
      p.gy1 = y;
    }
  }

  // Canonical link list: (x, i) with x + c_i a solid mask node, i.e. the pull of the
  // opposite direction bounces back from the body.  Off the first and last rows such
  // nodes lie in the general rectangle.
  p.links.clear();
  auto scan_links = [&](int y, int xa, int xb) {
    for (int x = xa; x <= xb; ++x) {
      const size_t k = size_t(y) * nx + x;
      if (p.node[k] & kSolidBit) continue;
      for (int i = 1; i < kQ; ++i)
        if (pull_code(p.node[k], kOpp[i]) == kBody) {
          p.links.push_back(int32_t(k));
          p.links.push_back(i);
        }
    }
  };
  for (int y = 0; y < ny; ++y) {
    if (y == 0 || y == ny - 1)
      scan_links(y, 0, nx - 1);
    else if (p.gx0 <= p.gx1 && y >= p.gy0 && y <= p.gy1)
      scan_links(y, p.gx0, p.gx1);
  }

  // Strips (strip_class) in row-major order, y then x: general strips holding a link
  // node or a node with a control-volume term own a force-partial slot (kPart sums);
  // box-interior strips own a slot of the box-momentum partials.  The slots are numbered
  // in this order whatever the tile shape, so every shape reduces the same partials in
  // the same order (bitwise the same forces).
  const int nsx = (nx + kStripW - 1) / kStripW;
  p.row_slot.assign(size_t(ny) * nsx, -1);
  p.nslots = p.njslots = p.ngeneral = 0;
  for (int y0 = 0; y0 < ny; ++y0)
    for (int sx = 0; sx < nsx; ++sx) {
      const int x0 = sx * kStripW;
      const int cls = p.has_box
                          ? strip_class(nx, ny, p.gx0, p.gx1, p.gy0, p.gy1, p.box[0], p.box[1],
                                        p.box[2], p.box[3], x0, y0)
                          : strip_class(nx, ny, p.gx0, p.gx1, p.gy0, p.gy1, 1, 0, 1, 0, x0, y0);
      int32_t& slot = p.row_slot[size_t(y0) * nsx + sx];
      if (cls == kStripPlain) continue;
      if (cls == kStripBoxInterior) {
        slot = p.njslots++;
        continue;
      }
      if (cls == kStripGeneral) ++p.ngeneral;
      bool forces = false;
      for (int x = x0; x < std::min(x0 + kStripW, nx); ++x) {
        const uint32_t wd = p.node[size_t(y0) * nx + x];
        bool link = false;
        if (!(wd & kSolidBit))
          for (int i = 1; i < kQ; ++i) link = link || pull_code(wd, i) == kBody;
        forces = forces || link || band(x, y0);
      }
      if (forces) slot = p.nslots++;
    }
  tile_slots(p, p.tile_rows, p.ntx, p.nty, p.strip_slot);
  p.ntiles = p.ntx * p.nty;
  p.box_bx = p.box_rows = 0;
  if (p.has_box) {
    p.box_bx = (p.box[1] - p.box[0] + kTileW - 1) / kTileW;
    p.box_rows = p.box[3] - p.box[2];
  }
}

}  // namespace

int build_plan(const lbm_grid& g, const uint8_t* mask, Plan& p, std::string& err) {
  Solids sol;
  const int rc = validate(g, mask, sol, err);
  if (rc != LBM_OK) return rc;
  p = Plan();
  set_geometry(p, g);
  p.node.assign(size_t(g.nx) * size_t(g.ny), 0u);
  for (int y = 0; y < g.ny; ++y)
    for (int x = 0; x < g.nx; ++x) p.node[size_t(y) * g.nx + x] = node_word(p, mask, x, y);
  derive(p, sol);
  return LBM_OK;
}

int replan(const lbm_grid& g, const uint8_t* mask, const std::vector<int32_t>& changed,
           Plan& p, Plan& np, PlanDelta& d, std::string& err) {
  Solids sol;
  const int rc = validate(g, mask, sol, err);
  if (rc != LBM_OK) return rc;
  // Node words that can change: those of the changed nodes and of their lattice
  // neighbours (a pull reads its source node, and the outlet rule the last column of
  // the neighbouring rows).
  Plan geo;
  set_geometry(geo, g);
  std::vector<int64_t> idx;
  idx.reserve(changed.size() * kQ);
  for (int32_t c : changed) {
    const int x = c % g.nx, y = c / g.nx;
    for (int i = 0; i < kQ; ++i) {
      int ax = x + kCx[i], ay = y + kCy[i];
      if (g.bc_x == LBM_BCX_PERIODIC) ax = (ax + g.nx) % g.nx;
      if (g.bc_y == LBM_BCY_PERIODIC) ay = (ay + g.ny) % g.ny;
      if (ax < 0 || ax >= g.nx || ay < 0 || ay >= g.ny) continue;
      idx.push_back(int64_t(ay) * g.nx + ax);
    }
  }
  std::sort(idx.begin(), idx.end());
  idx.erase(std::unique(idx.begin(), idx.end()), idx.end());
  d = PlanDelta();
  for (int64_t k : idx) {
    const uint32_t w = node_word(geo, mask, int(k % g.nx), int(k / g.nx));
    if (w == p.node[size_t(k)]) continue;
    d.idx.push_back(k);
    d.old_w.push_back(p.node[size_t(k)]);
    d.new_w.push_back(w);
  }
  // The new plan takes p's words (no copy) with the delta applied.
  apply_delta(p, d, true);
  np = Plan();
  set_geometry(np, g);
  np.node.swap(p.node);
  derive(np, sol);
  return LBM_OK;
}

namespace {

// Rows of the tables below, by storage.
int storage_row(int precision) {
  switch (precision) {
    case LBM_FP64: return 0;
    case LBM_FP32:
    case LBM_FP32DEV: return 1;
    case LBM_FP32SR: return 2;
    default: return 3;
  }
}

int strips_across(int nx) { return (nx + kStripW - 1) / kStripW; }

}  // namespace

void StepWork::add(const Plan& p, const FuseMap& m, int elem_bytes) {
  strips += double(strips_across(p.nx)) * kStripW * p.ny;
  nodes += double(p.nx) * p.ny;
  for (int k = 0; k < m.nrects; ++k) {
    const FuseRect& r = m.r[k];
    const int height = r.y1 - r.y0;
    double rows = height + 2.0 * kFuseM * ((height + r.rows - 1) / r.rows);
    if (p.bc_y == LBM_BCY_WALL)  // no rows are marched beyond a wall
      rows -= std::max(kFuseM - r.y0, 0) + std::max(kFuseM - (p.ny - r.y1), 0);
    const double lanes = 64.0 * r.nw * rows;
    if (r.kind == kFuseBody) {
      body += 2.0 * lanes;  // a wave for each half of a strip
      body_nodes += double(r.x1 - r.x0) * height;
    } else if (r.kind == kFusePlain) {
      plain += lanes * (8 / elem_bytes);
    } else {
      coded += lanes;
    }
  }
}

bool fuse_pays(int precision, int collision, bool forces, const StepWork& w, bool moving,
               bool batch) {
  // Both forms in us a step, as they were measured: a start, and us for a million lanes of strips
  // and nodes, or of the lanes and rows that windows of each kind march (they do about 1.4 times
  // the work in plain windows, 1.5 - 6 times at edges and bodies, for a third of the bytes; a narrow
  // lattice has few other windows).  No fused launch is shorter than its longest unit: `least`.
  // Fitted to 418 lattices and batches for each row of the table (242 in the lower half): widths 3 to
  // 20000, 2e5 to 8e6 nodes in all, cylinders, airfoils, porous blocks and small bodies, lattices and
  // members from 3 rows on.  Over those and 776 more lattices a row, half of them with spinning
  // bodies, the form picked (tiles among them) is on average 0.6 % slower than the fastest.
  // Measured, single : fused, with all forces (without): binary32 1024 x 512 10.4 : 10.0 (8.1 : 6.5),
  // 2048 x 1024 27 : 17, 8192 x 4096 397 : 177, 16 x 40000 23 : 40 (21 : 29), 37 x 14000 15 : 25
  // (13 : 21), 1000 lattices of 64 x 32 72 : 110 (30 : 60), of 43 000 nodes 16 20 : 19 (16 : 15), 256
  // 175 : 139 (170 : 106); binary64 16 x 40000 33 : 51 (31 : 40), 4096 x 2048 199 : 88; stochastically
  // rounded 2048 x 1024 27 : 31, 4096 x 2048 with an airfoil 100 : 85; binary16 3000 x 1500 31 : 38,
  // 5792 x 2896 101 : 98.
  // The stabilized collisions stay with single steps: regularized, binary32, 1024 x 512 without
  // forces 8.1 : 9.5, a moving airfoil with forces 12.4 : 13.3.
  // Bodies in motion slow a window more than a strip: a cylinder in 1300 x 650, binary64,
  // 25.5 : 15.9 at rest and 24.6 : 18.9 spinning, binary32 850 x 531 10.1 : 10.0 and 10.7 : 12.6.  In
  // batches it is the single steps that they slow: 32 lattices in binary32 30.9 : 28.1 at rest and
  // 50.7 : 30.8 spinning.  `kRatio` is the median of measured over fitted, of 388 lattices (against
  // that at rest) and 29 or 34 batches a row; of binary32 batches 4 to 12 % less, for the smallest:
  // 25 of 200 x 80 12.4 : 10.4 with forces, 8.4 : 7.4 without, 62 21.6 : 23.3 and 17.7 : 19.2 (spinning).
  struct Rates {
    double start, strips, nodes, body;                // single steps
    double least, begin, plain, coded, body_windows;  // fused launches
  };
  constexpr Rates kRates[4][2] = {
      {{2.4, 9.9, 15.5, 1.1, 5.4, 2.0, 5.8, 5.1, 4.8}, {4.2, 10.8, 13.7, 5.6, 10.2, 2.4, 6.0, 7.5, 13.9}},
      {{2.3, 6.8, 5.4, 0.6, 5.7, 2.8, 3.4, 3.5, 3.2}, {4.4, 8.0, 4.0, 4.7, 9.7, 4.0, 3.1, 5.1, 11.0}},
      {{3.1, 7.9, 3.4, 0.4, 8.1, 4.8, 6.0, 5.4, 5.6}, {4.8, 9.1, 2.1, 3.7, 12.0, 5.4, 5.8, 7.1, 13.0}},
      {{3.2, 5.5, 0.0, 0.8, 7.1, 3.8, 2.6, 5.5, 7.3}, {5.0, 5.6, 0.0, 4.6, 10.7, 4.4, 2.6, 6.5, 13.9}}};
  // Windows over single steps: lattices at rest and moving, batches at rest and moving.
  constexpr double kRatio[4][2][4] = {{{1.0, 1.1, 1.0, 1.05}, {1.0, 1.17, 1.0, 0.97}},
                                      {{1.0, 1.03, 0.96, 0.96}, {1.0, 1.17, 0.91, 0.58}},
                                      {{1.0, 1.0, 1.0, 1.05}, {1.0, 1.04, 0.85, 0.4}},
                                      {{1.0, 1.03, 1.0, 1.02}, {1.0, 1.0, 0.84, 0.7}}};
  // The fit is off by 5 % (median) and 18 % (one in ten) on lattices it was not made of, so what it
  // says of few nodes, or of many at bodies, is not followed: there windows measured 0.75 to 1.24 of
  // single steps (binary32 without forces 1020 x 317 7.0 : 7.7, with a spinning airfoil 1933 x 276
  // 10.2 : 12.6; stochastically rounded 3341 x 1371, periodic along x, 56 : 62).
  constexpr double kLeast[4] = {2.5e5, 4e5, 4e6, 1.5e7};
  constexpr double kBody[4] = {0.4, 0.2, 0.06, 0.04};
  if (collision != LBM_COLL_BGK) return false;
  const int row = storage_row(precision);
  if (w.nodes < kLeast[row] || w.body_nodes > kBody[row] * w.nodes) return false;
  const Rates& r = kRates[row][forces ? 1 : 0];
  const double single = r.start + 1e-6 * (r.strips * w.strips + r.nodes * w.nodes + r.body * w.body);
  const double windows =
      r.begin + 1e-6 * (r.plain * w.plain + r.coded * w.coded + r.body_windows * w.body);
  const double ratio = kRatio[row][forces ? 1 : 0][(batch ? 2 : 0) + (moving ? 1 : 0)];
  return ratio * std::max(r.least, windows) < single;
}

bool batch_tiles_pay(const StepWork& w) {
  // Windows of half strips do 2.3 times the work of the nodes they own, tiles 1.4 times, but take a
  // launch more.  Windows : tiles, in us a step of 256, 64, 32 and 16 lattices of 43 000 nodes, 11 %
  // of them in the body rectangles: binary32 148 : 139, 46 : 45, 28.7 : 27.1, 19.0 : 18.7; binary64
  // 232 : 210, 61 : 56, 39.6 : 38.1, 23.5 : 24.1.  Over 246 batches with bodies of 0.2 to 50 % the
  // ratio goes by the nodes of the body rectangles: tiles 1.1 - 1.2 times as slow below 3e4, even at
  // 1e5, 0.9 from 4e5 on.
  return w.body_nodes >= 1e5;
}

int tile_rows(int precision, int collision, bool forces, double summed, int nx, int ny, bool wide,
              bool moving) {
  // Small lattices are bound by latency: a launch of one step takes 3.4 us, with forces 5.2 as
  // each strip of the body sums 12 components, however few nodes there are.  Three steps of a
  // tile take 6 and 10, as long as there is no more than one block a CU; then a second round of
  // blocks begins, and the margins (12 rows of work for 8) cost more than the launches saved.
  // What counts are the blocks, of idle lanes too.  Measured in us a step with all forces (without),
  // single steps : tiles of 4 rows : of 8, and the blocks of 8 rows:
  //   binary64 200 x 100 (52) 6.6 : 4.6 : 5.2 (3.6 : 2.6 : 3.4), 512 x 256 (256) 7.5 : 6.2 : 5.4 (4.8 :
  //   3.8 : 2.9), 600 x 300 (380) 8.8 : 7.8 : 6.7 (6.3 : 5.9 : 5.1), 1024 x 512 (1024) 17.1 : 15.9 : 12.8
  //   (windows 13.0), 16 x 6250 (782) 8.6 : 11.0 : 9.2;
  //   binary32 512 x 256 6.8 : 5.8 : 5.2 (3.9 : 2.8 : 2.7), 724 x 362 (552) 7.8 : 9.0 : 7.6 (5.3 : 5.4 :
  //   5.6), 3 x 12500 (1563) 9.7 : 17.7 : 13.2 (8.2 : 11.1 : 10.2);
  //   stochastically rounded 600 x 300 7.6 : 8.4 : 7.0 (4.9 : 4.9 : 5.1), binary16 6.6 : 6.8 : 5.6 (4.1 :
  //   3.7 : 3.9);
  //   entropic 512 x 320 (320) binary64 9.1 : 9.6 : 8.8 (6.7 : 7.7 : 7.3), binary32 7.2 : 7.4 : 6.6 (4.7 :
  //   4.5 : 4.8), stochastically rounded 7.6 : 8.8 : 7.9 (5.2 : 5.5 : 6.1), 512 x 256 7.4 : 7.3 : 6.4 (4.6 :
  //   4.1 : 3.7).
  // The regularized collision is left to single steps: its compiled form rounds differently here.
  if (collision == LBM_COLL_REGULARIZED) return 0;
  // The most blocks of 8 rows, by storage: BGK without and with forces, entropic likewise.  512 are two
  // rounds of the chip: binary32 600 x 375 (470) 0.90 of single steps, 724 x 362 (552) 1.06; binary16
  // 0.87 and 1.11; entropic binary32 0.92 and 1.11.  Where a second round takes more than it gives, it
  // is 256: entropic binary64 515 x 234 (270) 1.33, stochastically rounded 1.18, binary16 640 x 234
  // (300) 1.08.
  constexpr int kMost[4][4] = {
      {400, 1100, 256, 400}, {512, 512, 512, 400}, {256, 400, 256, 256}, {512, 512, 256, 400}};
  const int row = storage_row(precision);
  const bool bgk = collision == LBM_COLL_BGK;
  const int strips = strips_across(nx), last = nx % kStripW;
  const int64_t blocks = int64_t(strips) * ((ny + 7) / 8);
  // A wave of at most 8 lanes takes longer than a full one, and it does here in every step, where a
  // single step's block of four strips hides it: entropic binary64 without forces, single steps :
  // tiles, 192 x 80 4.0 : 3.2, 193 x 80 to 200 x 80 3.9 : 4.8, 201 x 80 3.9 : 3.2; of five strips
  // or three no more than others (130 x 156 0.81, 385 x 100 0.81).
  if (row == 0 && !bgk && !forces && strips % 4 == 0 && last >= 1 && last <= 8) return 0;
  int most = kMost[row][(bgk ? 0 : 2) + (forces ? 1 : 0)];
  // Binary32 gains longer where a body's strips are summed: with forces 724 x 362 (552) without a body
  // 1.10 of single steps, with a cylinder or an airfoil (8 % of the strips) 0.96 and 0.99, with scattered
  // solids everywhere 0.73; 1700 x 212 (729) with a cylinder (3 %) 0.91; but 1.04 to 1.1 if it spins.
  if (row == 1 && bgk && forces && summed >= 0.025 && !moving) most = 730;
  // Binary16 without forces, 600 x 300 (380) with a spinning cylinder 1.07 to 1.15 of single steps (at
  // rest 0.99), 200 blocks 0.78.
  if (row == 3 && bgk && !forces && moving) most = 256;
  // Binary64 gains up to 2000 blocks where windows do not (37 x 12500 19.4 : 16.0 with forces, 18.1 : 14.2
  // without, windows 24.5 and 19.7), if the strips are at least half full.
  if (wide && row == 0 && bgk) most = 2000;
  if (int64_t(nx) * 2 < int64_t(strips) * kStripW) most = std::min(most, 400);
  if (blocks > most) return 0;
  return strips * ((ny + 3) / 4) <= 256 ? 4 : 8;
}

FuseMap step_map(const Plan& p, int precision, int collision, bool forces, int elem_bytes,
                 bool moving) {
  const double summed = p.nslots / (double(strips_across(p.nx)) * p.ny);
  if (const int rows = tile_rows(precision, collision, forces, summed, p.nx, p.ny, false, moving))
    return tile_map(p, rows);
  if (collision != LBM_COLL_BGK) return FuseMap{};
  const FuseMap m = fuse_map(p, elem_bytes, int64_t(p.nx) * p.ny);
  StepWork w;
  w.add(p, m, elem_bytes);
  if (fuse_pays(precision, collision, forces, w, moving, false)) return m;
  const int rows = tile_rows(precision, collision, forces, summed, p.nx, p.ny, true, moving);
  return rows ? tile_map(p, rows) : FuseMap{};
}

FuseMap keep_map(const Plan& p, int precision, int collision) {
  // 12 bytes read and 36 written a step and node in binary32, where single steps read 36 as well.
  // The recomputation for an adjoint run, which is beside the reverse steps, took, single steps :
  // tiles, in ms of the whole reverse sweep: binary32 1024 x 512 10.9 : 10.5, 2048 x 1024 13.0 :
  // 12.9, binary64 21.5 : 19.3, 26.2 : 23.7; stochastically rounded 16 x 12000, whose strips are a
  // quarter full, 6.8 : 7.5.
  int rows = tile_rows(precision, collision, false, 0.0, p.nx, p.ny, false, false);
  const bool full = p.nx * 2 >= strips_across(p.nx) * kStripW;
  const bool binary32 = precision == LBM_FP32 || precision == LBM_FP32DEV;
  if (rows == 0 && collision == LBM_COLL_BGK && full &&
      (precision == LBM_FP64 || (binary32 && double(p.nx) * p.ny <= 1e6)))
    rows = 8;
  return rows > 0 ? tile_map(p, rows) : FuseMap{};
}

FuseMap tile_map(const Plan& p, int rows) {
  FuseMap m{};
  m.tile_rows = rows;
  m.nblocks = strips_across(p.nx) * ((p.ny + rows - 1) / rows);
  return m;
}

FuseMap fuse_map(const Plan& p, int elem_bytes, int64_t nodes) {
  constexpr int kM = kFuseM;
  // Rows of a unit: in the plain rectangles few enough to give every SIMD three waves, many
  // enough to keep the margins (two rows of two steps) small; in the body rectangle as many as
  // a launch has time for (a row of three steps with forces takes 5 - 8 us, a launch of
  // 8192 x 4096 in binary32 500 us, of 1024 x 512 27 us).
  const int64_t bytes = nodes * kQ * elem_bytes;
  const int64_t lanes = bytes / (kQ * 8) / kFuseLanes;  // units of one row
  const int rows = int(std::clamp<int64_t>(lanes / 3072, 6, 12));
  const int body_rows = int(std::clamp<int64_t>(2 + bytes / 37000000, 2, 32));
  const int edge_rows = std::clamp(body_rows / 2, 2, 8);
  // The body rectangle (inclusive here): the general nodes with kM nodes of margin, so that
  // the other windows meet edge codes only, and the nodes with control-volume terms.
  int x0 = p.nx, x1 = -1, y0 = p.ny, y1 = -1;
  if (p.gx0 <= p.gx1) {
    x0 = p.gx0 - kM;
    x1 = p.gx1 + kM;
    y0 = p.gy0 - kM;
    y1 = p.gy1 + kM;
    // A margin across a periodic edge takes the whole axis.
    if (p.bc_x == LBM_BCX_PERIODIC && (x0 < 0 || x1 >= p.nx)) {
      x0 = 0;
      x1 = p.nx - 1;
    }
    if (p.bc_y == LBM_BCY_PERIODIC && (y0 < 0 || y1 >= p.ny)) {
      y0 = 0;
      y1 = p.ny - 1;
    }
  }
  if (p.has_box) {
    x0 = std::min(x0, p.box[0] - 1);
    x1 = std::max(x1, p.box[1]);
    y0 = std::min(y0, p.box[2] - 1);
    y1 = std::max(y1, p.box[3]);
  }
  FuseMap m{};
  auto add = [&](int kind, int ax0, int ax1, int ay0, int ay1) {
    if (ax0 >= ax1 || ay0 >= ay1) return;
    FuseRect& r = m.r[m.nrects++];
    r.x0 = ax0;
    r.x1 = ax1;
    r.y0 = ay0;
    r.y1 = ay1;
    r.kind = int16_t(kind);
    r.first = m.nblocks;
    const int per = kind == kFuseBody ? kStripW
                                      : (kind == kFuseEdge ? kFuseEdgeW : kFuseLanes * 8 / elem_bytes);
    r.rows = int16_t(kind == kFuseBody ? body_rows : (kind == kFusePlain ? rows : edge_rows));
    r.nw = kind == kFuseSides  ? 1
           : kind == kFuseBody ? (ax1 - ax0 / kStripW * kStripW + per - 1) / per
                               : (ax1 - ax0 + per - 1) / per;
    const int64_t units = int64_t(r.nw) * ((ay1 - ay0 + r.rows - 1) / r.rows);
    const int in_block = kind == kFuseBody ? kStrips / 2 : kStrips;
    m.nblocks += int32_t((units + in_block - 1) / in_block);
  };
  // The rectangles around the body: the rows before and after it, the columns beside it.
  struct Box {
    int x0, x1, y0, y1;
  };
  Box around[4];
  int n = 0;
  if (x0 <= x1) {
    x0 = std::max(x0, 0) / kHalf * kHalf;
    x1 = std::min((x1 / kHalf + 1) * kHalf, p.nx);
    y0 = std::max(y0, 0);
    y1 = std::min(y1 + 1, p.ny);
    add(kFuseBody, x0, x1, y0, y1);
    around[n++] = {0, p.nx, 0, y0};
    around[n++] = {0, x0, y0, y1};
    around[n++] = {x1, p.nx, y0, y1};
    around[n++] = {0, p.nx, y1, p.ny};
  } else {
    around[n++] = {0, p.nx, 0, p.ny};
  }
  // The nodes whose windows (margins included) stream plainly: kM + 1 nodes from the edges,
  // along x in whole 64-byte sectors (a window's first lanes are half a sector left of its
  // first column).
  const int sector = 64 / elem_bytes;
  const Box in = {sector, (p.nx - kM - 1) / sector * sector, kM + 1, p.ny - kM - 1};
  // The columns beside the interior, left and right of it in one window where both sides (with
  // their margins) fit one.
  const bool sides = in.x0 + kM <= kSideRight && p.nx - in.x1 + 2 * kM <= 64 - kM - kSideRight &&
                     in.x0 < in.x1;
  // Units that take longest start first.
  for (int pass = 0; pass < 3; ++pass)
    for (int k = 0; k < n; ++k) {
      const Box& b = around[k];
      if (b.x0 >= b.x1 || b.y0 >= b.y1) continue;
      const Box c = {std::max(b.x0, in.x0), std::min(b.x1, in.x1), std::max(b.y0, in.y0),
                     std::min(b.y1, in.y1)};
      // Beside the body: its left rectangle takes both sides if the right one reaches inside.
      const bool beside = n == 4 && (k == 1 || k == 2);
      const bool both = sides && c.y0 < c.y1 &&
                        (beside ? around[1].x1 >= in.x0 && around[2].x0 <= in.x1
                                : c.x0 < c.x1);
      const bool none = c.x0 >= c.x1 || c.y0 >= c.y1;
      if (pass == 2) {
        if (!none) add(kFusePlain, c.x0, c.x1, c.y0, c.y1);
      } else if (pass == 1) {
        if (both && k != 2) add(kFuseSides, in.x0, in.x1, c.y0, c.y1);
      } else if (both) {
        add(kFuseEdge, b.x0, b.x1, b.y0, c.y0);
        add(kFuseEdge, b.x0, b.x1, c.y1, b.y1);
      } else if (none) {
        add(kFuseEdge, b.x0, b.x1, b.y0, b.y1);
      } else {
        add(kFuseEdge, b.x0, b.x1, b.y0, c.y0);
        add(kFuseEdge, b.x0, b.x1, c.y1, b.y1);
        add(kFuseEdge, b.x0, c.x0, c.y0, c.y1);
        add(kFuseEdge, c.x1, b.x1, c.y0, c.y1);
      }
    }
  return m;
}

namespace {

// Blocks of kBatchTileRows rows of a strip's columns in the body rectangle of m, if it has one.
int body_tiles(const FuseMap& m) {
  const FuseRect& r = m.r[0];
  if (m.nrects == 0 || r.kind != kFuseBody) return 0;
  const int strips = (r.x1 + kStripW - 1) / kStripW - r.x0 / kStripW;
  return strips * ((r.y1 - r.y0 + kBatchTileRows - 1) / kBatchTileRows);
}

}  // namespace

bool BatchWork::set(size_t i, const Plan& p, int elem_bytes, int64_t nodes) {
  const FuseMap m = fuse_map(p, elem_bytes, nodes), &old = map[i];
  bool other = m.nrects != old.nrects || m.nblocks != old.nblocks || body_tiles(m) != body_tiles(old);
  for (int k = 0; k < m.nrects && !other; ++k)
    other = m.r[k].kind != old.r[k].kind || m.r[k].first != old.r[k].first;
  map[i] = m;
  work[i] = StepWork();
  work[i].add(p, m, elem_bytes);
  return other;
}

void BatchWork::list() {
  inst.clear();
  local.clear();
  auto add = [&](size_t i, int b) {
    inst.push_back(int32_t(i));
    local.push_back(b);
  };
  for (int kind = kFuseBody; kind <= kFusePlain; ++kind) {
    for (size_t i = 0; i < map.size(); ++i) {
      const FuseMap& f = map[i];
      for (int k = 0; k < f.nrects; ++k) {
        if (f.r[k].kind != kind) continue;
        const int end = k + 1 < f.nrects ? f.r[k + 1].first : f.nblocks;
        for (int b = f.r[k].first; b < end; ++b) add(i, b);
      }
    }
    if (kind == kFuseBody) nbody = inst.size();
  }
  nblocks = inst.size();
  for (size_t i = 0; i < map.size(); ++i)
    for (int b = 0; b < body_tiles(map[i]); ++b) add(i, b);
}

StepWork BatchWork::total() const {
  StepWork t;
  for (const StepWork& w : work) {
    t.strips += w.strips;
    t.nodes += w.nodes;
    t.plain += w.plain;
    t.coded += w.coded;
    t.body += w.body;
    t.body_nodes += w.body_nodes;
  }
  return t;
}

void tile_slots(const Plan& p, int rows, int& ntx, int& nty, std::vector<int32_t>& out) {
  const int tile_w = kTileW / rows;
  ntx = (p.nx + tile_w - 1) / tile_w;
  nty = (p.ny + rows - 1) / rows;
  const int nsx = (p.nx + kStripW - 1) / kStripW;
  out.assign(size_t(ntx) * nty * kStrips, -1);
  for (int tile = 0; tile < ntx * nty; ++tile)
    for (int w = 0; w < kStrips; ++w) {
      int x0 = 0, y0 = 0;
      strip_origin(tile, w, ntx, rows, x0, y0);
      if (y0 < p.ny && x0 < p.nx)
        out[size_t(tile) * kStrips + w] = p.row_slot[size_t(y0) * nsx + x0 / kStripW];
    }
}

void apply_delta(Plan& p, const PlanDelta& d, bool forward) {
  for (size_t j = 0; j < d.idx.size(); ++j)
    p.node[size_t(d.idx[j])] = forward ? d.new_w[j] : d.old_w[j];
}

void undo_replan(Plan& p, Plan& np, const PlanDelta& d) {
  p.node.swap(np.node);
  apply_delta(p, d, false);
}

void build_adjoint_codes(const Plan& p, std::vector<uint32_t>& adj) {
  adj.assign(p.node.size(), 0u);
  for (int y = 0; y < p.ny; ++y)
    for (int x = 0; x < p.nx; ++x) {
      const uint32_t w = p.node[size_t(y) * p.nx + x];
      if (w & kSolidBit) continue;
      for (int i = 1; i < kQ; ++i) {
        const uint32_t c = pull_code(w, i);
        int sx = x - kCx[i], sy = y - kCy[i];
        sx = (sx + p.nx) % p.nx;
        sy = (sy + p.ny) % p.ny;
        uint32_t bit = 0;
        if (c == kStream) {
          bit = kAdjStream;
        } else if (c == kWrap) {
          bit = kAdjWrap;
        } else if (c == kOutlet) {
          bit = kAdjOutlet;
          sx = p.nx - 1;
        } else {
          continue;  // bounce-back: read back from the node itself
        }
        adj[size_t(sy) * p.nx + sx] |= bit << (3 * (i - 1));
      }
    }
}

}  // namespace lbm

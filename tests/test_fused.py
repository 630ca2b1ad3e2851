"""Three steps per launch (the fused kernel): its cut of the grid on the CPU, and on the GPU
bitwise equality with single steps.

lbm_step takes the fused kernel on grids large enough to gain from it, for runs of three steps or
more; calls of one or two steps always take the single-step kernel, so a run in such calls is
the reference.  States are bitwise alike whatever the calls, and so are the momentum-exchange and
stress forces; the control-volume forces of a call's last step read a separately ordered sum
of the box momentum, so they agree to binary64 rounding of that sum."""
import os
import re
import subprocess

import numpy as np
import pytest

import workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2210_10377_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "plan.h"
using namespace lbm;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (%dx%d bc %d%d esz %d)\n", __LINE__, #c, g.nx, g.ny, g.bc_x, g.bc_y, esz); return 1; } } while (0)
int main() {
  std::mt19937 rng(7);
  auto pick = [&](int lo, int hi) { return lo + int(rng() % unsigned(hi - lo + 1)); };
  for (int it = 0; it < 600; ++it) {
    lbm_grid g{};
    const int big[] = {3, 4, 17, 63, 64, 65, 127, 128, 129, 200, 333, 700};
    g.nx = it % 3 ? big[pick(0, 11)] : pick(3, 500);
    g.ny = it % 5 ? pick(3, 90) : big[pick(0, 8)];
    g.bc_x = pick(0, 1);
    g.bc_y = pick(0, 1);
    g.precision = LBM_FP32;
    g.tile = pick(0, 2);
    for (int k = 0; k < 4; ++k) g.box[k] = -1;
    std::vector<uint8_t> mask(size_t(g.nx) * g.ny, 0);
    const int kind = pick(0, 3);
    if (kind >= 1) {
      const int n = kind == 3 ? g.nx * g.ny / 10 : 1 + pick(0, 3);
      for (int k = 0; k < n; ++k) mask[size_t(pick(0, g.ny - 1)) * g.nx + pick(0, g.nx - 1)] = 1;
    }
    if (kind == 2 && g.nx > 12 && g.ny > 12) {
      std::fill(mask.begin(), mask.end(), 0);
      const int x = pick(3, g.nx - 5), y = pick(3, g.ny - 5);
      mask[size_t(y) * g.nx + x] = 1;
      g.box[0] = x - 2; g.box[1] = x + 3; g.box[2] = y - 2; g.box[3] = y + 3;
    }
    Plan p;
    std::string err;
    int esz = 8;
    if (build_plan(g, mask.data(), p, err) != LBM_OK) continue;
    for (int e = 0; e < 3; ++e) {
      esz = e == 0 ? 8 : (e == 1 ? 4 : 2);
      const FuseMap m = fuse_map(p, esz, int64_t(pick(0, 1) ? 1 : 50000) * g.nx * g.ny);
      CHECK(m.nrects <= kFuseRects && m.nrects >= 1);
      std::vector<int> owner(mask.size(), 0), kindof(mask.size(), -1);
      int blocks = 0;
      for (int k = 0; k < m.nrects; ++k) {
        const FuseRect& r = m.r[k];
        CHECK(r.x0 >= 0 && r.x0 < r.x1 && r.x1 <= g.nx && r.y0 >= 0 && r.y0 < r.y1 && r.y1 <= g.ny);
        CHECK(r.first == blocks && r.rows >= 1);
        const int per = r.kind == kFuseBody ? kStripW : (r.kind == kFuseEdge ? kFuseEdgeW : kFuseLanes * 8 / esz);
        if (r.kind == kFuseSides) CHECK(r.nw == 1);
        else CHECK(r.nw == (r.x1 - (r.kind == kFuseBody ? r.x0 / kStripW * kStripW : r.x0) + per - 1) / per);
        const int units = r.nw * ((r.y1 - r.y0 + r.rows - 1) / r.rows);
        const int in = r.kind == kFuseBody ? kStrips / 2 : kStrips;
        blocks += (units + in - 1) / in;
        if (r.kind == kFuseBody) CHECK(k == 0 && r.x0 % kHalf == 0 && (r.x1 % kHalf == 0 || r.x1 == g.nx));
        if (r.kind == kFusePlain) CHECK(r.x0 * esz % 64 == 0);
        if (r.kind == kFuseSides) {
          // Both sides and their margins in lanes of their own.
          CHECK(r.x0 + kFuseM <= kSideRight);
          CHECK(kSideRight + kFuseM + (g.nx - r.x1) + kFuseM <= 64 - kFuseM);
        }
        for (int y = r.y0; y < r.y1; ++y)
          for (int x = r.kind == kFuseSides ? 0 : r.x0; x < (r.kind == kFuseSides ? g.nx : r.x1); ++x) {
            if (r.kind == kFuseSides && x >= r.x0 && x < r.x1) continue;
            ++owner[size_t(y) * g.nx + x];
            kindof[size_t(y) * g.nx + x] = r.kind;
          }
      }
      CHECK(blocks == m.nblocks);
      const int nsx = (g.nx + kStripW - 1) / kStripW;
      for (int y = 0; y < g.ny; ++y)
        for (int x = 0; x < g.nx; ++x) {
          const size_t at = size_t(y) * g.nx + x;
          CHECK(owner[at] == 1);                                // every node once
          // A node with a force term lies in the body rectangle.
          bool term = p.has_box && x >= p.box[0] - 1 && x <= p.box[1] && y >= p.box[2] - 1 && y <= p.box[3];
          for (int i = 1; i < kQ; ++i)
            term = term || (!(p.node[at] & kSolidBit) && pull_code(p.node[at], i) == kBody);
          if (term) CHECK(kindof[at] == kFuseBody);
          if (term) CHECK(p.row_slot[size_t(y) * nsx + x / kStripW] >= 0);
          // Within the margin of a node outside the body rectangle every code is the edge's;
          // around a plain node all stream.
          if (kindof[at] == kFuseBody) continue;
          const int mar = kFuseM;
          for (int dy = -mar; dy <= mar; ++dy)
            for (int dx = -mar; dx <= mar; ++dx) {
              int ax = x + dx, ay = y + dy;
              if (g.bc_x == LBM_BCX_PERIODIC) ax = ((ax % g.nx) + g.nx) % g.nx;
              if (g.bc_y == LBM_BCY_PERIODIC) ay = ((ay % g.ny) + g.ny) % g.ny;
              const bool out = ax < 0 || ax >= g.nx || ay < 0 || ay >= g.ny;
              if (kindof[at] == kFusePlain) CHECK(!out && p.node[size_t(ay) * g.nx + ax] == 0u);
              if (!out) CHECK(p.node[size_t(ay) * g.nx + ax] == edge_word(g.nx, g.ny, g.bc_x, g.bc_y, ax, ay));
            }
        }
    }
  }
  std::printf("ok\n");
  return 0;
}
"""


def test_work_map_owns_every_node_once_and_keeps_its_margins(tmp_path):
    """Random grids, masks, boundary codes and storages: every node in one rectangle, every
    strip with forces in the body rectangle, edge codes only within the margins of the other
    nodes, plain streaming only around the plain ones."""
    src = tmp_path / "driver.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "driver"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                           "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src),
                           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr


# The driver with a grid that the planner accepts (it refuses one without room for a force row),
# counting the plans that are built and the kinds of rectangle that occur, and its verdict.
COUNTED = (DRIVER
           .replace("  std::mt19937 rng(7);", "  std::mt19937 rng(7);\n  int built = 0, kinds[4] = {};")
           .replace("    g.tile = pick(0, 2);", "    g.tile = pick(0, 2);\n    g.max_record = 1;")
           .replace("    for (int e = 0; e < 3; ++e) {", "    ++built;\n    for (int e = 0; e < 3; ++e) {")
           .replace("        const FuseRect& r = m.r[k];", "        const FuseRect& r = m.r[k];\n        ++kinds[r.kind];")
           .replace('  std::printf("ok\\n");',
                    '  std::printf("%d %d %d %d %d\\n", built, kinds[0], kinds[1], kinds[2], kinds[3]);'))


def _run_map_driver(tmp_path, text):
    src = tmp_path / "driver.cpp"
    src.write_text(text)
    exe = tmp_path / "driver"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined",
                           "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src),
                           os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)


def test_work_map_checks_are_made_on_built_plans(tmp_path):
    """The same checks of the work map, over plans that are built: all 600, with rectangles of
    every kind among them."""
    out = _run_map_driver(tmp_path, COUNTED)
    assert out.returncode == 0, out.stdout + out.stderr
    built, *kinds = (int(v) for v in out.stdout.split())
    assert built == 600 and min(kinds) >= 100, (built, kinds)


def test_work_map_checks_notice_a_margin_too_small(tmp_path):
    """With one node of margin more asked for than the map has, the checks fail: they see where
    its rectangles end."""
    wider = COUNTED.replace("const int mar = kFuseM;", "const int mar = kFuseM + 1;")
    assert wider != COUNTED
    out = _run_map_driver(tmp_path, wider)
    assert out.returncode == 1 and out.stdout.startswith("line "), out.stdout + out.stderr


# One node's collision and rounding in every storage, for the BGK (0) and entropic (2) operators.
COLLIDE = r"""
#include "force_terms.h"
using namespace lbm;
using namespace lbm::dev;
template <int P, int COLL>
__global__ void node(StepArgs a, const typename Storage<P>::T* in, typename Storage<P>::T* out) {
  typename Storage<P>::C f[kQ];
  typename Storage<P>::T s[kQ];
  for (int i = 0; i < kQ; ++i) f[i] = unpack<P>(in[i * 64 + threadIdx.x], i);
  collide_pack<P, COLL>(a, f, a.step_key, int(threadIdx.x), 0, s);
  for (int i = 0; i < kQ; ++i) out[i * 64 + threadIdx.x] = s[i];
}
#define ALL(P) template __global__ void node<P, @>(StepArgs, const Storage<P>::T*, Storage<P>::T*);
ALL(LBM_FP64) ALL(LBM_FP32) ALL(LBM_FP32DEV) ALL(LBM_FP32SR) ALL(LBM_FP16DEV)
"""


@pytest.mark.parametrize("collision", ["LBM_COLL_BGK", "LBM_COLL_KBC"])
def test_collisions_leave_no_fused_operation_to_the_compiler(tmp_path, collision):
    """Kernels of one and of several steps give the same bits only if the collision names its
    fused operations: compiled with the build's flags it then has the arithmetic instructions
    that it has where the compiler may fuse none."""
    from paper_2210_10377_amd import build
    src = tmp_path / "node.hip"
    src.write_text(COLLIDE.replace("@", collision))
    counts = []
    for extra in ([], ["-ffp-contract=off"]):
        out = tmp_path / ("node%d.s" % len(extra))
        subprocess.check_call(["hipcc", *build._flags(), *extra, "-S", "--cuda-device-only", str(src),
                               "-o", str(out)], stderr=subprocess.DEVNULL)
        ops = re.findall(r"^\s+v_(add|sub|subrev|mul|fma|fmac|fmamk|fmaak|fma_mix|fma_mixlo|mad|mac)"
                         r"_(f16|f32|f64)", out.read_text(), re.M)
        fused = [("fma" if op.startswith(("fma", "mad", "mac")) else "other", t) for op, t in ops]
        counts.append({k: fused.count(k) for k in set(fused)})
    assert sum(counts[0].values()) > 500 and counts[0] == counts[1], counts


def test_tile_kernels_are_those_that_the_rule_can_take():
    """tile_rows never picks tiles for the regularized collision, whose rounding differs between
    kernels: the library holds tile kernels of the BGK and entropic collisions only (5 storages,
    with and without forces and motion, 2 heights each)."""
    from paper_2210_10377_amd import _capi as C
    names = subprocess.run(["nm", "-C", C.LIB_PATH], capture_output=True, text=True, check=True).stdout
    got = set(re.findall(r"__device_stub__tile_kernel<(\d), (\w+), (\d), (\w+), (\d)>", names))
    assert len(got) == 80 and {g[2] for g in got} == {str(C.LBM_COLL_BGK), str(C.LBM_COLL_KBC)}, sorted(got)


# The form that the planner picks for a lattice or a batch of equal ones, each with a small body.
FORM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "plan.h"
using namespace lbm;
int main() {
  int count, nx, ny, precision, collision, forces, moving, side;
  while (std::scanf("%d %d %d %d %d %d %d %d", &count, &nx, &ny, &precision, &collision, &forces, &moving,
                    &side) == 8) {
    lbm_grid g{};
    g.nx = nx;
    g.ny = ny;
    g.precision = precision;
    g.collision = collision;
    g.max_record = 1;
    for (int k = 0; k < 4; ++k) g.box[k] = -1;
    std::vector<uint8_t> mask(size_t(nx) * ny, 0);
    const int w = std::max(1, std::min(side, nx / 3)), h = std::max(1, std::min(side, ny / 3));
    for (int y = ny / 2; y < ny / 2 + h; ++y)
      for (int x = nx / 4; x < nx / 4 + w; ++x) mask[size_t(y) * nx + x] = 1;
    if (nx >= 12 && ny >= 12) {
      g.box[0] = std::max(1, nx / 4 - 2);
      g.box[1] = std::min(nx - 1, nx / 4 + w + 2);
      g.box[2] = std::max(1, ny / 2 - 2);
      g.box[3] = std::min(ny - 1, ny / 2 + h + 2);
    }
    Plan p;
    std::string err;
    if (build_plan(g, mask.data(), p, err) != LBM_OK) return 1;
    const int esz = precision == LBM_FP64 ? 8 : (precision == LBM_FP16DEV ? 2 : 4);
    if (count == 1) {
      const FuseMap m = step_map(p, precision, collision, forces != 0, esz, moving != 0);
      std::printf("%s\n", m.nblocks == 0 ? "single" : (m.tile_rows ? "tiles" : "windows"));
      continue;
    }
    StepWork one, all;
    one.add(p, fuse_map(p, esz, int64_t(count) * nx * ny), esz);
    for (int k = 0; k < count; ++k) all.add(p, fuse_map(p, esz, int64_t(count) * nx * ny), esz);
    if (all.nodes != count * one.nodes || one.nodes != double(nx) * ny) return 1;
    std::printf("%s\n", fuse_pays(precision, collision, forces != 0, all, moving != 0, true) ? "windows" : "single");
  }
  return 0;
}
"""
# (lattices, columns, rows, storage, collision, forces, form): where one form was measured to be
# faster than single steps, or slower, by 8 % or more (us a step single : the other form named).
FORMS = [
    (1, 16, 40000, "fp64", "bgk", 1, "single"),        # 33 : 51 windows
    (1, 16, 40000, "fp32", "bgk", 0, "single"),        # 21 : 29 windows
    (1, 37, 14000, "fp32", "bgk", 1, "single"),        # 15 : 25 windows
    (1, 64, 100000, "fp32", "bgk", 1, "single"),       # 91 : 129 windows
    (1, 3, 60000, "fp64", "bgk", 1, "single"),         # 48 : 59 tiles
    (1, 3, 60000, "fp32", "bgk", 0, "single"),         # 31 : 39 tiles
    (1, 9, 20000, "fp32", "bgk", 1, "single"),         # 14.6 : 18.0 tiles
    (1, 16, 12000, "fp32sr", "kbc", 1, "single"),      # 13.4 : 17.7 tiles
    (1, 3, 60000, "fp16dev", "kbc", 0, "single"),      # 35 : 51 tiles
    (1, 200, 80, "fp64", "kbc", 0, "single"),          # 4.1 : 4.9 tiles
    (1, 724, 206, "fp32sr", "kbc", 0, "single"),       # 5.2 : 6.0 tiles
    (1, 724, 362, "fp32", "kbc", 1, "single"),         # 7.9 : 8.9 tiles
    (1, 200, 80, "fp64", "bgk", 1, "tiles"),           # 5.2 : 3.4
    (1, 512, 256, "fp32", "bgk", 0, "tiles"),          # 3.9 : 2.7
    (1, 512, 256, "fp64", "kbc", 0, "tiles"),          # 5.7 : 4.2
    (1, 600, 300, "fp32", "bgk", 1, "tiles"),          # 7.5 : 5.8
    (1, 37, 12500, "fp64", "bgk", 1, "tiles"),         # 19.4 : 16.0
    (1, 2048, 1024, "fp64", "bgk", 1, "windows"),      # 52 : 29
    (1, 2048, 1024, "fp32", "bgk", 1, "windows"),      # 27 : 17
    (1, 8192, 4096, "fp32dev", "bgk", 0, "windows"),   # 390 : 164
    (1, 100000, 64, "fp32", "bgk", 1, "windows"),      # 80 : 41
    (1, 20000, 24, "fp64", "bgk", 0, "windows"),       # 14.5 : 6.9
    (1, 170003, 3, "fp32", "bgk", 0, "windows"),       # 8.5 : 6.5
    (1, 2200, 1100, "fp32sr", "bgk", 0, "single"),     # 30.6 : 33.3 windows
    (1, 3000, 1500, "fp16dev", "bgk", 1, "single"),    # 31 : 38 windows
    (1, 2048, 1024, "fp32", "regularized", 0, "single"),
    (1000, 64, 32, "fp64", "bgk", 1, "single"),        # 80 : 134 windows
    (1000, 64, 32, "fp32", "bgk", 0, "single"),        # 30 : 60
    (300, 64, 64, "fp32", "bgk", 1, "single"),         # 40 : 50
    (64, 40, 400, "fp64", "bgk", 1, "single"),         # 39 : 52
    (300, 33, 100, "fp32", "bgk", 1, "single"),        # 37 : 50
    (128, 96, 64, "fp32", "bgk", 0, "single"),         # 14.4 : 16.8
    (16, 400, 200, "fp32", "bgk", 0, "windows"),       # 19.1 : 14.3
    (8, 700, 350, "fp64", "bgk", 1, "windows"),        # 54 : 33
    (128, 96, 64, "fp64", "bgk", 0, "windows"),        # 26.4 : 22.4
    (1, 130, 156, "fp64", "kbc", 0, "tiles"),          # 4.4 : 3.5 (two columns in the last strip)
    (1, 490, 491, "fp32", "bgk", 0, "tiles"),          # two rounds of blocks
    (1, 515, 234, "fp64", "kbc", 0, "single"),         # 1.33 of it tiles
    (1, 515, 293, "fp32", "kbc", 0, "tiles"),
    (1, 1020, 317, "fp32", "bgk", 0, "single"),        # 7.0 : 7.7 windows
]
# Bodies of the given side, at rest and in motion (the same with their forms).
MOVING = [
    (1, 850, 531, "fp32", "bgk", 1, 44, "windows", "single"),    # 10.1 : 10.0, 10.7 : 12.6
    (1, 1700, 212, "fp32", "bgk", 1, 70, "tiles", "single"),     # 9.9 : 9.4, 9.6 : 10.7
    (1, 600, 300, "fp16dev", "bgk", 0, 20, "tiles", "single"),   # 4.0 : 3.8, 4.0 : 4.3
    (1, 2048, 1024, "fp32", "bgk", 1, 60, "windows", "windows"),
    (62, 200, 80, "fp32", "bgk", 1, 26, "single", "windows"),    # 22 : 28, 42 : 31
]


def test_form_goes_by_the_work_that_a_shape_leaves(tmp_path):
    """Narrow lattices, lattices that are all edges and batches of small members take the form
    that is faster for them: node counts alone do not tell."""
    from paper_2210_10377_amd.sim import COLLISIONS, PRECISIONS
    src = tmp_path / "form.cpp"
    src.write_text(FORM)
    exe = tmp_path / "form"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                           str(src), os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    cases = [case[:6] + (0, 12, case[-1]) for case in FORMS]
    for case in MOVING:
        cases += [case[:6] + (moving, case[6], case[7 + moving]) for moving in (0, 1)]
    lines = "".join("%d %d %d %d %d %d %d %d\n" % (n, nx, ny, PRECISIONS[p], COLLISIONS[c], f, moving, side)
                    for n, nx, ny, p, c, f, moving, side, _ in cases)
    out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, timeout=120)
    got = out.stdout.split()
    assert out.returncode == 0 and len(got) == len(cases)
    wrong = [(case, form) for case, form in zip(cases, got) if case[-1] != form]
    assert not wrong, wrong


def _case(name):
    z = lambda nx, ny: np.zeros((ny, nx), np.uint8)  # noqa: E731
    if name == "airfoil":            # 725 x 701, the box inside the grid
        w = workloads.naca_channel(725, 701, 181, 4.0, 500.0, 1)
        return w.mask, w.box
    if name == "two_bodies":         # at the outlet, at a wall and across the wrap; no box
        m = z(803, 640)
        m[300:320, 802] = 1
        m[0:3, 90:100] = 1
        m[400:405, 0:2] = 1
        return m, None
    if name == "thin_rows":          # three rows that are all edges
        return z(170003, 3), None
    if name == "narrow":             # narrower than a wave
        m = z(37, 14000)
        m[5000:5010, 12:20] = 1
        return m, workloads.default_box(m, 4)
    if name in ("cylinder_4m", "cylinder_15m"):  # large enough for the other storages
        nx, ny = (2803, 1499) if name == "cylinder_4m" else (6007, 2501)
        m = workloads.cylinder_mask(nx, ny, 900.0, 749.5, 60.5)
        return m, workloads.default_box(m, 20)
    raise KeyError(name)


CASES = [("airfoil", p, bx, by, c, s) for p in ("fp64", "fp32", "fp32dev")
         for bx, by, c, s in ((0, 0, "bgk", 0.0), (1, 1, "bgk", 1e-3))]
CASES += [("two_bodies", p, bx, by, "bgk", 0.0) for p in ("fp64", "fp32")
          for bx, by in ((0, 0), (1, 0), (0, 1), (1, 1))]
CASES += [("thin_rows", "fp32", bx, by, "bgk", 0.0) for bx, by in ((0, 0), (1, 1))]
CASES += [("narrow", p, 0, 0, "bgk", 0.0) for p in ("fp64", "fp32dev")]
CASES += [("cylinder_4m", "fp32sr", 0, 1, "bgk", 0.0), ("cylinder_15m", "fp16dev", 0, 1, "bgk", 0.0)]


@pytest.mark.gpu
@pytest.mark.parametrize("name,precision,bc_x,bc_y,collision,spin", CASES)
def test_fused_launches_bitwise_equal_single_steps(name, precision, bc_x, bc_y, collision, spin):
    from paper_2210_10377_amd import Sim
    mask, box = _case(name)
    ny, nx = mask.shape
    rng = np.random.default_rng(5)
    uin = 0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny))
    lines = 1 + 0.02 * rng.uniform(-1, 1, (9, ny, 1)) * rng.uniform(-1, 1, (9, 1, nx))
    S = workloads.NEAR_REST_BASE[:, None, None] * lines
    n = 7  # a single step and two fused launches
    runs = []
    for calls in ([n], [2, 2, 2, 1]):
        print(f"fused {name} {precision} bc {bc_x}{bc_y} {collision} calls {calls}", flush=True)
        sim = Sim(mask, 0.7, uin, precision=precision, bc_x=bc_x, bc_y=bc_y, box=box,
                  max_record=n, collision=collision)
        sim.set_populations(S)
        if spin:
            sim.set_body_motion(ux=0.01, omega=spin / 100, xc=nx / 3, yc=ny / 2)
        for k in calls:
            sim.step(k)
        runs.append((sim.populations(), sim.forces()))
        del sim
    (P0, F0), (P1, F1) = runs
    assert np.array_equal(P0, P1)
    assert np.array_equal(F0[:, [0, 1, 3]], F1[:, [0, 1, 3]])
    if box is not None:
        # The box momentum J sums up to N values of at most 0.45 a population: its rounding is
        # below N 2^-53 0.45 in any order, and a row holds two of them.
        N = (box[1] - box[0]) * (box[3] - box[2]) * 9
        assert np.abs(F0 - F1).max() <= 4 * N * 0.45 * 2.0 ** -53


# Tiles: columns and rows around the sizes of a tile (64, 4 and 8 rows), 380 blocks of 4 rows.
TILE_SIZES = [(5, 3), (63, 4), (65, 9), (130, 17), (200, 80), (600, 150)]


@pytest.mark.gpu
@pytest.mark.parametrize("precision,bc_x,bc_y,collision,spin", [
    ("fp64", 0, 0, "bgk", 0), ("fp64", 1, 1, "kbc", 0), ("fp32", 0, 1, "kbc", 1),
    ("fp32", 1, 0, "bgk", 0), ("fp32dev", 0, 0, "bgk", 1), ("fp32sr", 0, 0, "bgk", 0),
    ("fp32sr", 1, 0, "kbc", 0), ("fp16dev", 0, 1, "bgk", 1), ("fp16dev", 0, 0, "kbc", 0),
    ("fp32dev", 1, 1, "kbc", 0)])
def test_tiles_bitwise_equal_single_steps(precision, bc_x, bc_y, collision, spin):
    """Calls of 7 steps (a single step and two launches of three) against calls of one and two
    steps: bitwise, the forces included, as every strip sums in the same order; except DRTT,
    whose J of the step after a call comes from a sweep over the box in another order (bound as
    above)."""
    from paper_2210_10377_amd import Sim
    rng = np.random.default_rng(6)
    for nx, ny in TILE_SIZES:
        mask = np.zeros((ny, nx), np.uint8)
        box = None
        if nx >= 65:
            mask[ny // 2 - 1:ny // 2 + 2, nx // 2:nx // 2 + 5] = 1
            box = (nx // 2 - 3, nx // 2 + 9, ny // 2 - 3, ny // 2 + 4)
            if nx >= 200:
                box = (nx // 5, nx - 5, 2, ny - 2)  # strips wholly inside it
        else:
            mask[1, 2] = 1
        uin = 0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny))
        S = workloads.NEAR_REST_BASE[:, None, None] * (
            1 + 0.02 * rng.uniform(-1, 1, (9, ny, 1)) * rng.uniform(-1, 1, (9, 1, nx)))
        runs = []
        for calls in ([7], [2, 2, 2, 1]):
            print(f"tiles {nx}x{ny} {precision} bc {bc_x}{bc_y} {collision} {calls}", flush=True)
            sim = Sim(mask, 0.7, uin, precision=precision, bc_x=bc_x, bc_y=bc_y, box=box,
                      max_record=7, collision=collision)
            sim.set_populations(S)
            if spin:
                sim.set_body_motion(ux=0.01, omega=1e-4, xc=nx / 3, yc=ny / 2)
            for k in calls:
                sim.step(k)
            runs.append((sim.populations(), sim.forces()))
            del sim
        (P0, F0), (P1, F1) = runs
        np.testing.assert_array_equal(P0, P1)
        np.testing.assert_array_equal(F0[:, [0, 1, 3]], F1[:, [0, 1, 3]])
        if box is not None:
            N = (box[1] - box[0]) * (box[3] - box[2]) * 9
            assert np.abs(F0 - F1).max() <= 4 * N * 0.45 * 2.0 ** -53


BATCH_WORK = r"""
#include <algorithm>
#include <cstdio>
#include <set>
#include <string>
#include <utility>
#include <vector>
#include "plan.h"
using namespace lbm;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
static Plan lattice(int nx, int ny, int x, int y, bool body) {
  lbm_grid g{};
  g.nx = nx;
  g.ny = ny;
  g.precision = LBM_FP32;
  g.max_record = 1;
  for (int k = 0; k < 4; ++k) g.box[k] = -1;
  std::vector<uint8_t> mask(size_t(nx) * ny, 0);
  if (body) {
    for (int j = 0; j < 9; ++j)
      for (int i = 0; i < 9; ++i) mask[size_t(y + j) * nx + x + i] = 1;
    const int b[4] = {x - 3, x + 12, y - 3, y + 12};
    std::copy(b, b + 4, g.box);
  }
  Plan p;
  std::string err;
  build_plan(g, mask.data(), p, err);
  return p;
}
int main() {
  std::vector<Plan> m;
  for (int k = 0; k < 12; ++k) m.push_back(lattice(150 + 37 * k, 90 + 11 * k, 30 + k, 40, k % 4 != 3));
  int64_t nodes = 0;
  for (const Plan& p : m) nodes += int64_t(p.nx) * p.ny;
  BatchWork w(m.size());
  for (size_t i = 0; i < m.size(); ++i) CHECK(w.set(i, m[i], 4, nodes));
  w.list();
  auto whole = [&]() {  // every block of every map once, the longest kinds first
    std::set<std::pair<int, int>> seen;
    int last = 0;
    size_t blocks = 0;
    for (size_t k = 0; k < w.nblocks; ++k) {
      const FuseMap& f = w.map[w.inst[k]];
      int r = f.nrects - 1;
      while (r > 0 && w.local[k] < f.r[r].first) --r;
      if (w.local[k] < 0 || w.local[k] >= f.nblocks || f.r[r].kind < last) return false;
      if ((f.r[r].kind == kFuseBody) != (k < w.nbody)) return false;
      last = f.r[r].kind;
      if (!seen.insert({w.inst[k], w.local[k]}).second) return false;
    }
    for (const FuseMap& f : w.map) blocks += f.nblocks;
    return blocks == w.nblocks && w.inst.size() == w.local.size();
  };
  CHECK(whole());
  auto same = [&](const BatchWork& a) {
    bool maps = true;
    for (size_t i = 0; i < m.size(); ++i)
      for (int k = 0; k < a.map[i].nrects; ++k) {
        const FuseRect &p = a.map[i].r[k], &q = w.map[i].r[k];
        maps = maps && a.map[i].nrects == w.map[i].nrects && p.x0 == q.x0 && p.x1 == q.x1 && p.y0 == q.y0 &&
               p.y1 == q.y1 && p.kind == q.kind && p.rows == q.rows && p.nw == q.nw && p.first == q.first;
      }
    const StepWork s = a.total(), t = w.total();
    return maps && a.inst == w.inst && a.local == w.local && a.nbody == w.nbody && a.nblocks == w.nblocks &&
           s.plain == t.plain && s.coded == t.coded && s.body == t.body && s.body_nodes == t.body_nodes;
  };
  int kept = 0, listed = 0;
  for (int step = 0; step < 60; ++step) {  // bodies that move, appear and go, a node or many at a time
    const int i = step * 7 % 12;
    const int x = 30 + (step * 5) % 40, y = 40 + step % 3;
    m[i] = lattice(m[i].nx, m[i].ny, step % 2 ? 31 + i + step % 4 : x, y, step % 9 != 8);
    if (w.set(i, m[i], 4, nodes)) {
      w.list();
      ++listed;
    } else {
      ++kept;
    }
    BatchWork fresh(m.size());
    for (size_t k = 0; k < m.size(); ++k) fresh.set(k, m[k], 4, nodes);
    fresh.list();
    CHECK(same(fresh));
    CHECK(whole());
  }
  std::printf("%d %d\n", kept, listed);
  return 0;
}
"""


def test_batch_work_follows_one_member_at_a_time(tmp_path):
    """After a mask change of one member the maps and the list of blocks are those built from all
    members anew, and the list is kept where the member's blocks are as before."""
    src = tmp_path / "batch_work.cpp"
    src.write_text(BATCH_WORK)
    exe = tmp_path / "batch_work"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-I", CSRC,
                           "-I", os.path.join(ROOT, "include"), str(src), os.path.join(CSRC, "plan.cpp"),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    kept, listed = (int(v) for v in out.stdout.split())
    assert kept >= 10 and listed >= 10, (kept, listed)


def _small_body(nx, ny):
    """The body and control volume of FORM's lattices."""
    mask = np.zeros((ny, nx), np.uint8)
    w, h = max(1, min(12, nx // 6)), max(1, min(12, ny // 6))
    mask[ny // 2:ny // 2 + h, nx // 4:nx // 4 + w] = 1
    if nx < 12 or ny < 12:
        return mask, None
    return mask, (max(1, nx // 4 - 2), min(nx - 1, nx // 4 + w + 2),
                  max(1, ny // 2 - 2), min(ny - 1, ny // 2 + h + 2))


# Lattices that FORM's rule gives to windows, without forces and with them.
WINDOWS = [("fp64", 725, 701, 0), ("fp32", 725, 701, 0), ("fp32dev", 726, 703, 0), ("fp64", 1203, 605, 1),
           ("fp32", 1203, 605, 1), ("fp32", 170003, 3, 0), ("fp64", 20001, 24, 0), ("fp32sr", 2803, 1499, 0),
           ("fp32sr", 2803, 1499, 1), ("fp16dev", 6007, 2501, 0)]
# And to tiles: storage, collision, columns, rows, forces.
TILES = [(p, c, nx, ny, f) for p in ("fp64", "fp32", "fp32dev", "fp32sr", "fp16dev") for c in ("bgk", "kbc")
         for nx, ny in ((131, 17), (333, 60), (430, 250)) for f in (0, 1)]


def test_window_and_tile_cases_take_their_forms(tmp_path):
    """The lattices of the two tests below, by the planner's own rule."""
    from paper_2210_10377_amd.sim import COLLISIONS, PRECISIONS
    src = tmp_path / "form.cpp"
    src.write_text(FORM)
    exe = tmp_path / "form"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                           str(src), os.path.join(CSRC, "plan.cpp"), "-o", str(exe)])
    cases = [(1, nx, ny, PRECISIONS[p], 0, f, "windows") for p, nx, ny, f in WINDOWS]
    cases += [(1, nx, ny, PRECISIONS[p], COLLISIONS[c], f, "tiles") for p, c, nx, ny, f in TILES]
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d %d %d 0 12\n" % c[:6] for c in cases),
                         capture_output=True, text=True, timeout=120)
    got = out.stdout.split()
    wrong = [(c, g) for c, g in zip(cases, got) if c[6] != g]
    assert len(got) == len(cases) and not wrong, wrong


def _runs(precision, collision, nx, ny, bc, forces, spin, seed):
    """Populations and forces of 7 steps in one call and in calls of 2, 2, 2 and 1."""
    from paper_2210_10377_amd import Sim
    rng = np.random.default_rng(seed)
    mask, box = _small_body(nx, ny)
    uin = 0.05 * (1 + 0.1 * rng.uniform(-1, 1, ny))
    S = workloads.NEAR_REST_BASE[:, None, None] * (
        1 + 0.02 * rng.uniform(-1, 1, (9, ny, 1)) * rng.uniform(-1, 1, (9, 1, nx)))
    runs = []
    for calls in ([7], [2, 2, 2, 1]):
        print(f"{precision} {collision} {nx}x{ny} bc {bc} forces {forces} spin {spin} {calls}", flush=True)
        sim = Sim(mask, 0.55, uin, precision=precision, bc_x=bc[0], bc_y=bc[1], box=box, max_record=7,
                  collision=collision)
        sim.set_populations(S)
        if spin:
            sim.set_body_motion(ux=0.01, omega=1e-4, xc=nx / 3, yc=ny / 2)
        for k in calls:
            sim.step(k) if forces else sim.step(k, schemes=())
        runs.append((sim.populations(), sim.forces() if forces else None))
        del sim
    (P0, F0), (P1, F1) = runs
    np.testing.assert_array_equal(P0, P1)
    if forces:  # (DRTT as in the tests above)
        np.testing.assert_array_equal(F0[:, [0, 1, 3]], F1[:, [0, 1, 3]])
        if box is not None:
            N = (box[1] - box[0]) * (box[3] - box[2]) * 9
            assert np.abs(F0 - F1).max() <= 4 * N * 0.45 * 2.0 ** -53


@pytest.mark.gpu
@pytest.mark.parametrize("precision,nx,ny,forces", WINDOWS)
def test_windows_without_and_with_forces_bitwise_equal_single_steps(precision, nx, ny, forces):
    """Windows in every storage, also without forces: bounded, periodic and moving."""
    large = nx * ny > 3_000_000
    for bc, spin in ([((0, 0), 0)] if large else [((0, 0), 0), ((0, 1), 1), ((1, 0), 0)]):
        _runs(precision, "bgk", nx, ny, bc, forces, spin, 8)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32dev", "fp32sr", "fp16dev"])
@pytest.mark.parametrize("collision", ["bgk", "kbc"])
def test_tiles_without_and_with_forces_bitwise_equal_single_steps(precision, collision):
    """Tiles of both collisions in every storage, without forces and with them, of bodies at rest
    and in motion."""
    for p, c, nx, ny, forces in TILES:
        if (p, c) == (precision, collision):
            for bc, spin in (((0, 0), 0), ((0, 0), 1), ((1, 1), 0)):
                _runs(p, c, nx, ny, bc, forces, spin, 9)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32dev", "fp32sr"])
def test_kept_states_of_the_adjoint_equal_single_steps(precision):
    """Segments of two steps are recomputed by a single step each, longer ones by tiles that store
    every state: the objective and its gradients are bitwise alike."""
    import torch
    from paper_2210_10377_amd import Sim
    from paper_2210_10377_amd.autograd import ObjectiveSpec, objective
    for nx, ny in ((130, 37), (330, 90)):
        mask, box = _small_body(nx, ny)
        uin = 0.05 * (1 + 0.05 * np.random.default_rng(4).uniform(-1, 1, ny))
        got = []
        for every in (2, 11, 40):
            print(f"adjoint {precision} {nx}x{ny} every {every}", flush=True)
            sim = Sim(mask, 0.6, uin, precision=precision, box=box, max_record=8)
            u = torch.from_numpy(uin).cuda().requires_grad_()
            tau = torch.tensor(0.6, dtype=torch.float64, requires_grad=True)
            J = objective(u, tau, sim, ObjectiveSpec(40, every, 30, 10, (1.0, 0.25)))
            J.backward()
            got.append((J.item(), u.grad.cpu().numpy(), tau.grad.item()))
            del sim
        for J, g, t in got[1:]:
            assert J == got[0][0] and t == got[0][2]
            np.testing.assert_array_equal(g, got[0][1])

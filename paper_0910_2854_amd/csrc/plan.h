// plan.h -- how the sweeps of a table of boxes are cut into waves: the work shape
// of every kernel kind and each box's part of it.  Host arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <vector>

#include "layout.h"

namespace fish {

// What a plan takes from a box.
struct PlanBox {
  int n[3]{};
  int o[3]{};           // extra layer on outflow axes
  long long nelem = 0;  // elements per array
};

// The boxes of a table by form: boxes of the same cells and layers are planned
// together, so that a plan costs what the forms do and not what the boxes do
// (every change of the table makes one; 1000 boxes of 12^3: 4.1 ms with
// every segment length tried on every box, 0.02 ms so).
struct Forms {
  struct Form : PlanBox {
    long long count = 0;
    bool operator<(const Form& f) const {
      return std::lexicographical_compare(n, n + 3, f.n, f.n + 3) ||
             (std::equal(n, n + 3, f.n) && std::lexicographical_compare(o, o + 3, f.o, f.o + 3));
    }
  };
  std::vector<Form> forms;
  long long boxes = 0;

  void add(const PlanBox& b, long long count = 1) {
    boxes += count;
    if (!forms.empty() && std::equal(b.n, b.n + 3, forms.back().n) && std::equal(b.o, b.o + 3, forms.back().o)) {
      forms.back().count += count;
      return;
    }
    forms.emplace_back();
    static_cast<PlanBox&>(forms.back()) = b;
    forms.back().count = count;
  }
  // after the last box: equal forms that were not added one after another
  void merge() {
    if (forms.size() < 3) return;  // (of two, neither is the other)
    std::sort(forms.begin(), forms.end());
    std::vector<Form> all;
    all.swap(forms);
    boxes = 0;
    for (const Form& f : all) add(f, f.count);
  }
};

// Tuning targets per kernel kind: stream positions per wave for the x kinds
// (whole rows of the box fill it), the segment length along the sweep for
// the y/z kinds, cells per lane for the CFL check.
struct Tuning {
  int target[K_NUM];
  int remap[K_NUM];   // XCD-aware block order per kind (0/1)
  int groups[K_NUM];  // y/z kinds: waves of a block on consecutive rows; check kind: the
                      // step's CFL reduction in the check kernel instead of the last x
                      // sweep; x fluid kind: the strided layout (0/1)
};
inline Tuning default_tuning() {
  Tuning t;
  t.target[K_FLUID_X] = 1536;
  t.target[K_FIELD_X] = 384;
  t.target[K_FLUID_Y] = t.target[K_FLUID_Z] = 64;
  t.target[K_FIELD_Y] = t.target[K_FIELD_Z] = 64;
  t.target[K_CHECK] = 16;
  for (int k = 0; k < K_NUM; ++k) t.remap[k] = t.groups[k] = 0;
  // the y/z field sweeps read four neighbouring rows per row: 256^3 FP32
  // segments of 64, 145 -> 138 us (B_y) and 142 -> 134 us (B_z); 384^3 588 ->
  // 554 and 554 -> 520 us; the fluid sweeps read two, L_y 195 -> 206 us
  t.remap[K_FIELD_Y] = t.remap[K_FIELD_Z] = 1;
  return t;
}

inline long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }

// Waves of one box in the list of one kind, and the per-box parameter.
// Pencil waves of one segment of a y/z kind (strided_map's two orders).
inline long long strided_waves(long long nA, long long nO, int groups) {
  if (groups && nA >= 64) return ceil_div(nA, 64) * ceil_div(nO, 4) * 4;
  return ceil_div(nA * nO, 64);
}

inline long long kind_waves(const PlanBox& b, int kind, int target, int groups, int* par) {
  switch (kind) {
    case K_FLUID_X: {
      if (groups) {  // the strided policy along x: lanes along y, segments of the rows
        const int seg = std::max(1, std::min(target, b.n[0]));
        *par = seg;
        return strided_waves(b.n[1], b.n[2], groups) * ceil_div(b.n[0], seg);
      }
      const int rpw = std::max(1, target / (b.n[0] + 8));
      *par = rpw;
      return ceil_div((long long)b.n[1] * b.n[2], rpw);
    }
    case K_FIELD_X: {
      const int rpw = std::max(1, target / (b.n[0] + 8));
      *par = rpw;
      return ceil_div((long long)(b.n[1] + b.o[1]) * (b.n[2] + b.o[2]), rpw);
    }
    case K_FLUID_Y:
    case K_FLUID_Z: {
      const int D = kind - K_FLUID_X;
      const int seg = std::max(1, std::min(target, b.n[D]));
      *par = seg;
      return strided_waves(b.n[0], b.n[3 - D], groups) * ceil_div(b.n[D], seg);
    }
    case K_FIELD_Y:
    case K_FIELD_Z: {
      const int D = kind - K_FIELD_X;
      const int seg = std::max(1, std::min(target, b.n[D]));
      *par = seg;
      return strided_waves(b.n[0] + b.o[0], b.n[3 - D] + b.o[3 - D], groups) * ceil_div(b.n[D], seg);
    }
    default: {
      const int cpl = std::max(1, target);
      *par = cpl;
      return ceil_div((long long)b.n[0] * b.n[1] * b.n[2], 64ll * cpl);
    }
  }
}

// The work shape of a kind at its default, for the boxes of a table.  A launch
// of many waves takes the default as it is; a launch that leaves SIMDs idle is
// cut finer.
//   x kinds: halved while the boxes have fewer than 4096 waves, down to a row
// per wave (128^3 FP32 L_x: 35.2 us at 5 rows per wave, 32.7 at 2).
//   y/z kinds: a wave walks its segment and `halo` more positions, and a
// position takes it as long alone on its SIMD as `alone` waves that share one
// (latency against issue; more where the boxes come from HBM).  With fewer than
// 4096 waves at the default, the segment is the one whose rounds of resident
// waves take the shortest time.  Measured, L_z, at 64 halved to 2048 waves but
// no shorter than 8, and so: 32^3 FP32 18.0 -> 12.8 us (8 -> 2 cells), 64^3 FP32
// 20.0 -> 16.7 (8 -> 4), FP64 24.1 -> 21.2.  Boxes of several sizes are taken
// together, by the longest walk or the sum of the work.  The resident waves and
// `alone` are those of the plain scheme; FP64 with HSE, or with the
// loads ahead of the limiter switch and the irregular mesh, has one wave per SIMD
// and would take longer segments (L_y of 120^3 with HSE: 79 us at 32 cells, 91 at
// 16).
inline int planned_target(const Forms& table, int kind, int target, int groups, size_t esize) {
  int par = 1;
  auto waves_at = [&](int t) {
    long long w = 0;
    for (const Forms::Form& f : table.forms) w += f.count * kind_waves(f, kind, t, groups, &par);
    return w;
  };
  if (kind == K_CHECK) {
    while (target > 1 && waves_at(target) < 2048) target /= 2;
    return target;
  }
  if (kind == K_FIELD_X || (kind == K_FLUID_X && !groups)) {
    int lo = 0;
    for (const Forms::Form& f : table.forms) lo = std::max(lo, f.n[0] + 8);
    while (target / 2 >= lo && waves_at(target) < 4096) target /= 2;
    return target;
  }
  if (waves_at(target) >= 4096) return target;
  const int D = kind == K_FLUID_X ? 0 : kind <= K_FLUID_Z ? kind - K_FLUID_X : kind - K_FIELD_X;
  const int halo = kind <= K_FLUID_Z ? 6 : 8;
  long long bytes = 0;
  int longest_n = 1;
  std::vector<long long> segment_waves;
  for (const Forms::Form& f : table.forms) {
    bytes += 16ll * (long long)esize * f.nelem * f.count;
    longest_n = std::max(longest_n, f.n[D]);
    segment_waves.push_back(f.count * kind_waves(f, kind, f.n[D], groups, &par));
  }
  constexpr double kSimds = 1024.0;
  const double occupancy = esize == 8 ? 2.0 : 4.0;
  const double alone = (esize == 8 ? 1.15 : 1.75) * (bytes > (256ll << 20) ? 1.45 : 1.0);
  int best = target;
  double best_t = 0.0;
  for (int seg = target; seg >= 1; seg = std::min(seg, longest_n) - 1) {  // past the longest box all are alike
    double work = 0.0;
    long long w = 0;
    int longest = 0;
    for (size_t i = 0; i < segment_waves.size(); ++i) {
      const int n = table.forms[i].n[D], k = (n + seg - 1) / seg, even = (n + k - 1) / k;
      w += segment_waves[i] * k;
      work += (double)(segment_waves[i] * k) * (even + halo);
      longest = std::max(longest, even);
    }
    double t;
    if (table.boxes == 1) {
      const double n = std::ceil((double)w / kSimds), full = std::floor(n / occupancy), rest = n - full * occupancy;
      t = (longest + halo) * (full * std::max(alone, occupancy) + (rest > 0.0 ? std::max(alone, rest) : 0.0));
    } else {
      t = std::max((longest + halo) * alone, work / kSimds);
    }
    if (seg == target || t < best_t) {
      best_t = t;
      best = seg;
    }
  }
  return best;
}

// Segments per pencil of a y/z kind, ceil(n_d / segment length); 0 for the
// other kinds.
inline int kind_segments(const PlanBox& b, int kind, int par) {
  if (kind == K_FLUID_X) return (b.n[0] + par - 1) / par;  // read by the strided layout only
  if (kind == K_FLUID_Y || kind == K_FIELD_Y) return (b.n[1] + par - 1) / par;
  if (kind == K_FLUID_Z || kind == K_FIELD_Z) return (b.n[2] + par - 1) / par;
  return 0;
}

// Rows along the sweep of a y/z kind, the work of the lanes policy.
inline long long lane_rows(const PlanBox& b, int kind) {
  const bool field = kind >= K_FIELD_X;
  const int D = field ? kind - K_FIELD_X : kind - K_FLUID_X;
  const int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  return (long long)(b.n[t1] + (field ? b.o[t1] : 0)) * (b.n[t2] + (field ? b.o[t2] : 0));
}

// Whether a y/z kind takes the lanes policy: for boxes so small that a launch
// lasts as long as one wave's walk, which lanes along the sweep shorten to a
// window or two, and their uncoalesced accesses stay in the caches.  Double
// step, FP32, walks -> lanes of two cells: 32^3 113 -> 83 us (16^3 FP64 115 -> 70), 40^3 123
// -> 106, 48^3 128 -> 128, 56^3 147 -> 163, 64^3 161 -> 217.
//   The rows have to be short, since one is the least a wave gets: the four of a
// block are one window a wave up to 112 cells.  L_z, FP32, lanes and the best
// segments: 8x8 rows of 120 10.4 and 11.5 us, of 200 13.8 and 11.7, of 2000 (7x7)
// 131 and 13; FP64 12x12 rows of 130 13.3 and 13.7, of 400 29.6 and 15.4.  In y the
// lanes are n_x apart and share lines where that is little (and walks, whose lanes
// are along x, do not): n_x = 1, rows of 300 11.3 and 28.4, of 700 16.8 and 27.1;
// n_x = 3, rows of 300 11.9 and 16.7; n_x = 6, rows of 200 11.8 and 14.3; n_x = 4,
// rows of 500 19.6 and 14.2.
//   And there have to be few, since short ones leave three waves of a block without
// a window: L_y, FP64, 24000 rows of 4 24.6 us and in segments 16.2, 16000 of 6 18.6
// and 16.7, 14000 of 7 17.1 and 16.4 (the step of 2000x7x7 273 and 269 us, FP32
// 211 and 222).
inline int longest_lane_row(const PlanBox& b, int D) {
  if (D == 1 && b.n[0] <= 6) return b.n[0] == 1 ? 712 : b.n[0] <= 3 ? 352 : 232;
  return 128;
}
inline bool planned_lanes(const Forms& table, int kind) {
  if (kind == K_FLUID_X || kind == K_FIELD_X || kind == K_CHECK) return false;
  const int D = kind >= K_FIELD_X ? kind - K_FIELD_X : kind - K_FLUID_X;
  long long cells = 0, rows = 0;
  for (const Forms::Form& f : table.forms) {
    cells += f.count * f.n[0] * f.n[1] * f.n[2];
    rows += f.count * lane_rows(f, kind);
    if (f.n[D] < 4 || f.n[D] > longest_lane_row(f, D)) return false;
  }
  return cells <= 100000 && rows <= 14400;
}

// Segments of equal length (to a cell) instead of full ones and a remainder.
inline int even_segments(const PlanBox& b, int kind, int par) {
  const int k = kind_segments(b, kind, par);
  return k > 0 ? (b.n[kind <= K_FLUID_Z ? kind - K_FLUID_X : kind - K_FIELD_X] + k - 1) / k : par;
}

// How the boxes of a table are cut for a kind.
struct KindPlan {
  int target = 1;
  bool planned = false;  // the default target: the shape is planned
  bool lanes = false;    // y/z kinds: the lanes policy
};

// The default target of a kind stands for the shape planned for the boxes,
// whether it was left alone, set or found by the autotuner (whose output then
// sets it again); any other target is used as set.  A layout that is set keeps
// the kernel that has it: no lanes policy.
inline KindPlan plan_kind(const Forms& table, int kind, const Tuning& tuning, size_t esize) {
  KindPlan p;
  p.planned = table.boxes > 0 && tuning.target[kind] == default_tuning().target[kind];
  p.lanes = p.planned && !tuning.groups[kind] && planned_lanes(table, kind);
  p.target = tuning.target[kind];
  if (p.planned && !p.lanes) p.target = planned_target(table, kind, p.target, tuning.groups[kind], esize);
  return p;
}

// A box's part of a kind's list: BoxDesc::par and nseg, and its waves.
struct BoxShape {
  int par = 1, nseg = 0;
  long long waves = 0;
};

inline BoxShape box_shape(const PlanBox& b, int kind, const KindPlan& p, int groups) {
  BoxShape s;
  if (p.lanes) {
    s.waves = lane_rows(b, kind);
    return s;
  }
  s.waves = kind_waves(b, kind, p.target, groups, &s.par);
  if (p.planned && kind != K_FLUID_X) s.par = even_segments(b, kind, s.par);
  s.nseg = kind_segments(b, kind, s.par);
  return s;
}

// The variants of a kind that the autotuner times: the default target first, which
// stands for the planned shape, then set ones; each with both block orders and,
// for the y/z kinds, both pencil orders.  A variant that cuts every box as an
// earlier one does is left out.
struct Variant {
  int target, remap, groups;
};

inline std::vector<Variant> tuner_variants(const Forms& table, int kind, Tuning tuning, size_t esize) {
  const bool x = kind == K_FLUID_X || kind == K_FIELD_X;
  std::vector<int> targets = {default_tuning().target[kind]};
  for (int t : x ? std::vector<int>{256, 384, 512, 768, 1024, 1536, 2048, 3072, 4096, 6144}
                 : std::vector<int>{8, 16, 24, 32, 48, 64, 96, 128, 192, 256})
    if (t != targets[0]) targets.push_back(t);
  std::vector<Variant> out;
  std::vector<std::vector<long long>> seen;
  for (int t : targets)
    for (int g = 0; g < (x ? 1 : 2); ++g) {
      tuning.target[kind] = t;
      tuning.groups[kind] = g;
      const KindPlan p = plan_kind(table, kind, tuning, esize);
      std::vector<long long> cut = {g, p.lanes};
      for (const Forms::Form& f : table.forms) {
        const BoxShape s = box_shape(f, kind, p, g);
        cut.insert(cut.end(), {s.par, s.nseg, s.waves});
      }
      if (std::find(seen.begin(), seen.end(), cut) != seen.end()) continue;
      seen.push_back(cut);
      for (int r = 0; r < 2; ++r) out.push_back({t, r, g});
    }
  return out;
}

// A box alone in its table at the default tuning.  With more than max_waves
// waves the x field sweep takes several short rows per wave.
inline void plan_single_box(const int n[3], const int bc[3], size_t esize, long long max_waves, BoxShape shape[K_NUM],
                            bool lanes[K_NUM]) {
  PlanBox b;
  for (int a = 0; a < 3; ++a) {
    b.n[a] = n[a];
    b.o[a] = bc[a] == 1 ? 1 : 0;
  }
  b.nelem = (long long)(n[0] + b.o[0]) * (n[1] + b.o[1]) * (n[2] + b.o[2]);
  Forms table;
  table.add(b);
  const Tuning t = default_tuning();
  for (int k = 0; k < K_NUM; ++k) {
    KindPlan p = plan_kind(table, k, t, esize);
    shape[k] = box_shape(b, k, p, t.groups[k]);
    if (k == K_FIELD_X && shape[k].waves > max_waves) {
      p.target *= 2;
      shape[k] = box_shape(b, k, p, t.groups[k]);
    }
    lanes[k] = p.lanes;
  }
}

}  // namespace fish

// layout.h -- data structures shared by the host engine and the kernels:
// box geometry, per-box step scalars, the box table and the work lists.
#pragma once

namespace fish {

struct Geo {
  int n[3];
  int bc[3];          // 0 periodic, 1 outflow
  long long st[3];    // element strides, st[0] = 1
  double h[3];
};

// Device-resident step scalars.
struct Scalars {
  double dt;                    // step size of every sub-operator
  double t;                     // simulation time
  double t_end;                 // with has_end: the CFL step is clamped to land on t_end
  unsigned long long cmax_bits; // max CFL speed (FP64 bits; all values >= 0)
  int status;                   // sticky: 1 = bad state seen
  int has_end;
  int taken;                    // double steps taken with dt > 0
  int pad;
  double kh[3], kf[3];          // dt / (2 h_d) and dt / h_d per axis, set with dt
};

// ------------------------------------------------------------ work lists
// A launch covers every box of a batch.  Boxes live at element offset `off`
// of one pool per field; each kernel kind has a list giving the box of every
// wave, and the box gives the wave's position within it.  The box, its
// geometry and its offset are wave-uniform (scalar registers).
enum Kind { K_FLUID_X = 0, K_FLUID_Y, K_FLUID_Z, K_FIELD_X, K_FIELD_Y, K_FIELD_Z, K_CHECK, K_NUM };

struct BoxDesc {
  Geo g;
  long long off;      // element offset of the box in every pool
  double cfl;         // Courant number of Eq. (14)
  int slot;           // index of the box's Scalars
  int wave0[K_NUM];   // first wave of the box in each kind's list
  int par[K_NUM];     // lanes policy (x kinds, y/z kinds of small boxes): rows per wave; strided: segment length; check: cells per lane
  int nseg[K_NUM];    // strided policy: segments per pencil, ceil(n_d / par)
  long long woff[3];  // irregular meshes: element offset of the box's cell widths in each axis's width array
  double ih[3], i2h[3];  // 1 / h_d and 1 / (2 h_d)
};

// Whether the sweeps of boxes of `bytes` in all (both buffers) and rows of
// row_bytes treat what they touch once as streamed (WorkList::stream).  The
// rows have to be whole 128-byte lines: non-temporal stores of partly written
// lines are not merged (384^3 FP32 with rows of 385: 8.9 -> 9.5 ms per step).
// And the boxes have to outgrow the 256 MB cache of the memory, which otherwise
// holds one sweep's results for the next: per step, FP32, plain -> streamed,
// 128^3 (134 MB) 349 -> 381 us, 160^3 (262 MB) 600 -> 630, 192^3 (453 MB)
// 1041 -> 1001, 256^3 (1 GB) 2202 -> 2112.
inline bool stream_rule(long long bytes, long long row_bytes) {
  return row_bytes % 128 == 0 && bytes > (384ll << 20);
}

// Threads and waves of a block of every launch over a work list: constants,
// since the block and grid size of a running kernel are loads of its own.
constexpr int kBlock = 256;
constexpr int kBlockWaves = kBlock / 64;

// Whether the lanes policy gives a lane one cell of a row instead of two
// (WorkList::narrow): with no second wave for a SIMD (1024) a launch lasts as
// long as one window, which it halves, if a row still fits one (64 lanes with
// halos of 4).  Double step, two cells -> one: 16^3 FP64 59.5 -> 53.3 us, 24^3 74
// -> 66, 32^3 FP32 77.7 -> 71.8; but 40^3 (1600 waves) 97 -> 99 in y and z.
inline bool narrow_rule(long long waves, int longest_row) { return waves <= 1024 && longest_row <= 56; }
// The axis of a sweep kind's rows (0 for the check).
inline int kind_axis(int kind) {
  return kind >= K_FIELD_X && kind <= K_FIELD_Z ? kind - K_FIELD_X : kind <= K_FLUID_Z ? kind - K_FLUID_X : 0;
}

struct WorkList {
  const BoxDesc* boxes;
  const int* wave_box;  // table index of the box of every wave (not read with one)
  int one;              // 1: the table is one box, with its Scalars at slot (see work_item)
  int slot;
  int nwaves;
  int xcd_remap;        // 1: consecutive blocks of the list run on one XCD (see list_block)
  int reverse;          // 1: the blocks run from the last to the first (see list_block)
  int stream;           // 1: what a sweep reads or writes once passes the caches by (see ld_once)
  int row_groups;       // y/z kinds: 1 = a block's waves on consecutive rows (see strided_map)
  int lanes;            // y/z kinds: 1 = the lanes policy (par: rows per wave)
  int narrow;           // lanes policy: 1 = one cell per lane (narrow_rule)
};

}  // namespace fish

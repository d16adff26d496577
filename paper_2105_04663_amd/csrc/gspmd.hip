// C-ABI entry points of libgspmd (see include/gspmd.h) and the kernel launchers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "../../include/gspmd.h"
#include "kernels_basic.h"
#include "kernels_f32.h"
#include "launch.h"
#include "mfma_common.h"
#include "plan.h"
#include "testing.h"
#include "tile_index.h"

using namespace gspmd;

static_assert(kF32Tile == kGenTile && kF32Threads == 256, "dot_f32_kernel and dot_fallback_kernel share their tiles and launch");

namespace {

constexpr int64_t kWsAlign = 256;

// Workspace of gspmd_grouped_dot_noalloc: one copy per GPU the library is loaded on, held until the process ends.  In
// host code the array's name is only a handle: its device address is looked up once per device (scratch_address).
constexpr int64_t kScratchBytes = GSPMD_NOALLOC_MAX_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

void* scratch_address() {
  static std::once_flag once[kMaxDevices];
  static void* addr[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::call_once(once[dev], [dev] {
    void* p = nullptr;
    addr[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) == hipSuccess ? p : nullptr;
  });
  return addr[dev];
}

bool is_dtype(int32_t d) { return d == GSPMD_F32 || d == GSPMD_BF16; }

// A tensor with a zero-size dimension has no elements; its buffers may be null pointers.
bool has_no_elements(const gspmd_sharding* sh) {
  for (int i = 0; i < sh->rank; ++i) if (sh->global_shape[i] == 0) return true;
  return false;
}

int32_t check_buf(const gspmd_shard_buf* b) {
  if (!b) return GSPMD_ERR_NULL;
  if (!is_dtype(b->dtype)) return GSPMD_ERR_UNSUPPORTED;
  if (b->row_stride < 0) return GSPMD_ERR_BAD_BUFFER;
  return GSPMD_OK;
}

// Assign tile ids for tile edge (bm, bn) over the VALID extents; returns total tiles or -1 on overflow.  `chain`: of joined
// problems only the first has tiles (the ids after it start where its own end, so a search for the last entry that begins at
// or before an id never ends at the others).
int64_t assign_tiles(std::vector<Problem>& ps, int bm, int bn, bool chain = false) {
  int64_t t = 0;
  for (auto& p : ps) {
    const int64_t tm = (static_cast<int64_t>(p.Mv) + bm - 1) / bm, tn = (static_cast<int64_t>(p.Nv) + bn - 1) / bn;
    p.tile_begin = static_cast<int32_t>(t);
    p.tiles_n = static_cast<int32_t>(tn);
    if (!(chain && p.join_count > 1 && p.join_slot > 0)) t += tm * tn;
    if (t > INT32_MAX) return -1;
  }
  return t;
}

// Which contraction kernels a launch can take: those with direct global->LDS loads take rows of whole 32-bit words (even leading
// dimensions, pointers at multiples of 4 bytes), where a K-major operand's rows are not padded to 16 bytes only the rhs's and from one tile of
// columns on; the register-staged variant takes elements at any (even) address; longer rows (and fp32 operands) go to the scalar-FMA kernel.
enum KernelPath { kPathFallback = 0, kPathMfmaStaged = 1, kPathMfmaWords = 2, kPathMfmaDirect = 3 };

KernelPath kernel_path(const std::vector<Problem>& ps, int32_t in_dtype, int32_t layout, bool check_pointers = true) {
  if (in_dtype != GSPMD_BF16) return kPathFallback;
  // 32-bit byte offsets inside a tile: 256 rows of a K-contiguous operand (at most 64 in dot_split_kernel, 128 in dot_mid_kernel), 32 of
  // a K-major one
  const int32_t max_lda = (layout & GSPMD_LAYOUT_LHS_K_MAJOR) ? (1 << 24) : (1 << 22);
  const int32_t max_ldb = (layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) ? (1 << 22) : (1 << 24);
  KernelPath path = kPathMfmaDirect;
  for (const auto& p : ps) {
    const uintptr_t ptrs = check_pointers ? reinterpret_cast<uintptr_t>(p.A) | reinterpret_cast<uintptr_t>(p.B) : 0;
    if (p.lda > max_lda || p.ldb > max_ldb || (ptrs & 1)) return kPathFallback;
    const uintptr_t a = check_pointers ? reinterpret_cast<uintptr_t>(p.A) : 0, b = check_pointers ? reinterpret_cast<uintptr_t>(p.B) : 0;
    const bool a_loose = (a & 15) || (p.lda & 7), b_loose = (b & 15) || (p.ldb & 7);
    if (!a_loose && !b_loose) continue;
    const bool words = !((a | b) & 3) && !((p.lda | p.ldb) & 1) && !(a_loose && (layout & GSPMD_LAYOUT_LHS_K_MAJOR)) &&
                       !(b_loose && !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) && p.Nv < kMidTile);
    path = std::min(path, words ? kPathMfmaWords : kPathMfmaStaged);
  }
  return path;
}

// Run the contraction over all live tiles, then the zero fill of what the tiles do not cover.  Output tiles cover
// the valid extents only (rounded up to whole tiles, the kernel writes zeros inside a partly valid tile): tiles that
// would only write zeros are not interleaved with live ones, which would leave compute units idle (workgroups are
// placed in order), and cost no workgroup launches.  Tables of up to kInlineProblems problems and kInlineRects
// rectangles travel as kernel arguments; larger ones are uploaded into the workspace with a stream-ordered copy from
// a temporary host buffer (HIP stages a pageable source before the call returns).
// Where the MFMA kernel writes its per-workgroup timeline while gspmd_set_tile_timeline has one set (a profiling aid).
std::atomic<unsigned long long*> g_timeline{nullptr};
std::atomic<int> g_timeline_records{0};

// Workspace of a launch with joined problems: one arrival counter and join_count slots of kJoinSlotBytes per joined
// output tile.
constexpr int64_t kJoinSlotBytes = static_cast<int64_t>(kMfmaBM) * kMfmaBN * 4;
struct JoinSpace {
  uint32_t* counters = nullptr;
  float* partials = nullptr;
  int64_t tiles = 0;          // joined output tiles
  bool chain = false;         // dot_mid_kernel adds the members up in its registers: no counters, no slots
};

constexpr int64_t kJoinSlack = int64_t(64) << 20;
// counters of `tiles` joined output tiles, then `slots` slots
int64_t joined_bytes(int64_t tiles, int64_t slots) { return round_up(tiles * 4, kWsAlign) + slots * kJoinSlotBytes; }

int64_t tiles_of(const Problem& p, int bm, int bn) {
  return ((static_cast<int64_t>(p.Mv) + bm - 1) / bm) * ((static_cast<int64_t>(p.Nv) + bn - 1) / bn);
}

// Which kernel a bf16 launch takes, and dot_split_kernel's row blocks (of 16) per tile.
enum MfmaKernel : int32_t { kMfmaNone = GSPMD_TESTING_SCALAR, kMfmaBig = GSPMD_TESTING_MFMA, kMfmaMid = GSPMD_TESTING_MID, kMfmaSplit = GSPMD_TESTING_SPLIT, kMfmaPair = GSPMD_TESTING_PAIR };
struct MfmaChoice {
  MfmaKernel kernel;
  int row_blocks, col_blocks = 0;
  bool staged = false;      // dot_mfma_kernel, dot_mid_kernel: operands through registers
  bool loose = false;       // dot_pair_kernel: rows that are not padded to 16 bytes
};

// What this thread's launches are pinned to, and what its last one took (testing.h).
thread_local gspmd_testing_launch t_pin{GSPMD_TESTING_BY_RULE, 0, GSPMD_TESTING_BY_RULE, 0, 0, 0, 0, 0, 0};
thread_local gspmd_testing_launch t_last{GSPMD_TESTING_BY_RULE, 0, GSPMD_TESTING_BY_RULE, 0, 0, 0, 0, 0, 0};

// What a launch of dot_mfma_kernel or dot_mid_kernel takes, in us: straight lines through measured times.
// dot_mfma_kernel: rounds of 256 workgroups of 10 us and 1.3 us per 64-wide K step, where the chip is full and its clock drops, down to 0.85
//   in a round of few (short tiles: 0.75), 2 us for what is left of K.  From two full rounds on 1.25 us, and the last
//   round counts by its share, as the workgroups no longer start together.  Joined problems meet in slots: 4.6 us
//   per member, the last arriver at a tile reading the others' contributions one after the other, and 0.05 us per contribution to a tile, 0.1 beyond 256
//   (beyond the launch without: 2 members, 4 contributions 11 us; 2, 192: 17; 4, 24: 19; 4, 84: 25; 4, 256: 38; 8, 16: 38; 8, 512: 59).
// dot_mid_kernel: 2 us, and rounds of 512 workgroups of 4.5 us and 0.205 us per 32-wide step while a compute unit has one, 0.36 with two, 0.41 where the lhs is K-major; the members of
//   a joined sum follow each other in one workgroup, 1.8 us apart where they are not alike and whole K steps long; 0.25 us per 32-wide tile
//   that is left of K; in sums of more than one round of 512 0.44, and 0.30 in a last round of up to 256; a fifth more per step where a
//   K-contiguous operand's rows are not whole lines of 128 bytes (2112 x 8000 x 2112: 90 us, with rows of 8032 elements 117).  Fitted to drawn launches
//   together with dot_pair_kernel's line and the 256 x 256 tiles' 10 us; few of those had operands beyond 16 MB (drawn_us, below).  Over products drawn afresh the choice takes
//   0.8 % more than the best of all kernels pinned one after the other (150 experts' products), 1.3 % (50 of their weight gradients), 0.3 % and 1.5 % (80 feed-forward layers of up to
//   256 rows, 80 of more), 0.9 % (80 meshes of dense rows); 5.2 % where any extents are drawn (120, most of them of 4 to 12 us).
// Measured (one problem, M x K x N, us, dot_mfma_kernel / dot_mid_kernel): 2048 x 8192 x 2048: 120 / 62   512 x 8192 x 512: 117 / 45
//   2048 x 4096 x 4096: 66 / 60   2048 x 1024 x 4096: 22 / 19   4653 x 7168 x 4288: 255 / 267   1456 x 1415 x 3969, two of them: 38 / 45
//   2178 x 4736 x 1447, two: 76 / 72   1090 x 1333 x 1568, eight: 61 / 52   2112 x 8000 x 2112: 111 / 90   4096 x 512 x 8192, four, both K-major: 143 / 159
// Sums, slots / one after the other (K over all members): 2048 x 8192 x 2048 over 4: 78 / 64   1024 x 8192 x 2048 over 2, two groups: 75 / 59
//   both K-major 2085 x 3540 x 1652 over 2, two groups: 64 / 60   1770 x 3303 x 2085 over 2, two groups: 65 / 67   1572 x 4544 x 3328 over 8: 136 / 88
struct LaunchSize {
  int64_t rows = 0, k = 0, big = 0, mid = 0, pair = 0, members = 1;      // longest extents, tiles of 256 x 256, 128 x 128 and 256 x 128, most members of a sum
  int64_t cols = INT32_MAX, fewest_rows = INT32_MAX;
  int64_t loose_cols = INT32_MAX, loose_rows_of_lhs = INT32_MAX;      // fewest of a K-major operand whose rows are not padded to 16 bytes
  bool a_odd = false, b_odd = false;                           // an operand has elements at odd addresses
  int64_t in_bytes = 0;                                        // of the operands, each buffer once (one that comes round again in order, as on a mesh)
  bool broken_lines = false, whole_steps = true, whole_chunks = true;      // a K-contiguous operand's rows are not whole lines; all K are whole 64-wide steps
};
LaunchSize launch_size(const std::vector<Problem>& ps, int32_t layout) {
  LaunchSize s;
  bool a_again = false, b_again = false;
  for (const auto& p : ps) {
    const Problem* const before = &p > ps.data() ? &p - 1 : nullptr;
    if (!before || p.A != before->A) {
      a_again = a_again || (before && p.A == ps[0].A);
      if (!a_again) s.in_bytes += static_cast<int64_t>(p.Mv) * p.Kv * 2;
    }
    if (!before || p.B != before->B) {
      b_again = b_again || (before && p.B == ps[0].B);
      if (!b_again) s.in_bytes += static_cast<int64_t>(p.Nv) * p.Kv * 2;
    }
    s.rows = std::max<int64_t>(s.rows, p.Mv);
    s.k = std::max<int64_t>(s.k, p.Kv);
    s.cols = std::min<int64_t>(s.cols, p.Nv);
    s.fewest_rows = std::min<int64_t>(s.fewest_rows, p.Mv);
    if (!(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) && loose_rows(p.B, p.ldb)) s.loose_cols = std::min<int64_t>(s.loose_cols, p.Nv);
    if ((layout & GSPMD_LAYOUT_LHS_K_MAJOR) && loose_rows(p.A, p.lda)) s.loose_rows_of_lhs = std::min<int64_t>(s.loose_rows_of_lhs, p.Mv);
    s.a_odd = s.a_odd || (p.lda & 1) || (reinterpret_cast<uintptr_t>(p.A) & 2);
    s.b_odd = s.b_odd || (p.ldb & 1) || (reinterpret_cast<uintptr_t>(p.B) & 2);
    s.big += tiles_of(p, kMfmaBM, kMfmaBN);
    s.pair += tiles_of(p, kPairRows, kPairCols);
    if (p.join_slot == 0) {
      s.mid += tiles_of(p, kMidTile, kMidTile);
      s.members = std::max<int64_t>(s.members, p.join_count);
    }
    s.whole_steps = s.whole_steps && p.Kv % (2 * kMfmaBK) == 0;
    s.whole_chunks = s.whole_chunks && p.Kv % 8 == 0;
    s.broken_lines = s.broken_lines || (!(layout & GSPMD_LAYOUT_LHS_K_MAJOR) && (p.lda & 63)) || ((layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) && (p.ldb & 63));
  }
  return s;
}
double big_us(const LaunchSize& s, bool staged) {
  const double steps = static_cast<double>((s.k + 63) / 64), full = static_cast<double>(s.big / 256), part = static_cast<double>(s.big % 256) / 256.0;
  const double beside = 10.0 + (s.k % 64 ? 2.0 : 0.0);
  auto step = [&](double fill) { return s.rows <= 96 ? 0.75 : 0.85 + 0.45 * fill * fill; };
  const double first = static_cast<double>(std::min<int64_t>(s.big, 256)), later = static_cast<double>(s.big) - first;
  const double slots = s.members > 1 ? 4.6 * static_cast<double>(s.members) + 0.05 * first + 0.1 * later : 0.0;
  const double tile = std::min(s.loose_cols, s.loose_rows_of_lhs) < 8 ? 14.0 + steps * 7.0 : std::min(8.0 + steps * 3.4, 14.0 + steps * 2.0);
  if (staged) return tile * (full + (part == 0.0 ? 0.0 : full == 0.0 ? 1.0 : 0.8 + 0.2 * part)) + slots;
  if (s.rows > 96 && full >= 2.0) return (full + part) * (beside + steps * 1.25) + slots;
  return full * (beside + steps * step(1.0)) + (part > 0.0 ? beside + steps * step(part) : 0.0) + slots;
}
double mid_us(const LaunchSize& s, int32_t layout) {
  const double m = static_cast<double>(s.members), left = static_cast<double>((s.k % 64 + 31) / 32);
  const double steps = m * static_cast<double>((s.k + 31) / 32) * (s.broken_lines ? 1.2 : 1.0), beside = 4.5 + (s.whole_steps ? 0.0 : 1.8 * (m - 1.0)) + 0.25 * m * left;
  const int64_t part = s.mid % 512;
  const bool long_sum = s.members > 1 && s.mid > 512;
  const double one = long_sum ? 0.30 : 0.205, two = long_sum ? 0.44 : layout & GSPMD_LAYOUT_LHS_K_MAJOR ? 0.41 : 0.36;
  return 2.0 + static_cast<double>(s.mid / 512) * (beside + steps * two) + (part == 0 ? 0.0 : beside + steps * (part <= 256 ? one : two));
}
// Operands that take no direct loads, through registers.  dot_mfma_kernel: 14 us and 2.0 us per 64-wide step (8 and 3.4 up to four), a last round that is not full between 0.8 and 1 of
// that.  dot_mid_kernel: 4.7 us and per 32-wide step 0.27 us with one operand at odd addresses and 0.31 with both while a compute
// unit has one workgroup, 0.54 and 0.69 with two, a last round of more than 256 again in part.  Fitted to 40 drawn launches (us, 256 x 256 / 128 x 128 tiles;
// M x K x N): 5995 x 2709 x 877 103 / 61   six of 1432 x 2183 x 775 84 / 56   six of 354 x 817 x 2307 38 / 24   4330 x 146 x 4633 40 / 22   32 of 324 x 753 x 325
//   37 / 24   32 of 554 x 840 x 669 72 / 41   six of 1083 x 1389 x 1844 55 / 62   six of 975 x 889 x 2316 43 / 42   32 of 716 x 411 x 281 25 / 25
double mid_staged_us(const LaunchSize& s, double beside = 4.7) {
  const bool both = s.a_odd && s.b_odd, any = s.a_odd || s.b_odd;
  const double steps = static_cast<double>((s.k + 31) / 32), one = both ? 0.31 : any ? 0.27 : 0.16, two = both ? 0.69 : any ? 0.54 : 0.32;
  const int64_t full = s.mid / 512, part = s.mid % 512;
  const double last = part == 0 ? 0.0 : beside + steps * (part <= 256 ? one : two * (0.6 + 0.4 * static_cast<double>(part) / 512.0));
  return static_cast<double>(full) * (beside + steps * two) + last;
}

// dot_pair_kernel: 5.8 us, and rounds of 512 workgroups of 5.2 us and 0.70 us per 32-wide step, two of them on a compute unit, more where an operand is
//   K-contiguous (its half lines come twice from L2; the lhs is the larger part); in a last round about half of that per step
//   where every compute unit has one, 2.3 us and three quarters of it where only half of them have; 0.1 and 0.2 us more where rows are not padded to 16 bytes (six of 356 x
//   2088 x 2142: 34.6 / 37.1 / 38.5).  Measured (us, dot_mfma_kernel / dot_mid_kernel / dot_pair_kernel;
//   both K-major, then lhs K-contiguous): M x N = 2048 x 4096, K = 512 14.5 / 12.4 / 11.7, 14.2 / 12.0 / 12.1; 1024 21.2 / 19.1 / 18.1, 21.3 / 18.9 / 19.6; 2048 35.7 / 33.3 /
//   30.6, 35.5 / 32.2 / 34.2   4096 x 4096, K = 200 13.8 / 14.9 / 12.1, 13.6 / 15.1 / 13.7; 512 19.5 / 22.5 / 19.9, 19.2 / 22.2 / 21.7; 2048 53 / 65 / 57, 53 / 64 / 64
//   4096 x 8192, four of them, K = 64 69 / 61 / 55, 67 / 59 / 54; 200 96 / 103 / 85, 100 / 105 / 91; 512 143 / 159 / 138, 142 / 158 / 148; 1024 238 / 283 / 242, 237 / 282 / 265
double pair_us(const LaunchSize& s, int32_t layout, bool loose) {
  const double steps = static_cast<double>((s.k + 31) / 32);
  const bool a_lines = layout & GSPMD_LAYOUT_LHS_K_MAJOR, b_lines = !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS);
  const double rows = loose ? 0.1 : 0.0;
  const double two = 0.70 + (a_lines ? 0.0 : 0.13) + (b_lines ? 0.0 : a_lines ? 0.035 : 0.08) + 2.0 * rows, one = (a_lines ? 0.38 : b_lines ? 0.42 : 0.45) + rows;
  const int64_t part = s.pair % 512;
  const double fill = static_cast<double>(part) / 512.0, round = 5.2 + steps * two;
  double last = 0.0;
  if (part > 256) last = 5.2 + steps * two * (0.6 + 0.4 * fill);
  else if (part > 128) last = steps * one;
  else if (part > 0) last = 2.3 + steps * one * 0.75;
  return 5.8 + static_cast<double>(s.pair / 512) * round + std::max(last, fill * round);
}

// The kernels differ in what a launch pays beside its K loop, in how many workgroups it gives the chip, and in what
// a workgroup draws from L2 per flop, so the choice compares estimates: the lines above, and for dot_split_kernel rounds of 256 workgroups of
// 4 us (8.5 with 4 row blocks where rows are not padded to 16 bytes: six of 98 x 154 x 1092 11.3, dot_mid_kernel 7.8) and 1.0, 1.3, 1.7 us per eight 32-wide steps.  One problem, bf16, rows x K x N, us, dot_mfma_kernel / dot_split_kernel with 1, 2, 4 row
// blocks:
//   32 x 8192 x 8192: 101 / 43, 51, 54        64 x 8192 x 8192: 105 / 62, 47, 65      256 x 8192 x 8192: 135 / 222, 140, 97
//   32 x 2048 x 16384: 31 / 26, 19, 20        64 x 1024 x 1024: 14 / 6, 7, 10         256 x 2048 x 2048: 39 / 22, 13, 17
//   512 x 2048 x 2048: 39 / 41, 24, 16        1024 x 1024 x 4096: 23 / 89, 59, 40
// In tiles of 32 columns (1 and 2 row blocks; 0.75 and 1.05 us per eight steps, staged 0.8 and 0.9), where 64 leave compute units without a tile, or are more than
// an operand has (64 columns with 1, 2, 4 row blocks / 32 with 1, 2):
//   16 x 3648 x 2081: 13.9, 14.4, 16.2 / 11.4, 11.6     8 x 4096 x 1024: 10.3, 11.9, 15.2 / 7.6, 8.9      100 x 4096 x 1024: 11.9, 13.3, 17.7 / 10.5, 11.3
//   16 x 8192 x 8192: 41.7, 42.6, 44.9 / 38.4, 38.8     32 x 8192 x 8192: 39.5, 48.4, 51 / 65, 43         128 x 2048 x 2048: 8.9, 9.5, 12.5 / 12.7, 8.8
//   172 x 2361 x 559: 14.7, 17.7, 23.4 / 10.9, 13.1     300 x 1000 x 500: 7.9, 9.0, 11.8 / 8.5, 7.8       32 of 261 x 1486 x 59: 102, 86, 61 / 25, 26
// dot_split_kernel's order of summation is another one: partial sums along a contracting mesh dimension (`ordered`) stay with the
// first two, so that the joined sum, the two-launch sum and partials that a caller sums agree bit for bit; and beyond 256 rows it is taken
// from K = 1024 on (below, dot_mid_kernel is within 4 us).
// Operands that take no direct loads (kPathMfmaStaged) cost the address unit more: big_us, mid_staged_us; rounds of 3.2, 4.3, 8 us and 1.2, 1.25, 1.55 us
// per eight steps in the split kernel (256 x 256 staged tiles / 1, 2, 4 row blocks):
//   601 x 2001 x 601: 78 / 25, 15, 20     2001 x 1003 x 2001: 45 / 136, 82, 59     301 x 1001 x 301: 45 / 9, 10, 14
//   3826 x 102 x 538: 14 / 35, 25, 21     482 x 111 x 5292: 14 / 50, 34, 25        2289 x 293 x 885: 21 / 35, 23, 17
//   601 x 1203 x 697, six of them: 52 / -, -, 50     1083 x 1400 x 2367: 50 / 104, 60, 46     5990 x 3107 x 555: 117 / -, -, 107
// Where such a K-major operand has fewer columns (rows) than a tile of 64 columns, or fewer than 8 in one of 32, that kernel loads element by element (2.2 to 8.5 us per
// eight steps); 256 x 256 staged tiles below 8 columns too, 7 us a step.  32 of 268 x 2185 x N (256 x 256 / 64 columns with 1, 2, 4 row blocks / 32 columns with 1, 2):
//   N = 3: 236 / 98, 96, 60 / 57, 78     7: 270 / 134, 120, 69 / 74, 92     9: 88 / 148, 130, 72 / 24, 24     10: 79 / 148, 130, 73 / 17, 20     31: 88 / 148, 130, 76 / 24, 24
// While a timeline is recorded the launches that this gives to dot_mid_kernel, which writes no records, go to dot_mfma_kernel
// (with_records): the choice is the same with and without, so results are.
// Operands beyond 16 MB: 0.09 us per MB more in dot_mid_kernel and 0.04 in dot_pair_kernel than in 256 x 256 tiles, whose workgroups draw them from HBM (and from the memory-side
// cache) less often.  Without it, fitted to operands of which few were larger, launches that stream weights went to 128 x 128 tiles (us, dot_mfma_kernel / dot_mid_kernel): experts'
// products of 8 x 363 x 2176 x 3840 47 / 71, 16 x 339 x 1344 x 6144 94 / 126, 8 x 279 x 3968 x 6016 140 / 178, 4 x 369 x 1600 x 8064 37 / 55, unpadded 16 x 289 x 1600 x 5760 104 / 131,
// staged 32 x 2440 x 1759 x 665 291 / 352.
// Up to 128 rows 0.05 in dot_mid_kernel too, which then draws every weight once (dot_mfma_kernel / dot_mid_kernel; 4 x 35 x 3640 x 7781 63 / 46, 16 x 36 x 4057 x 1491 69 / 46,
// dot_split_kernel 68); and beyond them nothing where 256 x 256 tiles leave half of the compute units idle, which then draw less than HBM gives (16 x 272 x 3760 x 1280 with 64 to 128 of them 97 / 85,
// dot_pair_kernel 93; 16 x 269 x 2452 x 1072 61 / 62 / 67; 8 x 142 x 3904 x 2112 64 / 54).  Nor where the lhs is K-major: weight gradients have short K, and their outputs bound them, 8 x 3648 x 505 to 915 x
// 1152 64 / 57 / 53, 4 x 1152 x 528 to 578 x 7104 53 / 44 / 47, 8 x 1728 x 368 to 633 x 2896 63 / 60 / 53 (of 308 drawn ones none was faster with it).
constexpr int64_t kDrawnTiles = 128;
double drawn_us(const LaunchSize& s, int32_t layout, double narrow, double wide) {
  const double per_mb = layout & GSPMD_LAYOUT_LHS_K_MAJOR ? 0.0 : s.rows <= kMidTile ? narrow : s.big >= kDrawnTiles ? wide : 0.0;
  return per_mb * std::max(0.0, static_cast<double>(s.in_bytes) * 1e-6 - 16.0);
}
constexpr int32_t kMidShortK = 1024;      // members with something left of K that dot_mid_kernel runs through one loop
constexpr int64_t kSplitAnyKRows = 256, kSplitMinK = 1024;
// dot_mfma_kernel's direct variants take a K-major rhs with loose rows from one of their tiles of columns on
bool big_staged(const LaunchSize& size, KernelPath path, int32_t layout) {
  return path == kPathMfmaStaged || (path == kPathMfmaWords && !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) && size.cols < kMfmaBN);
}
// dot_mid_kernel's staged variant moves the last tiles of K-major operands back: from one of its tiles on, and no joined sums
bool mid_stages_whole(const LaunchSize& size, int32_t layout) {
  return ((layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) || size.cols >= kMidTile) && (!(layout & GSPMD_LAYOUT_LHS_K_MAJOR) || size.fewest_rows >= kMidTile);
}
// dot_pair_kernel's direct loads take what is left of K in chunks of eight, which reach into the padding of a K-contiguous operand's rows
bool pair_takes(const LaunchSize& size, KernelPath path, int32_t layout) {
  const bool kmajor = (layout & GSPMD_LAYOUT_LHS_K_MAJOR) && !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS);
  return size.members == 1 && (path == kPathMfmaDirect || (path == kPathMfmaWords && (size.whole_chunks || kmajor)));
}
MfmaChoice choose_mfma(const std::vector<Problem>& ps, KernelPath path, int32_t layout, bool ordered) {
  MfmaChoice choice{kMfmaBig, 0};
  const bool loose = path == kPathMfmaStaged;
  const LaunchSize size = launch_size(ps, layout);
  if (size.rows == 0) return choice;
  double best = big_us(size, choice.staged = big_staged(size, path, layout));
  if (!loose || (size.members == 1 && mid_stages_whole(size, layout))) {
    const double us = (loose ? mid_staged_us(size) : mid_us(size, layout)) + (size.members == 1 ? drawn_us(size, layout, 0.05, 0.09) : 0.0);
    if (us < 0.95 * best) { best = us; choice = MfmaChoice{kMfmaMid, 0, 0, loose}; }
  }
  if (pair_takes(size, path, layout)) {
    const double us = pair_us(size, layout, path == kPathMfmaWords) + drawn_us(size, layout, 0.04, 0.04);
    if (us < 0.95 * best) { best = us; choice = MfmaChoice{kMfmaPair, 0, 0, false, path == kPathMfmaWords}; }
  }
  if (!ordered && (loose || size.rows <= kSplitAnyKRows || size.k >= kSplitMinK)) {
    const double rounds8 = static_cast<double>((size.k + 255) / 256);
    const struct { int blocks, cols; double aligned, beside, unaligned, elements; } kinds[] = {
        {1, 4, 1.0, 3.2, 1.2, 5.0}, {2, 4, 1.3, 4.3, 1.25, 5.5}, {4, 4, 1.7, 8.0, 1.55, 8.5}, {1, 2, 0.75, 3.2, 0.8, 2.2}, {2, 2, 1.05, 4.3, 0.9, 4.5}};
    for (const auto& kind : kinds) {
      int64_t tiles = 0;
      for (const auto& p : ps) tiles += tiles_of(p, 16 * kind.blocks, 16 * kind.cols);
      const bool whole = kind.cols == 4;
      const bool elements = size.loose_cols < (whole ? 16 * kind.cols : 8) || size.loose_rows_of_lhs < (whole ? 16 * kind.blocks : 8);
      const double us = static_cast<double>((tiles + 255) / 256) * (loose ? kind.beside + rounds8 * (elements ? kind.elements : kind.unaligned) : (path == kPathMfmaWords && kind.blocks == 4 ? 8.5 : 4.0) + rounds8 * kind.aligned);
      if (us < best) { best = us; choice = MfmaChoice{kMfmaSplit, kind.blocks, kind.cols}; }
    }
  }
  return choice;
}

// Sums over a contracting mesh dimension are formed in one launch (joined problems) or in two: the members' products by themselves, in dense
// fp32 partials, then a sum kernel per out buffer.  Two, where that is estimated 15 % faster, or 5 % where one launch would take more than a round
// of dot_mid_kernel's tiles (kSeveralRounds: what a launch pays once no longer matters, and the lines are closer); the results are the same bits.
// Scattered over all members, slots / one after the other / two launches (us, all on one card): 4227 x 13543 x 3328 over 4: - / 416 / 371   4227 x
//   8192 x 3328 over 4: - / 238 / 250   3000 x 13543 x 3328 over 4: - / 348 / 272   8192 x 8000 x 2048 over 4: 328 / 299 / 290   6000 x 12000 x 4096
//   over 2: 461 / 660 / 490   4227 x 5000 x 3328 over 4: - / 180 / 211   4096 x 16384 x 4096 over 4: 461 / 513 / 448.  The rule takes the least in
//   all but the last, where it stays with the slots: its estimates are 4 % apart.
constexpr int64_t kSeveralRounds = 512;
constexpr double kStagedPartials = 7.0;      // us beside dot_mid_kernel's staged loop where it stores float32 partials (4.7 bf16 results): 1335 x 508 x 4085 over 2 members, unaligned: 46, in one launch 34
double sum_us(const std::vector<Problem>& ps, const MfmaChoice& choice, int32_t layout) {
  const LaunchSize size = launch_size(ps, layout);
  return choice.kernel == kMfmaMid ? choice.staged ? mid_staged_us(size, kStagedPartials) : mid_us(size, layout) : choice.kernel == kMfmaPair ? pair_us(size, layout, choice.loose) : big_us(size, choice.staged);
}
// What partials cost beside their launch: 1 us, 2.5 us per sum kernel (one per reduce group) and 0.31 us per MB written and read back.  Measured, one launch / two (us; M x K x N over members): 141 x 7248 x 463 over 8: 60 / 19;
// 659 x 4880 x 1316 over 2: 53 / 34; 727 x 205 x 74 over 8, unaligned: 51 / 19; 2048 x 8192 x 2048 over 4: 76 / 68, scattered: 77 / 76; 1335 x
// 508 x 4085 over 2, unaligned: 36 / 48; 1953 x 409 x 454 over 4: 15 / 20; 4023 x 8430 x 1215 over 8: 142 / 158.
double apart_us(int64_t partial_bytes, int64_t launches) {
  return 1.0 + 2.5 * static_cast<double>(launches) + 0.31e-6 * static_cast<double>(partial_bytes);
}

// The kernel of a launch of bf16 problems: by the rule above, unless a test has pinned one that may take them.
MfmaChoice pick_kernel(const std::vector<Problem>& ps, KernelPath path, int32_t layout, bool ordered) {
  if (path == kPathFallback) return MfmaChoice{kMfmaNone, 0};
  const MfmaKernel pin = static_cast<MfmaKernel>(t_pin.kernel);
  const LaunchSize size = launch_size(ps, layout);
  if (pin == kMfmaNone || pin == kMfmaBig || (pin == kMfmaMid && (path != kPathMfmaStaged || (size.members == 1 && mid_stages_whole(size, layout)))) ||
      (pin == kMfmaSplit && !ordered) || (pin == kMfmaPair && pair_takes(size, path, layout)))
    return MfmaChoice{pin, t_pin.row_blocks, t_pin.col_blocks ? t_pin.col_blocks : 4, pin == kMfmaBig ? big_staged(size, path, layout) : pin == kMfmaMid && path == kPathMfmaStaged};
  return choose_mfma(ps, path, layout, ordered);
}

// Whether four workgroups of dot_f32_kernel share a compute unit with two LDS stages each, not three with three: where its equal tiles come out
// even that way.  With four tiles each, three workgroups leave the fourth to itself (us, three / four): 2048 x 2048 x 2048 147 / 119, 2048 x 1500 x 2000
// 112 / 91, 2048 x 100 x 2000 16.5 / 15.0.  With more of them, where K is short and a round's start and end count: K = 300, seven each 47.8 /
// 43.0, eight 49.6 / 47.4, ten 63.8 / 60.5, thirteen 80.4 / 77.2, sixteen 97.1 / 90.7.  Elsewhere three: five each, K = 600 51.8 / 59.9; six 61.3 / 68.1,
// 2048 x 2048 x 3000 on 2 x 4 180 / 202; nine 90.6 / 96.4; eight, K = 1024 123 / 134, K = 1500 180 / 183.  Up to three each they are alike.
constexpr int64_t kF32ShortK = 512;
bool f32_four(int64_t tiles, int64_t k) {
  const int64_t each = (tiles + 255) / 256;
  return each == 4 || (each > 4 && k <= kF32ShortK && (each % 4 == 0 || each % 3 == 1));
}

// Rows that a load instruction of dot_f32_kernel (up to 8 of them) does not reach with 32-bit offsets.  Element by element such a product took three to four times as
// long (us, element by element / 64-bit offsets / rows within reach): 64 x 8192 x 4096 461 / 128 / 118, 64 x 2048 x 8192 118 / 36.5 / 33.4, 2048 x 4096 x 64 with a
// K-contiguous rhs 227 / 66 / 60.5.
bool f32_wide(const std::vector<Problem>& ps) {
  return std::any_of(ps.begin(), ps.end(), [](const Problem& p) { return std::max(p.lda, p.ldb) >= kF32MaxStride; });
}

// While a timeline is recorded dot_mid_kernel's launches go to dot_mfma_kernel, which takes whatever it takes and adds up in the same order.
MfmaKernel with_records(MfmaKernel kernel) {
  return (kernel == kMfmaMid || kernel == kMfmaPair) && g_timeline.load(std::memory_order_acquire) != nullptr ? kMfmaBig : kernel;
}

// Problems whose last tile column is moved back: those with loose rhs rows, and with one member of a sum all of them (the members are
// consecutive).  2048 x 8192 x 2050 over two members with rhs rows of 2056 and 2050 elements: both take columns 1794 .. 2049 for their last tile.
// Returns how many.
int32_t mark_moved_back(std::vector<Problem>& ps) {
  int32_t moved = 0;
  for (size_t i = 0; i < ps.size();) {
    const size_t end = i + static_cast<size_t>(std::max(ps[i].join_count, 1));
    bool loose = false;
    for (size_t m = i; m < end; ++m) loose = loose || loose_rows(ps[m].B, ps[m].ldb);
    for (; i < end; ++i)
      if (loose) {
        ps[i].flags |= kProblemMovesBack;
        ++moved;
      }
  }
  return moved;
}

// bf16 outputs of a launch that the caches do not hold for the next one (kernels_lines.h), and those of more than one round of dot_mid_kernel's workgroups: in the caches
// they take the place of operands that later tiles read (7592 x 3776 x 2240, 1080 tiles, us, through / past: 138.5 / 126.7, with a product of x 1024 that reads them 160 / 165).
// And those of a launch whose operands fill a quarter of the memory-side cache: what the outputs take there, operands lose that come round again (679 x 8000 x 4992, three sets of operands
// in turn, 68 / 55; 512 x 8192 x 5120 68.6 / 64.1, with a product of x 512 that reads them 98.8 / 97.2), and what the next kernel gains is little beside them (2000 x 9000 x 2000 on 2 x 2 84 / 84 and 124 /
// 127, the worst of eleven; below it is 6 to 18 %).
constexpr int64_t kPastBytes = 96000000, kPastTiles = 512, kPastInBytes = 64000000;

int32_t launch_problems(std::vector<Problem>& all, int32_t layout, int32_t in_dtype, int32_t out_dtype, int32_t epilogue,
                        bool ordered, void* workspace, int64_t workspace_bytes, hipStream_t stream, const JoinSpace* join = nullptr) {
  // problems with an empty static output block write nothing
  all.erase(std::remove_if(all.begin(), all.end(), [](const Problem& p) { return p.Ms == 0 || p.Ns == 0; }), all.end());
  if (all.empty()) return GSPMD_OK;
  if (in_dtype == GSPMD_F32 && out_dtype != GSPMD_F32) return GSPMD_ERR_UNSUPPORTED;
  std::vector<Problem> ps;
  for (const auto& p : all) if (p.Mv > 0) ps.push_back(p);      // Mv, Nv, Kv are all zero or all positive
  const KernelPath path = kernel_path(ps, in_dtype, layout);
  if (join && path == kPathFallback) return GSPMD_ERR_UNSUPPORTED;      // the caller checks before it joins problems
  // joined problems come with the caller's choice between the two kernels that keep the order of summation
  MfmaChoice choice = join ? MfmaChoice{join->chain ? kMfmaMid : kMfmaBig, 0} : pick_kernel(ps, path, layout, ordered);
  if (!join) choice.kernel = with_records(choice.kernel);
  choice.staged = choice.kernel == kMfmaBig ? big_staged(launch_size(ps, layout), path, layout) : choice.kernel == kMfmaMid && path == kPathMfmaStaged;
  const bool mfma = choice.kernel != kMfmaNone;
  const int split = choice.kernel == kMfmaSplit ? choice.row_blocks : 0;
  const bool mid = choice.kernel == kMfmaMid, pair = choice.kernel == kMfmaPair;
  const int bm = split ? 16 * split : mid ? kMidTile : pair ? kPairRows : mfma ? kMfmaBM : kGenTile;
  const int bn = split ? 16 * choice.col_blocks : mid ? kMidTile : pair ? kPairCols : mfma ? kMfmaBN : kGenTile;
  // Workgroups start in tile order and the launch ends when the last one does: problems whose tiles take longest
  // (the most K steps) go first, so that the compute units that are still busy at the end are busy with short tiles.
  if (!join)
    std::stable_sort(ps.begin(), ps.end(), [](const Problem& a, const Problem& b) { return a.Kv > b.Kv; });
  // Members of a sum run through one loop where their strides are equal and their K is, too, except that the last one's may be less (the part of
  // K that does not divide): 303 x 3900 x 7424 over eight members, 488 and 484 of K: 49.5 us, one after another with a drained ring 59.4.
  // K beyond whole 64-wide steps has to be one that the kernel masks; with two workgroups on a compute unit it has no registers for that.
  const bool short_members = mid && join && launch_size(ps, layout).mid <= kMidAlone;
  if (mid && join)
    for (size_t i = 0; i < ps.size(); i += std::max(ps[i].join_count, 1)) {     // the members of a sum are consecutive, in the order of summation
      const auto fits = [&](int32_t k) { return k % (2 * kMfmaBK) == 0 || (short_members && k <= kMidShortK && (path == kPathMfmaDirect || k % 8 == 0)); };
      bool alike = ps[i].join_count > 1 && fits(ps[i].Kv);
      for (int32_t m = 1; m < ps[i].join_count && alike; ++m) {
        const Problem &a = ps[i], &b = ps[i + static_cast<size_t>(m)];
        alike = a.lda == b.lda && a.ldb == b.ldb && (a.Kv == b.Kv || (m == ps[i].join_count - 1 && b.Kv > 0 && b.Kv < a.Kv && fits(b.Kv)));
      }
      if (alike) ps[i].flags |= kProblemRunsOn;
    }
  const bool moves = mfma && !split && !choice.staged && path == kPathMfmaWords && !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS);
  t_last.moved_back = moves ? mark_moved_back(ps) : 0;
  const int64_t tiles = assign_tiles(ps, bm, bn, mid);
  if (tiles < 0) return GSPMD_ERR_UNSUPPORTED;
  std::vector<ZeroRect> rects;
  for (const auto& p : all) {
    if (p.join_slot > 0) continue;                              // one of the joined problems speaks for their common output
    // rows that the contraction kernel's tiles write or clear; the MFMA kernel's last tile row also clears up to
    // kRowsBelow rows below its footprint
    const int32_t rows_done = mfma ? rows_cleared(p.Mv, p.Ms)
                                   : static_cast<int32_t>(std::min<int64_t>(p.Ms, (static_cast<int64_t>(p.Mv) + bm - 1) / bm * bm));
    const int32_t cols_done = static_cast<int32_t>(std::min<int64_t>(p.Ns, (static_cast<int64_t>(p.Nv) + bn - 1) / bn * bn));
    if (rows_done < p.Ms) rects.push_back(ZeroRect{p.C, p.ldc, rows_done, p.Ms, 0, p.Ns, 0});
    if (cols_done < p.Ns && rows_done > 0) rects.push_back(ZeroRect{p.C, p.ldc, 0, rows_done, cols_done, p.Ns, 0});
  }
  const bool inline_tables = ps.size() <= static_cast<size_t>(kInlineProblems) && rects.size() <= static_cast<size_t>(kInlineRects);
  const int64_t prob_bytes = static_cast<int64_t>(ps.size()) * sizeof(Problem);
  const int64_t table_bytes = prob_bytes + static_cast<int64_t>(rects.size()) * sizeof(ZeroRect);
  // the workspace contract does not depend on which way the tables travel
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kWsAlign - 1)) || workspace_bytes < table_bytes)
    return GSPMD_ERR_WORKSPACE;
  t_last.kernel = choice.kernel;
  t_last.row_blocks = choice.row_blocks;
  t_last.col_blocks = split ? choice.col_blocks : 0;
  t_last.one_launch = join ? 1 : 0;
  t_last.table_bytes = inline_tables ? 0 : table_bytes;
  if (t_pin.dry_run) return GSPMD_OK;
  const Problem* tab = nullptr;
  const ZeroRect* drects = nullptr;
  InlineProblems inl;
  InlineRects inl_rects;
  std::memset(&inl, 0, sizeof(inl));
  std::memset(&inl_rects, 0, sizeof(inl_rects));
  if (inline_tables) {
    if (!ps.empty()) std::memcpy(inl.p, ps.data(), static_cast<size_t>(prob_bytes));
    if (!rects.empty()) std::memcpy(inl_rects.r, rects.data(), rects.size() * sizeof(ZeroRect));
  } else {
    std::vector<char> host(static_cast<size_t>(table_bytes));
    if (prob_bytes) std::memcpy(host.data(), ps.data(), static_cast<size_t>(prob_bytes));
    if (!rects.empty()) std::memcpy(host.data() + prob_bytes, rects.data(), rects.size() * sizeof(ZeroRect));
    if (hipMemcpyAsync(workspace, host.data(), host.size(), hipMemcpyHostToDevice, stream) != hipSuccess)
      return GSPMD_ERR_DEVICE;
    tab = static_cast<const Problem*>(workspace);
    drects = reinterpret_cast<const ZeroRect*>(static_cast<const char*>(workspace) + prob_bytes);
  }
  const int n = static_cast<int>(ps.size());
  if (tiles > 0) {
    if (split) {
      MfmaLaunch l{&inl, tab, n, static_cast<int>(tiles), epilogue, nullptr, nullptr, g_timeline.load(std::memory_order_acquire),
                   g_timeline_records.load(std::memory_order_acquire)};
      // weights whose rows are whole multiples of what an L2's channels cover (32 x 8192 x 8192: 42.7 us in an eighth of the tiles at a time, 40.1
      // spread out; other rows gain nothing, 101 x 1793 x 2281 loses: 10.4, 11.2)
      l.spread = !(layout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) && std::all_of(ps.begin(), ps.end(), [](const Problem& p) { return p.ldb % 2048 == 0; });
      if (!launch_dot_split(l, layout, out_dtype, split, choice.col_blocks, stream)) return GSPMD_ERR_DEVICE;
    } else if (mid) {
      MfmaLaunch l{&inl, tab, n, static_cast<int>(tiles), epilogue, nullptr, nullptr, nullptr, 0};
      int64_t out_bytes = 0;
      for (const auto& p : ps) if (p.join_slot == 0) out_bytes += static_cast<int64_t>(p.Mv) * p.Nv * 2;
      l.past = out_bytes > kPastBytes || tiles > kPastTiles || launch_size(ps, layout).in_bytes > kPastInBytes;
      if (!launch_dot_mid(l, layout, out_dtype, join != nullptr, choice.staged, stream)) return GSPMD_ERR_DEVICE;
    } else if (pair) {
      const MfmaLaunch l{&inl, tab, n, static_cast<int>(tiles), epilogue, nullptr, nullptr, nullptr, 0};
      if (!launch_dot_pair(l, layout, out_dtype, stream)) return GSPMD_ERR_DEVICE;
    } else if (mfma) {
      if (join && join->tiles > 0) {
        const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((join->tiles + 255) / 256, 1024));
        hipLaunchKernelGGL(zero_words_kernel, dim3(blocks), dim3(256), 0, stream, join->counters, join->tiles);
        if (hipGetLastError() != hipSuccess) return GSPMD_ERR_DEVICE;
      }
      const MfmaLaunch l{&inl, tab, n, static_cast<int>(tiles), epilogue, join ? join->partials : nullptr, join ? join->counters : nullptr,
                         g_timeline.load(std::memory_order_acquire), g_timeline_records.load(std::memory_order_acquire)};
      if (!launch_dot_mfma(l, layout, out_dtype, choice.staged, stream)) return GSPMD_ERR_DEVICE;
    } else {
      const dim3 grid(static_cast<unsigned>(tiles)), block(256);
      if (in_dtype == GSPMD_F32) {
        auto go = [&](auto lean, auto wide) {
          constexpr bool kLean = decltype(lean)::value, kWide = decltype(wide)::value;
          switch (layout & 3) {
            case 0: hipLaunchKernelGGL((dot_f32_kernel<0, kLean, kWide>), grid, block, 0, stream, inl, tab, n, epilogue); break;
            case 1: hipLaunchKernelGGL((dot_f32_kernel<1, kLean, kWide>), grid, block, 0, stream, inl, tab, n, epilogue); break;
            case 2: hipLaunchKernelGGL((dot_f32_kernel<2, kLean, kWide>), grid, block, 0, stream, inl, tab, n, epilogue); break;
            default: hipLaunchKernelGGL((dot_f32_kernel<3, kLean, kWide>), grid, block, 0, stream, inl, tab, n, epilogue);
          }
        };
        if (f32_wide(ps)) go(std::false_type{}, std::true_type{});
        else if (f32_four(tiles, launch_size(ps, layout).k)) go(std::true_type{}, std::false_type{});
        else go(std::false_type{}, std::false_type{});
      } else if (out_dtype == GSPMD_F32)
        hipLaunchKernelGGL((dot_fallback_kernel<bf16_bits, float>), grid, block, 0, stream, inl, tab, n, layout, epilogue);
      else
        hipLaunchKernelGGL((dot_fallback_kernel<bf16_bits, bf16_bits>), grid, block, 0, stream, inl, tab, n, layout, epilogue);
      if (hipGetLastError() != hipSuccess) return GSPMD_ERR_DEVICE;
    }
  }
  if (!rects.empty()) {
    const int vec_elems = out_dtype == GSPMD_F32 ? 4 : 8;
    bool vec = true;
    int64_t most = 0;
    for (const auto& r : rects) {
      vec = vec && !(reinterpret_cast<uintptr_t>(r.C) & 15) && r.ldc % vec_elems == 0 && r.c0 % vec_elems == 0 &&
            (r.c1 - r.c0) % vec_elems == 0;
      most = std::max<int64_t>(most, static_cast<int64_t>(r.r1 - r.r0) * (r.c1 - r.c0));
    }
    const int64_t per_thread = vec ? vec_elems : 1;
    const unsigned gx = static_cast<unsigned>(std::min<int64_t>(std::max<int64_t>((most / per_thread + 255) / 256, 1), 2048));
    for (size_t first = 0; first < rects.size(); first += 65535) {       // grid.y is limited to 65535
      const unsigned gy = static_cast<unsigned>(std::min<size_t>(rects.size() - first, 65535));
      const dim3 grid(gx, gy), block(256);
      const ZeroRect* part = drects ? drects + first : nullptr;
      if (out_dtype == GSPMD_F32) {
        if (vec) hipLaunchKernelGGL((zero_rects_kernel<float, 4>), grid, block, 0, stream, inl_rects, part);
        else hipLaunchKernelGGL((zero_rects_kernel<float, 1>), grid, block, 0, stream, inl_rects, part);
      } else {
        if (vec) hipLaunchKernelGGL((zero_rects_kernel<bf16_bits, 8>), grid, block, 0, stream, inl_rects, part);
        else hipLaunchKernelGGL((zero_rects_kernel<bf16_bits, 1>), grid, block, 0, stream, inl_rects, part);
      }
    }
    if (hipGetLastError() != hipSuccess) return GSPMD_ERR_DEVICE;
  }
  return GSPMD_OK;
}

int32_t launch_reduce(const float* const* partials, int n_partials, int64_t rows, int64_t cols, int64_t ld_in,
                      void* out, int64_t ld_out, int32_t out_dtype, hipStream_t stream) {
  if (rows == 0 || cols == 0) return GSPMD_OK;
  PartialPtrs pp;
  uintptr_t bits = reinterpret_cast<uintptr_t>(out);
  for (int i = 0; i < kMaxPartials; ++i) pp.p[i] = nullptr;
  for (int i = 0; i < n_partials; ++i) { pp.p[i] = partials[i]; bits |= reinterpret_cast<uintptr_t>(partials[i]); }
  const bool vec = !(bits & 15) && !(cols & 3) && !(ld_in & 3) && !(ld_out & 3);
  const int64_t work = rows * (vec ? cols / 4 : cols);
  const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((work + 255) / 256, 1 << 20));   // one vector per thread up to 1 GiB of fp32
  const dim3 grid(blocks), block(256);
  if (out_dtype == GSPMD_F32) {
    if (vec) hipLaunchKernelGGL((reduce_partials_kernel<float, 4>), grid, block, 0, stream, pp, n_partials, rows, cols, ld_in, static_cast<float*>(out), ld_out);
    else hipLaunchKernelGGL((reduce_partials_kernel<float, 1>), grid, block, 0, stream, pp, n_partials, rows, cols, ld_in, static_cast<float*>(out), ld_out);
  } else {
    if (vec) hipLaunchKernelGGL((reduce_partials_kernel<bf16_bits, 4>), grid, block, 0, stream, pp, n_partials, rows, cols, ld_in, static_cast<bf16_bits*>(out), ld_out);
    else hipLaunchKernelGGL((reduce_partials_kernel<bf16_bits, 1>), grid, block, 0, stream, pp, n_partials, rows, cols, ld_in, static_cast<bf16_bits*>(out), ld_out);
  }
  return hipGetLastError() == hipSuccess ? GSPMD_OK : GSPMD_ERR_DEVICE;
}

// Largest extent whose index arithmetic (a padded dimension: partitions x shard size) stays within 31 bits.
constexpr int64_t kMoveMaxExtent = INT32_MAX >> 1;

// Launch shape of a move of `boxes` boxes (`dst_bits`: their addresses or-ed together) in 16-byte chunks of `vec` elements; fills in the shape's divisors, lanes per
// row and column block.  A row of fewer chunks than a wave has lanes shares the wave with other rows.  A workgroup takes
// at most kMoveUnroll chunks per lane of a row (columns beyond that go to another one), and loops over rows once there
// are more than 8192 workgroups (enough to fill the chip several times; more pay the set-up once more: a reshard of 537
// MB ran at 4.2 TB/s with 65536 and at 5.4 with 8192).
dim3 move_grid(MoveShape* s, uintptr_t dst_bits, int64_t boxes, int vec) {
  const int last = s->rank - 1;
  bool aligned = !(dst_bits & 15);
  for (int i = 0; i < last; ++i) aligned = aligned && s->dst_stride[i] % vec == 0;
  for (int i = 0; i < s->rank; ++i) {
    s->div_shard[i] = fast_div(static_cast<uint32_t>(s->shard[i]));
    s->div_per[i] = fast_div(static_cast<uint32_t>(s->src_per[i]));
  }
  // a row that does not start on 16 bytes in dst has a chunk more
  const int64_t chunks = (static_cast<int64_t>(s->shard[last]) + vec - 1) / vec + (aligned ? 0 : 1);
  int log_lanes = 0;
  while (log_lanes < 6 && (int64_t(1) << log_lanes) < chunks) ++log_lanes;
  const int64_t lanes = int64_t(1) << log_lanes, per_block = kMoveUnroll * lanes;
  const int64_t gx = (chunks + per_block - 1) / per_block;
  const int64_t each = ((chunks + gx - 1) / gx + lanes - 1) / lanes * lanes;        // even split in whole waves
  s->log_lanes = log_lanes;
  s->block_chunks = static_cast<int32_t>(each);
  const int64_t rows_per = 256 >> log_lanes, groups = (s->rows + rows_per - 1) / rows_per;
  const int64_t gy = std::min<int64_t>(std::min<int64_t>(groups, 65535), std::max<int64_t>(1, 8192 / (gx * boxes)));
  return dim3(static_cast<unsigned>(gx), static_cast<unsigned>(gy), static_cast<unsigned>(boxes));
}

bool is_contracting(int32_t c) { return c == GSPMD_AXIS_CONTRACTING || c == GSPMD_AXIS_CONTRACTING_SCATTER; }

bool has_contracting(const gspmd_mesh* mesh, const int32_t* cls) {
  for (int a = 0; a < mesh->rank; ++a) if (is_contracting(cls[a])) return true;
  return false;
}

bool has_scatter(const gspmd_mesh* mesh, const int32_t* cls) {
  for (int a = 0; a < mesh->rank; ++a) if (cls[a] == GSPMD_AXIS_CONTRACTING_SCATTER) return true;
  return false;
}

bool is_epilogue(int32_t e) { return e == GSPMD_EPILOGUE_NONE || e == GSPMD_EPILOGUE_RELU; }

// The sharding of a partition's partial sum: the out sharding with the dimensions that a scatter mesh dimension
// splits made whole again (the slice is taken after the sum).
void partial_mapping(const gspmd_mesh* mesh, const int32_t* cls, const gspmd_sharding* out_sh, int32_t* map) {
  for (int i = 0; i < out_sh->rank; ++i) {
    const int a = out_sh->dims_mapping[i];
    map[i] = (a >= 0 && a < mesh->rank && cls[a] == GSPMD_AXIS_CONTRACTING_SCATTER) ? -1 : a;
  }
}

// out shard of each of `pids` = epilogue(sum of the group's partials) restricted to the shard's place in them; all in one launch (out buffers
// whose rows are laid out differently in one each).
int32_t launch_reduce_scatter(const gspmd_mesh* mesh, const gspmd_sharding* out_sh, const gspmd_sharding* part_sh, const int64_t* pids, int n_out,
                              const float* const* partials, int n_partials, const gspmd_shard_buf* outs, int32_t epilogue,
                              hipStream_t stream) {
  for (int i = 1; i < n_out; ++i)
    if (outs[pids[i]].row_stride != outs[pids[0]].row_stride) {
      for (int j = 0; j < n_out; ++j) {
        const int32_t st = launch_reduce_scatter(mesh, out_sh, part_sh, pids + j, 1, partials, n_partials, outs, epilogue, stream);
        if (st != GSPMD_OK) return st;
      }
      return GSPMD_OK;
    }
  ScatterLaunch l;
  std::memset(&l, 0, sizeof(l));
  ScatterDesc& d = l.d;
  uintptr_t bits = 0;
  bool vec = true;
  int32_t st;
  for (int i = 0; i < n_out; ++i) {
    const gspmd_shard_buf& out = outs[pids[i]];
    Bounds ob, pb;
    if ((st = shard_bounds(mesh, out_sh, pids[i], &ob)) != GSPMD_OK) return st;
    if ((st = shard_bounds(mesh, part_sh, pids[i], &pb)) != GSPMD_OK) return st;
    const int r = ob.rank, last = r - 1;
    if (i == 0) {                         // static shapes and strides are the same for all
      d.rank = r;
      int64_t rows = 1, in_stride = 1;
      for (int k = last; k >= 0; --k) {
        if (ob.shard[k] > INT32_MAX) return GSPMD_ERR_UNSUPPORTED;
        d.shard[k] = static_cast<int32_t>(ob.shard[k]);
        d.in_stride[k] = in_stride;
        in_stride *= pb.shard[k];
        if (k < last) rows *= ob.shard[k];
      }
      if (rows > INT32_MAX) return GSPMD_ERR_UNSUPPORTED;
      d.rows = static_cast<int32_t>(rows);
      d.out_stride[last] = 1;
      if (r >= 2) {
        const int64_t rs = out.row_stride > 0 ? out.row_stride : ob.shard[last];
        if (rs < ob.shard[last]) return GSPMD_ERR_BAD_BUFFER;
        d.out_stride[r - 2] = rs;
        for (int k = r - 3; k >= 0; --k) d.out_stride[k] = d.out_stride[k + 1] * ob.shard[k + 1];
      }
      if (rows == 0 || ob.shard[last] == 0) return GSPMD_OK;
      vec = !(ob.shard[last] & 3) && !(pb.shard[last] & 3);
      for (int k = 0; k < last; ++k) vec = vec && !(d.in_stride[k] & 3) && !(d.out_stride[k] & 3);
    }
    if (!out.data) return GSPMD_ERR_NULL;
    ScatterOut& o = l.o[i];
    o.out = out.data;
    bits |= reinterpret_cast<uintptr_t>(out.data);
    for (int k = 0; k < r; ++k) {
      o.valid[k] = static_cast<int32_t>(ob.valid[k]);
      o.in_off[k] = ob.offset[k] - pb.offset[k];
    }
    vec = vec && !(o.in_off[last] & 3);
  }
  for (int i = 0; i < n_partials; ++i) { l.ptrs.p[i] = partials[i]; bits |= reinterpret_cast<uintptr_t>(partials[i]); }
  vec = vec && !(bits & 15);
  const int32_t cols = d.shard[d.rank - 1];
  const int64_t cols_v = (static_cast<int64_t>(cols) + (vec ? 3 : 0)) / (vec ? 4 : 1);
  // one vector per thread (a workgroup per 256 vectors of a row, or several short rows) up to the grid limit, beyond that each thread walks
  // down its column: measured faster than fewer workgroups with a loop (6.2 against 5.4 TB/s on 2.4 GB)
  while (d.log_lanes < 8 && (int64_t(1) << d.log_lanes) < cols_v) ++d.log_lanes;
  const int64_t gx = (cols_v + 255) / 256, rows_side = 256 >> d.log_lanes;
  const dim3 block(256), grid(static_cast<unsigned>(gx), static_cast<unsigned>(std::min<int64_t>((d.rows + rows_side - 1) / rows_side, 65535)), static_cast<unsigned>(n_out));
  if (outs[pids[0]].dtype == GSPMD_F32) {
    if (vec) hipLaunchKernelGGL((reduce_scatter_kernel<float, 4>), grid, block, 0, stream, l, n_partials, epilogue);
    else hipLaunchKernelGGL((reduce_scatter_kernel<float, 1>), grid, block, 0, stream, l, n_partials, epilogue);
  } else {
    if (vec) hipLaunchKernelGGL((reduce_scatter_kernel<bf16_bits, 4>), grid, block, 0, stream, l, n_partials, epilogue);
    else hipLaunchKernelGGL((reduce_scatter_kernel<bf16_bits, 1>), grid, block, 0, stream, l, n_partials, epilogue);
  }
  return hipGetLastError() == hipSuccess ? GSPMD_OK : GSPMD_ERR_DEVICE;
}

}  // namespace

extern "C" {

const char* gspmd_status_string(int32_t s) {
  switch (s) {
    case GSPMD_OK: return "ok";
    case GSPMD_ERR_NULL: return "null pointer";
    case GSPMD_ERR_BAD_MESH: return "bad device mesh";
    case GSPMD_ERR_BAD_SHARDING: return "bad sharding";
    case GSPMD_ERR_PARTITION_RANGE: return "partition id out of range";
    case GSPMD_ERR_BAD_DOT_DIMS: return "bad dot dimension numbers";
    case GSPMD_ERR_NEEDS_RESHARD: return "shardings need resharding";
    case GSPMD_ERR_UNSUPPORTED: return "unsupported dtype or layout";
    case GSPMD_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case GSPMD_ERR_DEVICE: return "HIP error";
    case GSPMD_ERR_BAD_BUFFER: return "bad shard buffer";
    case GSPMD_ERR_HOST_MEMORY: return "host allocation failed";
    default: return "unknown status";
  }
}

int32_t gspmd_shard_bounds(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t pid,
                           int64_t* offset, int64_t* valid_len, int64_t* shard_size) try {
  if (!offset || !valid_len) return GSPMD_ERR_NULL;
  int32_t st = validate_mesh(mesh, nullptr);
  if (st != GSPMD_OK) return st;
  if ((st = validate_sharding(mesh, sh)) != GSPMD_OK) return st;
  Bounds b;
  if ((st = shard_bounds(mesh, sh, pid, &b)) != GSPMD_OK) return st;
  for (int i = 0; i < b.rank; ++i) {
    offset[i] = b.offset[i];
    valid_len[i] = b.valid[i];
    if (shard_size) shard_size[i] = b.shard[i];
  }
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_classify_dot(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                           const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                           const gspmd_sharding* out_sh, int32_t* axis_class) try {
  if (!axis_class) return GSPMD_ERR_NULL;
  DotRoles r;
  int32_t cls[kMaxRank];
  const int32_t st = analyse_dot(mesh, dims, lhs_sh, rhs_sh, out_sh, &r, cls);
  if (st != GSPMD_OK) return st;
  for (int a = 0; a < mesh->rank; ++a) axis_class[a] = cls[a];
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_infer_out_sharding(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                                 const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                                 int32_t* out_mapping, int64_t* out_shape, int32_t* out_rank) try {
  if (!out_mapping || !dims) return GSPMD_ERR_NULL;
  int32_t st = validate_mesh(mesh, nullptr);
  if (st != GSPMD_OK) return st;
  if ((st = validate_sharding(mesh, lhs_sh)) != GSPMD_OK || (st = validate_sharding(mesh, rhs_sh)) != GSPMD_OK) return st;
  // a provisional, unsplit output lets analyse_dot check the dimension numbers and name the roles
  const int nb = dims->n_batch, nc = dims->n_contract;
  if (nb < 0 || nc < 0 || nb + nc > lhs_sh->rank || nb + nc > rhs_sh->rank) return GSPMD_ERR_BAD_DOT_DIMS;
  const int rank = lhs_sh->rank + rhs_sh->rank - nb - 2 * nc;
  if (rank <= 0 || rank > kMaxRank) return GSPMD_ERR_UNSUPPORTED;
  int64_t shape[kMaxRank];
  int32_t map[kMaxRank];
  std::vector<bool> lused(static_cast<size_t>(lhs_sh->rank), false), rused(static_cast<size_t>(rhs_sh->rank), false);
  for (int i = 0; i < nb; ++i) {
    const int a = dims->lhs_batch ? dims->lhs_batch[i] : -1, b = dims->rhs_batch ? dims->rhs_batch[i] : -1;
    if (a < 0 || a >= lhs_sh->rank || b < 0 || b >= rhs_sh->rank) return GSPMD_ERR_BAD_DOT_DIMS;
    lused[static_cast<size_t>(a)] = rused[static_cast<size_t>(b)] = true;
  }
  for (int i = 0; i < nc; ++i) {
    const int a = dims->lhs_contract ? dims->lhs_contract[i] : -1, b = dims->rhs_contract ? dims->rhs_contract[i] : -1;
    if (a < 0 || a >= lhs_sh->rank || b < 0 || b >= rhs_sh->rank) return GSPMD_ERR_BAD_DOT_DIMS;
    lused[static_cast<size_t>(a)] = rused[static_cast<size_t>(b)] = true;
  }
  int n = 0;
  for (int i = 0; i < nb; ++i) { shape[n] = lhs_sh->global_shape[dims->lhs_batch[i]]; map[n++] = -1; }
  for (int i = 0; i < lhs_sh->rank; ++i) if (!lused[static_cast<size_t>(i)]) { shape[n] = lhs_sh->global_shape[i]; map[n++] = -1; }
  for (int i = 0; i < rhs_sh->rank; ++i) if (!rused[static_cast<size_t>(i)]) { shape[n] = rhs_sh->global_shape[i]; map[n++] = -1; }
  if (n != rank) return GSPMD_ERR_BAD_DOT_DIMS;
  gspmd_sharding out{rank, shape, map};
  DotRoles r;
  // roles and size checks only: run the analysis on a 1-partition mesh so that no pattern is rejected yet
  const int64_t one = 1, zero = 0;
  gspmd_mesh unit{1, &one, &zero};
  std::vector<int32_t> lm(static_cast<size_t>(lhs_sh->rank), -1), rm(static_cast<size_t>(rhs_sh->rank), -1);
  gspmd_sharding l1{lhs_sh->rank, lhs_sh->global_shape, lm.data()}, r1{rhs_sh->rank, rhs_sh->global_shape, rm.data()};
  if ((st = analyse_dot(&unit, dims, &l1, &r1, &out, &r, nullptr)) != GSPMD_OK) return st;
  for (int a = 0; a < mesh->rank; ++a) {
    if (mesh->shape[a] == 1) continue;                // splits nothing
    int ld = -1, rd = -1;
    for (int i = 0; i < lhs_sh->rank; ++i) if (lhs_sh->dims_mapping[i] == a) ld = i;
    for (int i = 0; i < rhs_sh->rank; ++i) if (rhs_sh->dims_mapping[i] == a) rd = i;
    if (ld < 0 && rd < 0) continue;
    auto idx = [](const int* list, int cnt, int v) { for (int i = 0; i < cnt; ++i) if (list[i] == v) return i; return -1; };
    const int lb = ld >= 0 ? idx(r.lhs_batch, r.nb, ld) : -1, rbb = rd >= 0 ? idx(r.rhs_batch, r.nb, rd) : -1;
    const int lcn = ld >= 0 ? idx(r.lhs_contract, r.nc, ld) : -1, rcn = rd >= 0 ? idx(r.rhs_contract, r.nc, rd) : -1;
    const int lf = ld >= 0 ? idx(r.lhs_free, r.nlf, ld) : -1, rf = rd >= 0 ? idx(r.rhs_free, r.nrf, rd) : -1;
    if (lb >= 0 || rbb >= 0) {                        // a batch pair must be split alike on both sides
      if (lb < 0 || rbb != lb) return GSPMD_ERR_NEEDS_RESHARD;
      map[lb] = a;
    } else if (lcn >= 0 || rcn >= 0) {                // so must a contracting pair; the output is a partial sum
      if (lcn < 0 || rcn != lcn) return GSPMD_ERR_NEEDS_RESHARD;
    } else if (lf >= 0 && rf >= 0) {                  // one mesh dimension cannot split two output dimensions
      return GSPMD_ERR_NEEDS_RESHARD;
    } else if (lf >= 0) {
      map[r.nb + lf] = a;
    } else {
      map[r.nb + r.nlf + rf] = a;
    }
  }
  for (int i = 0; i < rank; ++i) { out_mapping[i] = map[i]; if (out_shape) out_shape[i] = shape[i]; }
  if (out_rank) *out_rank = rank;
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_plan_dot(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                       const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh, const gspmd_sharding* out_sh,
                       int64_t lhs_row_stride, int64_t rhs_row_stride, int64_t out_row_stride,
                       int64_t pid, const int64_t* lhs_fill,
                       gspmd_gemm_desc* descs, int64_t capacity, int64_t* count) try {
  if (!count || (capacity > 0 && !descs)) return GSPMD_ERR_NULL;
  if (capacity < 0 || lhs_row_stride < 0 || rhs_row_stride < 0 || out_row_stride < 0) return GSPMD_ERR_BAD_BUFFER;
  DotRoles r;
  int32_t cls[kMaxRank];
  int32_t st = analyse_dot(mesh, dims, lhs_sh, rhs_sh, out_sh, &r, cls);
  if (st != GSPMD_OK) return st;
  // plan against made-up base addresses far apart, with 1-byte elements, so that pointer differences are element offsets
  const uintptr_t base_a = uintptr_t(1) << 44, base_b = uintptr_t(2) << 44, base_c = uintptr_t(3) << 44;
  gspmd_shard_buf la{reinterpret_cast<void*>(base_a), GSPMD_F32, lhs_row_stride};
  gspmd_shard_buf rb{reinterpret_cast<void*>(base_b), GSPMD_F32, rhs_row_stride};
  gspmd_shard_buf oc{reinterpret_cast<void*>(base_c), GSPMD_F32, out_row_stride};
  std::vector<Problem> ps;
  int64_t elems = 0;
  int32_t layout = 0;
  if ((st = plan_partition(mesh, r, &la, lhs_sh, &rb, rhs_sh, &oc, out_sh, pid, lhs_fill, nullptr, &ps, &elems, &layout)) != GSPMD_OK) return st;
  *count = static_cast<int64_t>(ps.size());
  // the operand addresses here are made up: the path is named from the leading dimensions alone
  std::vector<Problem> live;
  for (const auto& p : ps) if (p.Mv > 0) live.push_back(p);
  const KernelPath kp = kernel_path(live, GSPMD_BF16, layout, false);
  const int32_t path = kp == kPathMfmaDirect ? GSPMD_KERNEL_MFMA : kp == kPathFallback ? GSPMD_KERNEL_SCALAR : GSPMD_KERNEL_MFMA_STAGED;
  for (int64_t i = 0; i < std::min<int64_t>(capacity, *count); ++i) {
    const Problem& p = ps[static_cast<size_t>(i)];
    gspmd_gemm_desc& d = descs[i];
    d.a_offset = static_cast<int64_t>(reinterpret_cast<uintptr_t>(p.A) - base_a) / 4;
    d.b_offset = static_cast<int64_t>(reinterpret_cast<uintptr_t>(p.B) - base_b) / 4;
    d.c_offset = static_cast<int64_t>(reinterpret_cast<uintptr_t>(p.C) - base_c) / 4;
    d.lda = p.lda; d.ldb = p.ldb; d.ldc = p.ldc;
    d.m_valid = p.Mv; d.n_valid = p.Nv; d.k_valid = p.Kv;
    d.m_static = p.Ms; d.n_static = p.Ns;
    d.layout = layout;
    d.kernel = path;
    d.reserved = 0;
  }
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_dot_workspace_bytes(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                                  const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                                  const gspmd_sharding* out_sh, int64_t pid, int32_t /*has_fill*/,
                                  int64_t* bytes) try {
  if (!bytes) return GSPMD_ERR_NULL;
  DotRoles r;
  int32_t cls[kMaxRank];
  int32_t st = analyse_dot(mesh, dims, lhs_sh, rhs_sh, out_sh, &r, cls);
  if (st != GSPMD_OK) return st;
  int64_t P = 1;
  for (int a = 0; a < mesh->rank; ++a) P *= mesh->shape[a];
  if (pid < -1 || pid >= P) return GSPMD_ERR_PARTITION_RANGE;
  int64_t n_prob = 0, partial_bytes = 0, tiles = 0;
  const bool contracting = has_contracting(mesh, cls);
  int32_t pmap[kMaxRank];
  partial_mapping(mesh, cls, out_sh, pmap);
  const gspmd_sharding part_sh{out_sh->rank, out_sh->global_shape, pmap};
  {                              // static shards: what is counted is the same for every partition
    const int64_t partitions = pid < 0 ? P : 1;
    int64_t n, e, t;
    if ((st = count_partition(mesh, r, lhs_sh, rhs_sh, &part_sh, std::max<int64_t>(pid, 0), &n, &e, &t, kMfmaBM)) != GSPMD_OK) return st;
    n_prob = n * partitions;
    tiles = std::min<int64_t>(t * partitions, int64_t(1) << 40);
    if (pid < 0 && contracting) partial_bytes = round_up(e * 4, kWsAlign) * partitions;
  }
  // A grouped call with a contracting mesh dimension keeps its partial sums either as one dense fp32 array per
  // partition or, when the problems can be joined in one launch, as one slot per output tile and partition plus a
  // counter per tile; the second layout is offered only while it stays within reach of the first.
  if (pid < 0 && contracting) {
    const int64_t joined = joined_bytes(tiles, tiles);
    if (joined <= 2 * partial_bytes + kJoinSlack) partial_bytes = std::max(partial_bytes, joined);
  }
  *bytes = round_up(std::max<int64_t>(n_prob, 1) * kTableBytesPerProblem, kWsAlign) + partial_bytes;
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_local_dot(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                        const gspmd_shard_buf* lhs, const gspmd_sharding* lhs_sh,
                        const gspmd_shard_buf* rhs, const gspmd_sharding* rhs_sh,
                        const gspmd_shard_buf* out, const gspmd_sharding* out_sh,
                        int64_t pid, const int64_t* lhs_fill, int32_t epilogue,
                        void* workspace, int64_t workspace_bytes, void* hip_stream) try {
  int32_t st;
  if (!is_epilogue(epilogue)) return GSPMD_ERR_UNSUPPORTED;
  if ((st = check_buf(lhs)) != GSPMD_OK || (st = check_buf(rhs)) != GSPMD_OK || (st = check_buf(out)) != GSPMD_OK) return st;
  DotRoles r;
  int32_t cls[kMaxRank];
  if ((st = analyse_dot(mesh, dims, lhs_sh, rhs_sh, out_sh, &r, cls)) != GSPMD_OK) return st;
  if (lhs->dtype != rhs->dtype) return GSPMD_ERR_UNSUPPORTED;
  if (has_contracting(mesh, cls) && (out->dtype != GSPMD_F32 || epilogue != GSPMD_EPILOGUE_NONE)) return GSPMD_ERR_UNSUPPORTED;
  if (has_scatter(mesh, cls)) return GSPMD_ERR_UNSUPPORTED;   // a slice of a sum exists only after the exchange
  std::vector<Problem> ps;
  int64_t elems = 0;
  int32_t layout = 0;
  if ((st = plan_partition(mesh, r, lhs, lhs_sh, rhs, rhs_sh, out, out_sh, pid, lhs_fill, nullptr, &ps, &elems, &layout)) != GSPMD_OK)
    return st;
  for (const auto& p : ps)
    if ((p.Kv && (!p.A || !p.B)) || !p.C) return GSPMD_ERR_NULL;
  t_last.sums_begin = t_last.sums_end = 0;
  return launch_problems(ps, layout, lhs->dtype, out->dtype, epilogue, has_contracting(mesh, cls), workspace, workspace_bytes,
                         static_cast<hipStream_t>(hip_stream));
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_grouped_dot(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                          const gspmd_shard_buf* lhs_shards, const gspmd_sharding* lhs_sh,
                          const gspmd_shard_buf* rhs_shards, const gspmd_sharding* rhs_sh,
                          const gspmd_shard_buf* out_shards, const gspmd_sharding* out_sh,
                          const int64_t* lhs_fill, int32_t epilogue,
                          void* workspace, int64_t workspace_bytes, void* hip_stream) try {
  if (!lhs_shards || !rhs_shards || !out_shards) return GSPMD_ERR_NULL;
  if (!is_epilogue(epilogue)) return GSPMD_ERR_UNSUPPORTED;
  DotRoles r;
  int32_t cls[kMaxRank];
  int32_t st;
  if ((st = analyse_dot(mesh, dims, lhs_sh, rhs_sh, out_sh, &r, cls)) != GSPMD_OK) return st;
  int64_t P = 1;
  for (int a = 0; a < mesh->rank; ++a) P *= mesh->shape[a];
  const int32_t in_dtype = lhs_shards[0].dtype, out_dtype = out_shards[0].dtype;
  for (int64_t p = 0; p < P; ++p) {
    if ((st = check_buf(&lhs_shards[p])) != GSPMD_OK || (st = check_buf(&rhs_shards[p])) != GSPMD_OK ||
        (st = check_buf(&out_shards[p])) != GSPMD_OK) return st;
    if (lhs_shards[p].dtype != in_dtype || rhs_shards[p].dtype != in_dtype || out_shards[p].dtype != out_dtype)
      return GSPMD_ERR_UNSUPPORTED;
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const bool contracting = has_contracting(mesh, cls);

  // workspace = [problem table][fp32 partial of partition 0][partial of partition 1]...
  int64_t need = 0;
  if ((st = gspmd_dot_workspace_bytes(mesh, dims, lhs_sh, rhs_sh, out_sh, -1, lhs_fill != nullptr, &need)) != GSPMD_OK) return st;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kWsAlign - 1)) || workspace_bytes < need) return GSPMD_ERR_WORKSPACE;
  int64_t n_bound = 0;
  std::vector<int64_t> elems(static_cast<size_t>(P), 0);
  int32_t pmap[kMaxRank];
  partial_mapping(mesh, cls, out_sh, pmap);
  const gspmd_sharding part_sh{out_sh->rank, out_sh->global_shape, pmap};   // == out_sh unless a sum is scattered
  if (contracting) {
    int64_t n, e;
    if ((st = count_partition(mesh, r, lhs_sh, rhs_sh, &part_sh, 0, &n, &e)) != GSPMD_OK) return st;
    n_bound = n * P;
    elems.assign(static_cast<size_t>(P), e);
  }
  char* partial_base = static_cast<char*>(workspace) + round_up(std::max<int64_t>(n_bound, 1) * kTableBytesPerProblem, kWsAlign);
  std::vector<float*> partial(static_cast<size_t>(P), nullptr);
  if (contracting) {
    int64_t off = 0;
    for (int64_t p = 0; p < P; ++p) {
      partial[static_cast<size_t>(p)] = reinterpret_cast<float*>(partial_base + off);
      off += round_up(elems[static_cast<size_t>(p)] * 4, kWsAlign);
    }
  }

  // Reduce groups: partitions that differ only along contracting mesh dimensions, in ascending mesh position.
  std::map<std::vector<int64_t>, std::vector<std::pair<int64_t, int64_t>>> groups;   // key -> (lin pos, pid)
  if (contracting) {
    for (int64_t p = 0; p < P; ++p) {
      int64_t coords[kMaxRank];
      if ((st = mesh_coords(mesh, p, coords)) != GSPMD_OK) return st;
      std::vector<int64_t> key;
      int64_t pos = 0;
      for (int a = 0; a < mesh->rank; ++a) {
        if (is_contracting(cls[a])) pos = pos * mesh->shape[a] + coords[a];
        else key.push_back(coords[a]);
      }
      groups[key].emplace_back(pos, p);
    }
    for (auto& kv : groups) std::sort(kv.second.begin(), kv.second.end());
  }

  // One launch for the whole sum (the AllReduce / ReduceScatter of Section 4.2 folded into the contraction): the
  // problems of a reduce group's members are joined -- every output tile gets one contribution per member, added in
  // ascending mesh position by whichever workgroup finishes last.  Two shapes qualify.  AllReduce: every member writes
  // the same out buffer and lowers to the same output blocks.  ReduceScatter along the output's last dimension, when
  // that is the only non-contracting rhs dimension and the scatter mesh dimension the only contracting one: each
  // member's problems are cut into the column ranges the members own, and the pieces for one owner are joined into that
  // owner's out shard.  Otherwise (other scattered sums, members with out buffers of their own, operands the MFMA
  // kernel cannot take, a workspace sized for the dense layout only) the partials go to dense arrays and a second
  // kernel sums them.
  int n_contracting_dims = 0;
  for (int a = 0; a < mesh->rank; ++a) n_contracting_dims += is_contracting(cls[a]) ? 1 : 0;
  const int last_out = out_sh->rank - 1;
  const bool scatter = has_scatter(mesh, cls);
  const bool scatter_by_columns = scatter && n_contracting_dims == 1 && r.nrf == 1 && out_sh->dims_mapping[last_out] >= 0 &&
                                  cls[out_sh->dims_mapping[last_out]] == GSPMD_AXIS_CONTRACTING_SCATTER;
  if (contracting && (!scatter || scatter_by_columns) && in_dtype == GSPMD_BF16) {
    std::vector<Problem> joined, apart;           // the sum in one launch; the members' products by themselves
    int32_t jlayout = 0;
    int64_t jtiles = 0, jslots = 0;
    bool ok = true;
    const size_t out_esize = out_dtype == GSPMD_BF16 ? 2 : 4;
    char* const dummy_c = reinterpret_cast<char*>(uintptr_t(1) << 44);      // never dereferenced: offsets are read off it
    for (auto& kv : groups) {
      const auto& members = kv.second;
      // the members' problems: against the shared out buffer, or (scattered) against a made-up dense partial
      std::vector<std::vector<Problem>> base(members.size());
      const gspmd_shard_buf& o0 = out_shards[members[0].second];
      for (size_t m = 0; m < members.size() && ok; ++m) {
        const int64_t p = members[m].second;
        if (!scatter) ok = out_shards[p].data == o0.data && out_shards[p].row_stride == o0.row_stride;
        if (!ok) break;
        int64_t e = 0;
        if ((st = plan_partition(mesh, r, &lhs_shards[p], lhs_sh, &rhs_shards[p], rhs_sh, &out_shards[p], scatter ? &part_sh : out_sh, p,
                                 lhs_fill, scatter ? dummy_c : nullptr, &base[m], &e, &jlayout)) != GSPMD_OK) return st;
        for (const auto& q : base[m])
          if ((q.Kv && (!q.A || !q.B)) || !q.C) return GSPMD_ERR_NULL;
        ok = base[m].size() == base[0].size();
      }
      if (!ok) break;
      for (const auto& list : base)
        for (const auto& q : list) if (q.Mv > 0) apart.push_back(q);
      // one round per owner of output columns: the one shared buffer, or every member's own slice
      for (size_t owner = 0; ok && owner < (scatter ? members.size() : 1); ++owner) {
        std::vector<std::vector<Problem>> pm = base;
        if (scatter) {
          const int64_t po = members[owner].second;
          Bounds ob;
          if ((st = shard_bounds(mesh, out_sh, po, &ob)) != GSPMD_OK) return st;
          if (!out_shards[po].data && ob.shard[last_out] > 0) return GSPMD_ERR_NULL;
          const int64_t off = ob.offset[last_out], width = ob.shard[last_out];
          const int64_t ldo = out_sh->rank >= 2 && out_shards[po].row_stride > 0 ? out_shards[po].row_stride : width;
          if (ldo < width || ldo > INT32_MAX || width > INT32_MAX) { ok = false; break; }
          for (auto& list : pm)
            for (auto& q : list) {
              const int64_t elem = (static_cast<char*>(q.C) - dummy_c) / 4;          // offset inside the dense partial
              if (q.Ns <= 0 || elem % q.Ns != 0) { ok = false; break; }
              const int64_t row = elem / q.Ns;
              const int64_t nv = std::max<int64_t>(0, std::min<int64_t>(ob.valid[last_out], static_cast<int64_t>(q.Nv) - off));
              const int64_t b_step = (jlayout & GSPMD_LAYOUT_RHS_K_CONTIGUOUS) ? off * q.ldb : off;
              q.B = static_cast<const char*>(q.B) + b_step * 2;
              q.C = static_cast<char*>(out_shards[po].data) + row * ldo * static_cast<int64_t>(out_esize);
              q.ldc = static_cast<int32_t>(ldo);
              q.Ns = static_cast<int32_t>(width);
              q.Nv = static_cast<int32_t>(nv);
              if (q.Mv == 0 || q.Nv == 0 || q.Kv == 0) q.Mv = q.Nv = q.Kv = 0;
            }
        }
        for (size_t i = 0; ok && i < pm[0].size(); ++i) {
          std::vector<size_t> live;
          for (size_t m = 0; m < members.size(); ++m) {
            const Problem &q = pm[m][i], &q0 = pm[0][i];
            ok = ok && q.C == q0.C && q.ldc == q0.ldc && q.Ms == q0.Ms && q.Ns == q0.Ns;
            if (q.Kv > 0) {
              if (!live.empty()) ok = ok && q.Mv == pm[live[0]][i].Mv && q.Nv == pm[live[0]][i].Nv;
              live.push_back(m);
            }
          }
          if (!ok || live.size() > static_cast<size_t>(kMaxPartials)) { ok = false; break; }
          if (live.size() <= 1) {
            joined.push_back(pm[live.empty() ? 0 : live[0]][i]);       // nothing to add up (a dead problem still has its zero fill)
            continue;
          }
          const int64_t t = tiles_of(pm[live[0]][i], kMfmaBM, kMfmaBN);
          for (size_t k = 0; k < live.size(); ++k) {
            Problem q = pm[live[k]][i];
            q.join_count = static_cast<int32_t>(live.size());
            q.join_slot = static_cast<int32_t>(k);
            q.join_first = static_cast<int32_t>(jtiles);
            joined.push_back(q);
          }
          jtiles += t;
          jslots += t * static_cast<int64_t>(live.size());
          if (jtiles > INT32_MAX) { ok = false; break; }
        }
      }
      if (!ok) break;
    }
    JoinSpace js;
    if (ok) {
      std::vector<Problem> live;
      for (const auto& q : joined) if (q.Mv > 0) live.push_back(q);
      const MfmaChoice one = pick_kernel(live, kernel_path(live, in_dtype, jlayout), jlayout, true);
      js.chain = jslots > 0 && with_records(one.kernel) == kMfmaMid;
      ok = one.kernel != kMfmaNone;
      if (ok && t_pin.one_launch >= 0) {
        ok = t_pin.one_launch == 1;
      } else if (ok && !apart.empty()) {
        const MfmaChoice two = pick_kernel(apart, kernel_path(apart, in_dtype, jlayout), jlayout, true);
        int64_t partial_bytes = 0, launches = 0;
        bool summable = true;       // the sum kernels take so many partials, those of members without any K among them
        for (int64_t e : elems) partial_bytes += 4 * e;
        for (const auto& kv : groups) {
          ++launches;
          summable = summable && kv.second.size() <= static_cast<size_t>(kMaxPartials);
        }
        ok = !summable || sum_us(live, one, jlayout) <= (launch_size(live, jlayout).mid > kSeveralRounds ? 1.05 : 1.15) * (sum_us(apart, two, jlayout) + apart_us(partial_bytes, launches));
      }
    }
    // Behind the launch tables come the counters, then the slots.  A scattered sum has more entries than the query counted (one
    // per member and owner), so tables too large for the kernel arguments may reach beyond the space it kept for them.
    int64_t table_area = partial_base - static_cast<char*>(workspace);
    if (joined.size() > static_cast<size_t>(kInlineProblems))
      table_area = std::max(table_area, round_up(static_cast<int64_t>(joined.size()) * kTableBytesPerProblem, kWsAlign));
    if (ok && table_area + (js.chain ? 0 : joined_bytes(jtiles, jslots)) <= workspace_bytes) {
      char* const counters = static_cast<char*>(workspace) + table_area;
      js.counters = reinterpret_cast<uint32_t*>(counters);
      js.partials = reinterpret_cast<float*>(counters + round_up(jtiles * 4, kWsAlign));
      js.tiles = jtiles;
      t_last.sums_begin = js.chain ? 0 : table_area;
      t_last.sums_end = js.chain ? 0 : table_area + joined_bytes(jtiles, jslots);
      // where only one member of every sum has any K nothing is joined: a launch like any other, by the kernel that the estimate was made for
      st = launch_problems(joined, jlayout, in_dtype, out_dtype, epilogue, true, workspace, workspace_bytes, stream, jslots > 0 ? &js : nullptr);
      t_last.one_launch = 1;
      return st;
    }
  }

  std::vector<Problem> ps;
  // Partitions that hold the same operands and write the same buffer (replicas along an
  // unused mesh dimension) need the product only once.
  std::map<std::array<const void*, 3>, int64_t> done;
  int32_t layout = 0;
  for (int64_t p = 0; p < P; ++p) {
    if (!contracting) {
      std::array<const void*, 3> key = {lhs_shards[p].data, rhs_shards[p].data, out_shards[p].data};
      if (done.count(key)) continue;
      done[key] = p;
    }
    int64_t e = 0;
    const size_t before = ps.size();
    st = plan_partition(mesh, r, &lhs_shards[p], lhs_sh, &rhs_shards[p], rhs_sh, &out_shards[p], &part_sh, p, lhs_fill,
                        contracting ? partial[static_cast<size_t>(p)] : nullptr, &ps, &e, &layout);
    if (st != GSPMD_OK) return st;
    for (size_t i = before; i < ps.size(); ++i)
      if ((ps[i].Kv && (!ps[i].A || !ps[i].B)) || !ps[i].C) return GSPMD_ERR_NULL;
  }
  t_last.sums_begin = t_last.sums_end = 0;
  if (contracting) {
    t_last.sums_begin = partial_base - static_cast<char*>(workspace);
    t_last.sums_end = t_last.sums_begin;
    for (int64_t e : elems) t_last.sums_end += round_up(e * 4, kWsAlign);
  }
  st = launch_problems(ps, layout, in_dtype, contracting ? GSPMD_F32 : out_dtype, contracting ? GSPMD_EPILOGUE_NONE : epilogue,
                       contracting, workspace, workspace_bytes, stream);
  if (st != GSPMD_OK || !contracting || t_pin.dry_run) return st;

  // Sum the partials of each reduce group, ascending in mesh position, into every distinct out buffer of the group.
  for (auto& kv : groups) {
    auto& members = kv.second;
    if (members.size() > static_cast<size_t>(kMaxPartials)) return GSPMD_ERR_UNSUPPORTED;
    std::vector<const float*> ptrs;
    for (auto& m : members) ptrs.push_back(partial[static_cast<size_t>(m.second)]);
    std::vector<int64_t> owners;          // one member per distinct out buffer
    for (auto& m : members) {
      bool seen = false;
      for (int64_t o : owners) seen = seen || out_shards[o].data == out_shards[m.second].data;
      if (!seen) owners.push_back(m.second);
    }
    if ((st = launch_reduce_scatter(mesh, out_sh, &part_sh, owners.data(), static_cast<int>(owners.size()), ptrs.data(),
                                    static_cast<int>(ptrs.size()), out_shards, epilogue, stream)) != GSPMD_OK)
      return st;
  }
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_grouped_dot_noalloc(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                                  const gspmd_shard_buf* lhs_shards, const gspmd_sharding* lhs_sh,
                                  const gspmd_shard_buf* rhs_shards, const gspmd_sharding* rhs_sh,
                                  const gspmd_shard_buf* out_shards, const gspmd_sharding* out_sh,
                                  const int64_t* lhs_fill, int32_t epilogue, void* hip_stream) try {
  int64_t need = 0;
  const int32_t st = gspmd_dot_workspace_bytes(mesh, dims, lhs_sh, rhs_sh, out_sh, -1, lhs_fill != nullptr, &need);
  if (st != GSPMD_OK) return st;
  if (need > kScratchBytes) return GSPMD_ERR_WORKSPACE;     // launch tables + fp32 partials do not fit the static array
  void* ws = scratch_address();
  if (!ws) return GSPMD_ERR_DEVICE;
  return gspmd_grouped_dot(mesh, dims, lhs_shards, lhs_sh, rhs_shards, rhs_sh, out_shards, out_sh, lhs_fill, epilogue,
                           ws, kScratchBytes, hip_stream);
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_reduce_partials(const void* const* partials, int32_t n_partials, int64_t n_elems,
                              void* out, int32_t out_dtype, void* hip_stream) try {
  if (!partials || !out) return GSPMD_ERR_NULL;
  if (n_partials < 1 || n_partials > kMaxPartials || n_elems < 0) return GSPMD_ERR_BAD_BUFFER;
  if (!is_dtype(out_dtype)) return GSPMD_ERR_UNSUPPORTED;
  for (int i = 0; i < n_partials; ++i) if (!partials[i]) return GSPMD_ERR_NULL;
  return launch_reduce(reinterpret_cast<const float* const*>(partials), n_partials, 1, n_elems, n_elems, out, n_elems,
                       out_dtype, static_cast<hipStream_t>(hip_stream));
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

static int32_t shard_copy(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t pid, const void* src_global,
                          void* dst_global, const gspmd_shard_buf* shard, uint32_t pad_bits, bool extract, void* hip_stream) try {
  int32_t st = validate_mesh(mesh, nullptr);
  if (st != GSPMD_OK) return st;
  if ((st = validate_sharding(mesh, sh)) != GSPMD_OK) return st;
  if ((st = check_buf(shard)) != GSPMD_OK) return st;
  if (has_no_elements(sh)) return GSPMD_OK;   // nothing to copy
  if (!shard->data || (extract ? !src_global : !dst_global)) return GSPMD_ERR_NULL;
  Bounds b;
  if ((st = shard_bounds(mesh, sh, pid, &b)) != GSPMD_OK) return st;
  CopyDesc d;
  std::memset(&d, 0, sizeof(d));
  d.rank = b.rank;
  int64_t total = 1, goff = 0, gs = 1;
  for (int i = b.rank - 1; i >= 0; --i) {
    d.shard[i] = b.shard[i];
    d.valid[i] = b.valid[i];
    d.gstride[i] = gs;
    goff += b.offset[i] * gs;
    gs *= sh->global_shape[i];
    total *= b.shard[i];
  }
  d.sstride[b.rank - 1] = 1;
  if (b.rank >= 2) {
    const int64_t rs = shard->row_stride > 0 ? shard->row_stride : b.shard[b.rank - 1];
    if (rs < b.shard[b.rank - 1]) return GSPMD_ERR_BAD_BUFFER;
    d.sstride[b.rank - 2] = rs;
    for (int i = b.rank - 3; i >= 0; --i) d.sstride[i] = d.sstride[i + 1] * b.shard[i + 1];
  }
  if (total == 0) return GSPMD_OK;
  // A partition wholly in the padding has an offset past the end; it reads/writes nothing
  // of the global tensor, so keep the base pointer in range.
  bool any_valid = true;
  for (int i = 0; i < b.rank; ++i) any_valid = any_valid && b.valid[i] > 0;
  if (!any_valid) goff = 0;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  // 32-bit index arithmetic in shard_move_kernel: extents and rows must fit
  int64_t rows = 1;
  bool fits = true;
  for (int i = 0; i < b.rank; ++i) {
    fits = fits && sh->global_shape[i] <= kMoveMaxExtent;
    if (i < b.rank - 1) rows = std::min<int64_t>(rows * (extract ? b.shard[i] : b.valid[i]), int64_t(INT32_MAX) + 1);
  }
  if (fits && rows <= INT32_MAX) {
    if (!extract && !any_valid) return GSPMD_OK;
    ShardCopy sc;
    std::memset(&sc, 0, sizeof(sc));
    sc.shape.rank = b.rank;
    sc.shape.rows = static_cast<int32_t>(rows);
    sc.shape.pad = pad_bits;
    // the tensor's side starts where the shard begins in it; either side is one src "shard" that holds everything
    const int64_t esz = shard->dtype == GSPMD_BF16 ? 2 : 4;
    if (extract) {
      sc.src = static_cast<const char*>(src_global) + goff * esz;
      sc.box.dst = shard->data;
    } else {
      sc.src = shard->data;
      sc.box.dst = static_cast<char*>(dst_global) + goff * esz;
    }
    for (int i = 0; i < b.rank; ++i) {
      sc.shape.shard[i] = static_cast<int32_t>(extract ? b.shard[i] : b.valid[i]);
      sc.box.valid[i] = static_cast<int32_t>(b.valid[i]);
      sc.shape.src_per[i] = INT32_MAX;
      sc.shape.dst_stride[i] = extract ? d.sstride[i] : d.gstride[i];
      sc.shape.src_stride[i] = extract ? d.gstride[i] : d.sstride[i];
    }
    const dim3 grid = move_grid(&sc.shape, reinterpret_cast<uintptr_t>(sc.box.dst), 1, static_cast<int>(16 / esz));
    if (shard->dtype == GSPMD_BF16) hipLaunchKernelGGL((shard_move_kernel<bf16_bits>), grid, dim3(256), 0, stream, sc);
    else hipLaunchKernelGGL((shard_move_kernel<uint32_t>), grid, dim3(256), 0, stream, sc);
    return hipGetLastError() == hipSuccess ? GSPMD_OK : GSPMD_ERR_DEVICE;
  }
  const unsigned blocks = static_cast<unsigned>(std::min<int64_t>((total + 255) / 256, 256 * 32));
  const dim3 grid(blocks), block(256);
  if (shard->dtype == GSPMD_BF16) {
    typedef bf16_bits T;
    if (extract) hipLaunchKernelGGL((shard_copy_kernel<T, true>), grid, block, 0, stream, d, static_cast<const T*>(src_global) + goff, static_cast<T*>(shard->data), static_cast<T>(pad_bits & 0xffffu), total);
    else hipLaunchKernelGGL((shard_copy_kernel<T, false>), grid, block, 0, stream, d, static_cast<const T*>(shard->data), static_cast<T*>(dst_global) + goff, static_cast<T>(0), total);
  } else {
    typedef uint32_t T;
    if (extract) hipLaunchKernelGGL((shard_copy_kernel<T, true>), grid, block, 0, stream, d, static_cast<const T*>(src_global) + goff, static_cast<T*>(shard->data), pad_bits, total);
    else hipLaunchKernelGGL((shard_copy_kernel<T, false>), grid, block, 0, stream, d, static_cast<const T*>(shard->data), static_cast<T*>(dst_global) + goff, 0u, total);
  }
  return hipGetLastError() == hipSuccess ? GSPMD_OK : GSPMD_ERR_DEVICE;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_shard_extract(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t pid, const void* global_data,
                            const gspmd_shard_buf* shard, uint32_t pad_bits, void* hip_stream) try {
  return shard_copy(mesh, sh, pid, global_data, nullptr, shard, pad_bits, true, hip_stream);
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_shard_assemble(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t pid, const gspmd_shard_buf* shard,
                             void* global_data, void* hip_stream) try {
  return shard_copy(mesh, sh, pid, nullptr, global_data, shard, 0, false, hip_stream);
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

// bytes of workspace per partition that the query asks for beside the src pointers (a MoveBox needs 80)
constexpr int64_t kReshardTableBytes = 312;
static_assert(sizeof(MoveBox) <= kReshardTableBytes, "the tables fit the workspace");

int32_t gspmd_reshard_workspace_bytes(const gspmd_mesh* mesh, int64_t* bytes) try {
  if (!bytes) return GSPMD_ERR_NULL;
  int64_t P = 0;
  const int32_t st = validate_mesh(mesh, &P);
  if (st != GSPMD_OK) return st;
  *bytes = round_up(P * 8, kWsAlign) + round_up(P * kReshardTableBytes, kWsAlign);
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_reshard(const gspmd_mesh* mesh, const gspmd_sharding* src_sh, const gspmd_shard_buf* src_shards,
                      const gspmd_sharding* dst_sh, const gspmd_shard_buf* dst_shards,
                      void* workspace, int64_t workspace_bytes, void* hip_stream) try {
  if (!src_shards || !dst_shards) return GSPMD_ERR_NULL;
  int64_t P = 0;
  int32_t st = validate_mesh(mesh, &P);
  if (st != GSPMD_OK) return st;
  if ((st = validate_sharding(mesh, src_sh)) != GSPMD_OK || (st = validate_sharding(mesh, dst_sh)) != GSPMD_OK) return st;
  if (src_sh->rank != dst_sh->rank) return GSPMD_ERR_BAD_SHARDING;
  const int rank = src_sh->rank, last = rank - 1;
  for (int i = 0; i < rank; ++i)
    if (src_sh->global_shape[i] != dst_sh->global_shape[i]) return GSPMD_ERR_BAD_SHARDING;
  if (P > 65535) return GSPMD_ERR_UNSUPPORTED;
  // 32-bit index arithmetic in the kernel: a padded dimension (partitions x shard size) must fit
  for (int i = 0; i < rank; ++i)
    if (src_sh->global_shape[i] > (INT32_MAX >> 1)) return GSPMD_ERR_UNSUPPORTED;
  const int32_t dtype = src_shards[0].dtype;
  for (int64_t p = 0; p < P; ++p) {
    if ((st = check_buf(&src_shards[p])) != GSPMD_OK || (st = check_buf(&dst_shards[p])) != GSPMD_OK) return st;
    if (src_shards[p].dtype != dtype || dst_shards[p].dtype != dtype) return GSPMD_ERR_UNSUPPORTED;
    if (src_shards[p].row_stride != src_shards[0].row_stride || dst_shards[p].row_stride != dst_shards[0].row_stride)
      return GSPMD_ERR_BAD_BUFFER;
    if (!has_no_elements(src_sh) && (!src_shards[p].data || !dst_shards[p].data)) return GSPMD_ERR_NULL;
  }
  if (has_no_elements(src_sh)) return GSPMD_OK;   // same global shape on both sides: nothing to move
  int64_t need = 0;
  if ((st = gspmd_reshard_workspace_bytes(mesh, &need)) != GSPMD_OK) return st;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kWsAlign - 1)) || workspace_bytes < need) return GSPMD_ERR_WORKSPACE;

  int64_t mesh_stride[kMaxRank];
  for (int a = mesh->rank - 1, acc = 1; a >= 0; --a) { mesh_stride[a] = acc; acc *= static_cast<int>(mesh->shape[a]); }
  bool src_uses[kMaxRank] = {false};
  for (int i = 0; i < rank; ++i) if (src_sh->dims_mapping[i] >= 0) src_uses[src_sh->dims_mapping[i]] = true;

  // strides of the src shards (one row_stride for all) from any partition's static shape
  Bounds sb0;
  if ((st = shard_bounds(mesh, src_sh, 0, &sb0)) != GSPMD_OK) return st;
  int64_t src_stride[kMaxRank];
  src_stride[last] = 1;
  if (rank >= 2) {
    const int64_t rs = src_shards[0].row_stride > 0 ? src_shards[0].row_stride : sb0.shard[last];
    if (rs < sb0.shard[last]) return GSPMD_ERR_BAD_BUFFER;
    src_stride[rank - 2] = rs;
    for (int i = rank - 3; i >= 0; --i) src_stride[i] = src_stride[i + 1] * sb0.shard[i + 1];
  }

  InlineReshard inl;
  std::memset(&inl, 0, sizeof(inl));
  MoveShape& shape = inl.shape;
  std::vector<MoveBox> boxes;
  std::vector<void*> seen;
  for (int64_t p = 0; p < P; ++p) {
    void* dst = dst_shards[p].data;
    if (std::find(seen.begin(), seen.end(), dst) != seen.end()) continue;   // replicas sharing a buffer: fill it once
    seen.push_back(dst);
    Bounds db;
    if ((st = shard_bounds(mesh, dst_sh, p, &db)) != GSPMD_OK) return st;
    int64_t coords[kMaxRank];
    if ((st = mesh_coords(mesh, p, coords)) != GSPMD_OK) return st;
    MoveBox d;
    std::memset(&d, 0, sizeof(d));
    d.dst = dst;
    for (int i = 0; i < rank; ++i) {
      if (db.shard[i] > INT32_MAX) return GSPMD_ERR_UNSUPPORTED;
      d.valid[i] = static_cast<int32_t>(db.valid[i]);
      d.dst_off[i] = static_cast<int32_t>(db.offset[i]);
    }
    for (int a = 0; a < mesh->rank; ++a) if (!src_uses[a]) d.base_pos += static_cast<int32_t>(coords[a] * mesh_stride[a]);
    if (boxes.empty()) {                     // static shapes and strides are the same for every partition
      int64_t rows = 1, total = 1;
      shape.rank = rank;
      for (int i = 0; i < rank; ++i) {
        shape.shard[i] = static_cast<int32_t>(db.shard[i]);
        shape.src_per[i] = static_cast<int32_t>(std::max<int64_t>(sb0.shard[i], 1));
        shape.src_stride[i] = src_stride[i];
        const int a = src_sh->dims_mapping[i];
        shape.pos_stride[i] = a >= 0 ? static_cast<int32_t>(mesh_stride[a]) : 0;
        if (i < last) rows *= db.shard[i];
        total *= db.shard[i];
      }
      shape.dst_stride[last] = 1;
      if (rank >= 2) {
        const int64_t rs = dst_shards[0].row_stride > 0 ? dst_shards[0].row_stride : db.shard[last];
        if (rs < db.shard[last]) return GSPMD_ERR_BAD_BUFFER;
        shape.dst_stride[rank - 2] = rs;
        for (int i = rank - 3; i >= 0; --i) shape.dst_stride[i] = shape.dst_stride[i + 1] * db.shard[i + 1];
      }
      if (total == 0) return GSPMD_OK;
      if (rows > INT32_MAX) return GSPMD_ERR_UNSUPPORTED;
      shape.rows = static_cast<int32_t>(rows);
    }
    boxes.push_back(d);
  }

  // tables: [src shard of the partition at each mesh position][dst boxes]; as kernel arguments when they fit, else
  // uploaded into the workspace (stream-ordered copy from a temporary host buffer)
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const void* const* d_ptrs = nullptr;
  const MoveBox* d_boxes = nullptr;
  if (P <= kInlineReshardSrc && boxes.size() <= static_cast<size_t>(kInlineReshardDescs)) {
    for (int64_t pos = 0; pos < P; ++pos) inl.src[pos] = src_shards[mesh->device_ids[pos]].data;
    std::memcpy(inl.d, boxes.data(), boxes.size() * sizeof(MoveBox));
  } else {
    const int64_t ids_bytes = round_up(P * 8, kWsAlign);
    std::vector<char> host(static_cast<size_t>(ids_bytes + boxes.size() * sizeof(MoveBox)), 0);
    for (int64_t pos = 0; pos < P; ++pos) std::memcpy(host.data() + pos * 8, &src_shards[mesh->device_ids[pos]].data, 8);
    std::memcpy(host.data() + ids_bytes, boxes.data(), boxes.size() * sizeof(MoveBox));
    if (hipMemcpyAsync(workspace, host.data(), host.size(), hipMemcpyHostToDevice, stream) != hipSuccess) return GSPMD_ERR_DEVICE;
    const char* ws = static_cast<const char*>(workspace);
    d_ptrs = reinterpret_cast<const void* const*>(ws);
    d_boxes = reinterpret_cast<const MoveBox*>(ws + ids_bytes);
  }
  uintptr_t dst_bits = 0;
  for (const MoveBox& d : boxes) dst_bits |= reinterpret_cast<uintptr_t>(d.dst);
  const dim3 grid = move_grid(&shape, dst_bits, static_cast<int64_t>(boxes.size()), dtype == GSPMD_BF16 ? 8 : 4);
  if (dtype == GSPMD_BF16) hipLaunchKernelGGL((reshard_kernel<bf16_bits>), grid, dim3(256), 0, stream, inl, d_boxes, d_ptrs);
  else hipLaunchKernelGGL((reshard_kernel<uint32_t>), grid, dim3(256), 0, stream, inl, d_boxes, d_ptrs);
  return hipGetLastError() == hipSuccess ? GSPMD_OK : GSPMD_ERR_DEVICE;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

namespace {

// Roles of the Dot's dimensions without any sharding in play (unit mesh, unsplit tensors).
int32_t dot_roles(const gspmd_dot_dims* dims, const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                  const gspmd_sharding* out_sh, DotRoles* r) {
  const int64_t one = 1, zero = 0;
  gspmd_mesh unit{1, &one, &zero};
  int32_t none[kMaxRank];
  for (int i = 0; i < kMaxRank; ++i) none[i] = -1;
  if (!lhs_sh || !rhs_sh || !out_sh) return GSPMD_ERR_NULL;
  if (lhs_sh->rank > kMaxRank || rhs_sh->rank > kMaxRank || out_sh->rank > kMaxRank) return GSPMD_ERR_BAD_SHARDING;
  gspmd_sharding l{lhs_sh->rank, lhs_sh->global_shape, none}, rr{rhs_sh->rank, rhs_sh->global_shape, none},
      o{out_sh->rank, out_sh->global_shape, none};
  return analyse_dot(&unit, dims, &l, &rr, &o, r, nullptr);
}

int index_in(const int* list, int n, int v) {
  for (int i = 0; i < n; ++i) if (list[i] == v) return i;
  return -1;
}

// Static shard shape and bytes (rows padded to 8 elements) of one partition's temporary under `sh`.
int64_t temp_shard_bytes(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t pid, size_t esize, int64_t* row_stride) {
  Bounds b;
  if (shard_bounds(mesh, sh, pid, &b) != GSPMD_OK) return -1;
  const int last = b.rank - 1;
  const int64_t ld = round_up(std::max<int64_t>(b.shard[last], 1), 8);
  int64_t rows = 1;
  for (int i = 0; i < last; ++i) rows *= b.shard[i];
  if (row_stride) *row_stride = b.rank >= 2 ? ld : 0;
  return round_up(std::max<int64_t>(rows, 1) * ld * static_cast<int64_t>(esize), kWsAlign);
}

bool same_mapping(const gspmd_sharding* sh, const int32_t* map) {
  for (int i = 0; i < sh->rank; ++i) if (sh->dims_mapping[i] != map[i]) return false;
  return true;
}

// Temporaries of one resharded operand: one buffer per distinct shard position (replicas share), laid out from `base`.
// Returns the bytes used; fills `bufs` (P entries) when base is non-null.
int64_t layout_temps(const gspmd_mesh* mesh, const gspmd_sharding* sh, int64_t P, int32_t dtype, char* base,
                     std::vector<gspmd_shard_buf>* bufs) {
  const size_t esize = dtype == GSPMD_BF16 ? 2 : 4;
  std::map<std::vector<int64_t>, int64_t> at;     // shard offset -> byte offset of its buffer
  int64_t used = 0;
  for (int64_t p = 0; p < P; ++p) {
    Bounds b;
    if (shard_bounds(mesh, sh, p, &b) != GSPMD_OK) return -1;
    std::vector<int64_t> key(b.offset, b.offset + b.rank);
    int64_t rs = 0;
    const int64_t bytes = temp_shard_bytes(mesh, sh, p, esize, &rs);
    if (bytes < 0) return -1;
    auto it = at.find(key);
    if (it == at.end()) {
      it = at.emplace(key, used).first;
      used += bytes;
    }
    if (bufs) (*bufs)[static_cast<size_t>(p)] = gspmd_shard_buf{base ? base + it->second : nullptr, dtype, rs};
  }
  return used;
}

}  // namespace

int32_t gspmd_compatible_operand_shardings(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                                           const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                                           const gspmd_sharding* out_sh, int32_t* lhs_mapping, int32_t* rhs_mapping) try {
  if (!lhs_mapping || !rhs_mapping) return GSPMD_ERR_NULL;
  int32_t st = validate_mesh(mesh, nullptr);
  if (st != GSPMD_OK) return st;
  if ((st = validate_sharding(mesh, lhs_sh)) != GSPMD_OK || (st = validate_sharding(mesh, rhs_sh)) != GSPMD_OK ||
      (st = validate_sharding(mesh, out_sh)) != GSPMD_OK) return st;
  DotRoles r;
  if ((st = dot_roles(dims, lhs_sh, rhs_sh, out_sh, &r)) != GSPMD_OK) return st;
  for (int i = 0; i < lhs_sh->rank; ++i) lhs_mapping[i] = -1;
  for (int i = 0; i < rhs_sh->rank; ++i) rhs_mapping[i] = -1;
  for (int a = 0; a < mesh->rank; ++a) {
    if (mesh->shape[a] == 1) continue;            // splits nothing
    int ld = -1, rd = -1, od = -1;
    for (int i = 0; i < lhs_sh->rank; ++i) if (lhs_sh->dims_mapping[i] == a) ld = i;
    for (int i = 0; i < rhs_sh->rank; ++i) if (rhs_sh->dims_mapping[i] == a) rd = i;
    for (int i = 0; i < out_sh->rank; ++i) if (out_sh->dims_mapping[i] == a) od = i;
    // a contracting pair split alike on both sides stays: partial sums (scattered if the output is split on it too)
    const int ci = ld >= 0 ? index_in(r.lhs_contract, r.nc, ld) : -1;
    const bool contracting = ci >= 0 && r.rhs_contract[ci] == rd;
    if (contracting) {
      lhs_mapping[ld] = a;
      rhs_mapping[rd] = a;
      continue;
    }
    if (od < 0) continue;                         // output whole on this mesh dimension: so are the operands
    if (od < r.nb) {                              // batch: all three split alike
      lhs_mapping[r.lhs_batch[od]] = a;
      rhs_mapping[r.rhs_batch[od]] = a;
    } else if (od < r.nb + r.nlf) {
      lhs_mapping[r.lhs_free[od - r.nb]] = a;
    } else {
      rhs_mapping[r.rhs_free[od - r.nb - r.nlf]] = a;
    }
  }
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_resharded_dot_workspace_bytes(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                                            const gspmd_sharding* lhs_sh, const gspmd_sharding* rhs_sh,
                                            const gspmd_sharding* out_sh, int32_t in_dtype, int64_t* bytes) try {
  if (!bytes) return GSPMD_ERR_NULL;
  if (!is_dtype(in_dtype)) return GSPMD_ERR_UNSUPPORTED;
  int32_t lmap[kMaxRank], rmap[kMaxRank];
  int32_t st = gspmd_compatible_operand_shardings(mesh, dims, lhs_sh, rhs_sh, out_sh, lmap, rmap);
  if (st != GSPMD_OK) return st;
  int64_t P = 0;
  if ((st = validate_mesh(mesh, &P)) != GSPMD_OK) return st;
  const gspmd_sharding l2{lhs_sh->rank, lhs_sh->global_shape, lmap}, r2{rhs_sh->rank, rhs_sh->global_shape, rmap};
  int64_t total = 0, n = 0;
  if ((st = gspmd_reshard_workspace_bytes(mesh, &n)) != GSPMD_OK) return st;
  total += 2 * n;
  if (!same_mapping(lhs_sh, lmap)) {
    if ((n = layout_temps(mesh, &l2, P, in_dtype, nullptr, nullptr)) < 0) return GSPMD_ERR_UNSUPPORTED;
    total += n;
  }
  if (!same_mapping(rhs_sh, rmap)) {
    if ((n = layout_temps(mesh, &r2, P, in_dtype, nullptr, nullptr)) < 0) return GSPMD_ERR_UNSUPPORTED;
    total += n;
  }
  if ((st = gspmd_dot_workspace_bytes(mesh, dims, &l2, &r2, out_sh, -1, 1, &n)) != GSPMD_OK) return st;
  *bytes = total + n;
  return GSPMD_OK;
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_resharded_dot(const gspmd_mesh* mesh, const gspmd_dot_dims* dims,
                            const gspmd_shard_buf* lhs_shards, const gspmd_sharding* lhs_sh,
                            const gspmd_shard_buf* rhs_shards, const gspmd_sharding* rhs_sh,
                            const gspmd_shard_buf* out_shards, const gspmd_sharding* out_sh,
                            const int64_t* lhs_fill, int32_t epilogue,
                            void* workspace, int64_t workspace_bytes, void* hip_stream) try {
  if (!lhs_shards || !rhs_shards || !out_shards) return GSPMD_ERR_NULL;
  int32_t lmap[kMaxRank], rmap[kMaxRank];
  int32_t st = gspmd_compatible_operand_shardings(mesh, dims, lhs_sh, rhs_sh, out_sh, lmap, rmap);
  if (st != GSPMD_OK) return st;
  int64_t P = 0;
  if ((st = validate_mesh(mesh, &P)) != GSPMD_OK) return st;
  if ((st = check_buf(&lhs_shards[0])) != GSPMD_OK || (st = check_buf(&rhs_shards[0])) != GSPMD_OK) return st;
  const int32_t in_dtype = lhs_shards[0].dtype;
  if (rhs_shards[0].dtype != in_dtype) return GSPMD_ERR_UNSUPPORTED;
  int64_t need = 0;
  if ((st = gspmd_resharded_dot_workspace_bytes(mesh, dims, lhs_sh, rhs_sh, out_sh, in_dtype, &need)) != GSPMD_OK) return st;
  if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & (kWsAlign - 1)) || workspace_bytes < need) return GSPMD_ERR_WORKSPACE;
  const gspmd_sharding l2{lhs_sh->rank, lhs_sh->global_shape, lmap}, r2{rhs_sh->rank, rhs_sh->global_shape, rmap};
  char* ws = static_cast<char*>(workspace);
  int64_t rs_bytes = 0;
  if ((st = gspmd_reshard_workspace_bytes(mesh, &rs_bytes)) != GSPMD_OK) return st;
  char* rs_ws[2] = {ws, ws + rs_bytes};
  ws += 2 * rs_bytes;
  std::vector<gspmd_shard_buf> ltmp(static_cast<size_t>(P)), rtmp(static_cast<size_t>(P));
  const gspmd_shard_buf* luse = lhs_shards;
  const gspmd_shard_buf* ruse = rhs_shards;
  if (!same_mapping(lhs_sh, lmap)) {
    const int64_t n = layout_temps(mesh, &l2, P, in_dtype, ws, &ltmp);
    if (n < 0) return GSPMD_ERR_UNSUPPORTED;
    ws += n;
    if ((st = gspmd_reshard(mesh, lhs_sh, lhs_shards, &l2, ltmp.data(), rs_ws[0], rs_bytes, hip_stream)) != GSPMD_OK) return st;
    luse = ltmp.data();
  }
  if (!same_mapping(rhs_sh, rmap)) {
    const int64_t n = layout_temps(mesh, &r2, P, in_dtype, ws, &rtmp);
    if (n < 0) return GSPMD_ERR_UNSUPPORTED;
    ws += n;
    if ((st = gspmd_reshard(mesh, rhs_sh, rhs_shards, &r2, rtmp.data(), rs_ws[1], rs_bytes, hip_stream)) != GSPMD_OK) return st;
    ruse = rtmp.data();
  }
  const int64_t left = workspace_bytes - (ws - static_cast<char*>(workspace));
  return gspmd_grouped_dot(mesh, dims, luse, &l2, ruse, &r2, out_shards, out_sh, lhs_fill, epilogue, ws, left, hip_stream);
} catch (...) { return GSPMD_ERR_HOST_MEMORY; }

int32_t gspmd_testing_pin(const gspmd_testing_launch* pin) {
  if (!pin) return GSPMD_ERR_NULL;
  const bool split = pin->kernel == GSPMD_TESTING_SPLIT;
  const bool known = (pin->kernel >= GSPMD_TESTING_BY_RULE && pin->kernel <= GSPMD_TESTING_SPLIT) || pin->kernel == GSPMD_TESTING_PAIR;
  if (!known || pin->one_launch < GSPMD_TESTING_BY_RULE || pin->one_launch > 1 ||
      (split ? pin->row_blocks != 1 && pin->row_blocks != 2 && pin->row_blocks != 4 : pin->row_blocks != 0)) return GSPMD_ERR_UNSUPPORTED;
  if (pin->dry_run != 0 && pin->dry_run != 1) return GSPMD_ERR_UNSUPPORTED;
  if (pin->col_blocks != 0 && !(split && (pin->col_blocks == 4 || (pin->col_blocks == 2 && pin->row_blocks <= 2)))) return GSPMD_ERR_UNSUPPORTED;
  t_pin = *pin;
  return GSPMD_OK;
}

int32_t gspmd_testing_last(gspmd_testing_launch* last) {
  if (!last) return GSPMD_ERR_NULL;
  *last = t_last;
  return GSPMD_OK;
}

int32_t gspmd_set_tile_timeline(void* device_records, int64_t n_records) try {
  if (n_records < 0 || n_records > INT32_MAX) return GSPMD_ERR_BAD_BUFFER;
  if (device_records == nullptr || n_records == 0) {
    g_timeline.store(nullptr, std::memory_order_release);
    g_timeline_records.store(0, std::memory_order_release);
    return GSPMD_OK;
  }
  if (reinterpret_cast<uintptr_t>(device_records) & 7) return GSPMD_ERR_BAD_BUFFER;
  g_timeline_records.store(static_cast<int>(n_records), std::memory_order_release);
  g_timeline.store(static_cast<unsigned long long*>(device_records), std::memory_order_release);
  return GSPMD_OK;
} catch (...) {
  return GSPMD_ERR_HOST_MEMORY;
}

}  // extern "C"

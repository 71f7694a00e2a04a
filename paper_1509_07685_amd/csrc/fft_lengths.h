// Which transform lengths run on which plans: the compile-time plans, the rules
// that plan creation and the launchers share, and the limits of the pass
// kernels.  Plain C++ (no device code), so that a host-only test can hold plan
// creation's choices against the plans that the kernels are built with.
#ifndef DKS_FFT_LENGTHS_H
#define DKS_FFT_LENGTHS_H

#include <stddef.h>

namespace dks {

constexpr int kMaxPass = 12;        // radix passes per transform (N <= 4096)
constexpr int kMaxLength = 4096;    // longest transform length
constexpr int kLdsBytes = 65536;    // LDS budget per FFT workgroup
constexpr size_t kLdsHardware = 163840;   // LDS per workgroup on gfx950 (160 KiB)

// Lanes of the runtime plan's kernels, and the most of the compile-time ones'.
template <typename T> struct PassLanes {
  static constexpr int value = sizeof(T) == 4 ? 512 : 256;
};

// ---------------------------------------------------------------------------
// Compile-time plans.  For the lengths of static_radices (every 2^a 3^b from
// 16 to 512) the kernels are instantiated with the whole plan known at
// compile time (length, tile width, LDS stride, radix order, lanes), so
// butterfly indexing, twiddle offsets and guards fold to constants; the
// runtime plan (DynPlan) serves every other shape.  A launcher uses a
// compile-time plan only when the host plan matches it exactly.
// ---------------------------------------------------------------------------
constexpr int ilog2(int v) { return v <= 1 ? 0 : 1 + ilog2(v >> 1); }
constexpr int cmin(int a, int b) { return a < b ? a : b; }
constexpr int cmax(int a, int b) { return a > b ? a : b; }

struct DynPlan {
  static constexpr bool is_static = false;
};

// Radix order of a length with a compile-time plan (n = 0: none, the length
// runs on the runtime plan).  At most three passes, the two or three radices
// near equal so that every pass keeps about the same lanes busy; the first
// radix of an even length is even (a zero-padded forward transform then skips
// its whole upper half), the last one too where the factors allow it.
// Against the runtime plan, whose time went to index arithmetic, guards and
// passes of radix 3 (the five passes of a solve): 96 x 96 x 192
// FP64 180 -> 91 us, 8 x 48^3 FP32 in one batch 115 -> 36 us, 144 x 128 x 96
// FP32 106 -> 56 us; raw 216 x 144 x 96 x 4 FP64, there and back, 410 -> 288 us.
struct RadixList {
  int n;
  int r[3];
};
constexpr RadixList static_radices(int N) {
  switch (N) {
    case 16: return {2, {4, 4, 1}};
    case 18: return {2, {6, 3, 1}};
    case 24: return {2, {6, 4, 1}};
    case 27: return {2, {9, 3, 1}};
    case 32: return {2, {8, 4, 1}};
    case 36: return {2, {6, 6, 1}};
    case 48: return {2, {8, 6, 1}};
    case 54: return {2, {6, 9, 1}};
    case 64: return {2, {8, 8, 1}};
    case 72: return {2, {12, 6, 1}};
    case 81: return {2, {9, 9, 1}};
    case 96: return {2, {8, 12, 1}};
    case 108: return {2, {12, 9, 1}};
    case 128: return {2, {16, 8, 1}};
    case 144: return {2, {12, 12, 1}};
    case 162: return {3, {6, 3, 9}};
    case 192: return {2, {16, 12, 1}};
    case 216: return {3, {6, 6, 6}};
    case 243: return {3, {9, 9, 3}};
    case 256: return {3, {8, 8, 4}};
    case 288: return {3, {8, 6, 6}};
    case 324: return {3, {6, 9, 6}};
    case 384: return {3, {8, 6, 8}};
    case 432: return {3, {6, 9, 8}};
    case 486: return {3, {6, 9, 9}};
    case 512: return {3, {8, 8, 8}};
    default: return {0, {1, 1, 1}};
  }
}

// Lengths with compile-time kernels in the convolution: x rows (pairs of
// reals: even lengths) up to 256, y and z pencils (doubled extents) from 32,
// where the intermediates' element offsets fit 32 bits.
constexpr bool static_row(int N) { return N % 2 == 0 && N <= 256 && static_radices(N).n > 0; }
constexpr bool static_pencil(int N) { return N % 2 == 0 && N >= 32 && static_radices(N).n > 0; }

// The lengths above, for switches over them.
#define DKS_STATIC_LENGTHS(F) \
  F(16) F(18) F(24) F(27) F(32) F(36) F(48) F(54) F(64) F(72) F(81) F(96) F(108) F(128) F(144) F(162) F(192) F(216) \
  F(243) F(256) F(288) F(324) F(384) F(432) F(486) F(512)

// Compile-time plan of length N (radix order static_radices, REV reversed:
// the inverse z transform), W pencils per tile with LDS stride LD, at most
// CAP lanes per workgroup.  TH lanes run the tile: the widest pass's
// butterflies in the fewest rounds that CAP allows, so a short transform does
// not carry idle wavefronts through its barriers.
template <int N_, int W_, int LD_, bool REV_, int CAP_>
struct SPlan {
  static constexpr bool is_static = true;
  static constexpr int N = N_, W = W_, LD = LD_, logW = ilog2(W_);
  static constexpr RadixList list = static_radices(N_);
  static_assert(list.n > 0 && list.r[0] * list.r[1] * list.r[2] == N_, "radices of a compile-time plan");
  static constexpr int npass = list.n;
  static constexpr int R(int p) { return REV_ ? list.r[npass - 1 - p] : list.r[p]; }
  static constexpr int Ns(int p) { return p == 0 ? 1 : Ns(p - 1) * R(p - 1); }
  static constexpr int tw_off(int p) { return p <= 1 ? 0 : tw_off(p - 1) + Ns(p - 1) * (R(p - 1) - 1); }
  static constexpr int widest() {
    int m = 0;
    for (int p = 0; p < npass; ++p) m = N / R(p) > m ? N / R(p) : m;
    return m * W;
  }
  static constexpr int rounds = (widest() + CAP_ - 1) / CAP_;
  static constexpr int TH = ((widest() + rounds - 1) / rounds + 63) / 64 * 64;
  // the first radix is even, so the first pass's upper half inputs are r >= R/2
  static constexpr bool even_first = R(0) % 2 == 0;
  using Reversed = SPlan<N_, W_, LD_, !REV_, CAP_>;
};

template <class SP, class Plan> inline bool plan_matches(const Plan& h) {
  if (h.N != SP::N || h.W != SP::W || h.LD != SP::LD || h.npass != SP::npass) return false;
  for (int p = 0; p < h.npass; ++p)
    if (h.R[p] != SP::R(p) || h.Ns[p] != SP::Ns(p) || h.tw_off[p] != SP::tw_off(p)) return false;
  return true;
}

// Radices the runtime plan's passes are written for.
constexpr bool runtime_radix(int R) { return R == 2 || R == 3 || R == 4 || R == 8; }

// Whether the kernels of the runtime plan can run host plan h.
template <class Plan> inline bool runtime_plan(const Plan& h) {
  for (int p = 0; p < h.npass; ++p)
    if (!runtime_radix(h.R[p])) return false;
  return true;
}

// ---------------------------------------------------------------------------
// Plans of the convolution: tiles of 128 bytes, x rows padded by one column.
// Each length of the switch below is tried where its rule above holds; a
// length without a compile-time plan takes the runtime plan, and a plan that
// neither can run is refused (the functions return false without a call).
// ---------------------------------------------------------------------------
template <typename T, int PAD, bool X, int N, class Plan, class F> bool try_plan(const Plan& h, F&& f) {
  constexpr int W = 128 / (2 * (int)sizeof(T));
  if constexpr (X ? static_row(N) : static_pencil(N)) {
    using SP = SPlan<N, W, W + PAD, false, PassLanes<T>::value>;
    if (plan_matches<SP>(h)) {
      f(SP{});
      return true;
    }
  }
  return false;
}
// X: plans of the x rows; otherwise of the y and z pencils.  allow: the
// compile-time kernels' 32-bit element offsets suffice (offsets_fit32).
template <typename T, int PAD, bool X, class Plan, class F> bool with_plan(const Plan& h, F&& f, bool allow = true) {
  bool done = false;
  if (allow) switch (h.N) {
#define DKS_TRY(N) case N: done = try_plan<T, PAD, X, N>(h, f); break;
    DKS_STATIC_LENGTHS(DKS_TRY)
#undef DKS_TRY
    default: break;
  }
  if (done) return true;
  if (!runtime_plan(h)) return false;
  f(DynPlan{});
  return true;
}

// ---------------------------------------------------------------------------
// Plans of the raw transforms.
// ---------------------------------------------------------------------------
// Tile width of an x (row) tile: the widest power of two <= w whose padded
// tile (N (W + 1) complex values) fits the LDS budget.
constexpr int row_width(int N, int c, int w) { return (w > 1 && N * (w + 1) * c > kLdsBytes) ? row_width(N, c, w / 2) : w; }

// 32-bit offsets inside a pencil tile when the whole array is addressable with them.
inline bool cols_fit32(size_t elems) { return elems < 0x7fffffffULL; }

// Column tiles of 256 instead of 128 bytes per row, for lengths up to 256 (the
// tile then still takes at most 64 KiB) of arrays of 64 MiB and more: the
// segments of a strided pencil pass lie a row or a plane apart, and twice the
// run per segment raised the z pass of 512 x 512 x 256 FP32 from 3.7 to 4.8
// TB/s (290 -> 222 us) and the 216 x 144 x 96 x 4 FP64 columns from 50 and 49
// to 30 and 40 us.  Smaller arrays stay in the caches and want the larger
// number of tiles (96^3 FP64: 22.7 against 25.5 us for the three passes).  Over
// a length of 192 only two of the wide tiles fit a CU's LDS, which costs more
// than the run gains unless the narrow segments are ragged (rows that are no
// multiple of 64 bytes) or the array is of 192 MiB and more (the last-level
// cache holds 256).  There and back, 128 against 256 bytes: aligned 256^3 FP32
// (128 MiB) 258 / 268 us, 256 x 256 x 128 FP64 (128) 257 / 265, 216^3 FP64 (154)
// 333 / 340, but 192^3 x 2 FP32 (108) 216 / 212, 256 x 256 x 192 FP64 (192) 412 /
// 409 and 256^3 x 2 FP32 (256) 562 / 551; ragged 243^3 FP32 (109) 337 / 299.
constexpr int kWideMaxLength = 256;
inline bool wide_columns(int N, size_t elems, size_t csize, size_t row_bytes) {
  const size_t bytes = elems * csize;
  if (N > kWideMaxLength || static_radices(N).n == 0 || !cols_fit32(elems) || bytes < ((size_t)64 << 20)) return false;
  return N <= 192 || row_bytes % 64 != 0 || bytes >= ((size_t)192 << 20);
}

// Real rows of even length whose half has compile-time kernels.
inline bool real_rows_half(int nx) { return nx % 2 == 0 && static_radices(nx / 2).n > 0; }

template <typename T, int N> using RowPlan =
    SPlan<N, row_width(N, 2 * (int)sizeof(T), 128 / (2 * (int)sizeof(T))),
          row_width(N, 2 * (int)sizeof(T), 128 / (2 * (int)sizeof(T))) + 1, false, PassLanes<T>::value>;
// Column tiles of 128 bytes per row of the array, or 256 (WIDE).
template <typename T, int N, bool WIDE> using ColPlan =
    SPlan<N, (WIDE ? 256 : 128) / (2 * (int)sizeof(T)), (WIDE ? 256 : 128) / (2 * (int)sizeof(T)), false,
          PassLanes<T>::value>;

// Call f with the compile-time plan equal to host plan h, or with DynPlan;
// false where neither can run it.  Plan creation gives a length the radices of
// static_radices exactly where the compile-time kernels run it: every row, and
// columns whose array is addressable with 32-bit element offsets.
template <class SP, class Plan, class F> bool try_raw(const Plan& h, F&& f) {
  if (!plan_matches<SP>(h)) return false;
  f(SP{});
  return true;
}
template <typename T, class Plan, class F> bool with_row_plan(const Plan& h, F&& f) {
  bool done = false;
  switch (h.N) {
#define DKS_TRY(N) case N: done = try_raw<RowPlan<T, N>>(h, f); break;
    DKS_STATIC_LENGTHS(DKS_TRY)
#undef DKS_TRY
    default: break;
  }
  if (done) return true;
  if (!runtime_plan(h)) return false;
  f(DynPlan{});
  return true;
}

template <typename T, class Plan, class F> bool with_col_plan(const Plan& h, F&& f, bool off32) {
  bool done = false;
  if (off32) switch (h.N) {
#define DKS_TRY(N)                                                                           \
  case N:                                                                                    \
    if constexpr (N <= kWideMaxLength) done = try_raw<ColPlan<T, N, true>>(h, f);            \
    if (!done) done = try_raw<ColPlan<T, N, false>>(h, f);                                   \
    break;
    DKS_STATIC_LENGTHS(DKS_TRY)
#undef DKS_TRY
    default: break;
  }
  if (done) return true;
  if (!runtime_plan(h)) return false;
  f(DynPlan{});
  return true;
}

}  // namespace dks

#endif  // DKS_FFT_LENGTHS_H

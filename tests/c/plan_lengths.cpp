// Host-only harness of csrc/fft_lengths.h: plans built by the rules that plan
// creation uses (compile-time radices, 128- and 256-byte tiles, half-length
// real rows), for every length the library accepts, held against the choice
// the launchers make.  For each dtype and role it prints how many plans run on
// a compile-time plan, on the runtime plan, are refused, or break an invariant
// of the pass kernels, and then what happens to planted mistakes.
//
//   g++ -std=c++17 -I paper_1509_07685_amd/csrc tests/c/plan_lengths.cpp -o plan_lengths
#include <cstdio>
#include <cstring>
#include <vector>

#include "fft_lengths.h"
#include "fft_plan_check.h"

using namespace dks;

struct Plan {
  int N, npass, W, logW, LD;
  int R[kMaxPass], Ns[kMaxPass], tw_off[kMaxPass];
};

static bool is23(int n) {
  if (n < 1) return false;
  while (n % 2 == 0) n /= 2;
  while (n % 3 == 0) n /= 3;
  return n == 1;
}

static std::vector<int> radices(int N, bool fixed) {
  const RadixList l = static_radices(N);
  if (fixed && l.n > 0) return std::vector<int>(l.r, l.r + l.n);
  int a = 0, b = 0;
  while (N % 2 == 0) { N /= 2; ++a; }
  while (N % 3 == 0) { N /= 3; ++b; }
  std::vector<int> r;
  while (a >= 3) { r.push_back(8); a -= 3; }
  if (a == 2) r.push_back(4);
  if (a == 1) r.push_back(2);
  for (int i = 0; i < b; ++i) r.push_back(3);
  return r;
}

static Plan make(int N, const std::vector<int>& r, int W, int LD) {
  Plan P;
  std::memset(&P, 0, sizeof(P));
  P.N = N;
  P.npass = (int)r.size();
  P.W = W;
  while ((1 << P.logW) < W) ++P.logW;
  P.LD = LD;
  int Ns = 1, off = 0;
  for (size_t p = 0; p < r.size(); ++p) {
    P.R[p] = r[p];
    P.Ns[p] = Ns;
    P.tw_off[p] = off;
    if (p > 0) off += Ns * (r[p] - 1);
    Ns *= r[p];
  }
  return P;
}

// Tile width of the convolution's plans (plan creation's rule).
static int width(int N, int c, bool padded) {
  int W = 128 / c;
  while (W > 1 && (long long)N * (padded ? W + 1 : W) * c > kLdsBytes) W >>= 1;
  return W;
}

struct Count {
  int fixed = 0, runtime = 0, refused = 0, broken = 0;
};

template <class Pick> static bool see(Count& n, Pick&& pick) {
  bool fixed = false;
  const bool ok = pick([&](auto sp) { fixed = decltype(sp)::is_static; });
  ++(!ok ? n.refused : fixed ? n.fixed : n.runtime);
  return fixed;
}

template <typename T> static void run(const char* name) {
  const int c = 2 * (int)sizeof(T), wmax = 128 / c;
  EngineLimits L;
  L.threads = PassLanes<T>::value;
  L.emax = kLdsBytes / c / L.threads;
  L.max_length = kMaxLength;
  L.max_pass = kMaxPass;
  L.lds_hw = kLdsHardware;
  Count x, pencil, far_pencil, rows, half, cols, far_cols;
  for (int n = 1; n <= kMaxLength; ++n) {
    if (!is23(n)) continue;
    if (n >= 2 && n <= kMaxLength / 2) {           // mesh extents: x rows of n, pencils of 2 n
      const int W = width(n, c, true);
      const Plan px = make(n, radices(n, static_row(n)), W, W + 1);
      const bool f = see(x, [&](auto g) { return with_plan<T, 1, true>(px, g); });
      x.broken += fft_plan_violation(px, L, c, n, 16, (size_t)(n + 1) * c, f) != kPlanOk;
      const int N = 2 * n, Wp = width(N, c, false);
      for (int fit = 0; fit < 2; ++fit) {
        Count& k = fit ? pencil : far_pencil;
        std::vector<int> r = radices(N, fit && static_pencil(N));
        const Plan pp = make(N, r, Wp, Wp);
        const bool fp = see(k, [&](auto g) { return with_plan<T, 0, false>(pp, g, fit != 0); });
        const Plan pi = make(N, std::vector<int>(r.rbegin(), r.rend()), Wp, Wp);
        bool same = !fp;                            // the inverse z plan, reversed
        if (fp)
          with_plan<T, 0, false>(pp, [&](auto sp) {
            if constexpr (decltype(sp)::is_static) same = plan_matches<typename decltype(sp)::Reversed>(pi);
          });
        else
          same = runtime_plan(pi);
        k.broken += fft_plan_violation(pp, L, c, 0, 0, 0, fp) != kPlanOk ||
                    fft_plan_violation(pi, L, c, 0, 0, 0, fp) != kPlanOk || !same;
      }
    }
    // raw rows, whole and (for real rows of 2 n) half-length
    const int Wr = row_width(n, c, wmax);
    const bool padded = (size_t)n * (Wr + 1) * c <= (size_t)kLdsBytes;
    const Plan pr = make(n, radices(n, true), Wr, padded ? Wr + 1 : Wr);
    const bool fr = see(rows, [&](auto g) { return with_row_plan<T>(pr, g); });
    rows.broken += fft_plan_violation(pr, L, c, n, L.emax, 0, fr) != kPlanOk;
    if (2 * n <= kMaxLength && real_rows_half(2 * n)) {
      const bool fh = see(half, [&](auto g) { return with_row_plan<T>(pr, g); });
      half.broken += !fh || fft_plan_violation(pr, L, c, n, L.emax, (size_t)(n + 1) * c, fh) != kPlanOk;
    }
    // raw columns of small, large and not 32-bit addressable arrays
    for (size_t elems : {(size_t)n * 64, (size_t)1 << 27, (size_t)1 << 31}) {
      const bool fit = cols_fit32(elems);
      int W = wide_columns(n, elems, c, 64) ? 2 * wmax : wmax;
      while (W > 1 && (size_t)n * W * c > (size_t)kLdsBytes) W >>= 1;
      const Plan pc = make(n, radices(n, fit), W, W);
      Count& k = fit ? cols : far_cols;
      const bool fc = see(k, [&](auto g) { return with_col_plan<T>(pc, g, fit); });
      k.broken += fft_plan_violation(pc, L, c, 0, 0, 0, fc) != kPlanOk;
    }
  }
  const auto line = [&](const char* role, const Count& k) {
    std::printf("%s %s %d %d %d %d\n", name, role, k.fixed, k.runtime, k.refused, k.broken);
  };
  line("x", x);
  line("pencil", pencil);
  line("far_pencil", far_pencil);
  line("rows", rows);
  line("half", half);
  line("cols", cols);
  line("far_cols", far_cols);
  // a radix order that only a compile-time plan knows, on a tile that none has
  const Plan odd = make(216, {6, 6, 6}, wmax / 2, wmax / 2);
  bool called = false;
  const auto mark = [&](auto) { called = true; };
  const bool a = with_plan<T, 0, false>(odd, mark), b = with_col_plan<T>(odd, mark, true);
  const Plan fixed = make(216, {6, 6, 6}, wmax, wmax);
  const bool d = with_plan<T, 0, false>(fixed, mark, false), e = with_col_plan<T>(fixed, mark, false);
  const Plan row = make(216, {6, 6, 6}, wmax / 2, wmax / 2 + 1);
  const bool f = with_row_plan<T>(row, mark), g = with_plan<T, 1, true>(row, mark);
  std::printf("%s planted %d %d %d %d\n", name, a || b || d || e || f || g, called,
              fft_plan_violation(odd, L, c, 0, 0, 0), fft_plan_violation(fixed, L, c, 0, 0, 0, true));
}

int main() {
  run<float>("f32");
  run<double>("f64");
  return 0;
}

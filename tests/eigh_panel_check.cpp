// Host-only check of the two parts of the block eigensolver whose workgroups wait for
// one another (no GPU), built from the geometry header the kernels use.
//
// panel n j0 seed ring: k_panel of the panel at column j0 of an FP64 block of n rows.
//   The workgroups run as state machines that a random scheduler steps: what each
//   polls, publishes and restores per column, word by word, in the exchange region.
//   Words are tagged with the column they belong to.  Asserted: every index lies in
//   its part of its ring slot; a word is published only where the last one has been
//   restored; a poll never sees the word of another column; nobody waits for ever.
//   Restores are stores in flight: they land at any time up to the point where the
//   kernel waits for its stores.  ring is the number of slots (the kernel's: 4); with
//   fewer the check must fail.  seed 0 is the form in which one workgroup runs every
//   part in turn.
// layout n K: the exchange region is the last of the workspace, without it the layout
//   is the one of launches per column, and every panel fits what the kernel assumes.
// chase n: the sweeps of k_sb_chase.  Every band word a task touches lies in the band;
//   once task (i, k) may start, no task of an earlier sweep that may still be running or
//   to come touches a word of it; counters and kept reflectors lie in their regions.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <random>
#include <utility>
#include <vector>

#include "eigh_geometry.h"

using namespace bse;

namespace {

[[noreturn]] void stop(const char *what, int64_t a = 0, int64_t b = 0) {
  std::printf("FAILED: %s (%lld, %lld)\n", what, (long long)a, (long long)b);
  std::exit(1);
}

// ---------------------------------------------------------------------------
// k_panel
// ---------------------------------------------------------------------------
struct Panel {
  int n, j0, m, RW, G, ring;
  PanParts<int64_t> o;
  std::vector<int> tag;  // per word: 0 none, else column + 1

  Panel(int n_, int j0_, int ring_) : n(n_), j0(j0_), ring(ring_), o(g_pan_parts<int64_t>(0, n_)) {
    m = n - j0 - 1;
    RW = g_pan_rows(m);
    G = g_pan_wgs(m);
    tag.assign(size_t(g_pan_words(n)), 0);
  }
  // word k of part [lo, hi) of the slot of column i
  size_t word(int i, int64_t lo, int64_t hi, int64_t k) const {
    if (k < 0 || lo + k >= hi) stop("word outside its part", lo + k, hi);
    const int64_t w = 2 * g_pan_ctrl(n) + (i % ring) * g_pan_ring(n) + lo + k;
    if (w < 2 * g_pan_ctrl(n) || w >= g_pan_words(n)) stop("word outside the region", w);
    return size_t(w);
  }
  size_t col(int i, int r, int c) const { return word(i, o.col, o.rec, 2 * int64_t(r) + c); }
  size_t rec(int i, int g, int s, int c) const {
    return word(i, o.rec, o.pa, 2 * (int64_t(g) * 2 * NBK + s) + c);
  }
  size_t pa(int i, int g, int c) const { return word(i, o.pa, o.bred, 2 * g + c); }
  size_t bred(int i, int s, int c) const { return word(i, o.bred, o.head, 2 * s + c); }
  size_t head(int i, int t, int c) const { return word(i, o.head, o.yj, 2 * t + c); }
  size_t yj(int i, int c) const { return word(i, o.yj, o.end, c); }

  bool there(size_t w, int i) const {  // a poll for column i
    if (tag[w] == 0) return false;
    if (tag[w] != i + 1) stop("stale word read: column, found", i, tag[w] - 1);
    return true;
  }
  void put(size_t w, int i) {
    if (tag[w] != 0) stop("published over a word: column, found", i, tag[w] - 1);
    tag[w] = i + 1;
  }
};

struct Group {  // one workgroup
  Panel &P;
  int g, rb, nr, i = 0, phase = 0;
  bool done = false;
  std::deque<size_t> flight;  // restores not landed yet
  Group(Panel &p, int g_) : P(p), g(g_) {
    rb = P.j0 + 1 + g * P.RW;
    nr = std::min(P.RW, P.n - rb);
    if (nr < 1) stop("workgroup without rows", g);
  }
  void land() {
    P.tag[flight.front()] = 0;
    flight.pop_front();
  }
  bool owns(int r) const { return r >= rb && r < rb + nr; }

  bool step() {  // one step; false: it has to wait
    const int jn = P.j0 + i, m0 = jn + 1;
    switch (phase) {
      case 0:  // the column and the head rows
        if (i > 0) {
          for (int r = jn; r < P.n; ++r)
            if (!P.there(P.col(i, r, 0), i) || !P.there(P.col(i, r, 1), i)) return false;
          for (int t = 0; t < 2 * NBK; ++t)
            if ((t & (NBK - 1)) < i)
              for (int c = 0; c < 2; ++c)
                if (!P.there(P.head(i, t, c), i)) return false;
        }
        break;
      case 1:  // the dot products of this workgroup, four lanes of 64 records each at most
        if (P.G > 4 * 64 || P.G > ENT) stop("more workgroups than a poll covers", P.G);
        for (int s = g; s < 2 * i; s += P.G)
          for (int h = 0; h < P.G; ++h)
            if (!P.there(P.rec(i, h, s, 0), i) || !P.there(P.rec(i, h, s, 1), i)) return false;
        for (int s = g; s < 2 * i; s += P.G)
          for (int c = 0; c < 2; ++c) P.put(P.bred(i, s, c), i);
        break;
      case 2:
        for (int c = 0; c < 2; ++c) P.put(P.pa(i, g, c), i);
        if (owns(m0))
          for (int c = 0; c < 2; ++c) P.put(P.yj(i, c), i);
        break;
      case 3:  // every sum, every dot product, y[m0]; then the stores in flight
        for (int c = 0; c < 2; ++c) {
          for (int h = 0; h < P.G; ++h)
            if (!P.there(P.pa(i, h, c), i)) return false;
          for (int s = 0; s < 2 * i; ++s)
            if (!P.there(P.bred(i, s, c), i)) return false;
          if (!P.there(P.yj(i, c), i)) return false;
        }
        while (!flight.empty()) land();
        break;
      case 4:  // the next column
        if (i + 1 < NBK) {
          for (int r = std::max(rb, m0); r < rb + nr; ++r)
            for (int c = 0; c < 2; ++c) P.put(P.col(i + 1, r, c), i + 1);
          for (int s = 0; s < 2 * (i + 1); ++s)
            for (int c = 0; c < 2; ++c) P.put(P.rec(i + 1, g, s, c), i + 1);
          if (owns(m0 + 1))
            for (int t = 0; t < 2 * NBK; ++t)
              if ((t & (NBK - 1)) <= i)
                for (int c = 0; c < 2; ++c) P.put(P.head(i + 1, t, c), i + 1);
        }
        break;
      case 5:  // column i - 1 back to none
        if (i > 0) {
          for (int t = 0; t < 2 * nr; ++t) flight.push_back(P.word(i - 1, P.o.col, P.o.rec, 2 * rb + t));
          for (int t = 0; t < 4 * NBK; ++t)
            flight.push_back(P.word(i - 1, P.o.rec, P.o.pa, int64_t(g) * 4 * NBK + t));
          for (int t = 0; t < 2; ++t) {
            flight.push_back(P.pa(i - 1, g, t));
            for (int s = g; s < 2 * NBK; s += P.G) flight.push_back(P.bred(i - 1, s, t));
          }
          if (owns(jn)) {
            for (int t = 0; t < 4 * NBK; ++t) flight.push_back(P.word(i - 1, P.o.head, P.o.yj, t));
            for (int t = 0; t < 2; ++t) flight.push_back(P.yj(i - 1, t));
          }
        }
        break;
    }
    if (++phase == 6) {
      phase = 0;
      if (++i == NBK) done = true;
    }
    return true;
  }
};

int panel(int n, int j0, unsigned seed, int ring) {
  if (!g_pan(n, j0, true) || ring < 1 || ring > PAN_RING) stop("not a panel", n, j0);
  Panel P(n, j0, ring);
  std::vector<Group> W;
  for (int g = 0; g < P.G; ++g) W.emplace_back(P, g);
  if (W.back().rb + W.back().nr != n) stop("rows not covered", n);
  if (seed == 0) {  // given up: part A of every workgroup, then part B of every workgroup
    for (int i = 0; i < NBK; ++i)
      for (int half = 0; half < 2; ++half)
        for (Group &w : W) {
          for (int k = 0; k < 3; ++k)
            if (!w.step()) stop("the lone workgroup waits for itself: column, part", i, 3 * half + k);
          while (!w.flight.empty()) w.land();
        }
    return 0;
  }
  std::mt19937 rng(seed);
  // some workgroups are slow, and some hold back their stores
  std::vector<int> pace(size_t(P.G)), hold(size_t(P.G));
  for (int g = 0; g < P.G; ++g) {
    pace[size_t(g)] = rng() % 4 == 0 ? 8 : 1;
    hold[size_t(g)] = int(rng() % 3);
  }
  int64_t left = P.G;
  for (int64_t idle = 0; left > 0;) {
    bool moved = false;
    for (int k = 0; k < P.G && left > 0; ++k) {
      const size_t g = rng() % size_t(P.G);
      Group &w = W[g];
      if (hold[g] == 0 || (hold[g] == 1 && rng() % 8 == 0))
        while (!w.flight.empty()) w.land();
      if (w.done || rng() % unsigned(pace[g])) continue;
      if (!w.step()) continue;
      moved = true;
      if (w.done) --left;
    }
    idle = moved ? 0 : idle + 1;
    if (idle > 2000) stop("the workgroups wait for ever", left);
  }
  return 0;
}

int layout(int64_t n, int64_t K) {
  std::vector<char> buf(ws_layout(n, true, nullptr, nullptr, K));
  Desc D{};
  ws_layout(n, true, &D, buf.data(), K);
  const size_t words = size_t(g_pan_bytes(n, true));
  if (g_tail0(n) == 0) return D.px || words ? (stop("words without a panel", n), 1) : 0;
  if (reinterpret_cast<char *>(D.px) + words != buf.data() + buf.size()) stop("px is not last", n);
  if (g_pan_parts<int64_t>(0, n).end != g_pan_ring(n)) stop("parts of a ring slot", n);
  if (words < size_t(g_pan_words(n)) * 8 || (reinterpret_cast<char *>(D.px) - buf.data()) % 8)
    stop("px too small or not aligned", n);
  for (int64_t j0 = 0; j0 < g_tail0(n); j0 += NBK) {
    if (2 * (j0 / NBK) + 1 >= 2 * g_pan_ctrl(n)) stop("entry counter", j0);
    if (!g_pan(n, j0, true)) continue;
    const int64_t m = n - j0 - 1;
    if (j0 + NBK >= n) stop("panel without rows below it", n, j0);
    if (g_pan_wgs(m) > g_pan_gmax(n) || g_pan_wgs(m) > PAN_WGS) stop("workgroups", n, j0);
    if (m + 1 > PAN_M + 1) stop("rows of the column in LDS", n, j0);
    if ((m + 1) * D.lda > INT32_MAX || (NBK + 1) * D.ldv > INT32_MAX) stop("32-bit index", n, j0);
    if (kind_wgs<double>(K_PANEL, n, j0, 4) != g_pan_wgs(m)) stop("kind_wgs", n, j0);
  }
  for (int64_t s : {0, 3, 4, 96, 512, 768, 4096})
    if (g_pan_limit(s) > PAN_WGS || 4 * g_pan_limit(s) > s || g_pan_batch(s) + g_pan_limit(s) > s)
      stop("panel limits", s);
  return 0;
}

// ---------------------------------------------------------------------------
// k_sb_chase
// ---------------------------------------------------------------------------
typedef std::vector<std::pair<int, int>> Words;  // (column, row)

Words task(int n, int i, int k) {
  const int rk = i + 1 + k * SBW, rp = k > 0 ? rk - SBW : i, L = std::min(SBW, n - rk);
  Words w;
  if (L < 1) stop("task without rows", i, k);
  for (int p = 0; p < SBW; ++p)
    for (int q = 0; q < SBW; ++q) {
      // the loads of every lane (those of masked lanes are dropped)
      const int64_t a = k > 0 ? int64_t(rp + q) * LDB + SBW + p - q : int64_t(i) * LDB + 1 + p;
      const int64_t b = int64_t(std::min(rk + q, n - 1)) * LDB + (p >= q ? p - q : 0);
      if (a < 0 || a >= int64_t(n) * LDB || b < 0 || b >= int64_t(n) * LDB) stop("band", i, k);
      if (p < L && (k > 0 || q == 0)) {
        if (k > 0 && (SBW + p - q < 1 || SBW + p - q >= LDB)) stop("outside the column", i, k);
        w.emplace_back(k > 0 ? rp + q : i, rk + p);
      }
      if (q <= p && p < L) w.emplace_back(rk + q, rk + p);
    }
  std::sort(w.begin(), w.end());
  return w;
}

bool meet(const Words &a, const Words &b) {
  size_t x = 0, y = 0;
  while (x < a.size() && y < b.size()) {
    if (a[x] == b[y]) return true;
    if (a[x] < b[y]) ++x;
    else ++y;
  }
  return false;
}

int chase(int n) {
  constexpr int BACK = 4;  // earlier sweeps looked at
  auto kmax = [&](int i) { return (int)g_bc_kmax(n, i); };
  auto want = [&](int i, int k) {  // tasks of sweep i - 1 that (i, k) waits for
    return i > 0 ? std::min(k + 2, kmax(i - 1) + 1) : 0;
  };
  std::vector<std::vector<Words>> T;  // of the last sweeps
  for (int i = 0; i + 1 < n; ++i) {
    std::vector<Words> now;
    for (int k = 0; k <= kmax(i); ++k) now.push_back(task(n, i, k));
    if (n - 1 - i > (kmax(i) + 1) * SBW || n - 1 - i <= kmax(i) * SBW) stop("rows of a sweep", i);
    for (int k = 0; k <= kmax(i); ++k) {
      // sweep i - d has finished this many tasks, at least
      int fin = want(i, k);
      for (int d = 1; d <= BACK && i - d >= 0; ++d) {
        for (int q = fin; q <= kmax(i - d); ++q)
          if (meet(now[size_t(k)], T[T.size() - size_t(d)][size_t(q)])) stop("tasks meet", i, k);
        if (fin > 0 && i - d > 0) fin = want(i - d, fin - 1);
        else if (i - d > 0) fin = 0;
      }
      if (g_bc_off(n, i) + k * SBW + std::min(SBW, n - (i + 1 + k * SBW)) > g_bc_off(n, i + 1))
        stop("kept reflector outside its sweep", i, k);
    }
    T.push_back(std::move(now));
    if (T.size() > BACK) T.erase(T.begin());
  }
  std::vector<char> buf(ws_layout(n, true, nullptr, nullptr, 0, true));
  Desc D{};
  ws_layout(n, true, &D, buf.data(), 0, true);
  const char *last = reinterpret_cast<char *>(D.rfl + int64_t(n - 1) * SBW) + sizeof(int);
  if (last > reinterpret_cast<char *>(D.rtau)) stop("sweep counter", n);
  return 0;
}

}  // namespace

int main(int argc, char **argv) {
  auto num = [&](int a) { return a < argc ? std::atoll(argv[a]) : 0; };
  int done = 0;
  for (int a = 1; a < argc; ++done) {
    if (!std::strcmp(argv[a], "panel") && a + 4 < argc) {
      panel((int)num(a + 1), (int)num(a + 2), (unsigned)num(a + 3), (int)num(a + 4));
      a += 5;
    } else if (!std::strcmp(argv[a], "layout") && a + 2 < argc) {
      layout(num(a + 1), num(a + 2));
      a += 3;
    } else if (!std::strcmp(argv[a], "chase") && a + 1 < argc) {
      chase((int)num(a + 1));
      a += 2;
    } else {
      std::fprintf(stderr, "usage: %s panel n j0 seed ring | layout n K | chase n ...\n", argv[0]);
      return 2;
    }
  }
  std::printf("%d checks passed\n", done);
  return 0;
}

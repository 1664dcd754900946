// Evaluates the index maps of the binary64 tile kernel on the host, for every
// shape and operand layout: prints one line per finding, "ok <count>" at the end.
#include <cstdio>
#include <utility>
#include <vector>

#include "bgemm_tiles.h"

using namespace bg;

static int bad = 0, shapes = 0;
#define CHECK(cond, ...)                \
  do {                                  \
    if (!(cond) && ++bad <= 40) {       \
      std::printf(__VA_ARGS__);         \
      std::printf("\n");                \
    }                                   \
  } while (0)

// An operand tile: the value (mn, k) that each of the two places of a unit holds.
template <class T, int EXT, bool KC>
static std::vector<std::pair<int, int>> staged(const char* what, int chunks, int nw, int per_wave) {
  std::vector<std::pair<int, int>> held(2 * 64 * chunks, {-1, -1});
  for (int i = 0; i < per_wave; ++i)
    for (int wave = 0; wave < nw; ++wave)
      for (int lane = 0; lane < 64; ++lane) {
        const int p = (i * nw + wave) % chunks * 64 + lane;
        int mn = 0, k = 0;
        T::at(p, mn, k);
        held[2 * p] = {mn, k};
        held[2 * p + 1] = KC ? std::make_pair(mn, k + 1) : std::make_pair(mn + 1, k);
      }
  std::vector<int> seen(EXT * 16, 0);
  for (auto& e : held) {
    CHECK(e.first >= 0 && e.first < EXT && e.second >= 0 && e.second < 16,
          "%s: a unit holds (%d, %d)", what, e.first, e.second);
    if (e.first >= 0 && e.first < EXT && e.second >= 0 && e.second < 16)
      ++seen[e.first * 16 + e.second];
  }
  for (int x : seen) CHECK(x == 1, "%s: a value is staged %d times", what, x);
  return held;
}

template <class CF, bool TA, bool TB>
static void layout(const char* name) {
  constexpr bool AK = TA, BKC = !TB;
  using At = PTile<CF::BM, CF::BK, AK, true>;
  using Bt = PTile<CF::BN, CF::BK, BKC, false>;
  const auto a = staged<At, CF::BM, AK>(name, CF::CA, CF::NW, CF::PA);
  const auto b = staged<Bt, CF::BN, BKC>(name, CF::CB, CF::NW, CF::PB);
  // Units one pointer serves in turn differ by a fixed k at the same mn.
  auto steps = [&](auto tile, int chunks, int per_wave) {
    using T = decltype(tile);
    if (CF::NW * 64 % T::UR || chunks % CF::NW) return;
    for (int p = 0; p < CF::NW * 64; ++p)
      for (int i = 1; i < per_wave; ++i) {
        int m0, k0, m1, k1;
        T::at(p, m0, k0);
        T::at(p + i * CF::NW * 64, m1, k1);
        CHECK(m0 == m1 && k1 == k0 + i * (CF::NW * 64 / T::UR), "%s: units of one pointer", name);
      }
  };
  if (!AK) steps(At{}, CF::CA, CF::PA);
  if (!BKC) steps(Bt{}, CF::CB, CF::PB);

  std::vector<int> read(CF::BM * CF::BN, 0), wide(CF::BM * CF::BN, 0), edge(CF::BM * CF::BN, 0);
  std::vector<int> product(CF::BM * CF::BN, 0);
  auto touch = [&](std::vector<int>& c, int row, int col, const char* what) {
    CHECK(row >= 0 && row < CF::BM && col >= 0 && col < CF::BN, "%s: %s reaches (%d, %d)", name,
          what, row, col);
    if (row >= 0 && row < CF::BM && col >= 0 && col < CF::BN) ++c[row * CF::BN + col];
  };
  for (int wave = 0; wave < CF::NW; ++wave) {
    const int wm0 = CF::wave_row(wave), wn0 = CF::wave_col(wave);
    // the fragments of every lane: (row, k) and (column, k) per slab and group
    for (int tp = 0; tp < 2; ++tp)
      for (int u = 0; u < 2; ++u) {
        std::vector<std::pair<int, int>> P(64 * CF::FP), Q(64 * CF::GQ);
        for (int lane = 0; lane < 64; ++lane) {
          for (int s = 0; s < CF::FP / 2; ++s)
            for (int r = 0; r < 2; ++r) {   // read r of the pair
              const int v = AK ? 2 * tp + r : 0;
              const int unit = At::p_base(wm0, lane, v) + At::p_offset(tp, r, s);
              // KC: slab 2s + r at k of u; else slabs 2s, 2s + 1 at k of r
              if (AK) P[64 * (2 * s + r) + lane] = a[2 * unit + u];
              else if (r == u)
                for (int x = 0; x < 2; ++x) P[64 * (2 * s + x) + lane] = a[2 * unit + x];
            }
          for (int h = 0; h < CF::GQ; h += 2)
            for (int r = 0; r < 2; ++r) {
              const int unit = Bt::q_base(wn0, lane, BKC ? 0 : (h / 2) & 1) + Bt::q_offset(tp, r, h);
              if (BKC) Q[64 * (h + r) + lane] = b[2 * unit + u];
              else if (r == u)
                for (int x = 0; x < 2; ++x) Q[64 * (h + x) + lane] = b[2 * unit + x];
            }
        }
        // lane 16 s + 4 b + i: P(i of block b, k_s) and Q(i, k_s); the result's
        // lane 16 i + 4 b + j sums P of lanes 16 s + 4 b + i, Q of lanes 16 s + 4 b + j
        for (int lane = 0; lane < 64; ++lane) {
          const int i = lane >> 4, blk = (lane >> 2) & 3, j = lane & 3;
          for (int s = 0; s < 4; ++s)
            for (int f = 0; f < CF::FP; ++f)
              for (int g = 0; g < CF::GQ; ++g) {
                const auto p = P[64 * f + 16 * s + 4 * blk + i], q = Q[64 * g + 16 * s + 4 * blk + j];
                CHECK(p.second == q.second && p.second == 2 * s + 8 * tp + u, "%s: k of a product",
                      name);
                CHECK(p.first == CF::lane_row(wm0, lane) + 32 * (f / 2) + (f & 1) &&
                          q.first == CF::lane_col(BKC, wn0, lane, g),
                      "%s: lane %d sums C(%d, %d) and stores it elsewhere", name, lane, p.first,
                      q.first);
                touch(product, p.first, q.first, "a product");
              }
        }
      }
    // what the epilogue reads and writes, group by group as it steps
    for (int lane = 0; lane < 64; ++lane)
      for (int s = 0; s < CF::FP / 2; ++s)
        for (int x = 0; x < 2; ++x) {
          const int row = CF::lane_row(wm0, lane) + 32 * s + x;
          for (int g0 = 0; g0 < CF::GQ; g0 += CF::GE)
            for (int g = 0; g < CF::GE; ++g) {
              touch(wide, row, CF::lane_col(BKC, wn0, lane, g0 + g), "an interior tile");
              CHECK(g0 + g < CF::GQ, "%s: column group %d of %d", name, g0 + g, CF::GQ);
            }
          for (int g0 = 0; g0 < CF::GQ; g0 += CF::GB)
            for (int g = 0; g < CF::GB; ++g) {
              touch(edge, row, CF::lane_col(BKC, wn0, lane, g0 + g), "an edge tile");
              CHECK(g0 + g < CF::GQ, "%s: column group %d of %d", name, g0 + g, CF::GQ);
            }
        }
  }
  for (int e = 0; e < CF::BM * CF::BN; ++e) {
    CHECK(product[e] == 16, "%s: C(%d, %d) sums %d of 16 k", name, e / CF::BN, e % CF::BN, product[e]);
    CHECK(wide[e] == 1 && edge[e] == 1, "%s: C(%d, %d) is written %d and %d times", name,
          e / CF::BN, e % CF::BN, wide[e], edge[e]);
  }
}

template <class CF>
static void shape() {
  char name[64];
  std::snprintf(name, sizeof name, "%dx%d in %dx%d", CF::BM, CF::BN, CF::WM, CF::WN);
  layout<CF, false, false>(name);
  layout<CF, false, true>(name);
  layout<CF, true, false>(name);
  layout<CF, true, true>(name);
  ++shapes;
}

int main() {
  shape<P128>();
  shape<P128x64>();
  shape<P128x48>();
  shape<P64>();
  shape<P64x32>();
  shape<P32x64>();
  shape<P32>();
  shape<P32x16>();
#define SHAPE(...) shape<PCfg<__VA_ARGS__>>();
  TUNED_SHAPES
  std::printf(bad ? "%d findings\n" : "ok %d\n", bad ? bad : shapes);
  return bad != 0;
}

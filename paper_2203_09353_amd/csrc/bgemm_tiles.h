// Tile shapes of the binary64 tile kernel and its index maps: which unit of an
// operand each thread stages, which unit each lane's fragment read takes, and
// which elements of C each lane holds.  Plain constexpr C++, so that the host
// test of these maps evaluates the very functions the kernels use.
#pragma once

namespace bg {

// Largest part, up to `most`, that `groups` column groups split into evenly: the
// epilogue takes them a part at a time, and a part that did not divide them
// would reach past the tile.
constexpr int even_part(int groups, int most) {
  int c = most;
  while (groups % c) --c;
  return c;
}

// C tile BM x BN per workgroup in waves of WM x WN.
template <int BM_, int BN_, int WM_, int WN_>
struct PCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = 2, BK = 16;
  static constexpr int WAVES_M = BM / WM, NW = WAVES_M * (BN / WN), NT = 64 * NW;
  static constexpr int FP = WM / 16, GQ = WN / 4;    // slabs, column groups per wave
  static constexpr int GE = even_part(GQ, 8);        // groups of C in flight, interior tiles
  static constexpr int GB = even_part(GQ, 4);        // ... edge tiles
  static constexpr int CA = BM * BK / 128, CB = BN * BK / 128;   // 1 KB chunks per stage
  static constexpr int PA = (CA + NW - 1) / NW, PB = (CB + NW - 1) / NW;   // per wave
  static constexpr int STAGE = (BM + BN) * BK / 2;   // units
  static constexpr int LDS = NS * STAGE * 2;         // doubles
  // workgroups that fit a CU's LDS, and the waves per SIMD they make
  static constexpr int WGS = 163840 / (LDS * 8 + 64);
  static constexpr int WAVES = WGS * NW / 4 > 8 ? 8 : (WGS * NW / 4 < 1 ? 1 : WGS * NW / 4);
  static_assert(BM % WM == 0 && BN % WN == 0, "tile");
  static_assert(WM == 32 || WM == 64, "one or two slab pairs");
  static_assert(WN % 16 == 0, "a wave starts at a whole turn of the Q swizzle");
  static_assert(GQ % GE == 0 && GQ % GB == 0, "the epilogue ends where the wave's columns do");

  // First of the wave's rows and columns in the tile.
  static constexpr int wave_row(int wave) { return wave % WAVES_M * WM; }
  static constexpr int wave_col(int wave) { return wave / WAVES_M * WN; }
  // The lane's part of C: rows lane_row + 32 a and the next (slabs 2a, 2a + 1), one
  // column per group.
  static constexpr int lane_row(int wm0, int lane) {
    return wm0 + 2 * (4 * ((lane >> 2) & 3) + (lane >> 4));
  }
  static constexpr int lane_col(bool b_kc, int wn0, int lane, int g) {
    return wn0 + (b_kc ? 4 * g + (lane & 3) : 8 * (g / 2) + 2 * (lane & 3) + (g & 1));
  }
};

// An operand tile in LDS: EXT values of its product dimension x BK of k, in units
// of two values along the operand's contiguous dimension.
template <int EXT, int BK, bool KC, bool ROLE_P>
struct PTile {
  static_assert(BK == 16, "rows of eight units");
  static constexpr int UR = KC ? BK / 2 : EXT / 2;   // units per row
  static constexpr int rho(int mn) { return (mn & ~3) | ((mn & 1) << 1) | ((mn >> 1) & 1); }
  static constexpr int f(int mn) { return (ROLE_P ? (mn >> 2) & 7 : 0) ^ (2 * (mn & 1)); }
  // first element of the unit at position p
  static constexpr void at(int p, int& mn, int& k) {
    if (KC) {
      mn = rho(p / UR);
      k = 2 * ((p % UR) ^ f(mn));
    } else {
      k = p / UR;
      mn = 2 * ((p % UR) ^ (ROLE_P ? 0 : 4 * ((k >> 1) & 1)));
    }
  }

  // Fragment reads.  Half slice tp of a step holds k = 2 ls + 8 tp and the next
  // for lane group ls, unit ls + 4 tp of a K-contiguous row.  A read's unit is a
  // lane address (BASES of them) and a constant offset.
  static constexpr int BASES = KC ? (ROLE_P ? 4 : 1) : (ROLE_P ? 1 : 2);
  // P, slab pair a of the wave at w0.  KC: one of rows 2 lr + u at both k (v = 2 tp
  // + u); else both rows at k + u.
  static constexpr int p_base(int w0, int lane, int v) {
    const int ls = lane >> 4, lr = lane & 15, row = 2 * lr + (v & 1);
    return KC ? (w0 + rho(row)) * 8 + ((ls + 4 * (v >> 1)) ^ f(row)) : 2 * ls * UR + w0 / 2 + lr;
  }
  static constexpr int p_offset(int tp, int u, int a) {
    return KC ? 32 * a * 8 : (8 * tp + u) * UR + 16 * a;
  }
  // Q, column groups h and h + 1 (h even) of the wave at w0.  KC: column 4 (h + u) +
  // lj at both k; else both groups' columns at k + u (v = h / 2 mod 2).
  static constexpr int q_base(int w0, int lane, int v) {
    const int ls = lane >> 4, lj = lane & 3;
    return KC ? (w0 + rho(lj)) * 8 + (ls ^ f(lj)) : 2 * ls * UR + w0 / 2 + lj + 4 * ((ls & 1) ^ v);
  }
  static constexpr int q_offset(int tp, int u, int h) {
    return KC ? 4 * (h + u) * 8 + 4 * tp : (8 * tp + u) * UR + 8 * (h / 4);
  }
};

// Shapes: BM, BN, WM, WN.
using P128 = PCfg<128, 128, 64, 64>;
using P128x64 = PCfg<128, 64, 64, 32>;
using P128x48 = PCfg<128, 48, 32, 48>;
using P64 = PCfg<64, 64, 32, 32>;
using P64x32 = PCfg<64, 32, 32, 16>;
using P32x64 = PCfg<32, 64, 32, 16>;
using P32 = PCfg<32, 32, 32, 16>;
using P32x16 = PCfg<32, 16, 32, 16>;

}  // namespace bg

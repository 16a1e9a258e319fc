// Operator fragments of the nodal matrix-core form, shared by the host setup
// and the stage kernel: the 16x4 tiles of Dr, Ds, Dt and LIFT in the order of
// use, without the tiles of the derivatives that are zero.
//
// D_a[i][j] (a = 1, 2, 3 for r, s, t) is zero unless b_m(j) <= b_m(i) for the
// three barycentrics m != a, or for the three m != 0 (by the product form of
// the lattice's Lagrange basis, whose factor in each barycentric vanishes at
// the smaller lattice values), and on the diagonal where b_a = b_0: 376 of
// 1225 entries at order 4 are left.  Rows may stand in any order in the tiles;
// the one taken gathers rows with the same zero tiles greedily, starting with
// the incomplete tile, and leaves 59 of 81 tiles at order 4, 251 of 378 at
// order 6.  Products keep their order, so a left-out tile changes no result.
#pragma once

#include <cstdint>

namespace dgw {

template <int N>
struct Nodal {
  static constexpr int Np = (N + 1) * (N + 2) * (N + 3) / 6;
  static constexpr int Nfp = (N + 1) * (N + 2) / 2, NF = 4 * Nfp;
  static constexpr int MT = (Np + 15) / 16;   // row tiles
  static constexpr int KS = (Np + 3) / 4;     // k-steps per reference direction
  static constexpr int KL = NF / 4;           // k-steps of the lift
  static_assert(3 * KS <= 64, "a mask of k-steps fits 64 bits");

  struct Tab {
    uint8_t row[16 * MT] = {};     // node of each tile row, 255 past the last
    uint64_t need[MT] = {};        // bit a KS + ks: the tile is not zero
  };
  static constexpr Tab make() {
    Tab T;
    int b[Np][4] = {};
    int n = 0;
    for (int k = 0; k <= N; ++k)
      for (int j = 0; j <= N - k; ++j)
        for (int i = 0; i <= N - j - k; ++i, ++n) {
          b[n][0] = N - i - j - k;
          b[n][1] = i;
          b[n][2] = j;
          b[n][3] = k;
        }
    uint64_t z[Np] = {};
    for (int i = 0; i < Np; ++i)
      for (int j = 0; j < Np; ++j) {
        bool le[4] = {};
        for (int m = 0; m < 4; ++m) le[m] = b[j][m] <= b[i][m];
        for (int a = 1; a < 4; ++a) {
          const int p = a == 1 ? 2 : 1, q = a == 3 ? 2 : 3;   // the other two of 1..3
          const bool nz = (le[p] && le[q] && (le[0] || le[a]));
          if (nz && !(i == j && b[i][a] == b[i][0]))
            z[i] |= uint64_t(1) << ((a - 1) * KS + j / 4);
        }
      }
    bool used[Np] = {};
    int left = Np;
    for (int tile = 0; tile < MT; ++tile) {
      const int at = (tile + MT - 1) % MT;   // the incomplete tile is the last
      const int size = tile == 0 ? Np - 16 * (MT - 1) : 16;
      uint64_t u = 0;
      for (int c = 0; c < 16; ++c) T.row[16 * at + c] = 255;
      for (int c = 0; c < size && left > 0; ++c, --left) {
        int best = -1, add = 0, own = 0;
        for (int i = 0; i < Np; ++i) {
          if (used[i]) continue;
          const int a = __builtin_popcountll(z[i] & ~u), o = __builtin_popcountll(z[i]);
          // the first row: the one with the fewest tiles; then the fewest new
          // tiles, the most tiles of its own
          if (best < 0 || a < add || (a == add && c > 0 && o > own)) {
            best = i;
            add = a;
            own = o;
          }
        }
        used[best] = true;
        u |= z[best];
        T.row[16 * at + c] = (uint8_t)best;
      }
      T.need[at] = u;
    }
    return T;
  }
  static constexpr Tab tab = make();
  static constexpr bool need(int s, int mt) { return s >= 3 * KS || (tab.need[mt] >> s & 1); }

  // steps a KS + ks of the volume, then the lift's; chunks of steps that the
  // kernel stages in LDS, starting at a multiple of four fragments
  static constexpr int nsteps = 3 * KS + KL;
  static constexpr int step_frags(int s) {
    int n = 0;
    for (int mt = 0; mt < MT; ++mt) n += need(s, mt) ? 1 : 0;
    return n;
  }
  // fragments a chunk; two chunks lie beside the tile, so a longer one costs
  // work-groups a CU and a shorter one barriers (FP32 stage launch with 16, 24,
  // 36: order 4, 82944 elements, 167, 164, 180 us; order 5, 48000 elements, 24
  // and 36, 176, 200; order 6, 24576 elements, 185, 177, 173)
  static constexpr int kLimit = N <= 3 ? 64 : N <= 5 ? 24 : 36;
  struct Layout {
    int chunk[nsteps + 1] = {}, at[nsteps] = {};
    int begin[nsteps + 1] = {};
    int chunks = 0;
  };
  static constexpr Layout lay() {
    Layout L;
    int f = 0, in = kLimit + 1;
    for (int s = 0; s < nsteps; ++s) {
      if (in + step_frags(s) > kLimit) {
        f = (f + 3) / 4 * 4;
        L.begin[L.chunks++] = f;
        in = 0;
      }
      L.chunk[s] = L.chunks - 1;
      L.at[s] = f;
      f += step_frags(s);
      in += step_frags(s);
    }
    L.chunk[nsteps] = -1;
    L.begin[L.chunks] = (f + 3) / 4 * 4;
    return L;
  }
  static constexpr Layout layout = lay();
  static constexpr int chunks = layout.chunks, frags = layout.begin[chunks];
  static constexpr int chunk_frags(int c) { return layout.begin[c + 1] - layout.begin[c]; }
  static constexpr int max_chunk() {
    int m = 0;
    for (int c = 0; c < chunks; ++c) m = chunk_frags(c) > m ? chunk_frags(c) : m;
    return m;
  }
};

}  // namespace dgw

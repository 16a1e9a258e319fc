// The lattice under the Klein four-group of the tetrahedron, shared by the
// host setup (operator fragments) and the matrix-core stage kernel.
//
// The double transpositions g_1 = (01)(23), g_2 = (02)(13), g_3 = (03)(12) of
// the four barycentrics, with g_0 = id, map the equispaced lattice onto
// itself; g_f maps vertex 0 to vertex f and face 0 to face f.  The four
// characters are x_i(g_j) = +1 where i = 0, j = 0 or i = j, else -1, and
// x_i x_j = x_(i xor j).  A nodal vector q is stored per orbit o (with
// representative node b_o) by its transform
//   q^_i(o) = sum_j x_i(g_j) q(g_j b_o),  q(g_j b_o) = 1/4 sum_i x_i(g_j) q^_i(o)
// (for short orbits the nodes repeat and the components that the stabiliser
// forbids are zero).  The derivative operators
//   T_p = p_1 D_r + p_2 D_s + p_3 D_t,  p_a = x_p(g_a),  p = 1, 2, 3
// satisfy g T_p g^-1 = x_p(g) T_p, so T_p takes component i to component
// i xor p only, and the four faces' lifts are one matrix: component i of the
// lifted flux needs component i of the flux's transform over the faces only.
// In these components the volume term of a column is 12 blocks of about
// Np/4 x Np/4 and the lift 4 blocks of Np/4 x Nfp, a quarter of the products
// of the nodal form.
#pragma once

#include <cstdint>

namespace dgw {

// x_i(g_j)
constexpr int sym_sign(int i, int j) { return i == 0 || j == 0 || i == j ? 1 : -1; }

template <int N>
struct Sym {
  static constexpr int Np = (N + 1) * (N + 2) * (N + 3) / 6;
  static constexpr int Nfp = (N + 1) * (N + 2) / 2;

  // node of the lattice point with barycentrics (b1, b2, b3) (b0 the rest)
  static constexpr int node(int b1, int b2, int b3) {
    int n = 0;
    for (int k = 0; k <= N; ++k)
      for (int j = 0; j <= N - k; ++j)
        for (int i = 0; i <= N - j - k; ++i, ++n)
          if (i == b1 && j == b2 && k == b3) return n;
    return -1;
  }
  // g_j applied to barycentrics: component a of the image is b[a xor j]
  struct Tab {
    int n = 0;                 // orbits: full ones, then size 2 by stabiliser, then size 1
    uint8_t at[Np][4] = {};    // at[o][j] = node g_j b_o
    uint8_t stab[Np] = {};     // 0 full; 1..3 fixed by that g; 4 fixed by all
    uint8_t slot[4 * Nfp] = {};  // face node (f, m) -> 4 j + f, j its face-0 preimage
  };
  static constexpr Tab make() {
    Tab T;
    for (int kind = 0; kind < 5; ++kind)
      for (int k = 0; k <= N; ++k)
        for (int j = 0; j <= N - k; ++j)
          for (int i = 0; i <= N - j - k; ++i) {
            const int b[4] = {N - i - j - k, i, j, k};
            int im[4] = {};
            for (int g = 0; g < 4; ++g) im[g] = node(b[1 ^ g], b[2 ^ g], b[3 ^ g]);
            int first = im[0];
            for (int g = 1; g < 4; ++g) first = im[g] < first ? im[g] : first;
            if (first != im[0]) continue;
            int st = 0;
            for (int g = 1; g < 4; ++g)
              if (im[g] == im[0]) st = st == 0 ? g : 4;
            if (st != kind) continue;
            for (int g = 0; g < 4; ++g) T.at[T.n][g] = (uint8_t)im[g];
            T.stab[T.n] = (uint8_t)st;
            ++T.n;
          }
    // face f's nodes ascending in node order; the preimage of (f, m) is the
    // face-0 node g_f x
    for (int f = 0; f < 4; ++f) {
      int m = 0;
      for (int k = 0; k <= N; ++k)
        for (int j = 0; j <= N - k; ++j)
          for (int i = 0; i <= N - j - k; ++i) {
            const int b[4] = {N - i - j - k, i, j, k};
            if (b[f] != 0) continue;
            const int want = node(b[1 ^ f], b[2 ^ f], b[3 ^ f]);
            int c = 0, at = -1;
            for (int k2 = 0; k2 <= N; ++k2)
              for (int j2 = 0; j2 <= N - k2; ++j2)
                for (int i2 = 0; i2 <= N - j2 - k2; ++i2) {
                  if (i2 + j2 + k2 != N) continue;
                  if (node(i2, j2, k2) == want) at = c;
                  ++c;
                }
            T.slot[f * Nfp + m] = (uint8_t)(4 * at + f);
            ++m;
          }
    }
    return T;
  }
  static constexpr Tab tab = make();
  static constexpr int nO = tab.n;
  static constexpr int MT = (nO + 15) / 16;   // row tiles of 16 orbits
  static constexpr int KS = (nO + 3) / 4;     // k-steps of 4 orbits
  static constexpr int KF = (Nfp + 3) / 4;    // k-steps of the lift
  // whether orbit o has a component i
  static constexpr bool has(int o, int i) {
    return o < nO && (tab.stab[o] == 0 || i == 0 || tab.stab[o] == i);
  }
  static constexpr bool kstep(int ks, int i) {
    for (int o = 4 * ks; o < 4 * ks + 4; ++o)
      if (has(o, i)) return true;
    return false;
  }
  // fragments of 64 entries: volume in the order (ks, p, i, row tile) of the
  // k-steps that exist, then lift in the order (ks, i, row tile)
  static constexpr int volume_frags() {
    int n = 0;
    for (int ks = 0; ks < KS; ++ks)
      for (int p = 1; p < 4; ++p)
        for (int i = 0; i < 4; ++i) n += kstep(ks, i) ? MT : 0;
    return n;
  }
  static constexpr int frags() { return volume_frags() + 4 * KF * MT; }
};

}  // namespace dgw

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
    uint8_t face[4 * Nfp] = {};  // (f, j) -> face node (f, m) with face-0 preimage j
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
            T.face[f * Nfp + at] = (uint8_t)(f * Nfp + m);
            ++m;
          }
    }
    return T;
  }
  static constexpr Tab tab = make();
  static constexpr int nO = tab.n;
  static constexpr int KS = (nO + 3) / 4;     // steps of four orbits
  static constexpr int KF = (Nfp + 3) / 4;    // steps of the lift
  // full orbits, and size-2 orbits of each type (stabiliser)
  static constexpr int count(int st) {
    int n = 0;
    for (int o = 0; o < nO; ++o) n += tab.stab[o] == st ? 1 : 0;
    return n;
  }
  static constexpr int nf = count(0), nt = count(1);
  // Component x has dim(x) values: index n < nf is orbit n, then come the
  // size-2 orbits that have the component (type x; component 0 has all, type
  // by type, and the size-1 orbit last, so its index is the orbit).
  static constexpr int dim(int x) { return x == 0 ? nO : nf + nt; }
  static constexpr int steps(int x) { return (dim(x) + 3) / 4; }
  static constexpr int orbit(int x, int n) {
    return n >= dim(x) ? -1 : n < nf || x == 0 ? n : nf + (x - 1) * nt + n - nf;
  }
  // index in component 0 (and lane group mod 4, step) of the first type-t
  // orbit; in component t its index is nf.  shift(t): lane groups from the
  // latter's to the former's
  static constexpr int home(int t) { return nf + (t - 1) * nt; }
  static constexpr int shift(int t) { return home(t) % 4 - nf % 4; }
  // nt consecutive indices from nf, and from home(t), lie in one step
  static constexpr bool aligned() {
    return nt == 0 || (nf % 4 + nt <= 4 && home(2) % 4 + nt <= 4 && home(3) % 4 + nt <= 4);
  }
  static_assert(aligned() && count(2) == nt && count(3) == nt, "short orbits within a step");
  // Operator fragments of 16 entries (4 rows x 4 products), step by step: the
  // volume's steps from the last down, each in the order (p, input component
  // i, row step of component i xor p), then the lift's, each in the order
  // (component, row step).  The steps are grouped in chunks that the kernel
  // stages in LDS one after the other (orders 3 and 4: all in one), each
  // starting at an even fragment.
  static constexpr int nsteps = KS + KF;
  static constexpr int step_frags(int s) {
    if (s >= KS) return steps(0) + steps(1) + steps(2) + steps(3);
    int n = 0;
    for (int p = 1; p < 4; ++p)
      for (int i = 0; i < 4; ++i) n += KS - 1 - s < steps(i) ? steps(i ^ p) : 0;
    return n;
  }
  static constexpr int kLimit = N <= 4 ? 100 : N == 5 ? 48 : 78;
  struct Layout {
    int chunk[nsteps] = {}, at[nsteps] = {};   // chunk and first fragment of a step
    int begin[nsteps + 1] = {};                // first fragment of a chunk
    int chunks = 0;
  };
  static constexpr Layout lay() {
    Layout L;
    int f = 0, in = kLimit + 1;
    for (int s = 0; s < nsteps; ++s) {
      if (in + step_frags(s) > kLimit) {
        f += f % 2;
        L.begin[L.chunks++] = f;
        in = 0;
      }
      L.chunk[s] = L.chunks - 1;
      L.at[s] = f;
      f += step_frags(s);
      in += step_frags(s);
    }
    L.begin[L.chunks] = f + f % 2;
    return L;
  }
  static constexpr Layout layout = lay();
  static constexpr int chunks = layout.chunks;
  static constexpr int frags = layout.begin[chunks];
  static constexpr int chunk_frags(int c) { return layout.begin[c + 1] - layout.begin[c]; }
  static constexpr int max_chunk() {
    int m = 0;
    for (int c = 0; c < chunks; ++c) m = chunk_frags(c) > m ? chunk_frags(c) : m;
    return m;
  }
};

}  // namespace dgw

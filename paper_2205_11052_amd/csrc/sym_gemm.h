// GEMM of the FP64 kernels in the symmetry components of the lattice (sym.h).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "sym.h"

namespace dgw {
namespace stagec {

// fn(integral_constant) for every index of [I, E), as straight code
template <int I, int E, class F>
__device__ __forceinline__ void unroll(F &&fn) {
  if constexpr (I < E) {
    fn(std::integral_constant<int, I>{});
    unroll<I + 1, E>(fn);
  }
}

// The transform over the Klein four-group (sym.h), its own inverse up to 4.
template <typename real>
__device__ __forceinline__ void sym4(const real (&a)[4], real (&t)[4]) {
  const real s = a[0] + a[1], d = a[0] - a[1], u = a[2] + a[3], v = a[2] - a[3];
  t[0] = s + u;
  t[1] = s - u;
  t[2] = d + v;
  t[3] = d - v;
}

// One column per lane of a 16-column tile, one tile per wave (the first NT
// waves of a work-group of THREADS).  A column is a nodal vector
//   sum_a D_a (sum_m C_a[m] q_m) + LIFT F
// with M fields q_m in LDS (qf[m]), cs[p][m] the sum of the two C_a[m], a != p,
// and F on face n, node j the combination sum_m cf[n][m] fl[m][n Nfp + j] of
// three LDS rows (nodes in the order of their face-0 preimages).  The caller
// sets qf, fl and cs.
template <int N, int M, int NT, int THREADS>
struct SymGemm {
  using S = Sym<N>;
  static constexpr int Np = S::Np, Nfp = S::Nfp, KS = S::KS;
  static constexpr int ROW = 4 * Nfp | 1;   // flux row, odd against bank conflicts
  // operator buffer: one chunk, or two where there are more
  static constexpr int OPS1 = 16 * S::max_chunk(), OPS = OPS1 * (S::chunks > 1 ? 2 : 1);
  static constexpr int OV = (8 * S::max_chunk() + THREADS - 1) / THREADS;
  typedef double vec2 __attribute__((ext_vector_type(2)));
  static_assert(NT <= THREADS / 64, "one column tile per wave");
  int g, w, lane;
  const uint32_t (&nodes)[KS];   // of this lane's orbits, four to a word
  const double *qf[M], *fl[3], *Ab;
  vec2 op, opv[OV];
  double cs[4][M];
  double acc[4][KS];   // acc[x][r] exists for r < S::steps(x)

  __device__ __forceinline__ SymGemm(const double *sop, const uint32_t (&nd)[KS], int tid)
      : nodes(nd) {
    lane = tid & 63;
    g = lane >> 4;
    w = tid >> 6;
    Ab = sop + 2 * (4 * g + (lane & 3));
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int r = 0; r < KS; ++r) acc[x][r] = 0.0;
  }
  // column of this lane
  __device__ __forceinline__ int column() const { return w * 16 + (lane & 15); }

  // Staging of the operator chunks (sym.h): thread tid's vectors of chunk c
  // into registers, and from there to its LDS buffer; chunk 0 comes with the
  // block's first loads, chunk c + 1 while chunk c is used.
  static __device__ __forceinline__ void load_ops(const double *ops, int c, int tid,
                                                  vec2 (&v)[OV]) {
    const vec2 *src = (const vec2 *)ops + 8 * S::layout.begin[c];
#pragma unroll
    for (int u = 0; u < OV; ++u) {
      const int t = tid + u * THREADS;
      v[u] = src[t < 8 * S::chunk_frags(c) ? t : 0];
    }
  }
  static __device__ __forceinline__ void store_ops(double *sop, int c, int tid,
                                                   const vec2 (&v)[OV]) {
#pragma unroll
    for (int u = 0; u < OV; ++u) {
      const int t = tid + u * THREADS;
      if (t < 8 * S::chunk_frags(c)) ((vec2 *)(sop + (c & 1) * OPS1))[t] = v[u];
    }
  }

  // acc += fragment f x y
  template <int s>
  __device__ __forceinline__ void mma(int n, double y, double &c) {
    // fragment n of step s, in pairs of one 16-byte read
    constexpr int ch = S::layout.chunk[s];
    const int f = S::layout.at[s] - S::layout.begin[ch] + n;
    if (f % 2 == 0 || n == 0) op = *(const vec2 *)(Ab + (ch & 1) * OPS1 + 32 * (f / 2));
    c = __builtin_amdgcn_mfma_f64_4x4x4f64(op[f % 2], y, c, 0, 0, 0);
  }
  // the value of the lane `shift` groups on, for the same column
  __device__ __forceinline__ double from(double v, int shift) const {
    return __shfl(v, (lane + 16 * shift) & 63);
  }

  // runs step s around fn, with the staging of the next chunk
  template <int s, class F>
  __device__ __forceinline__ void step(const double *ops, double *sop, int tid, F &&fn) {
    constexpr int c = S::layout.chunk[s];
    constexpr bool next = c + 1 < S::chunks;
    if constexpr (next && (s == 0 || S::layout.chunk[s > 0 ? s - 1 : 0] != c))
      load_ops(ops, c + 1, tid, opv);
    if (w < NT) fn();
    if constexpr (next && S::layout.chunk[s + 1 < S::nsteps ? s + 1 : s] != c) {
      store_ops(sop, c + 1, tid, opv);
      __syncthreads();
    }
  }

  __device__ __forceinline__ void volume(const double *ops, double *sop, int tid) {
    double mv[4][M];   // components 2 and 3 of their short orbits, at their indices' lanes
    unroll<0, KS>([&](auto I) {
      constexpr int s = decltype(I)::value, ks = KS - 1 - s;
      step<s>(ops, sop, tid, [&] {
        double qt[M][4];
#pragma unroll
        for (int m = 0; m < M; ++m) {
          double v[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = qf[m][(nodes[ks] >> (8 * j)) & 255];
          sym4(v, qt[m]);
#pragma unroll
          for (int t = 2; t < 4; ++t) {
            if (S::nt > 0 && ks == S::home(t) / 4) mv[t][m] = from(qt[m][t], S::shift(t));
            if (S::nt > 0 && ks == S::nf / 4)
              qt[m][t] = g >= S::nf % 4 && g < S::nf % 4 + S::nt ? mv[t][m] : qt[m][t];
          }
        }
        int n = 0;   // a constant at every use once unrolled
#pragma unroll
        for (int p = 1; p < 4; ++p)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (ks >= S::steps(i)) continue;
            double y = cs[p][0] * qt[0][i];
#pragma unroll
            for (int m = 1; m < M; ++m) y += cs[p][m] * qt[m][i];
#pragma unroll
            for (int r = 0; r < S::steps(i ^ p); ++r) mma<s>(n++, y, acc[i ^ p][r]);
          }
      });
    });
  }

  // face(cf) gives the column's flux on face n as sum_m cf[n][m] fl[m]
  template <class F>
  __device__ __forceinline__ void lift(const double *ops, double *sop, int tid, F &&face) {
    double cf[4][3];
    face(cf);
    unroll<0, S::KF>([&](auto I) {
      constexpr int ks = decltype(I)::value, s = KS + ks;
      step<s>(ops, sop, tid, [&] {
        // the rows past Nfp of the last step read a valid node; their
        // operator entries are zero
        const int j = 4 * ks + g, jj = j < Nfp ? j : Nfp - 1;
        double v[4], ft[4];
#pragma unroll
        for (int n = 0; n < 4; ++n)
          v[n] = cf[n][0] * fl[0][n * Nfp + jj] + cf[n][1] * fl[1][n * Nfp + jj] +
                 cf[n][2] * fl[2][n * Nfp + jj];
        sym4(v, ft);
        int n = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
          for (int r = 0; r < S::steps(x); ++r) mma<s>(n++, ft[x], acc[x][r]);
      });
    });
  }

  // the column's nodal values to out (where ok)
  __device__ __forceinline__ void store(double *out, bool ok) const {
    if (w >= NT) return;
    double mv[4] = {};
    if (S::nt > 0)
#pragma unroll
      for (int t = 2; t < 4; ++t) mv[t] = from(acc[t][S::nf / 4], -S::shift(t));
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      double a[4], t[4];
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        a[x] = ks < S::steps(x) ? acc[x][ks] : (double)0;
        if (S::nt > 0 && x >= 2) {
          if (ks == S::nf / 4 && g >= S::nf % 4 && g < S::nf % 4 + S::nt) a[x] = (double)0;
          if (ks == S::home(x) / 4 && g >= S::home(x) % 4 && g < S::home(x) % 4 + S::nt)
            a[x] = mv[x];
        }
      }
      sym4(a, t);
      if (4 * ks + g < S::nO && ok)
#pragma unroll
        for (int j = 0; j < 4; ++j) out[(nodes[ks] >> (8 * j)) & 255] = t[j];
    }
  }
};

}  // namespace stagec
}  // namespace dgw

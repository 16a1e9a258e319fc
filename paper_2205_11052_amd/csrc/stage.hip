// Fused right-hand side + LSERK stage kernel for gfx950.
//
// Work item: a block of BE consecutive elements of one shot.  The items of
// all shots form one flat list.  The hardware dispatches work-groups to the 8
// XCDs round-robin, so the linear work-group id is remapped to give every XCD
// one contiguous range of items: face neighbours (same element, same cube,
// adjacent cubes) are then mostly processed on the same XCD and their traces
// are L2 hits.  Two launch forms share the item code: one work-group per item,
// or a persistent grid of a multiple of 8 work-groups that loop over the
// items (each work-group stays on one XCD).  They are separate instantiations
// so the one-item form carries no loop.
//
// Per item (256 threads):
//   1. every global read of the item's fields is issued at once: the block's
//      fields q[BE][9][Np] (contiguous in HBM, coalesced) and per-element data
//      go to LDS, and each thread gathers the neighbour traces of its face
//      nodes (the neighbour element from the face connectivity, the node from
//      a per-face-node table, so no load waits on a table lookup) into
//      registers;
//   2. one thread per (element, face node): exact Riemann flux in jump form
//      (optionally blended with the central flux; for anisotropic elements
//      from the face's impedance matrices) from the own trace (LDS) and the
//      neighbour's (registers); six quantities go to LDS, the velocity flux
//      and the velocity change dv (the stress flux is lambda (n.dv) I +
//      mu (dv n^T + n dv^T), n constant per face, so it is formed from the
//      lifted dv or on the way into the lift), or all nine components;
//   3. the volume terms and the lifted flux, by one of three forms: one thread
//      per (element, node) on the vector ALUs (phase3_nodes); a GEMM on the
//      matrix cores in nodal form (NodalGemm: FP32, and FP64 at orders 1 and
//      2); a GEMM in the symmetry components of the lattice (StageGemm: FP64
//      from order 3).  Then + point source, res = a res + dt rhs and
//      q_out = q_in + b res.
// q_in and q_out are distinct buffers (neighbour traces are read from q_in
// while other blocks write q_out); res is element-local and updated in place.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "dgw_internal.h"
#include "stage_common.h"
#include "nodal.h"
#include "sym_gemm.h"

namespace dgw {

namespace {

constexpr int kThreads = 256;
// Whether the matrix-core form works in symmetry components (StageGemm).
template <int N, typename real>
constexpr bool kSymForm = stage_symmetric(N, 8 * (int)sizeof(real));
using namespace stagec;

// Residual and update of a block's contiguous span by 16-byte vectors; the
// right-hand side comes from LDS in the block's (element, field, node) order.
//
// Streaming at order >= 4: the residual (read and written once per stage)
// and the FP64 output state move with non-temporal loads and stores, so
// they do not evict the neighbour traces and operators.  Measured on the
// order-4 82944-element workload (whose streams exceed the 256 MB
// last-level cache): FP64 370 -> 351 us, FP32 213 -> 204 us (FP32 keeps
// its output state cached, which measured faster).  The order-3
// 24576-element gradient workload fits that cache and ran 5% slower with
// them, so lower orders keep ordinary accesses.
template <int N, typename real, int BE>
struct Update {
  static constexpr int Np = Sz<N>::Np;
  static constexpr bool kStream = N >= 4;
  using SP = Span16<real>;
  static constexpr int UV = (BE * 9 * Np / SP::VW + kThreads - 1) / kThreads;
  SP sp{0, 0};
  bool first;
  real *rs, *qo;
  int tl0;
  typename SP::vec rv[UV];
  real rh, rt;

  // residual loads of this thread's update items, all issued together
  __device__ __forceinline__ void load(const StageArgs<real> &A, int64_t k0, int shot, int nE,
                                       real *qout, real *res, int tid) {
    sp = SP(shot * A.shot_stride + k0 * 9 * Np, nE * 9 * Np);
    first = A.rk_a == 0.0;
    rs = res + k0 * 9 * Np;
    qo = qout + k0 * 9 * Np;
#pragma unroll
    for (int u = 0; u < UV; ++u) {
      const int j = tid + u * kThreads;
      if (!first && j < sp.nv) {
        const typename SP::vec *rp = (const typename SP::vec *)(rs + sp.hd) + j;
        if constexpr (kStream)
          rv[u] = __builtin_nontemporal_load(rp);
        else
          rv[u] = *rp;
      }
      else rv[u] = typename SP::vec{};
    }
    tl0 = sp.hd + SP::VW * sp.nv;
    rh = (!first && tid < sp.hd) ? rs[tid] : (real)0;
    rt = (!first && tid < sp.tl) ? rs[tl0 + tid] : (real)0;
  }

  // LSERK update over the contiguous span, with the point source (element
  // es of the block) and the sponge where the block has them: a plain block
  // needs no element and node of each value, whose divisions were a third of
  // the update's instructions
  __device__ __forceinline__ void apply(const StageArgs<real> &A, const real *sq,
                                        const real *sfl, const double *ssig, int nE,
                                        int64_t es, int shot, int64_t step, int tid) {
    if ((es >= 0 && es < nE) || A.sponge)
      sweep<true>(A, sq, sfl, ssig, nE, es, shot, step, tid);
    else
      sweep<false>(A, sq, sfl, ssig, nE, es, shot, step, tid);
  }

  template <bool EXTRA>
  __device__ __forceinline__ void sweep(const StageArgs<real> &A, const real *sq,
                                        const real *sfl, const double *ssig, int nE,
                                        int64_t es, int shot, int64_t step, int tid) {
    const real ra = (real)A.rk_a, rb = (real)A.rk_b, rdt = (real)A.dt;
    double s = 0.0;
    const double *spar = A.src_par + 10 * shot;
    if (EXTRA && es >= 0 && es < nE)
      s = ricker_d(((double)step + A.rk_c) * A.dt, spar[6], spar[7], spar[8]);
    auto update = [&](int t, real rold) -> real2v<real> {
      real rhs = sfl[t];
      if constexpr (EXTRA) {
        const int e = t / (9 * Np), ci = t - e * 9 * Np, c = ci / Np, i = ci - c * Np;
        if (e == es && c >= 3) rhs += (real)(s * spar[c - 3] * A.src_vec[shot * Np + i]);
        if (A.sponge) rhs -= (real)ssig[e] * sq[t];
      }
      const real rn = first ? rdt * rhs : ra * rold + rdt * rhs;
      return {rn, sq[t] + rb * rn};
    };
#pragma unroll
    for (int u = 0; u < UV; ++u) {
      const int j = tid + u * kThreads;
      if (j >= sp.nv) continue;
      const int b = sp.hd + SP::VW * j;
      typename SP::vec nr, nq;
#pragma unroll
      for (int l = 0; l < SP::VW; ++l) {
        const real2v<real> o = update(b + l, rv[u][l]);
        nr[l] = o.r;
        nq[l] = o.q;
      }
      if constexpr (kStream) {
        __builtin_nontemporal_store(nr, (typename SP::vec *)(rs + b));
        if constexpr (sizeof(real) == 8)
          __builtin_nontemporal_store(nq, (typename SP::vec *)(qo + b));
        else
          *(typename SP::vec *)(qo + b) = nq;
      } else {
        *(typename SP::vec *)(rs + b) = nr;
        *(typename SP::vec *)(qo + b) = nq;
      }
    }
    if (tid < sp.hd) {
      const real2v<real> o = update(tid, rh);
      if constexpr (kStream)
        __builtin_nontemporal_store(o.r, rs + tid);
      else
        rs[tid] = o.r;
      qo[tid] = o.q;
    }
    if (tid < sp.tl) {
      const real2v<real> o = update(tl0 + tid, rt);
      if constexpr (kStream)
        __builtin_nontemporal_store(o.r, rs + tl0 + tid);
      else
        rs[tl0 + tid] = o.r;
      qo[tl0 + tid] = o.q;
    }
  }
};

// A column (element, field k) of the block's right-hand side.  By linearity
// the element's metric and material factors move to the input side: every
// component is rhs_k = sum_a D_a u_{k,a} + LIFT F_k, with
// u_{k,a} = sum_m c_{a,m} q_{f(m)} a per-node combination of at most three
// fields (for example u_{vx,a} = (1/rho) sum_b X^-1[a][b] sigma_{xb} and
// u_{sxx,a} = (lambda + 2 mu) X^-1[a][0] vx + lambda X^-1[a][1] vy +
// lambda X^-1[a][2] vz).
template <typename real>
struct Column {
  int f[3];
  real c[3][3];
};

template <typename real, bool AN>
__device__ __forceinline__ void column_setup(const StageArgs<real> &A, const double *gm,
                                             int64_t k0e, int k, Column<real> &o) {
  // input-side coefficients of this column, c[a][m] = s_m X^-1[a][x_m],
  // with the material factor s_m and the metric column x_m of each of
  // the three combined fields f_m given per component k by packed tables
  // (branch-free: the sixteen lanes of a column tile hold different k):
  //   k = 0..2 (vx, vy, vz):   f = sigma row k, s = 1/rho, x = (0, 1, 2)
  //   k = 3..5 (sxx..szz):      f = (vx, vy, vz), s = lambda + 2 mu on
  //                             x = k - 3, lambda elsewhere, x = (0, 1, 2)
  //   k = 6 (syz): f = (vy, vz), s = mu, x = (2, 1)
  //   k = 7 (sxz): f = (vx, vz), s = mu, x = (2, 0)
  //   k = 8 (sxy): f = (vx, vy), s = mu, x = (1, 0)
  // fields (4 bits per k, m = 0, 1, 2)
  constexpr uint64_t F0 = 0x001000783ull, F1 = 0x122111648ull, F2 = 0x210222567ull;
  // metric columns (2 bits per k) and material factor ids (3 bits per k:
  // 0 1/rho, 1 lambda + 2 mu, 2 lambda, 3 mu, 4 zero)
  constexpr uint32_t X0 = 0x1a000u, X1 = 0x01555u, X2 = 0x2aaaau;
  constexpr uint32_t S0 = 0x36d2200u, S1 = 0x36d1400u, S2 = 0x490a400u;
  int f0 = (int)((F0 >> (4 * k)) & 15), f1 = (int)((F1 >> (4 * k)) & 15),
      f2 = (int)((F2 >> (4 * k)) & 15);
  const real ri = (real)gm[M_RHOINV], la = (real)gm[M_LAM], mu = (real)gm[M_MU];
  const real l2 = la + 2 * mu;
  auto fac = [&](uint32_t S) -> real {
    const int id = (int)((S >> (3 * k)) & 7);
    return id == 0 ? ri : id == 1 ? l2 : id == 2 ? la : id == 3 ? mu : (real)0;
  };
  const real s0 = fac(S0), s1 = fac(S1), s2 = fac(S2);
  const int x0 = (int)((X0 >> (2 * k)) & 3), x1 = (int)((X1 >> (2 * k)) & 3),
            x2 = (int)((X2 >> (2 * k)) & 3);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const real r0 = (real)gm[M_XINV + 3 * a], r1 = (real)gm[M_XINV + 3 * a + 1],
               r2 = (real)gm[M_XINV + 3 * a + 2];
    auto pick = [&](int x) { return x == 0 ? r0 : x == 1 ? r1 : r2; };
    o.c[a][0] = s0 * pick(x0);
    o.c[a][1] = s1 * pick(x1);
    o.c[a][2] = s2 * pick(x2);
  }
  if constexpr (AN) {
    // anisotropic stress rows (k >= 3, Voigt row I = k - 3): the fields
    // are (vx, vy, vz) and c[a][m] = sum_b C[I][voigt(m, b)] X^-1[a][b]
    // (selects, so the column setup stays branch-free)
    const bool st = k >= 3;
    const int I = st ? k - 3 : 0;
    const double *Cu = A.aniso + k0e * DGW_ANI + A_C;
    real cr[6];
#pragma unroll
    for (int J = 0; J < 6; ++J) {
      const int i = I < J ? I : J, j = I < J ? J : I;   // upper triangle
      cr[J] = (real)Cu[i * (11 - i) / 2 + j];
    }
    constexpr int VG[3][3] = {{0, 5, 4}, {5, 1, 3}, {4, 3, 2}};   // voigt(m, b)
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        real v = 0;
#pragma unroll
        for (int b = 0; b < 3; ++b) v += cr[VG[m][b]] * (real)gm[M_XINV + 3 * a + b];
        o.c[a][m] = st ? v : o.c[a][m];
      }
    f0 = st ? 0 : f0;
    f1 = st ? 1 : f1;
    f2 = st ? 2 : f2;
  }
  o.f[0] = f0;
  o.f[1] = f1;
  o.f[2] = f2;
}

// Phase 3 on the matrix cores in nodal form: the block's right-hand side is one
// GEMM, rhs[i][(e,k)] = [Dr Ds Dt LIFT][i][.] x [u_r; u_s; u_t; F][.][(e,k)],
// whose operator side is shared by all elements.  Each wave owns one or two
// tiles of 16 columns (element, field) and feeds both from every fragment it
// reads; rows are nodes, in the order of nodal.h.  The fragments are staged in
// LDS in chunks, one while the other is used, without the zero tiles; the data
// side is formed in registers from the LDS tile.  The accumulators go through
// LDS (the flux buffer, dead by then) so that the update and the stores run
// over the block's contiguous span, fully coalesced.
// It is bound by the matrix instructions and the passes through LDS around
// them.  FP32 stage launch, fragments of every tile from L2 -> this: order 4,
// 82944 elements, 190 -> 158 us (without the fragment loads 112); order 5, 118
// -> 94; order 6, 24576 elements, 221 -> 169 us.  A value that is not finite
// spreads over its element in a few stages instead of one, as zero tiles are
// left out; after a whole step the values that are not finite are the same.
template <int N, typename real, int BE, bool AN>
struct NodalGemm {
  using S = Nodal<N>;
  using M = Mma<real>;
  using v4 = typename M::v4;
  static constexpr int Np = S::Np, NF = S::NF, MT = S::MT, KS = S::KS;
  static constexpr int NT = (9 * BE + 15) / 16;      // column tiles
  static constexpr int NW = kThreads / 64;
  static constexpr int HT = (NT + NW - 1) / NW;      // column tiles per wave
  static constexpr int VW = 16 / (int)sizeof(real);  // fragments per 16-byte read
  static constexpr int OPS1 = 64 * S::max_chunk();
  // At orders 1 and 2 the few fragments come from L2 as they are used, and the
  // residual is loaded after the products: staged and early, FP64 order 2 took
  // 79 us instead of 74 (82944 elements), order 1 21.9 instead of 20.5 (24576).
  static constexpr bool kStaged = N >= 3;
  static constexpr int OPS = kStaged ? OPS1 * (S::chunks > 1 ? 2 : 1) : 4;
  static constexpr int OV = kStaged ? (OPS1 / VW + kThreads - 1) / kThreads : 1;
  typedef real vec __attribute__((ext_vector_type(VW)));
  static_assert(9 * Np <= 9 * NF, "the flux buffer holds the right-hand side");
  int lane, g, w, cols;
  const uint32_t (&rows)[MT];   // nodes of this lane's accumulator rows, four to a word
  const real *qf[HT][3], *fl[HT], *Ab;
  Column<real> C[HT];
  vec op, opv[OV];
  v4 acc[HT][MT];

  __device__ __forceinline__ NodalGemm(const StageArgs<real> &A, const real *sq,
                                       const real *sfl, const real *sop,
                                       const double *smeta, int nE, int64_t k0,
                                       const uint32_t (&rw)[MT], int tid)
      : rows(rw) {
    lane = tid & 63;
    g = lane >> 4;
    w = tid >> 6;
    cols = 9 * nE;
    Ab = sop + VW * lane;
#pragma unroll
    for (int h = 0; h < HT; ++h) {
      const int col = column(h);
      const bool cok = col < cols;
      const int e = cok ? col / 9 : 0, k = cok ? col - 9 * (col / 9) : 0;
      column_setup<real, AN>(A, smeta + e * DGW_META, k0 + e, k, C[h]);
#pragma unroll
      for (int m = 0; m < 3; ++m) qf[h][m] = sq + (e * 9 + C[h].f[m]) * Np;
      fl[h] = sfl + (e * 9 + k) * NF;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[h][mt] = v4{0, 0, 0, 0};
    }
  }
  __device__ __forceinline__ int column(int h) const { return (w + h * NW) * 16 + (lane & 15); }

  // staging of the chunks, as in SymGemm
  static __device__ __forceinline__ void load_ops(const real *ops, int c, int tid,
                                                  vec (&v)[OV]) {
    const vec *src = (const vec *)ops + 64 / VW * S::layout.begin[c];
#pragma unroll
    for (int u = 0; u < OV; ++u) {
      const int t = tid + u * kThreads;
      if constexpr (kStaged) v[u] = src[t < 64 / VW * S::chunk_frags(c) ? t : 0];
    }
  }
  static __device__ __forceinline__ void store_ops(real *sop, int c, int tid,
                                                   const vec (&v)[OV]) {
#pragma unroll
    for (int u = 0; u < OV; ++u) {
      const int t = tid + u * kThreads;
      if (kStaged && t < 64 / VW * S::chunk_frags(c)) ((vec *)(sop + (c & 1) * OPS1))[t] = v[u];
    }
  }

  // step s (nodal.h): acc += its fragments x b
  template <int s, class F>
  __device__ __forceinline__ void step(const real *ops, real *sop, int tid, F &&fb) {
    constexpr int c = S::layout.chunk[s];
    constexpr bool next = c + 1 < S::chunks;
    if constexpr (next && (s == 0 || S::layout.chunk[s > 0 ? s - 1 : 0] != c))
      load_ops(ops, c + 1, tid, opv);
    if (w < NT && S::step_frags(s) > 0) {
      real b[HT];
#pragma unroll
      for (int h = 0; h < HT; ++h) b[h] = fb(h);
      int f = S::layout.at[s] - S::layout.begin[c];   // constants once unrolled
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        if (!S::need(s, mt)) continue;
        if (f % VW == 0)
          op = *(const vec *)(kStaged ? Ab + (c & 1) * OPS1 + 64 * f : ops + VW * lane + 64 * f);
#pragma unroll
        for (int h = 0; h < HT; ++h) acc[h][mt] = M::mma(op[f % VW], b[h], acc[h][mt]);
        ++f;
      }
    }
    if constexpr (next && S::layout.chunk[s + 1] != c) {
      store_ops(sop, c + 1, tid, opv);
      __syncthreads();
    }
  }

  // volume: three reference directions, K = Np (padded to a multiple of 4)
  __device__ __forceinline__ void volume(const real *ops, real *sop, int tid) {
    // each value once from LDS for the three directions
    real q[HT][3][KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      // rows past Np of the last k-step read a valid node and are zeroed
      const int j = 4 * ks + g, jj = j < Np ? j : Np - 1;
#pragma unroll
      for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int m = 0; m < 3; ++m) q[h][m][ks] = qf[h][m][jj];
    }
    stagec::unroll<0, 3 * KS>([&](auto I) {
      constexpr int s = decltype(I)::value, a = s / KS, ks = s % KS;
      const int j = 4 * ks + g;
      step<s>(ops, sop, tid, [&](int h) {
        // written out: the bits must not hang on how a compiler contracts it
        const real v = fma(C[h].c[a][2], q[h][2][ks],
                           fma(C[h].c[a][0], q[h][0][ks], C[h].c[a][1] * q[h][1][ks]));
        return j < Np ? v : (real)0;
      });
    });
  }
  // lift: the column's flux on the 4 Nfp face nodes
  __device__ __forceinline__ void lift(const real *ops, real *sop, int tid) {
    stagec::unroll<0, S::KL>([&](auto I) {
      constexpr int ks = decltype(I)::value;
      step<3 * KS + ks>(ops, sop, tid, [&](int h) { return fl[h][4 * ks + g]; });
    });
  }

  // right-hand side to LDS in the block's (element, field, node) order
  __device__ __forceinline__ void store(real *out) const {
    if (w >= NT) return;
#pragma unroll
    for (int h = 0; h < HT; ++h) {
      const int col = column(h);
      if (col >= cols) continue;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = (rows[mt] >> (8 * r)) & 255;
          if (i < Np) out[col * Np + i] = acc[h][mt][r];
        }
    }
  }
};

// Phase 3 on the vector ALUs: one thread per (element, node).  AN:
// anisotropic elements, whose stress rate is C times the strain rate of the
// volume term plus that of the lifted face terms (N(n_f) times the lifted
// dv of each face), with C from the anisotropic per-element data.
template <int N, typename real, int BE, bool AN>
__device__ __forceinline__ void phase3_nodes(const StageArgs<real> &A, const real *sq,
                                             const real *sfl, const double *smeta,
                                             const double *ssig, int nE, int64_t k0,
                                             int shot, int64_t step,
                                             real *qout, real *res, int oz, int tid) {
  constexpr int Np = Sz<N>::Np, Nfp = Sz<N>::Nfp, NF = 4 * Sz<N>::Nfp;
  constexpr int UJ = Np % 7 == 0 ? 7 : Np % 5 == 0 ? 5 : 4;  // divides Np
  for (int t = tid; t < nE * Np; t += kThreads) {
    const int e = t / Np, i = t - e * Np;
    const real *qe = sq + e * 9 * Np;
    const double *g = smeta + e * DGW_META;
    real dr[9], ds[9], dt[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) dr[c] = ds[c] = dt[c] = (real)0;
    // column i of the transposed operators, walked in chunks of UJ rows:
    // inside a chunk every offset is an immediate
    const real *pr = A.DrT + i + oz, *ps = A.DsT + i + oz, *pt = A.DtT + i + oz;
#pragma unroll 1   // a short chunk loop unrolled would hoist every load
    for (int j0 = 0; j0 < Np; j0 += UJ) {
#pragma unroll
      for (int u = 0; u < UJ; ++u) {
        const real a0 = pr[u * Np], a1 = ps[u * Np], a2 = pt[u * Np];
#pragma unroll
        for (int c = 0; c < 9; ++c) {
          const real v = qe[c * Np + j0 + u];
          dr[c] += a0 * v;
          ds[c] += a1 * v;
          dt[c] += a2 * v;
        }
      }
      pr += UJ * Np;
      ps += UJ * Np;
      pt += UJ * Np;
    }
    const int64_t k = k0 + e;
    // the residual loads are issued here, after the volume loop has freed
    // its registers, so their latency overlaps the lift
    real rold[9];
#pragma unroll
    for (int c = 0; c < 9; ++c)
      rold[c] = (A.rk_a == 0.0) ? (real)0 : res[(k * 9 + c) * Np + i];
    real X[9];
#pragma unroll
    for (int u = 0; u < 9; ++u) X[u] = (real)g[M_XINV + u];
    // d/dx_b of field c
    auto D = [&](int c, int b) -> real {
      return X[b] * dr[c] + X[3 + b] * ds[c] + X[6 + b] * dt[c];
    };
    const real ri = (real)g[M_RHOINV], la = (real)g[M_LAM], mu = (real)g[M_MU];
    real rhs[9];
    rhs[0] = (D(3, 0) + D(8, 1) + D(7, 2)) * ri;
    rhs[1] = (D(8, 0) + D(4, 1) + D(6, 2)) * ri;
    rhs[2] = (D(7, 0) + D(6, 1) + D(5, 2)) * ri;
    // anisotropic: the Voigt strain rate (engineering shears), times C below
    real ev[6];
    if constexpr (AN) {
      ev[0] = D(0, 0);
      ev[1] = D(1, 1);
      ev[2] = D(2, 2);
      ev[3] = D(1, 2) + D(2, 1);
      ev[4] = D(0, 2) + D(2, 0);
      ev[5] = D(0, 1) + D(1, 0);
    } else {
      const real divv = D(0, 0) + D(1, 1) + D(2, 2);
      rhs[3] = la * divv + 2 * mu * D(0, 0);
      rhs[4] = la * divv + 2 * mu * D(1, 1);
      rhs[5] = la * divv + 2 * mu * D(2, 2);
      rhs[6] = mu * (D(1, 2) + D(2, 1));
      rhs[7] = mu * (D(0, 2) + D(2, 0));
      rhs[8] = mu * (D(0, 1) + D(1, 0));
    }
    // lift: velocity flux over all faces; lifted dv per face, then the
    // stress components from it and the face normal
    const real *fle = sfl + e * NF * 6;
    const real *pl = A.LIFTT + i + oz;
    real V0 = 0, V1 = 0, V2 = 0;
#pragma unroll 1   // unrolled, the persistent form hoists too much and spills
    for (int f = 0; f < 4; ++f) {
      real U0 = 0, U1 = 0, U2 = 0;
      // the face's lift entries in chunks of LC, each chunk's loads issued
      // before its first use (one by one, every entry cost a round trip)
      constexpr int LC = Nfp % 7 == 0 ? 7 : Nfp % 5 == 0 ? 5 : Nfp;
#pragma unroll
      for (int m0 = 0; m0 < Nfp; m0 += LC) {
        real l[LC];
#pragma unroll
        for (int u = 0; u < LC; ++u) l[u] = pl[(f * Nfp + m0 + u) * Np];
#pragma unroll
        for (int u = 0; u < LC; ++u) {
          const real *s6 = fle + (f * Nfp + m0 + u) * 6;
          V0 += l[u] * s6[0];
          V1 += l[u] * s6[1];
          V2 += l[u] * s6[2];
          U0 += l[u] * s6[3];
          U1 += l[u] * s6[4];
          U2 += l[u] * s6[5];
        }
      }
      const real nx = (real)g[M_NORMAL + 3 * f], ny = (real)g[M_NORMAL + 3 * f + 1],
                 nz = (real)g[M_NORMAL + 3 * f + 2];
      if constexpr (AN) {
        ev[0] += nx * U0;
        ev[1] += ny * U1;
        ev[2] += nz * U2;
        ev[3] += nz * U1 + ny * U2;
        ev[4] += nz * U0 + nx * U2;
        ev[5] += ny * U0 + nx * U1;
      } else {
        const real nU = nx * U0 + ny * U1 + nz * U2;
        rhs[3] += la * nU + 2 * mu * U0 * nx;
        rhs[4] += la * nU + 2 * mu * U1 * ny;
        rhs[5] += la * nU + 2 * mu * U2 * nz;
        rhs[6] += mu * (U1 * nz + U2 * ny);
        rhs[7] += mu * (U0 * nz + U2 * nx);
        rhs[8] += mu * (U0 * ny + U1 * nx);
      }
    }
    rhs[0] += V0;
    rhs[1] += V1;
    rhs[2] += V2;
    if constexpr (AN) {
      // stress rate C ev, C symmetric from its upper triangle
      const double *Cu = A.aniso + k * DGW_ANI + A_C;
      int u = 0;
      real cm[6][6];
#pragma unroll
      for (int a = 0; a < 6; ++a)
#pragma unroll
        for (int b = a; b < 6; ++b) cm[a][b] = cm[b][a] = (real)Cu[u++];
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        real acc = 0;
#pragma unroll
        for (int b = 0; b < 6; ++b) acc += cm[a][b] * ev[b];
        rhs[3 + a] = acc;
      }
    }
    if (A.sponge) {
      const real sg = (real)ssig[e];
#pragma unroll
      for (int c = 0; c < 9; ++c) rhs[c] -= sg * qe[c * Np + i];
    }
    if (A.src_elem[shot] == k) {
      const double *sp = A.src_par + 10 * shot;
      const double s = ricker_d(((double)step + A.rk_c) * A.dt, sp[6], sp[7], sp[8]);
      const double w = s * A.src_vec[shot * Np + i];
#pragma unroll
      for (int c = 0; c < 6; ++c) rhs[3 + c] += (real)(w * sp[c]);
    }
    const real ra = (real)A.rk_a, rb = (real)A.rk_b, rdt = (real)A.dt;
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      const int64_t idx = (k * 9 + c) * Np + i;
      // stage 1 (a = 0) never reads res, so stale values cannot leak in
      const real r = (A.rk_a == 0.0) ? rdt * rhs[c] : ra * rold[c] + rdt * rhs[c];
      res[idx] = r;
      qout[idx] = qe[c * Np + i] + rb * r;
    }
  }
}

// Phase 3 on the matrix cores in FP64 from order 3: the block's right-hand side
// as one GEMM in the symmetry components of the lattice (sym.h).  With cs_p
// the sum of the two coefficients c_a, a != p, of a column, component x of its
// right-hand side is
//   r_x = sum_p A_{x,p} (sum_m cs_p[m] q^_{m, x xor p}) + B_x F^_x,
// the factor -1/8 in A and 1/4 in B.  Rows and products run over the
// components' indices (sym.h) in steps of four: lane group g supplies index
// 4 ks + g of an operand and holds row 4 r + g of accumulator r, so a lane
// reads the four nodes of its own orbits from the LDS tile and transforms
// them in registers (which serves all twelve blocks), and transforms its
// results back.  The flux of a face node and its three images is one
// transform too.  The values of the size-2 orbits sit in other lanes in
// component 0 than in their own, and move between them.
//
// The instruction is the four-block 4x4x4: its four blocks take the sixteen
// columns of a 16x16x4 with the four rows of A repeated, so rows come in fours
// (the components have 11, 8, 8 and 8 at order 4), and it is the faster one:
// 19.6 cycles for 256 products against 122.7 for 1024 (a loop on every SIMD, in
// cycles of 2.4 GHz).  Matrix and vector instructions of one wave do not
// overlap, those of two waves do.
//
// Its operand traffic is what the layout is made for.  Read from global memory
// per wave, the fragments took 45 of 267 us (512 bytes to the registers for
// 128 in memory, and every wave reads all), and no other load could be in
// flight behind them.  So a work-group stages them in LDS (12.3 KB at order 4;
// in chunks, one while the other is used, at orders 5 and 6: 37 and 61 KB),
// the lifted flux keeps six quantities per face node instead of nine, which
// leaves three work-groups a CU at order 4 (226 -> 212 us), and the residual
// is loaded with the neighbour traces, its trip over before the update waits
// for it (259 -> 225 us with two work-groups a CU).
//
// Measured, FP64 stage launch, nodal form on 16x16x4 (at order 6 the faster
// node-per-thread form) -> these components on 16x16x4 with operators from
// global memory -> this: order 4, 82944 elements, 348 -> 268 -> 212 us (983 MB
// of traffic, 4.6 of the 5.3 TB/s a copy reaches), anisotropic 462 -> 362 ->
// 256 us; order 3, 24576 elements, 54 -> 58 -> 49 us; order 5, 24576
// elements, 211 -> 137 -> 128 us; order 6, 24576 elements, 476 -> 282 -> 217
// us.  Orders 1 and 2 keep the nodal form, whose operators are a few
// fragments: 34 against 44 us at order 1 and 53 against 56 us at order 2
// (55566 elements).
template <int N, int BE, bool AN>
struct StageGemm : SymGemm<N, 3, (9 * BE + 15) / 16, kThreads> {
  using G = SymGemm<N, 3, (9 * BE + 15) / 16, kThreads>;
  bool vel, ok;

  __device__ __forceinline__ StageGemm(const StageArgs<double> &A, const double *sq,
                                       const double *sfl, const double *sop,
                                       const double *smeta, int nE, int64_t k0,
                                       const uint32_t (&nd)[G::KS], int tid)
      : G(sop, nd, tid) {
    const int col = G::column();
    ok = col < 9 * nE;
    const int e = ok ? col / 9 : 0, k = ok ? col - 9 * (col / 9) : 0;
    Column<double> C;
    column_setup<double, AN>(A, smeta + e * DGW_META, k0 + e, k, C);
    vel = k < 3;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      G::qf[m] = sq + (e * 9 + C.f[m]) * G::Np;
      G::cs[1][m] = C.c[1][m] + C.c[2][m];
      G::cs[2][m] = C.c[0][m] + C.c[2][m];
      G::cs[3][m] = C.c[0][m] + C.c[1][m];
      G::fl[m] = sfl + (e * 6 + (vel ? k : 3 + C.f[m])) * G::ROW;
    }
  }

  // a stress column's flux on face n is sum_m cf[n][m] dv_m with the same
  // coefficients as its volume term on Fscale_n n_n = -4 grad lambda_n, the
  // transform of cs; a velocity column's flux is stored as it is
  __device__ __forceinline__ void lift(const double *ops, double *sop, int tid) {
    G::lift(ops, sop, tid, [&](double (&cf)[4][3]) {
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        const double c[4] = {0.0, G::cs[1][m], G::cs[2][m], G::cs[3][m]};
        double t[4];
        sym4(c, t);
#pragma unroll
        for (int n = 0; n < 4; ++n) cf[n][m] = vel ? (double)(m == 0) : t[n];
      }
    });
  }
  // right-hand side to LDS in the block's (element, field, node) order
  __device__ __forceinline__ void store(double *out) const {
    G::store(out + G::column() * G::Np, ok);
  }
};

// Face tables of a block for this thread's face items: the packed
// connectivity code and, for interior faces, the neighbour trace's offset
// in the shot's field array.  Loaded ahead of the gathers (by the persistent
// form one block early).  Both tables are read unconditionally (the index is
// clamped into the block) so every table load is in flight at once.
template <int N, int BE>
struct FaceTab {
  static constexpr int FI = (BE * 4 * Sz<N>::Nfp + kThreads - 1) / kThreads;
  int cn[FI];
  int64_t gb[FI];
  int n1[FI];   // the face node's volume node in its own element
};

// SY: with each face's nodes in the order of their face-0 preimages (sym.h)
template <int N, typename real, int BE, bool SY>
__device__ __forceinline__ void face_tables(const StageArgs<real> &A, int64_t item,
                                            int64_t nblk, int64_t total,
                                            FaceTab<N, BE> &T) {
  constexpr int Np = Sz<N>::Np, Nfp = Sz<N>::Nfp, NF = 4 * Nfp;
  const int slot = slot_of(item, nblk, total);
  const int64_t k0 = (item - (int64_t)slot * nblk) * BE;
  const int nE = (int)((A.K - k0) < BE ? (A.K - k0) : BE);
  const uint8_t *nbn = SY ? A.nbsym : A.nbnode;
  const int32_t *own = SY ? A.fsym : A.fmask;
#pragma unroll
  for (int u = 0; u < FaceTab<N, BE>::FI; ++u) {
    const int t = threadIdx.x + u * kThreads;
    const bool ok = k0 < A.K && t < nE * NF;
    const int tt = ok ? t : 0;
    const int e = tt / NF, fm = tt - e * NF, f = fm / Nfp;
    const int64_t k = ok ? k0 + e : 0;
    const int cn = A.conn[k * 4 + f];
    const int nb = nbn[k * NF + fm];
    T.cn[u] = ok ? cn : CONN_ABSORB;
    T.n1[u] = own[fm];
    // masked arithmetic rather than a select, so the compiler keeps the
    // node-table load unconditional (not behind a wait for cn)
    const int64_t live = -(int64_t)(ok && cn >= 0);
    T.gb[u] = ((int64_t)(cn >> 5) * 9 * Np + nb) & live;
  }
}

// The block's own fields (16-byte vectors over its contiguous span, scalar
// head and tail) and per-element data, loaded into registers: every load is
// issued before any is waited for.
template <int N, typename real, int BE>
struct BlockLoad {
  using SP = Span16<real>;
  static constexpr int QV = (BE * 9 * Sz<N>::Np / SP::VW + kThreads - 1) / kThreads;
  static constexpr int MV = (BE * DGW_META / 2 + kThreads - 1) / kThreads;
  typename SP::vec q[QV];
  real qh, qt;
  double2 m[MV];
  double sg;   // damping rate of element tid of the block (threads < BE)
};

template <int N, typename real, int BE>
__device__ __forceinline__ void block_loads(const StageArgs<real> &A, int64_t item,
                                            int64_t nblk, int64_t total,
                                            BlockLoad<N, real, BE> &B) {
  constexpr int Np = Sz<N>::Np;
  using BL = BlockLoad<N, real, BE>;
  using SP = typename BL::SP;
  const int slot = slot_of(item, nblk, total);
  const int shot = A.shot_map ? A.shot_map[slot] : slot;
  const int64_t k0 = (item - (int64_t)slot * nblk) * BE;
  const int nE = (int)((A.K - k0) < BE ? (A.K - k0) : BE);
  const int tid = threadIdx.x;
  // every load is unconditional, with out-of-range lanes clamped to an
  // in-bounds index (their values are never stored): a load under a branch
  // makes the compiler's wait counting conservative, and the neighbour
  // gathers would wait for these loads
  const bool ok = k0 < A.K;
  const int64_t off = ok ? shot * A.shot_stride + k0 * 9 * Np : 0;
  const SP sp(off, ok ? nE * 9 * Np : 1);
  const real *src = A.q_in + off;
  const int nv1 = sp.nv > 0 ? sp.nv - 1 : 0;
  const typename SP::vec *sv = (const typename SP::vec *)(src + sp.hd);
#pragma unroll
  for (int u = 0; u < BL::QV; ++u) {
    const int j = tid + u * kThreads;
    B.q[u] = sv[j < sp.nv ? j : nv1];
  }
  B.qh = src[tid < sp.hd ? tid : 0];
  B.qt = src[tid < sp.tl ? sp.hd + SP::VW * sp.nv + tid : 0];
  const double2 *mv = (const double2 *)(A.meta + (ok ? k0 : 0) * DGW_META);
#pragma unroll
  for (int u = 0; u < BL::MV; ++u) {
    const int j = tid + u * kThreads;
    B.m[u] = mv[j < nE * DGW_META / 2 ? j : 0];
  }
  // the sponge rate: read unconditionally (from the per-element data when
  // there is no sponge, then discarded)
  const double *sgp = A.sponge ? A.sponge : A.meta;
  const double sgv = sgp[(ok ? k0 : 0) + (tid < nE ? tid : 0)];
  B.sg = A.sponge ? sgv : 0.0;
}

template <int N, typename real, int BE, int V>
constexpr bool kSymV = (V == 1 || V == 3) && kSymForm<N, real>;

// Exact Riemann flux of one face node: own trace from LDS, neighbour trace qp
// (registers), lifted quantities to LDS at d: six adjacent values (the
// node-per-thread forms), or at stride st six (symmetry components, dv without
// Fscale) or all nine components (nodal GEMM).
template <int N, typename real, int V>
__device__ __forceinline__ void face_flux(const StageArgs<real> &A, const real *qe,
                                          const double *g, int64_t k, int cn, int n1, int f,
                                          const real (&qp)[9], real *d, int st) {
  constexpr int Np = Sz<N>::Np;
  real qm[9], p[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) qm[c] = qe[c * Np + n1];
  if (cn >= 0) {
#pragma unroll
    for (int c = 0; c < 9; ++c) p[c] = qp[c];
  } else if (cn == CONN_FREE) {
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = qm[c];
#pragma unroll
    for (int c = 3; c < 9; ++c) p[c] = -qm[c];
  } else {
#pragma unroll
    for (int c = 0; c < 9; ++c) p[c] = (real)0;
  }
  const real nx = (real)g[M_NORMAL + 3 * f], ny = (real)g[M_NORMAL + 3 * f + 1],
             nz = (real)g[M_NORMAL + 3 * f + 2];
  // jumps [v] = v+ - v-, [t] = (sigma+ - sigma-) n
  const real dvx = p[0] - qm[0], dvy = p[1] - qm[1], dvz = p[2] - qm[2];
  const real dsxx = p[3] - qm[3], dsyy = p[4] - qm[4], dszz = p[5] - qm[5];
  const real dsyz = p[6] - qm[6], dsxz = p[7] - qm[7], dsxy = p[8] - qm[8];
  const real dtx = dsxx * nx + dsxy * ny + dsxz * nz;
  const real dty = dsxy * nx + dsyy * ny + dsyz * nz;
  const real dtz = dsxz * nx + dsyz * ny + dszz * nz;
  const real ri = (real)g[M_RHOINV], fs = (real)g[M_FSCALE + f];
  // traction change t* - t- (w) and velocity change dv = v* - v- (u) of
  // the flux states: tu times the exact Riemann states' plus (1 - tu)
  // times the central states' (half the jumps); tu = 1 (upwind) leaves
  // exactly the Riemann terms (1 x + 0 = x)
  const real tu = A.ftau, hc = ((real)1 - tu) * (real)0.5;
  real wx, wy, wz, ux, uy, uz;
  if constexpr (V == 2 || V == 3) {
    // anisotropic: dv = W ([t] + Z+ [v]) and t* - t- = Z- dv with the
    // face's impedance matrices (symmetric 3x3: xx yy zz yz xz xy)
    const double *za = A.aniso + k * DGW_ANI + A_FACE + A_FSTRIDE * f;
    auto smv = [](const double *Z, real x, real y, real z, real (&o)[3]) {
      const real xx = (real)Z[0], yy = (real)Z[1], zz = (real)Z[2], yz = (real)Z[3],
                 xz = (real)Z[4], xy = (real)Z[5];
      o[0] = xx * x + xy * y + xz * z;
      o[1] = xy * x + yy * y + yz * z;
      o[2] = xz * x + yz * y + zz * z;
    };
    real zj[3], dv[3], dtr[3];
    smv(za + A_ZP, dvx, dvy, dvz, zj);
    smv(za + A_W, dtx + zj[0], dty + zj[1], dtz + zj[2], dv);
    smv(za + A_ZM, dv[0], dv[1], dv[2], dtr);
    wx = tu * dtr[0] + hc * dtx;
    wy = tu * dtr[1] + hc * dty;
    wz = tu * dtr[2] + hc * dtz;
    ux = tu * dv[0] + hc * dvx;
    uy = tu * dv[1] + hc * dvy;
    uz = tu * dv[2] + hc * dvz;
  } else {
    const real dvn = dvx * nx + dvy * ny + dvz * nz;
    const real dtn = dtx * nx + dty * ny + dtz * nz;
    const real zp = (real)g[M_ZP], zs = (real)g[M_ZS];
    const real zpn = (real)g[M_ZPNB + f], zsn = (real)g[M_ZSNB + f];
    const real izp = (real)g[M_IZPS + f], izs = (real)g[M_IZSS + f];
    // normal and tangential Riemann amplitudes
    const real kn = (dtn + zpn * dvn) * izp;
    const real kTx = (dtx - dtn * nx + zsn * (dvx - dvn * nx)) * izs;
    const real kTy = (dty - dtn * ny + zsn * (dvy - dvn * ny)) * izs;
    const real kTz = (dtz - dtn * nz + zsn * (dvz - dvn * nz)) * izs;
    wx = tu * (zp * kn * nx + zs * kTx) + hc * dtx;
    wy = tu * (zp * kn * ny + zs * kTy) + hc * dty;
    wz = tu * (zp * kn * nz + zs * kTz) + hc * dtz;
    ux = tu * (kn * nx + kTx) + hc * dvx;
    uy = tu * (kn * ny + kTy) + hc * dvy;
    uz = tu * (kn * nz + kTz) + hc * dvz;
  }
  // velocity flux (t* - t-)/rho and the velocity change dv; the stress
  // flux is lambda (n.dv) I + mu (dv n^T + n dv^T) (anisotropic: C N(n) dv)
  // with n constant on the face, so lifting dv is enough for all six
  // stress components
  if constexpr (kSymV<N, real, 1, V>) {
    d[0 * st] = fs * wx * ri;
    d[1 * st] = fs * wy * ri;
    d[2 * st] = fs * wz * ri;
    d[3 * st] = ux;
    d[4 * st] = uy;
    d[5 * st] = uz;
  } else if constexpr (V == 0 || V == 2) {
    d[0] = fs * wx * ri;
    d[1] = fs * wy * ri;
    d[2] = fs * wz * ri;
    d[3] = fs * ux;
    d[4] = fs * uy;
    d[5] = fs * uz;
  } else {
    // all nine lifted components, field-major (the GEMM's data side)
    const real Dvx = fs * ux, Dvy = fs * uy, Dvz = fs * uz;
    d[0 * st] = fs * wx * ri;
    d[1 * st] = fs * wy * ri;
    d[2 * st] = fs * wz * ri;
    if constexpr (V == 3) {
      // C N(n) dv
      const real ev[6] = {nx * Dvx, ny * Dvy, nz * Dvz, nz * Dvy + ny * Dvz,
                          nz * Dvx + nx * Dvz, ny * Dvx + nx * Dvy};
      const double *Cu = A.aniso + k * DGW_ANI + A_C;
      real cm[6][6];
      int uu = 0;
#pragma unroll
      for (int a = 0; a < 6; ++a)
#pragma unroll
        for (int b = a; b < 6; ++b) cm[a][b] = cm[b][a] = (real)Cu[uu++];
#pragma unroll
      for (int a = 0; a < 6; ++a) {
        real acc = 0;
#pragma unroll
        for (int b = 0; b < 6; ++b) acc += cm[a][b] * ev[b];
        d[(3 + a) * st] = acc;
      }
    } else {
      const real la = (real)g[M_LAM], mu = (real)g[M_MU];
      const real ndv = nx * Dvx + ny * Dvy + nz * Dvz;
      d[3 * st] = la * ndv + 2 * mu * Dvx * nx;
      d[4 * st] = la * ndv + 2 * mu * Dvy * ny;
      d[5 * st] = la * ndv + 2 * mu * Dvz * nz;
      d[6 * st] = mu * (Dvy * nz + Dvz * ny);
      d[7 * st] = mu * (Dvx * nz + Dvz * nx);
      d[8 * st] = mu * (Dvx * ny + Dvy * nx);
    }
  }
}

template <int N, typename real, int BE, int V>
__device__ __forceinline__ void stage_item(const StageArgs<real> &A, int64_t item,
                                           int64_t nblk, int64_t total,
                                           const FaceTab<N, BE> &T,
                                           const BlockLoad<N, real, BE> &B) {
  constexpr int Np = Sz<N>::Np, Nfp = Sz<N>::Nfp, NF = 4 * Nfp;
  constexpr bool SY = kSymV<N, real, BE, V>;
  constexpr int FI = FaceTab<N, BE>::FI;      // face items per thread
  // flux row of an (element, field) in the matrix-core forms
  constexpr int ROW = SY ? NF | 1 : NF;
  // lifted flux, and in the matrix-core forms then the right-hand side
  constexpr int FL = SY ? 6 * ROW : V == 1 || V == 3 ? 9 * NF : 6 * NF;
  constexpr int SF = BE * (SY && FL < 9 * Np ? 9 * Np : FL);
  // declared here (not passed in) so every access stays an LDS access
  __shared__ real sq[BE * 9 * Np];
  __shared__ __attribute__((aligned(16))) real sfl[SF];
  __shared__ double smeta[BE * DGW_META];
  __shared__ double ssig[BE];
  // the matrix-core form's GEMM
  constexpr bool MC = V == 1 || V == 3;
  using GM = std::conditional_t<SY, StageGemm<N, SY ? BE : 1, V == 3>,
                                NodalGemm<N, real, MC && !SY ? BE : 1, V == 3>>;
  __shared__ __attribute__((aligned(16))) real sop[MC ? GM::OPS : 4];
  const int slot = slot_of(item, nblk, total);
  const int shot = A.shot_map ? A.shot_map[slot] : slot;
  const int64_t step = A.shot_step[shot];
  const int64_t src = A.src_elem[shot];
  if (step >= A.shot_len[shot]) return;            // uniform per work-group
  const int64_t k0 = (item - (int64_t)slot * nblk) * BE;
  // never taken (items cover the mesh exactly), but it bounds nE to
  // [1, BE] for the compiler, which keeps the register count low
  if (k0 >= A.K) return;
  const int nE = (int)((A.K - k0) < BE ? (A.K - k0) : BE);
  const real *__restrict__ qin = A.q_in + shot * A.shot_stride;
  real *__restrict__ qout = A.q_out + shot * A.shot_stride;
  real *__restrict__ res = A.res + shot * A.shot_stride;
  const int tid = threadIdx.x;
  // an opaque zero added to the operator addresses: in the persistent form
  // the compiler would otherwise hoist every operator load (they depend on
  // the thread only) out of the item loop, far beyond the register file
  int oz;
  asm volatile("v_mov_b32 %0, 0" : "=v"(oz));

  // ---- 1. all global reads of the item's fields are in flight together ----
  // neighbour traces of this thread's face nodes go to registers; read
  // unconditionally (boundary and idle face items have offset 0, an
  // in-bounds read of the first element that is never used), so no branch
  // makes the compiler wait on earlier loads
  // the first operator chunk
  std::remove_reference_t<decltype(GM::op)> opv[GM::OV];
  const real *ops = SY ? A.Asym : A.Anod;
  if constexpr (MC) GM::load_ops(ops, 0, tid, opv);
  real qp[FI][9];
#pragma unroll
  for (int u = 0; u < FI; ++u) {
#pragma unroll
    for (int c = 0; c < 9; ++c) qp[u][c] = qin[T.gb[u] + c * Np];
  }
  // From order 3 on the matrix-core forms read their operators from LDS, so
  // nothing waits behind the residual and it is loaded here.
  Update<N, real, BE> U;
  if constexpr (MC && N >= 3) U.load(A, k0, shot, nE, qout, res, tid);
  // the block's own fields and per-element data (loads issued by
  // block_loads) to LDS
  {
    using BL = BlockLoad<N, real, BE>;
    using SP = typename BL::SP;
    const SP sp(shot * A.shot_stride + k0 * 9 * Np, nE * 9 * Np);
#pragma unroll
    for (int u = 0; u < BL::QV; ++u) {
      const int j = tid + u * kThreads;
      if (j < sp.nv)
#pragma unroll
        for (int l = 0; l < SP::VW; ++l) sq[sp.hd + SP::VW * j + l] = B.q[u][l];
    }
    if (tid < sp.hd) sq[tid] = B.qh;
    if (tid < sp.tl) sq[sp.hd + SP::VW * sp.nv + tid] = B.qt;
#pragma unroll
    for (int u = 0; u < BL::MV; ++u) {
      const int j = tid + u * kThreads;
      if (j < nE * DGW_META / 2) {
        smeta[2 * j] = B.m[u].x;
        smeta[2 * j + 1] = B.m[u].y;
      }
    }
    if (tid < nE) ssig[tid] = B.sg;
    if constexpr (MC) GM::store_ops(sop, 0, tid, opv);
  }
  __syncthreads();

  // ---- 2. faces: exact Riemann flux ----
  // the nodes of this lane's orbits (sym.h) or rows (nodal.h), four to a word
  constexpr int TW = SY ? Sym<N>::KS : Nodal<N>::MT;
  uint32_t nodes[TW];
  if constexpr (MC) {
    const uint32_t *tab = SY ? A.symnode : A.rowtab;
#pragma unroll
    for (int u = 0; u < TW; ++u) nodes[u] = tab[4 * u + ((tid & 63) >> 4)];
  }
  auto flux = [&] {
#pragma unroll
    for (int u = 0; u < FI; ++u) {
      const int t = tid + u * kThreads;
      if (t >= nE * NF) continue;
      const int e = t / NF, fm = t - e * NF;
      real *d = V == 0 || V == 2 ? sfl + t * 6 : sfl + e * (SY ? 6 : 9) * ROW + fm;
      face_flux<N, real, V>(A, sq + e * 9 * Np, smeta + e * DGW_META, k0 + e, T.cn[u], T.n1[u],
                            fm / Nfp, qp[u], d, ROW);
    }
  };
  // ---- 3. volume, lift, update ----
  if constexpr (MC) {
    // In FP32 from order 4 on the flux, which waits for the neighbour traces,
    // runs after the volume (order 4, 82944 elements, 162 -> 158 us).  FP64 has
    // no registers to hold the traces that long (order 3 spills, order 4 loses
    // a work-group a CU), and below order 4 nothing is gained.
    constexpr bool late = V == 1 && N >= 4 && sizeof(real) == 4;
    if constexpr (!late) flux();
    GM G(A, sq, sfl, sop, smeta, nE, k0, nodes, tid);
    G.volume(ops, sop, tid);
    if constexpr (late) flux();
    __syncthreads();
    G.lift(ops, sop, tid);
    if constexpr (N < 3) U.load(A, k0, shot, nE, qout, res, tid);
    __syncthreads();   // every wave is done with the flux buffer
    G.store(sfl);
    __syncthreads();
    U.apply(A, sq, sfl, ssig, nE, src - k0, shot, step, tid);
  } else {
    flux();
    __syncthreads();
    phase3_nodes<N, real, BE, V == 2>(A, sq, sfl, smeta, ssig, nE, k0, shot, step, qout, res,
                                      oz, tid);
  }
}

// Waves per SIMD that the registers have to leave room for.  At order 3 in FP64
// the LDS holds four work-groups a CU: with 128 registers instead of 136 they
// fit (48 -> 45 us, 24576 elements).  At order 4 it holds three, which the
// registers do anyway.
template <int N, typename real, int V>
constexpr int kWaves = V == 1 && N == 3 && sizeof(real) == 8 ? 4 : 1;

// One work-group per item.
template <int N, typename real, int BE, int V>
__global__ void __launch_bounds__(kThreads, (kWaves<N, real, V>))
stage_kernel(StageArgs<real> A, int64_t nblk, int64_t total) {
  const int64_t item = xcd_item(blockIdx.x, total);
  FaceTab<N, BE> T;
  face_tables<N, real, BE, kSymV<N, real, BE, V>>(A, item, nblk, total, T);
  BlockLoad<N, real, BE> B;
  block_loads<N, real, BE>(A, item, nblk, total, B);
  stage_item<N, real, BE, V>(A, item, nblk, total, T, B);
}

// Persistent grid (a multiple of 8 work-groups) looping over the items;
// the next item's face tables are loaded while the current one is processed.
template <int N, typename real, int BE, int V>
__global__ void __launch_bounds__(kThreads)
stage_kernel_persistent(StageArgs<real> A, int64_t nblk, int64_t total) {
  int64_t L = blockIdx.x;
  FaceTab<N, BE> T;
  if (L < total) face_tables<N, real, BE, kSymV<N, real, BE, V>>(A, xcd_item(L, total), nblk, total, T);
  for (; L < total; L += gridDim.x) {
    const int64_t item = xcd_item(L, total);
    FaceTab<N, BE> Tn;
    if (L + gridDim.x < total)
      face_tables<N, real, BE, kSymV<N, real, BE, V>>(A, xcd_item(L + gridDim.x, total), nblk, total, Tn);
    BlockLoad<N, real, BE> B;
    block_loads<N, real, BE>(A, item, nblk, total, B);
    stage_item<N, real, BE, V>(A, item, nblk, total, T, B);
    __syncthreads();   // LDS is reused by the next item
    T = Tn;
  }
}

// Elements per work-group for variant V: the largest BE with one thread per
// element node (V = 0, 2: BE * Np <= 256) or one MFMA column per (element,
// field) (V = 1, 3: 9 BE <= 64, four waves of 16 columns) for which the fields,
// the lifted quantities (six per face node, nine in V = 1 and 3) and the
// per-element data take at most 64 KB; and half of it.  That sum was the
// nodal form's LDS in FP64 when its operators came from L2, and the blocks are
// part of the launch shapes that callers set and tuners store, so it stays
// the rule; it is not the LDS of every form.  The symmetry components
// store six quantities and stage their operators beside them (order 4, 7
// elements, 53,176 bytes; order 5, 6 elements, 63,312; order 6, 4 elements,
// 69,920), the FP32 nodal form stages its fragments (order 4, 14 elements,
// 65,664; order 6, 7 elements, 70,568).
template <int N, typename real, int V>
struct Shapes {
  static constexpr int Np = Sz<N>::Np, NF = 4 * Sz<N>::Nfp;
  static constexpr int per =
      (9 * Np + (V == 1 || V == 3 ? 9 : 6) * NF) * (int)sizeof(real) + DGW_META * 8;
  static constexpr int cap1 =
      V == 0 || V == 2 ? kThreads / Np : kThreads / 64 * 16 / 9;
  static constexpr int cap2 = 65536 / per;
  static constexpr int a0 = cap1 < cap2 ? cap1 : cap2;
  // matrix-core FP32: two column tiles per wave (14 elements), both fed from
  // each operator fragment, where the sum above allows it, and the one-tile
  // block as the second choice
  static constexpr bool two = (V == 1 || V == 3) && sizeof(real) == 4 && cap2 >= 2 * cap1;
  static constexpr int a = two ? 2 * cap1 : a0;
  static constexpr int b = two ? cap1 : (a0 / 2 > 0 ? a0 / 2 : 1);
};

template <int N, typename real, int BE, int V>
void launch_be(int64_t grid, bool persistent, int64_t nblk, int64_t total,
               const StageArgs<real> &a, hipStream_t st) {
  if (persistent)
    hipLaunchKernelGGL((stage_kernel_persistent<N, real, BE, V>), dim3((unsigned)grid),
                       dim3(kThreads), 0, st, a, nblk, total);
  else
    hipLaunchKernelGGL((stage_kernel<N, real, BE, V>), dim3((unsigned)grid),
                       dim3(kThreads), 0, st, a, nblk, total);
}

template <int N, typename real, int V>
hipError_t launch_t(int be, int wpc, int ncu, int nshots, const StageArgs<real> &a,
                    hipStream_t st) {
  constexpr int A_ = Shapes<N, real, V>::a, B_ = Shapes<N, real, V>::b;
  if (be != A_ && be != B_) return hipErrorInvalidValue;
  if ((V == 1 || V == 3) && (kSymForm<N, real> ? a.Asym == nullptr || a.nbsym == nullptr
                                             : a.Anod == nullptr || a.rowtab == nullptr))
    return hipErrorInvalidValue;
  const int64_t nblk = (a.K + be - 1) / be;
  const int64_t total = nblk * nshots;
  const int64_t pers = ((int64_t)ncu * wpc + 7) / 8 * 8;
  const bool persistent = wpc > 0 && pers < total;
  const int64_t grid = persistent ? pers : total;
  if (be == A_)
    launch_be<N, real, A_, V>(grid, persistent, nblk, total, a, st);
  else
    launch_be<N, real, B_, V>(grid, persistent, nblk, total, a, st);
  return hipGetLastError();
}

template <typename real, int V>
hipError_t launch_r(int N, int be, int wpc, int ncu, int nshots, const void *args,
                    hipStream_t st) {
  const StageArgs<real> &a = *(const StageArgs<real> *)args;
  switch (N) {
    case 1: return launch_t<1, real, V>(be, wpc, ncu, nshots, a, st);
    case 2: return launch_t<2, real, V>(be, wpc, ncu, nshots, a, st);
    case 3: return launch_t<3, real, V>(be, wpc, ncu, nshots, a, st);
    case 4: return launch_t<4, real, V>(be, wpc, ncu, nshots, a, st);
    case 5: return launch_t<5, real, V>(be, wpc, ncu, nshots, a, st);
    case 6: return launch_t<6, real, V>(be, wpc, ncu, nshots, a, st);
  }
  return hipErrorInvalidValue;
}

template <typename real, int V>
std::vector<int> choices_r(int N) {
  switch (N) {
    case 1: return {Shapes<1, real, V>::a, Shapes<1, real, V>::b};
    case 2: return {Shapes<2, real, V>::a, Shapes<2, real, V>::b};
    case 3: return {Shapes<3, real, V>::a, Shapes<3, real, V>::b};
    case 4: return {Shapes<4, real, V>::a, Shapes<4, real, V>::b};
    case 5: return {Shapes<5, real, V>::a, Shapes<5, real, V>::b};
    case 6: return {Shapes<6, real, V>::a, Shapes<6, real, V>::b};
  }
  return {};
}

}  // namespace

hipError_t launch_stage(int kernel, int N, int precision, int be, int wpc, int ncu,
                        int nshots, const void *args, hipStream_t st) {
  if (!stage_kernel_supported(kernel, N, precision)) return hipErrorInvalidValue;
  if (kernel == 2) {
    if (be != stage_split_block() || wpc != 0) return hipErrorInvalidValue;
    return launch_stage_split(N, precision, nshots, args, st);
  }
  if (kernel == 0 && stage_zero_is_one(N, precision)) {
    const std::vector<int> own = stage_block_choices(0, N, precision),
                           one = stage_block_choices(1, N, precision);
    if (std::find(own.begin(), own.end(), be) == own.end()) return hipErrorInvalidValue;
    kernel = 1;
    const int64_t elems = ((const StageArgs<double> *)args)->K * nshots;
    be = 3 * ((elems + one[0] - 1) / one[0]) < ncu ? one[1] : one[0];
  }
  // anisotropic elements: instantiations 2 (node per thread) and 3 (matrix
  // cores)
  const bool an = precision == 64 ? ((const StageArgs<double> *)args)->aniso != nullptr
                                  : ((const StageArgs<float> *)args)->aniso != nullptr;
  if (an) {
    if (precision == 64)
      return kernel == 0 ? launch_t<1, double, 2>(be, wpc, ncu, nshots,
                                                  *(const StageArgs<double> *)args, st)
                         : launch_r<double, 3>(N, be, wpc, ncu, nshots, args, st);
    return kernel == 0 ? launch_r<float, 2>(N, be, wpc, ncu, nshots, args, st)
                       : launch_r<float, 3>(N, be, wpc, ncu, nshots, args, st);
  }
  if (precision == 64)
    return kernel == 0 ? launch_t<1, double, 0>(be, wpc, ncu, nshots,
                                                *(const StageArgs<double> *)args, st)
                       : launch_r<double, 1>(N, be, wpc, ncu, nshots, args, st);
  return kernel == 0 ? launch_r<float, 0>(N, be, wpc, ncu, nshots, args, st)
                     : launch_r<float, 1>(N, be, wpc, ncu, nshots, args, st);
}

// Kernel 0 in FP64 from order 2 runs kernel 1's code (each element's results do
// not depend on the block): the node-per-thread form is slower there at every
// size.  Stage launch, node per thread -> kernel 1: order 2, 55566 elements, 58
// -> 54 us, 384 elements 10.8 -> 7.7; order 3, 384 elements, 14.9 -> 9.4, 7986
// elements 26 -> 23; order 4, 82944 elements, 433 -> 212; order 6, 7986
// elements, 151 -> 78.  The larger block, but the smaller one where that
// leaves two thirds of the CUs without a work-group (order 4, 384 elements,
// 12.0 -> 10.7 us; 1296 elements 12.9 against 13.7).  Order 1 keeps it: 30
// against 35 us at 55566 elements.
bool stage_zero_is_one(int N, int precision) { return precision == 64 && N >= 2; }

bool stage_kernel_supported(int kernel, int N, int precision) {
  if (kernel == 2) return stage_split_supported(N, precision);
  return (kernel == 0 || kernel == 1) && N >= 1 && N <= DGW_MAX_ORDER &&
         (precision == 64 || precision == 32);
}

std::vector<int> stage_block_choices(int kernel, int N, int precision) {
  if (kernel == 2)
    return stage_split_supported(N, precision) ? std::vector<int>{stage_split_block()}
                                               : std::vector<int>{};
  if (kernel == 1) return precision == 64 ? choices_r<double, 1>(N) : choices_r<float, 1>(N);
  if (kernel == 0) return precision == 64 ? choices_r<double, 0>(N) : choices_r<float, 0>(N);
  return {};
}

int default_block(int kernel, int N, int precision) {
  std::vector<int> c = stage_block_choices(kernel, N, precision);
  return c.empty() ? 0 : c[0];
}

}  // namespace dgw

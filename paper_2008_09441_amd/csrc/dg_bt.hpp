// Fused DG elastic-wave stage for orders 5-7 on tiles of 16 elements (gfx950).
//
// At these orders the operators (0.2-0.8 MB of split fragments) are larger
// than the data of an element, so what bounds a stage is how often their
// fragments are read.  One workgroup owns 16 consecutive elements, the columns
// of every v_mfma_f32_16x16x32_bf16 product, so that a fragment serves 16
// elements; the column is the element in every accumulator, and the chain rule,
// the material operator and the trace stay within a lane.  Waves own 16-row
// node tiles of LIFT and the derivatives, and groups of components in the
// quadrature.
//
// Products are split products of P bf16 parts per operand, A B as the sum of
// the leading part products with FP32 accumulation.  P = 2 (BF16x3: hi hi,
// hi lo, lo hi) and P = 3 (FP32: three parts hold every bit of an FP32 value; six
// of the nine part products, see kProd in dg_bx.hpp, of 16 cycles each per 32 K
// slots against eight of 32 for v_mfma_f32_16x16x4_f32).  With three parts,
// elements of odd index carry the opposite sign from their fluxes and metric terms
// to the result, so that what the products cut off downwards (kProd) does not add
// up over the steps of a run.
//
// Measured against one element per workgroup (dg_be.hpp), us per stage on
// 24,576 elements: BF16x3 order 5 307 -> 109, order 6 593 -> 292, order 7
// 926 -> 402; FP32 order 5 464 -> 173, order 6 1006 -> 376.  The relative error
// of an FP32 right-hand side of a smooth state against FP64 went from 1.23e-6 to
// 6.9e-7 (order 5) and from 1.77e-6 to 9.5e-7 (order 6).
// What bounds it now (order 7, cycles of a workgroup's 151,000): state and
// neighbour loads 21,000, fluxes 18,000, LIFT and derivatives 23,000 (22
// cycles a product on a SIMD that could start one every 16), quadrature 65,000
// (fragment reads through the L1, 8 of 64 KiB each K step, and products),
// parts and update 25,000.  Registers (8 waves of 244) and LDS leave one
// workgroup per CU at orders 6 and 7, so the memory phases overlap with
// nothing.  Tried and slower or equal: quadrature rows split over the waves
// with the weighted values exchanged through LDS (order 5 110, order 6 322,
// order 7 375), eight fragments in flight instead of four (432 at order 7).
//
// The B operands live in LDS, split once by whoever produces them, as
// [component][K step][part][64 lanes][8] in the lane order of the product, so
// that a wave reads 16 bytes per lane without bank conflicts; lane (g, e) of K
// step s sits at 16 g + (e ^ (4 (s % 4) + g)), which spreads the stores of
// consecutive rows of one element over the banks.
// Phases, with a workgroup barrier after each:
//   1  the state in FP32 in LDS, face fluxes [WSG10] from its traces and the
//      gathered neighbour traces, one thread per face node, then the fluxes
//      into LDS (over the state);
//   2  r = LIFT f [HW08, Ch. 10];
//   3  the state, split, into LDS (over the fluxes);
//   4  D_r q, D_s q, D_t q of the nine fields, chain rule: r += ...;
//   5  r into LDS (over the state);
//   6  V_q r, the weight-adjusted material operator [CHW17, C18] and P_q per
//      wave, for one group of components and one part of the points;
//   7  the parts summed, right-hand side store or LSRK(5,4) update [CK94].
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dg_be.hpp"

namespace dgb {

// a float4 in memory at any 4-byte alignment (the caller's states need no more)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// loads and stores at a lane's 32-bit byte offset from a uniform base (a 64-bit
// address per lane and access would take two registers each)
template <typename V>
__device__ __forceinline__ V bt_ld(const void* base, unsigned off) {
  return *reinterpret_cast<const V*>(static_cast<const char*>(base) + off);
}
// four floats at any 4-byte alignment (a template argument would drop the
// alignment of the type)
__device__ __forceinline__ f32x4 bt_ldu(const void* base, unsigned off) {
  return *reinterpret_cast<const f32x4u*>(static_cast<const char*>(base) + off);
}
__device__ __forceinline__ void bt_stu(void* base, unsigned off, const f32x4& v) {
  *reinterpret_cast<f32x4u*>(static_cast<char*>(base) + off) = v;
}

// a workgroup barrier that no instruction moves across (conversions and cleared
// accumulators of the next phase would otherwise fill the registers of this one)
__device__ __forceinline__ void bt_sync() {
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();
  __builtin_amdgcn_sched_barrier(0);
}

template <int N, int P>
struct TOrd {
  static constexpr int Np = (N + 1) * (N + 2) * (N + 3) / 6;
  static constexpr int Nfp = (N + 1) * (N + 2) / 2;
  static constexpr int NF4 = 4 * Nfp;
  static constexpr int Nq = (N + 1) * (N + 1) * (N + 1);
  static constexpr int RT = (Np + 15) / 16;         // node row tiles
  static constexpr int KN = (Np + 31) / 32;         // K steps over nodes
  static constexpr int KF = (NF4 + 31) / 32;        // K steps over face nodes
  static constexpr int KQ = (Nq + 31) / 32;         // K steps over quadrature points
  // LIFT and derivatives: one node tile per wave, split into DH groups of
  // components (2: the strains from the velocities, and the velocity rows
  // from the stresses), to fill the SIMDs where LDS leaves one workgroup per CU
  static constexpr int DH = N == 5 && P == 3 ? 2 : 1;
  static constexpr int WV = RT * DH;                // waves
  static constexpr int TH = 64 * WV;
  // quadrature: G groups of components times QH parts of the points
  static constexpr int G = WV % 4 == 0 ? 4 : 3;
  static constexpr int QH = WV / G;
  static_assert(WV == G * QH && QH <= 2 && RT % QH == 0, "waves cover the components");
  static_assert(Np % 4 == 0, "lanes hold four nodes");
  // the state stays in registers from phase 1 to phase 3 where they suffice
  static constexpr bool KEEPQ = N == 5;
  // fragments of P parts (the layout of EOrd at P = 2)
  static constexpr int OFF_D = 0;
  static constexpr int OFF_L = OFF_D + 3 * RT * KN;
  static constexpr int OFF_V = OFF_L + RT * KF;
  static constexpr int OFF_P = OFF_V + 2 * KQ * KN;
  static constexpr int NFRAG = P * (OFF_P + RT * KQ);   // of 64 lanes x 16 bytes
  // LDS, in 16-byte units: the FP32 state [9][16][Np], the fluxes, the split
  // state and then r, the partial results of the two parts of the points
  static constexpr int LQ = 9 * kTile * Np / 4;
  static constexpr int LF = 9 * KF * P * 64;
  static constexpr int LN = 9 * KN * P * 64;
  static constexpr int LX = QH == 2 ? 9 * RT * 64 : 0;
  static constexpr int LM = LQ > LF ? LQ : LF, LO = LN > LX ? LN : LX;
  static constexpr int USED = 16 * (LM > LO ? LM : LO);
  // padded as the other stage kernels are: the workgroups of a CU never use
  // more than 128 KiB of LDS together
  static constexpr int FLOOR =
      USED <= 43690 ? 40976 : USED <= 65536 ? 54630 : USED <= 81920 ? 81936 : 0;
  static constexpr int BYTES = USED > FLOOR ? USED : FLOOR;
  static_assert(BYTES <= 131072, "LDS of one workgroup");
};

// components of group grp of G groups (the trace couples the normal stresses
// 3-5): {0,1 | 2,6 | 3,4,5 | 7,8} or {0,1,2 | 3,4,5 | 6,7,8}.  The group is a
// wave's own, uniform value.
__device__ __forceinline__ int bt_comp(int G, int grp, int i) {
  return G == 3 ? 3 * grp + i : grp == 1 ? (i == 0 ? 2 : 6) : (grp == 0 ? 0 : grp == 2 ? 3 : 7) + i;
}

// LIFT and derivatives, group h of DH: components C0 ... C0 + NC - 1 from the
// fields F0 ... F0 + NF - 1
struct BtRole {
  int c0, nc, f0, nf;
};
__host__ __device__ constexpr BtRole bt_role(int DH, int h) {
  return DH == 1 ? BtRole{0, 9, 0, 9} : h == 0 ? BtRole{3, 6, 0, 3} : BtRole{0, 3, 3, 6};
}

template <int P>
__device__ __forceinline__ void bt_split(const float* v, int n, __bf16 (&o)[P]) {
  float r = v[n];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    o[p] = __bf16(r);
    r -= float(o[p]);
  }
}

template <int P>
__device__ __forceinline__ void bt_frag(const FragBuf& F, int f, u32x4 (&a)[P]) {
#pragma unroll
  for (int p = 0; p < P; ++p)
    a[p] = F.load(f * P + p);
}

// B operand of component c, K step s (of KS) from a buffer; l0 = 16 g + (e ^ g)
template <int P>
__device__ __forceinline__ void bt_bread(const bf16x8* buf, int KS, int c, int s, int l0,
                                         bf16x8 (&b)[P]) {
#pragma unroll
  for (int p = 0; p < P; ++p) b[p] = buf[((c * KS + s) * P + p) * 64 + (l0 ^ (4 * (s & 3)))];
}

// Items j < NJ of a phase in order: each reads the B operand parts of GS
// components (or fields) and multiplies.  The reads run one item ahead and no
// further (left alone, the scheduler hoists them until registers spill); an
// item's products go part by part over all of its accumulators, since a
// product that takes the accumulator of the one before it waits for it.
template <int NJ, int GS, int P, typename BRead, typename Mul>
__device__ __forceinline__ void bt_pipe(BRead bread, Mul mul) {
  bf16x8 b[2][GS][P];
  bread(0, b[0]);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (j + 1 < NJ) bread(j + 1, b[(j + 1) & 1]);
    mul(j, b[j & 1]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// four consecutive rows (16 t + 4 g + j, j < 4) of component c and column e
// into a buffer of KS K steps
template <int P>
__device__ __forceinline__ void bt_put4(bf16x8* buf, int KS, int c, int t, int g, int e,
                                        const f32x4& v) {
  const int s = t >> 1, gb = 2 * (t & 1) + (g >> 1);
  const int at = 16 * gb + (e ^ (4 * (s & 3) + gb));
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  f32x4 r = v;
  bf16x4 o[P];
#pragma unroll
  for (int p = 0; p < P; ++p) {
    o[p] = __builtin_convertvector(r, bf16x4);
    r -= __builtin_convertvector(o[p], f32x4);
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    reinterpret_cast<bf16x4*>(buf + ((c * KS + s) * P + p) * 64 + at)[g & 1] = o[p];
}

// LIFT f and the derivatives at one node tile t for the components of group h:
// r[i] += rows 4 g + j of component C0 + i
template <int N, int P, int H>
__device__ __forceinline__ void bt_lift(const FragBuf& F, const bf16x8* sf, int t, int l0,
                                        f32x4 (&r)[9]) {
  using O = TOrd<N, P>;
  constexpr BtRole R = bt_role(O::DH, H);
#pragma unroll
  for (int c = 0; c < R.nc; ++c) r[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 fa[2][P];
  bt_frag<P>(F, O::OFF_L + t * O::KF, fa[0]);
  constexpr int GS = 3, NG = R.nc / GS;
  bt_pipe<O::KF * NG, GS, P>(
      [&](int j, bf16x8(&b)[GS][P]) {
#pragma unroll
        for (int k = 0; k < GS; ++k)
          bt_bread<P>(sf, O::KF, R.c0 + j % NG * GS + k, j / NG, l0, b[k]);
      },
      [&](int j, const bf16x8(&b)[GS][P]) {
        const int s = j / NG;
        if (j % NG == 0 && s + 1 < O::KF)
          bt_frag<P>(F, O::OFF_L + t * O::KF + s + 1, fa[(s + 1) & 1]);
#pragma unroll
        for (int x = 0; x < kProd<P>; ++x)
#pragma unroll
          for (int k = 0; k < GS; ++k) {
            const int c = j % NG * GS + k;
            r[c] = mma(fa[s & 1][prod_a(P, x)], b[k][prod_b(P, x)], r[c]);
          }
      });
}

// D_r q, D_s q, D_t q of the group's fields, then the chain rule
// r_c += sum_d sum_j G_dj w(c, j) D_d q_{f(c,j)}
template <int N, int P, int H>
__device__ __forceinline__ void bt_deriv(const FragBuf& F, const bf16x8* sn, int t, int l0,
                                         const float (&Ge)[9], f32x4 (&r)[9]) {
  using O = TOrd<N, P>;
  constexpr BtRole R = bt_role(O::DH, H);
  constexpr int RT = O::RT, KN = O::KN;
  f32x4 d[3][R.nf];
#pragma unroll
  for (int x = 0; x < 3; ++x)
#pragma unroll
    for (int f = 0; f < R.nf; ++f) d[x][f] = f32x4{0.f, 0.f, 0.f, 0.f};
  // one K step ahead, registers allowing
  constexpr int NB = P == 3 && O::DH == 1 ? 1 : 2;
  u32x4 fa[NB][3][P];
#pragma unroll
  for (int x = 0; x < 3; ++x) bt_frag<P>(F, O::OFF_D + (x * RT + t) * KN, fa[0][x]);
  // with three parts, the five small products of every K step come before the
  // leading product of any: the accumulators then round at full size KN times,
  // not 6 KN times (a derivative's sum cancels, so its roundings weigh most)
  constexpr int NY = P == 3 ? kProd<P> - 1 : kProd<P>;
  bt_pipe<KN * R.nf, 1, P>(
      [&](int j, bf16x8(&b)[1][P]) { bt_bread<P>(sn, KN, R.f0 + j % R.nf, j / R.nf, l0, b[0]); },
      [&](int j, const bf16x8(&b)[1][P]) {
        const int f = j % R.nf, s = j / R.nf;
        auto next = [&]() {
#pragma unroll
          for (int x = 0; x < 3; ++x)
            bt_frag<P>(F, O::OFF_D + (x * RT + t) * KN + s + 1, fa[(s + 1) % NB][x]);
        };
        if (NB == 2 && f == 0 && s + 1 < KN) next();
#pragma unroll
        for (int y = 0; y < NY; ++y)
#pragma unroll
          for (int x = 0; x < 3; ++x)
            d[x][f] = mma(fa[s % NB][x][prod_a(P, y)], b[0][prod_b(P, y)], d[x][f]);
        if (NB == 1 && f == R.nf - 1 && s + 1 < KN) next();
      });
  if constexpr (P == 3) {
    u32x4 fh[KN][3];
#pragma unroll
    for (int s = 0; s < KN; ++s)
#pragma unroll
      for (int x = 0; x < 3; ++x)
        fh[s][x] = F.load((O::OFF_D + (x * RT + t) * KN + s) * P);
    bt_pipe<KN * R.nf, 1, 1>(
        [&](int j, bf16x8(&b)[1][1]) {
          b[0][0] = sn[((R.f0 + j % R.nf) * KN + j / R.nf) * P * 64 + (l0 ^ (4 * (j / R.nf & 3)))];
        },
        [&](int j, const bf16x8(&b)[1][1]) {
#pragma unroll
          for (int x = 0; x < 3; ++x)
            d[x][j % R.nf] = mma(fh[j / R.nf][x], b[0][0], d[x][j % R.nf]);
        });
  }
#pragma unroll
  for (int i = 0; i < R.nc; ++i) {
    const int c = R.c0 + i;
#pragma unroll
    for (int x = 0; x < 3; ++x)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if (comp_weight(c, j) != 0.f)
          r[i] += (Ge[x * 3 + j] * comp_weight(c, j)) * d[x][comp_field(c, j) - R.f0];
  }
}

// r of the group's components into LDS.  The accumulator rows past Np are zero
// (zero operator rows).
template <int N, int P, int H>
__device__ __forceinline__ void bt_rput(bf16x8* sn, int t, int g, int e, const f32x4 (&r)[9]) {
  using O = TOrd<N, P>;
  constexpr BtRole R = bt_role(O::DH, H);
#pragma unroll
  for (int i = 0; i < R.nc; ++i) bt_put4<P>(sn, O::KN, R.c0 + i, t, g, e, r[i]);
  static_assert(2 * O::KN == O::RT, "node tiles fill the K steps");
}

// The weight-adjusted mass inverse for the NC components of group grp and the K
// steps kb <= c < ke of quadrature points (32 each): V_q r (B operands from
// LDS), the weights, and P_q with the accumulators as B operand (the fragments
// of P_q hold, at K slot 8 g + j of step c, point 32 c + 16 (j / 4) + 4 g + j % 4,
// which is where the lane's accumulators have it), so that no wave waits for
// another.  A K step is 2 KN items of V_q and RT items of P_q, one operator
// fragment each, fetched PD items ahead.
template <int N, int P, int NC>
__device__ __forceinline__ void bt_quad(const BeArgs& A, const FragBuf& F, const bf16x8* sn,
                                        int64_t e0, int er, int g, int l0, int grp, int kb, int ke,
                                        f32x4 (&out)[TOrd<N, P>::RT][3]) {
  using O = TOrd<N, P>;
  constexpr int KN = O::KN, RT = O::RT, Nq = O::Nq, NV = 2 * KN, NI = NV + RT, PD = 4;
  static_assert(NI % PD == 0, "the fragment ring closes over a K step");
  const bool normal = grp == (O::G == 4 ? 2 : 1);
  // the two weights: lam and mu for the normal stresses (lam tr + 2 mu), else
  // 1/rho or 2 mu for each of two components (three components share the first)
  const int c0 = bt_comp(O::G, grp, 0), c1 = bt_comp(O::G, grp, 1);
  // (values first: a choice between the fields of A would keep a batch's copy of
  // it in memory)
  const float *irho = A.irho, *lam = A.lam, *mu = A.mu;
  const float* wf[2] = {(normal ? lam : c0 < 3 ? irho : mu) + e0 * Nq,
                        (normal ? mu : c1 < 3 ? irho : mu) + e0 * Nq};
  const float ws[2] = {!normal && c0 >= 3 ? 2.f : 1.f, normal || c1 >= 3 ? 2.f : 1.f};
  auto weights = [&](int c, f32x4 (&m)[2][2]) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int p0 = 32 * c + 16 * u + 4 * g, me = er * Nq;   // points past Nq weigh zeros
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        if constexpr (Nq % 4 == 0) {
          m[u][f] = bt_ldu(wf[f], 4u * unsigned(me + min(p0, Nq - 4)));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            m[u][f][j] = bt_ld<float>(wf[f], 4u * unsigned(me + min(p0 + j, Nq - 1)));
        }
      }
    }
  };
  u32x4 fr[PD][P];
  auto fetch = [&](int c, int j) {   // item j (maybe of the next K step)
    const int cc = j < NI ? c : min(c + 1, ke - 1), i = j < NI ? j : j - NI;
    bt_frag<P>(F, i < NV ? O::OFF_V + (2 * cc + i / KN) * KN + i % KN : O::OFF_P + (i - NV) * O::KQ + cc,
               fr[j % PD]);
  };
  const bf16x8* sc[NC];
#pragma unroll
  for (int k = 0; k < NC; ++k) sc[k] = sn + bt_comp(O::G, grp, k) * (KN * P * 64);
  f32x4 m[2][2];
  weights(kb, m);
#pragma unroll
  for (int j = 0; j < PD; ++j) fetch(kb, j);
#pragma unroll 1
  for (int c = kb; c < ke; ++c) {
    f32x4 w[2][NC] = {};
    bf16x8 b[2][NC][P];
    auto bread = [&](int s, bf16x8(&x)[NC][P]) {
#pragma unroll
      for (int k = 0; k < NC; ++k) bt_bread<P>(sc[k], KN, 0, s, l0, x[k]);
    };
    bread(0, b[0]);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if (j + 1 < NV) bread((j + 1) % KN, b[(j + 1) & 1]);
#pragma unroll
      for (int x = 0; x < kProd<P>; ++x)
#pragma unroll
        for (int k = 0; k < NC; ++k)
          w[j / KN][k] = mma(fr[j % PD][prod_a(P, x)], b[j & 1][k][prod_b(P, x)], w[j / KN][k]);
      fetch(c, j + PD);
      __builtin_amdgcn_sched_barrier(0);
    }
    // the weights, then the lane's eight points as the B operand of P_q
    bf16x8 q[NC][P];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      f32x4 tr = {0.f, 0.f, 0.f, 0.f}, m1 = ws[1] * m[u][1];
      if constexpr (NC == 3) {
        if (normal) tr = m[u][0] * (w[u][0] + w[u][1] + w[u][2]);
        else m1 = ws[0] * m[u][0];
      }
#pragma unroll
      for (int k = 0; k < NC; ++k)
        w[u][k] = NC == 2 && k == 0 ? (ws[0] * m[u][0]) * w[u][k] : tr + m1 * w[u][k];
    }
    weights(min(c + 1, ke - 1), m);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = w[j / 4][k][j % 4];
      split8<P>(v, q[k]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int j = NV + t;
#pragma unroll
      for (int x = 0; x < kProd<P>; ++x)
#pragma unroll
        for (int k = 0; k < NC; ++k)
          out[t][k] = mma(fr[j % PD][prod_a(P, x)], q[k][prod_b(P, x)], out[t][k]);
      fetch(c, j + PD);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The stage of one tile: launch position bid of a grid of G tiles
template <int N, int P>
__device__ __forceinline__ void stage_bt_run(const BeArgs& A, int64_t G, int64_t bid) {
  using O = TOrd<N, P>;
  constexpr int Np = O::Np, Nfp = O::Nfp, NF4 = O::NF4, Nq = O::Nq;
  constexpr int RT = O::RT, KN = O::KN, KF = O::KF, KQ = O::KQ, WV = O::WV, TH = O::TH;
  constexpr int QH = O::QH;
  __shared__ __align__(16) unsigned char smem[O::BYTES];
  float* sq = reinterpret_cast<float*>(smem);              // FP32 state (phase 1)
  bf16x8* sf = reinterpret_cast<bf16x8*>(smem);            // fluxes (phase 2)
  bf16x8* sn = reinterpret_cast<bf16x8*>(smem);            // state, then r (3-6)
  f32x4* sx = reinterpret_cast<f32x4*>(smem);              // partial results (7)

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int e = lane & 15, g = lane >> 4, l0 = 16 * g + (e ^ g);
  // XCD-aware order: each XCD takes one contiguous range of tiles
  const int64_t xcd = bid & 7, per = G >> 3, rem8 = G & 7;
  const int64_t tile = xcd * per + (xcd < rem8 ? xcd : rem8) + (bid >> 3);
  const int64_t K = A.K, KNp = K * Np, e0 = tile * kTile;
  const int ne = int((K - e0) < kTile ? (K - e0) : kTile);
  const int er = min(e, ne - 1);   // lanes past the last element repeat it
  // per-lane offsets are 32-bit, from uniform bases
  const float* qt = A.q_in + e0 * Np;

  // 1: the tile's state in FP32 in LDS, then the fluxes, kept split in
  // registers until every wave has read its traces.  Lane (g, e) of state task
  // (field, K step) holds nodes 32 s + 8 g ... + 7 of element e, also for
  // phase 3; face-node task idx is element idx / FK, face node idx % FK (rows
  // past NF4 are zero: the products read them).
  constexpr int QI = (9 * KN + WV - 1) / WV;
  constexpr int FK = 32 * KF, TF = kTile * FK, IF = (TF + TH - 1) / TH;
  f32x4 qv[QI][2];
  auto load_q = [&]() {
#pragma unroll
    for (int i = 0; i < QI; ++i) {
      const int task = min(wave + i * WV, 9 * KN - 1);
      const int f = task / KN, n0 = 32 * (task - f * KN) + 8 * g;
#pragma unroll
      for (int h = 0; h < 2; ++h)
        qv[i][h] = bt_ldu(qt + f * KNp, 4u * unsigned(er * Np + min(n0 + 4 * h, Np - 4)));
    }
  };
  __bf16 fx[IF][9][P];
  {
    unsigned nbi[IF], vM[IF];
    float fg[IF][4], qP[IF][9], zM[IF][2], zP[IF][2];
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = min(tid + it * TH, TF - 1);
      const int el = min(idx / FK, ne - 1), jf = min(idx - (idx / FK) * FK, NF4 - 1);
      nbi[it] = bt_ld<unsigned>(A.nbn + e0 * NF4, 4u * unsigned(el * NF4 + jf));
      vM[it] = unsigned(el * Np + bt_ld<int>(A.fmask, 4u * unsigned(jf)));
      const f32x4 v = bt_ld<f32x4>(A.fgeo + e0 * 16, 16u * unsigned(el * 4 + jf / Nfp));
#pragma unroll
      for (int j = 0; j < 4; ++j) fg[it][j] = v[j];
    }
    __builtin_amdgcn_sched_barrier(0);
    load_q();
    __builtin_amdgcn_sched_barrier(0);
    const unsigned r0 = unsigned(e0 * Np);
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      // a neighbour inside the tile is read from LDS below; its lanes load the
      // tile's first row instead (one hot line)
      const unsigned lr = nbi[it] - r0 < unsigned(kTile * Np) ? r0 : nbi[it];
#pragma unroll
      for (int f = 0; f < 9; ++f) qP[it][f] = (A.q_in + f * KNp)[lr];
      zM[it][0] = bt_ld<float>(A.zp + e0 * Np, 4u * vM[it]);
      zM[it][1] = bt_ld<float>(A.zs + e0 * Np, 4u * vM[it]);
      zP[it][0] = A.zp[nbi[it]];
      zP[it][1] = A.zs[nbi[it]];
    }
#pragma unroll
    for (int i = 0; i < QI; ++i) {
      const int task = wave + i * WV;
      const int f = task / KN, n0 = 32 * (task - f * KN) + 8 * g;
      if (task < 9 * KN) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (n0 + 4 * h < Np)
            *reinterpret_cast<f32x4*>(sq + (f * kTile + e) * Np + n0 + 4 * h) = qv[i][h];
      }
    }
    bt_sync();
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      __builtin_amdgcn_sched_barrier(0);   // one task at a time: registers
      const int idx = tid + it * TH;
      const int jf = idx - (idx / FK) * FK;
      const unsigned rl = nbi[it] - r0;
      const bool inT = rl < unsigned(kTile * Np);
      const unsigned rc = inT ? rl : 0u;
      float M[9], Q[9];
#pragma unroll
      for (int f = 0; f < 9; ++f) {
        M[f] = sq[f * kTile * Np + vM[it]];
        const float x = sq[f * kTile * Np + rc];
        Q[f] = inT ? x : qP[it][f];
      }
      const float nx = fg[it][0], ny = fg[it][1], nz = fg[it][2];
      const float fs = P == 3 && idx / FK % 2 ? -fg[it][3] : fg[it][3];
      const float jtx = (Q[3] - M[3]) * nx + (Q[8] - M[8]) * ny + (Q[7] - M[7]) * nz;
      const float jty = (Q[8] - M[8]) * nx + (Q[4] - M[4]) * ny + (Q[6] - M[6]) * nz;
      const float jtz = (Q[7] - M[7]) * nx + (Q[6] - M[6]) * ny + (Q[5] - M[5]) * nz;
      const float jvx = Q[0] - M[0], jvy = Q[1] - M[1], jvz = Q[2] - M[2];
      float dvx, dvy, dvz, dtx, dty, dtz;
      if (A.upwind) {
        const float zpM = zM[it][0], zsM = zM[it][1], zpP = zP[it][0], zsP = zP[it][1];
        const float jvn = jvx * nx + jvy * ny + jvz * nz;
        const float jtn = jtx * nx + jty * ny + jtz * nz;
        const float dvn = (zpP * jvn + jtn) * rcp_t(zpM + zpP);
        const float ivs = rcp_t(zsM + zsP);
        const float dvtx = (zsP * (jvx - jvn * nx) + (jtx - jtn * nx)) * ivs;
        const float dvty = (zsP * (jvy - jvn * ny) + (jty - jtn * ny)) * ivs;
        const float dvtz = (zsP * (jvz - jvn * nz) + (jtz - jtn * nz)) * ivs;
        dvx = dvn * nx + dvtx;
        dvy = dvn * ny + dvty;
        dvz = dvn * nz + dvtz;
        const float dtn = zpM * dvn;
        dtx = dtn * nx + zsM * dvtx;
        dty = dtn * ny + zsM * dvty;
        dtz = dtn * nz + zsM * dvtz;
      } else {
        dvx = 0.5f * jvx; dvy = 0.5f * jvy; dvz = 0.5f * jvz;
        dtx = 0.5f * jtx; dty = 0.5f * jty; dtz = 0.5f * jtz;
      }
      float fl[9];
      fl[0] = fs * dtx;
      fl[1] = fs * dty;
      fl[2] = fs * dtz;
      fl[3] = fs * dvx * nx;
      fl[4] = fs * dvy * ny;
      fl[5] = fs * dvz * nz;
      fl[6] = fs * 0.5f * (dvy * nz + dvz * ny);
      fl[7] = fs * 0.5f * (dvx * nz + dvz * nx);
      fl[8] = fs * 0.5f * (dvx * ny + dvy * nx);
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        if (jf >= NF4) fl[c] = 0.f;   // whatever the clamped traces are
        bt_split<P>(fl, c, fx[it][c]);
      }
    }
  }
  bt_sync();
#pragma unroll
  for (int it = 0; it < IF; ++it) {
    const int idx = tid + it * TH;
    const int el = idx / FK, jf = idx - el * FK;
    if (idx < TF) {
      const int s = jf >> 5, gb = (jf >> 3) & 3, j = jf & 7;
      const int at = 16 * gb + (el ^ (4 * (s & 3) + gb));
#pragma unroll
      for (int c = 0; c < 9; ++c)
#pragma unroll
        for (int p = 0; p < P; ++p)
          reinterpret_cast<__bf16*>(sf + ((c * KF + s) * P + p) * 64 + at)[j] = fx[it][c][p];
    }
  }
  if constexpr (!O::KEEPQ) load_q();   // again, from L2: registers
  float Ge[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    Ge[i] = bt_ld<float>(A.geo + e0 * 9, 4u * unsigned(er * 9 + i));
    if (P == 3 && e % 2) Ge[i] = -Ge[i];
  }
  bt_sync();

  const FragBuf F(A.frags, O::NFRAG, lane);

  // 2: r = LIFT f
  const int dt = wave % RT, dh = wave / RT;
  f32x4 r[9] = {};
  if (O::DH == 1 || dh == 0) bt_lift<N, P, 0>(F, sf, dt, l0, r);
  else bt_lift<N, P, O::DH - 1>(F, sf, dt, l0, r);
  mma_done(r);
  bt_sync();

  // 3: the state into LDS, rows past Np zero
#pragma unroll
  for (int i = 0; i < QI; ++i) {
    const int task = wave + i * WV;
    const int f = task / KN, s = task - f * KN, n0 = 32 * s + 8 * g;
    if (task < 9 * KN) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = n0 + 4 * (j / 4) < Np ? qv[i][j / 4][j % 4] : 0.f;
      bf16x8 o[P];
      split8<P>(v, o);
#pragma unroll
      for (int p = 0; p < P; ++p) sn[((f * KN + s) * P + p) * 64 + (l0 ^ (4 * (s & 3)))] = o[p];
    }
  }
  bt_sync();

  // 4: derivatives; 5: r into LDS
  if (O::DH == 1 || dh == 0) bt_deriv<N, P, 0>(F, sn, dt, l0, Ge, r);
  else bt_deriv<N, P, O::DH - 1>(F, sn, dt, l0, Ge, r);
  mma_done(r);
  bt_sync();
  if (O::DH == 1 || dh == 0) bt_rput<N, P, 0>(sn, dt, g, e, r);
  else bt_rput<N, P, O::DH - 1>(sn, dt, g, e, r);

  // 6: the mass inverse, one group of components and one part of the points
  // per wave.  The groups of the two parts are shifted, so that those of three
  // components run on different SIMDs.
  const int qh = wave / O::G, grp = (wave + qh) % O::G;
  const int kb = qh * ((KQ + QH - 1) / QH), ke = qh + 1 == QH ? KQ : (KQ + QH - 1) / QH;
  const bool three = O::G == 3 || grp == 2;
  f32x4 out[RT][3] = {};
  bt_sync();
  if (three) bt_quad<N, P, 3>(A, F, sn, e0, er, g, l0, grp, kb, ke, out);
  else bt_quad<N, P, 2>(A, F, sn, e0, er, g, l0, grp, kb, ke, out);

  // 7: the parts of the points together (part h finishes node tiles h RT / 2
  // ...), then the store or stage update: nodes 16 t + 4 g + j of element e
  const int64_t t0 = e0 * Np;
  constexpr int TW = RT / QH;
  const int tb = qh * TW;
  f32x4 rv[TW][3], qo[TW][3];
  if (A.lsrk) {
#pragma unroll
    for (int u = 0; u < TW; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int64_t fb = t0 + bt_comp(O::G, grp, three ? k : min(k, 1)) * KNp;
        const unsigned at = 4u * unsigned(er * Np + min(16 * (tb + u) + 4 * g, Np - 4));
        rv[u][k] = bt_ldu(A.res + fb, at);
        qo[u][k] = bt_ldu(A.q_in + fb, at);
      }
  }
  f32x4 fin[TW][3];
  if constexpr (QH == 2) {
    bt_sync();   // every wave has read r
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if ((t < TW) == (qh == 1) && (k < 2 || three))
          sx[(bt_comp(O::G, grp, k) * RT + t) * 64 + lane] = out[t][k];
    bt_sync();
#pragma unroll
    for (int u = 0; u < TW; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        fin[u][k] = (qh == 0 ? out[u][k] : out[TW + u][k]) +
                    sx[(bt_comp(O::G, grp, k < 2 || three ? k : 0) * RT + tb + u) * 64 + lane];
  } else {
#pragma unroll
    for (int u = 0; u < TW; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k) fin[u][k] = out[u][k];
  }
#pragma unroll
  for (int u = 0; u < TW; ++u) {
    const int n0 = 16 * (tb + u) + 4 * g;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if ((k == 2 && !three) || n0 >= Np || e >= ne) continue;
      const int64_t fb = t0 + bt_comp(O::G, grp, k) * KNp;
      const unsigned at = 4u * unsigned(e * Np + n0);
      const f32x4 rr = P == 3 && e % 2 ? -fin[u][k] : fin[u][k];
      if (A.lsrk) {
        const f32x4 rn = A.a * rv[u][k] + A.dt * rr;
        bt_stu(A.res + fb, at, rn);
        bt_stu(A.q_out + fb, at, qo[u][k] + A.b * rn);
      } else {
        bt_stu(A.rhs_out + fb, at, rr);
      }
    }
  }
}

template <int N, int P>
__global__ __launch_bounds__((TOrd<N, P>::TH), 2) void stage_bt(BeArgs A) {
  stage_bt_run<N, P>(A, gridDim.x, blockIdx.x);
}

}  // namespace dgb

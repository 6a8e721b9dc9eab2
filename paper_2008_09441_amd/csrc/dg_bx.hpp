// Fused DG elastic-wave stage with BF16x3 matrix-core contractions (gfx950),
// component-group design.
//
// Every dense contraction of the stage -- reference derivatives plus LIFT,
// interpolation to the quadrature points (V_q) and projection back (P_q) --
// runs on v_mfma_f32_16x16x32_bf16 as a split product: each FP32 operand x is
// written x = hi + lo with hi = bf16(x), lo = bf16(x - hi), and
// A B ~ A_hi B_hi + A_hi B_lo + A_lo B_hi with FP32 accumulation (relative
// error ~2^-16 per product).  Fluxes, the chain rule, material weights and
// the LSRK(5,4) update [CK94] are FP32.  FP32 runs the same phases on three bf16
// parts at orders 3 and 4 (see kProd) and on FP32 products at orders 1 and 2 and
// in the adjoint, FP64 in double precision on the FP64 products.
//
// One workgroup (four waves) owns a tile of 16 consecutive elements; the
// MFMA column index is the element, so a lane keeps the same element through
// the whole stage.  Each wave owns a fixed set of output components of the
// right-hand side and carries them through every contraction without any
// exchange with the other waves:
//   wave 0: v_x, v_y          (1/rho weights)
//   wave 1: v_z, s_yz         (1/rho and 2 mu weights)
//   wave 2: s_xx, s_yy, s_zz  (lam tr(e) + 2 mu e: the trace couples them)
//   wave 3: s_xz, s_xy        (2 mu weights)
// Phases (barriers only between the shared ones):
//   A  stage q[9][Np][16] and the metric terms in LDS (coalesced reads);
//   B  face fluxes [9][4 Nfp][16] in LDS, one thread per element face node:
//      own trace from LDS, neighbour trace gathered through the (neighbour,
//      trace pattern) tables, exact-Riemann upwind or central flux [WSG10],
//      scaled by Fscale;
//   C  per wave: r_c = sum_d D_d U_{c,d} + LIFT f_c as one K loop over the
//      concatenated [D_r|D_s|D_t|LIFT] operator [HW08, Ch. 10], with
//      U_{c,d} = sum_j G_dj w_cj q_{f_cj} folding the element's constant
//      metric terms into the inputs (div sigma rows, eps(v) rows);
//   D  per wave, for each chunk of 32 quadrature points: V_q r, the pointwise
//      weight-adjusted material operator [CHW17, C18], accumulation of P_q;
//      the accumulators of one contraction are the B operand of the next
//      (K slots permuted on the host), so values never leave their lane;
//   E  right-hand side store or fused stage update, coalesced over [9][K][Np].
// Operator fragments (hi/lo, in lane order) are read from global memory and
// stay in the L2/L1 caches; the material is stored blocked by element tile in
// the lane order of phase D, so its loads are whole 1 KiB wave transactions.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "dg_bx_layout.hpp"

namespace dgb {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

// four values of the working precision: the MFMA accumulator of a lane and
// one lane's entry of an FP32 / FP64 operator fragment
template <typename T> struct Vec4;
template <> struct Vec4<float> { typedef f32x4 type; };
template <> struct Vec4<double> { typedef f64x4 type; };
template <typename T> using v4_t = typename Vec4<T>::type;

constexpr int kThreads = 256;   // four waves
constexpr int kTile = 16;       // elements per workgroup
constexpr int kES = 17;         // LDS stride of a row of 16 element values (odd)

// Arguments of the stage in working precision T (float: BF16x3 or FP32
// matrix-core products; double: FP64 matrix-core products)
template <typename T>
struct BxArgsT {
  const T* q_in;         // [9][K][Np]
  T* q_out;              // [9][K][Np] (LSRK mode)
  T* res;                // [9][K][Np] (LSRK mode)
  T* rhs_out;            // [9][K][Np] (rhs mode)
  const T* geo;          // [K][9]: d(r,s,t)_i / d(x,y,z)_j at i*3+j
  const T* fgeo;         // [K][4][4]: outward unit normal, Fscale
  const int32_t* nbn;    // [K][4 Nfp]: neighbour volume node nb * Np + vP of each face node
  const int32_t* fmask;  // [4][Nfp]
  const int32_t* torder; // [ceil(K/16)]: tile processed at each launch position
  const T* mat;          // [ceil(K/16)][3][MATS]: 1/rho, lam, mu blocked
  const T* zp;           // [K][Np]
  const T* zs;
  const u32x4* frags;    // BF16x3: [NFRAG][64] u32x4; FP32 / FP64: FOrd fragments of T
  int64_t K;
  T a, b, dt;
  int lsrk;              // 0: write rhs_out; 1: fused LSRK update
  int upwind;            // 1 upwind, 0 central
  T* r_out;              // stage_bx_r: the raw right-hand side R q [9][K][Np]
  T* j_out;              // stage_bx_r, if not null: velocity and traction jumps of
                         // every face node, [K][4 Nfp][8] (jv, jt, 0, 0)
};
typedef BxArgsT<float> BxArgs;


// Output component c (vx vy vz sxx syy szz syz sxz sxy) of the volume term
// is sum_d D_d U_{c,d} with U_{c,d} = sum_j G_dj w(c,j) q_{f(c,j)}: the stress
// row (sigma_{c x}, sigma_{c y}, sigma_{c z}) for the velocity components,
// the symmetrised velocity pattern for the strain components.
__host__ __device__ constexpr int comp_field(int c, int j) {
  return c == 0 ? (j == 0 ? 3 : j == 1 ? 8 : 7)
       : c == 1 ? (j == 0 ? 8 : j == 1 ? 4 : 6)
       : c == 2 ? (j == 0 ? 7 : j == 1 ? 6 : 5)
       : c == 3 ? 0
       : c == 4 ? 1
       : c == 5 ? 2
       : c == 6 ? (j == 1 ? 2 : 1)
       : c == 7 ? (j == 0 ? 2 : 0)
       : (j == 0 ? 1 : 0);
}
__host__ __device__ constexpr float comp_weight(int c, int j) {
  return c < 3 ? 1.f
       : c < 6 ? (j == c - 3 ? 1.f : 0.f)
       : (j == c - 6 ? 0.f : 0.5f);
}

// components owned by wave W
__host__ __device__ constexpr int wave_ncomp(int W) { return W == 2 ? 3 : 2; }
__host__ __device__ constexpr int wave_comp(int W, int i) {
  return W == 0 ? i : W == 1 ? (i == 0 ? 2 : 6) : W == 2 ? 3 + i : 7 + i;
}

__device__ __forceinline__ f32x4 mma(const u32x4& a, const bf16x8& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), b, c, 0, 0, 0);
}

// x as P bf16 parts, each the rounding (to nearest even) of what the parts before
// leave, converted in pairs (one packed conversion per pair and part): two parts
// hold 16 bits, three all 24 of an FP32 value
template <int P>
__device__ __forceinline__ void split8(const float* v, bf16x8 (&o)[P]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f32x2 r = {v[2 * k], v[2 * k + 1]};
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const bf16x2 h = __builtin_convertvector(r, bf16x2);
      if (p + 1 < P) r = r - __builtin_convertvector(h, f32x2);
      o[p][2 * k] = h[0];
      o[p][2 * k + 1] = h[1];
    }
  }
}

// The part products of a split product A B: A part prod_a and B part prod_b of
// product k < kProd<P>.  P = 2 (BF16x3): hi hi, hi lo, lo hi.  P = 3 (FP32): six
// of nine, from the smallest up; a part is at most 2^-9 of the one before it, so
// the three left out (second by third part, both ways, and third by third) are at
// most 2^-27 of the product.
//   What three parts have to mind: v_mfma_f32_16x16x32_bf16 adds four groups of
// eight products to the accumulator in turn, and an accumulator smaller than the
// largest product of a group is first cut off at that product's last FP32 bit,
// downwards.  The error is small but has one sign, so that it adds up over the
// steps of a run where rounding to nearest averages out (v_mfma_f32_16x16x4_f32
// rounds to nearest).  Left alone, a right-hand side of order 4 is off by 1.8e-7
// of its norm in the mean of 200 steps (5.9e-8 on FP32 products) and a state of
// 3,072 elements by 3.2e-6 after 800 steps and 1.0e-5 after 3,200 (2.3e-6, 4.7e-6);
// order 3 2.0e-6 and 5.3e-6 (1.8e-6, 3.9e-6).  Therefore:
//   - an accumulator that holds whole products takes the leading product, and the
//     five small ones have one of their own (mma_split);
//   - every second K step is negated, and the accumulator with it, so that what is
//     cut off cancels (the results then have the sign of the step count);
//   - elements of odd index have the opposite sign from their fluxes and metric
//     terms to the result, so that what is left cancels over neighbours;
//   - the derivatives are taken of the state less its value at node mid_node, which
//     they do not change: their products are large and nearly cancel.
// 4.9e-8 so in the mean, and 2.3e-6 and 4.9e-6 (order 3 1.8e-6 and 3.7e-6); a stage
// of 82,944 elements takes 125 us at order 3 and 288 at order 4 (124 and 282
// without, 153 and 386 on FP32 products).
template <int P>
constexpr int kProd = P == 2 ? 3 : 6;
__host__ __device__ constexpr int prod_a(int P, int k) {
  return P == 2 ? (k == 2 ? 1 : 0) : (k == 0 ? 2 : k == 2 || k == 3 ? 1 : 0);
}
__host__ __device__ constexpr int prod_b(int P, int k) {
  return P == 2 ? (k == 1 ? 1 : 0) : (k == 1 ? 2 : k == 2 || k == 4 ? 1 : 0);
}
// c + A B, with FLIP its negative (three parts)
template <int P, bool FLIP = false>
__device__ __forceinline__ f32x4 mma_split(const u32x4 (&a)[P], const bf16x8 (&b)[P], f32x4 c) {
  if constexpr (P == 2) {
#pragma unroll
    for (int k = 0; k < kProd<P>; ++k) c = mma(a[prod_a(P, k)], b[prod_b(P, k)], c);
    return c;
  } else {
    f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k + 1 < kProd<P>; ++k) d = mma(a[prod_a(P, k)], b[prod_b(P, k)], d);
    c = mma(a[0], b[0], c);
    return FLIP ? -c - d : c + d;
  }
}
// a node near the element's centre: (1, 1, 1) of orders 3 on
__host__ __device__ constexpr int mid_node(int N) { return (N + 1) * (N + 2) / 2 + N + 1; }

// Uses accumulators where they are complete: products have no side effect, and
// the compiler sinks those whose result is read in a later block into it, with
// all their operands kept in registers until then.
template <int M>
__device__ __forceinline__ void mma_done(f32x4 (&v)[M]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int i = 0; i < M; ++i) asm volatile("" : "+v"(v[i]));
#endif
}

// operator fragments (64 lanes x 16 bytes each): a buffer descriptor, a uniform
// fragment offset and the lane's slot, so that one register addresses them all
// (BF16x3, order 4: 233 registers and 1685 us at 663,552 elements, against 247
// and 1714 with a 64-bit address per fragment row)
template <typename V>
struct FragBufV {
  __amdgpu_buffer_rsrc_t r;
  int lane16;
  __device__ FragBufV(const void* frags, int count, int lane)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(frags), 0, count * 1024, 0x00020000)),
        lane16(lane * 16) {}
  __device__ __forceinline__ V load(int f, int i = 0) const {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, lane16, (f + i) * 1024, 0));
  }
};
using FragBuf = FragBufV<u32x4>;

// the same for the four-value fragments of FOrd in FP64 (64 lanes x 4 doubles).
// With 64-bit addresses the FP64 stage takes 876 us at order 4 and 384 at order 3
// (82,944 elements), with these 848 and 377.
struct FragBufD {
  __amdgpu_buffer_rsrc_t r;
  int off;
  __device__ FragBufD(const void* frags, int count, int lane)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(frags), 0, count * 2048, 0x00020000)),
        off(lane * 32) {}
  __device__ __forceinline__ f64x4 load(int f, int k = 0) const {
    union {
      u32x4 u[2];
      f64x4 v;
    } x;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      x.u[i] = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, (f + k) * 2048, 0);
    return x.v;
  }
};

// fragments of 64 lanes x V by address: FP32 and BF16x3 at orders 1 and 2, whose
// few fragments take more registers with a descriptor than they save (order 2, FP32,
// 3,075 elements: 7.86 us a stage so, 7.93 with one)
template <typename V>
struct FragPtr {
  const V* p;
  int lane;
  __device__ FragPtr(const void* frags, int, int l) : p(static_cast<const V*>(frags)), lane(l) {}
  __device__ __forceinline__ V load(int f, int i = 0) const { return (p + f * 64)[i * 64 + lane]; }
};

// the form at order N of split products, and of FOrd fragments
template <int N>
using FragsS = std::conditional_t<(N <= 2), FragPtr<u32x4>, FragBuf>;
template <int N, typename T>
using FragsF = std::conditional_t<sizeof(T) == 8, FragBufD,
                                  std::conditional_t<(N <= 2), FragPtr<f32x4>, FragBufV<f32x4>>>;

// LDS use of one workgroup, in values of T, and its padded allocation in bytes
template <int N, typename T = float>
struct BLds {
  using O = BOrd<N>;
  static constexpr int SQ = 9 * O::Np * kES;             // q       [9][Np][17]
  static constexpr int SG = kTile * 9;                   // metric  [16][9]
  static constexpr int SZ = 2 * O::Np * kES;             // Z_p, Z_s [2][Np][17]
  static constexpr int SF = 9 * O::NF4 * kES;            // fluxes  [9][4 Nfp][17]
  static constexpr int SR = 9 * O::Np * kES;             // result  [9][Np][17] (over the fluxes)
  // the three-component wave keeps its V_q B operands (hi/lo, lane order)
  // in LDS behind the result rows during phase D
  static constexpr int RO = (SR + 3) & ~3;
  static constexpr int SRL = sizeof(T) == 4 ? 3 * O::SVQ * 2 * 64 * 4 : 0;
  static constexpr int SU = SF > RO + SRL ? SF : RO + SRL;
  static constexpr int OFF_U = (SQ + SG + SZ + 3) & ~3;  // 16-byte aligned union
  static constexpr int USED = (OFF_U + SU) * int(sizeof(T));
  // Padded so that the workgroups one CU can hold (160 KiB of LDS) never use
  // more than 128 KiB together (at most 3 per CU at >40 KiB each, 2 at
  // >53.3 KiB each, or 1 at >80 KiB each).
  static constexpr int FLOOR =
      USED <= 43690 ? 40976 : USED <= 65536 ? 54630 : USED <= 81920 ? 81936 : 0;
  static constexpr int BYTES = USED > FLOOR ? USED : FLOOR;
};

// Phase C for wave W: acc[i][t] = rows 16 t + 4 g + j of r_{comp i}, in three parts
// negated where kNegC<N>
template <int N>
constexpr bool kNegC = (BOrd<N>::SVL - 1) & 1;
template <int N, int W, int P>
__device__ __forceinline__ void vol_lift(const BxArgs& A, const FragsS<N>& F, const float* sq, const float* sg,
                                         const float* sF, int lane, f32x4 (&acc)[3][BOrd<N>::RT]) {
  using O = BOrd<N>;
  constexpr int Np = O::Np, NF4 = O::NF4, RT = O::RT, SN = O::SN, SVL = O::SVL;
  constexpr int NC = wave_ncomp(W);
  const int e = lane & 15, g = lane >> 4;
  float G[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) G[i] = sg[e * 9 + i];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // three parts: the state at the middle node (see kProd)
  float q0[NC][3];
  if constexpr (P == 3) {
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        q0[i][j] = sq[(comp_field(wave_comp(W, i), j) * Np + mid_node(N)) * kES + e];
  }

  // operator fragments are prefetched one K step ahead (the fragment reads
  // hit L2; without the prefetch each step waits for its own)
  u32x4 fc[RT][P], fn[RT][P];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int h = 0; h < P; ++h) fc[t][h] = F.load((O::OFF_V + t * SVL) * P + h);
#pragma unroll
  for (int s = 0; s < SVL; ++s) {
    if (s + 1 < SVL) {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int h = 0; h < P; ++h)
          fn[t][h] = F.load((O::OFF_V + t * SVL + s + 1) * P + h);
    }
    __builtin_amdgcn_sched_barrier(0);
    float bv[NC][8];
    if (s < SN) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        // node slots: entries beyond Np meet zero operator columns, so the
        // clamped node only has to be a finite value
        const int m = min(g + 4 * (2 * s + h), Np - 1);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = wave_comp(W, i);
          float a[3];
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            a[j] = 0.f;
            if (comp_weight(c, j) != 0.f) {
              a[j] = sq[(comp_field(c, j) * Np + m) * kES + e];
              if constexpr (P == 3) a[j] -= q0[i][j];
              a[j] *= comp_weight(c, j);
            }
          }
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            float u = 0.f;
#pragma unroll
            for (int j = 0; j < 3; ++j)
              if (comp_weight(c, j) != 0.f) u += G[d * 3 + j] * a[j];
            bv[i][3 * h + d] = u;
          }
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int jf = min(g + 4 * (2 * s + h), NF4 - 1);
#pragma unroll
        for (int i = 0; i < NC; ++i) bv[i][6 + h] = sF[(wave_comp(W, i) * NF4 + jf) * kES + e];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int jf = min(g + 4 * (2 * SN + 8 * (s - SN) + j), NF4 - 1);
#pragma unroll
        for (int i = 0; i < NC; ++i) bv[i][j] = sF[(wave_comp(W, i) * NF4 + jf) * kES + e];
      }
    }
    bf16x8 b[NC][P];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (P == 3 && s % 2) {
#pragma unroll
        for (int j = 0; j < 8; ++j) bv[i][j] = -bv[i][j];
      }
      split8<P>(bv[i], b[i]);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
#pragma unroll
      for (int i = 0; i < NC; ++i)
        acc[i][t] = s + 1 < SVL ? mma_split<P, P == 3>(fc[t], b[i], acc[i][t])
                                : mma_split<P>(fc[t], b[i], acc[i][t]);
      if (P == 3) __builtin_amdgcn_sched_barrier(0);   // registers
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int h = 0; h < P; ++h) fc[t][h] = fn[t][h];
  }
  if constexpr (P == 3) {
#pragma unroll
    for (int i = 0; i < NC; ++i) mma_done(acc[i]);
  }
}

// Material samples of chunk ch for this lane: m[f][u] holds quadrature
// points 32 ch + 16 u + 4 g + j (j < 4) of field f (1/rho, lam, mu); only the
// fields wave W uses are loaded
template <int N, int W, typename T = float>
__device__ __forceinline__ void mat_chunk(const BxArgsT<T>& A, int64_t tile, int lane, int ch,
                                          v4_t<T> (&m)[3][2]) {
  using O = BOrd<N>;
  constexpr bool need[3] = {W == 0 || W == 1, W == 2, W != 0};
  const v4_t<T>* mat = reinterpret_cast<const v4_t<T>*>(A.mat) + tile * 3 * (O::MATS / 4);
#pragma unroll
  for (int f = 0; f < 3; ++f)
#pragma unroll
    for (int u = 0; u < 2; ++u)
      m[f][u] = need[f] ? mat[f * (O::MATS / 4) + (ch * 2 + u) * 64 + lane] : v4_t<T>{0, 0, 0, 0};
}

// Phase D for wave W: V_q, material, P_q; the nodal result goes to sr.  m0
// holds the material of chunk 0 (loaded before phase C).
template <int N, int W, int P>
__device__ __forceinline__ void quad_proj(const BxArgs& A, const FragsS<N>& F, int64_t tile, int lane,
                                          const f32x4 (&acc)[3][BOrd<N>::RT],
                                          const f32x4 (&m0)[3][2], float* sr, bf16x8* srl) {
  using O = BOrd<N>;
  constexpr int Np = O::Np, RT = O::RT, QT = O::QT, QC = O::QC, SVQ = O::SVQ;
  constexpr int NC = wave_ncomp(W);
  const int e = lane & 15, g = lane >> 4;

  // V_q B operands: K slot 8 g + j of step s holds row 4 g + j % 4 of node
  // tile 2 s + j / 4, which is where this lane's accumulator already has it.
  // The three-component wave parks two parts in LDS (register budget).
  constexpr int PK = NC == 3 ? 2 : 0;   // parts parked
  auto pk = [&](int i, int s, int h) { return srl + ((i * SVQ + s) * 2 + h) * 64 + lane; };
  bf16x8 r[NC][SVQ][P];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int s = 0; s < SVQ; ++s) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int t = 2 * s + j / 4;
        v[j] = t < RT ? acc[i][t][j % 4] : 0.f;
      }
      split8<P>(v, r[i][s]);
#pragma unroll
      for (int h = 0; h < PK; ++h) *pk(i, s, h) = r[i][s][h];
    }

  f32x4 out[NC][RT];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t) out[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // V_q fragments of chunk 0; inside the loop the P_q fragments and the next
  // chunk's material are issued at the top of a chunk, the next chunk's V_q
  // fragments after its V_q products, so every fetch is covered by MFMA work.
  // With three parts (registers) the V_q fragments come one quadrature tile
  // ahead and the P_q fragments after the V_q products.
  constexpr int FU = P == 3 ? 1 : 2;   // quadrature tiles of V_q fragments held
  u32x4 fv[2][SVQ][P];
  auto load_v = [&](int qt, u32x4(&f)[SVQ][P]) {
#pragma unroll
    for (int s = 0; s < SVQ; ++s)
#pragma unroll
      for (int h = 0; h < P; ++h)
        f[s][h] = qt < QT ? F.load((O::OFF_Q + qt * SVQ + s) * P + h)
                          : u32x4{0u, 0u, 0u, 0u};
  };
#pragma unroll
  for (int u = 0; u < FU; ++u) load_v(u, fv[u]);
  f32x4 m[3][2];
#pragma unroll
  for (int f = 0; f < 3; ++f) m[f][0] = m0[f][0], m[f][1] = m0[f][1];
#pragma unroll
  for (int ch = 0; ch < QC; ++ch) {
    u32x4 fp[RT][P];
    auto load_p = [&]() {
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int h = 0; h < P; ++h)
          fp[t][h] = F.load((O::OFF_P + t * QC + ch) * P + h);
    };
    if (P == 2) load_p();
    f32x4 mn[3][2];
    if (P == 2 && ch + 1 < QC) mat_chunk<N, W>(A, tile, lane, ch + 1, mn);
    __builtin_amdgcn_sched_barrier(0);
    const f32x4* mi = m[0];
    const f32x4* ml = m[1];
    const f32x4* mm = m[2];
    f32x4 w[NC][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (P == 3) {
        // the next tile's fragments (of the next chunk after u = 1)
        if (2 * ch + u + 1 < QT) load_v(2 * ch + u + 1, fv[(u + 1) & 1]);
        if (u == 1) load_p();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < NC; ++i) w[i][u] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (2 * ch + u < QT) {
#pragma unroll
        for (int s = 0; s < SVQ; ++s) {
#pragma unroll
          for (int i = 0; i < NC; ++i) {
#pragma unroll
            for (int h = 0; h < PK; ++h) r[i][s][h] = *pk(i, s, h);
            if constexpr (P == 2) {
              w[i][u] = mma_split<P>(fv[u][s], r[i][s], w[i][u]);
            } else {
#pragma unroll
              for (int k = 0; k + 1 < kProd<P>; ++k)
                w[i][u] = mma(fv[u][s][prod_a(P, k)], r[i][s][prod_b(P, k)], w[i][u]);
            }
          }
        }
        if constexpr (P == 3) {   // the leading products on their own
          f32x4 wl[NC];
#pragma unroll
          for (int i = 0; i < NC; ++i) wl[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < SVQ; ++s)
#pragma unroll
            for (int i = 0; i < NC; ++i) {
              if (PK > 0) r[i][s][0] = *pk(i, s, 0);
              wl[i] = mma(fv[u][s][0], r[i][s][0], wl[i]);
            }
#pragma unroll
          for (int i = 0; i < NC; ++i) w[i][u] += wl[i];
        }
      }
      if (P == 3) __builtin_amdgcn_sched_barrier(0);
    }
    if (P == 2 && ch + 1 < QC) {
#pragma unroll
      for (int u = 0; u < 2; ++u) load_v(2 * (ch + 1) + u, fv[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // pointwise weight-adjusted material operator
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if constexpr (W == 0) {
        w[0][u] *= mi[u];
        w[1][u] *= mi[u];
      } else if constexpr (W == 1) {
        w[0][u] *= mi[u];
        w[1][u] *= 2.f * mm[u];
      } else if constexpr (W == 2) {
        const f32x4 tr = w[0][u] + w[1][u] + w[2][u];
        const f32x4 m2 = 2.f * mm[u];
#pragma unroll
        for (int i = 0; i < 3; ++i) w[i][u] = ml[u] * tr + m2 * w[i][u];
      } else {
        w[0][u] *= 2.f * mm[u];
        w[1][u] *= 2.f * mm[u];
      }
    }
    // three parts: the next chunk's material over this one's (registers)
    if (P == 3 && ch + 1 < QC) mat_chunk<N, W>(A, tile, lane, ch + 1, m);
    // P_q B operands: K slot 8 g + j of chunk ch is row 4 g + j % 4 of
    // quadrature tile 2 ch + j / 4
    bf16x8 p[NC][P];
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = P == 3 && ch % 2 ? -w[i][j / 4][j % 4] : w[i][j / 4][j % 4];
      split8<P>(v, p[i]);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int i = 0; i < NC; ++i)
        out[i][t] = ch + 1 < QC ? mma_split<P, P == 3>(fp[t], p[i], out[i][t])
                                : mma_split<P>(fp[t], p[i], out[i][t]);
    if (P == 2 && ch + 1 < QC) {
#pragma unroll
      for (int f = 0; f < 3; ++f) m[f][0] = mn[f][0], m[f][1] = mn[f][1];
    }
  }
  // the signs of both phases and of odd elements
  const bool neg = P == 3 && (kNegC<N> + QC - 1 + e) % 2;
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = 16 * t + 4 * g + j;
        if (n < Np) sr[(wave_comp(W, i) * Np + n) * kES + e] = neg ? -out[i][t][j] : out[i][t][j];
      }
}

__device__ __forceinline__ f32x4 mma_f(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f64x4 mma_f(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// 1 / x: the hardware reciprocal (1 ulp) in FP32, a division in FP64
__device__ __forceinline__ float rcp_t(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp_t(double x) { return 1.0 / x; }

// Phase C of the FP32 / FP64 kernel for wave W: acc[i][t] = rows
// 16 t + 4 g + j of r_{comp i}, one K slot per lane and step (the order of
// FOrd); operator fragments are fetched one group of four steps ahead.
template <int N, int W, typename T>
__device__ __forceinline__ void vol_lift_f(const FragsF<N, T>& F, const T* sq, const T* sg,
                                           const T* sF, int lane,
                                           v4_t<T> (&acc)[3][BOrd<N>::RT]) {
  using O = FOrd<N>;
  using V4 = v4_t<T>;
  constexpr int Np = O::Np, NF4 = O::NF4, RT = O::RT, NB = O::NB, SV = O::SV, SV4 = O::SV4;
  constexpr int NC = wave_ncomp(W);
  const int e = lane & 15, g = lane >> 4;
  T G[9];
#pragma unroll
  for (int i = 0; i < 9; ++i) G[i] = sg[e * 9 + i];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[i][t] = V4{0, 0, 0, 0};
  V4 fc[RT], fn[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) fc[t] = F.load(O::OFF_V / 64, t * SV4);
#pragma unroll
  for (int q = 0; q < SV4; ++q) {
    if (q + 1 < SV4) {
#pragma unroll
      for (int t = 0; t < RT; ++t) fn[t] = F.load(O::OFF_V / 64, t * SV4 + q + 1);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int s = 4 * q + j;
      if (s >= SV) break;
      T b[NC];
      if (s < 3 * NB) {
        // U_{c,d} at node 4 (s / 3) + g (clamped: beyond Np the operator is zero)
        const int d = s % 3, m = min(4 * (s / 3) + g, Np - 1);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
          const int c = wave_comp(W, i);
          T u = 0;
#pragma unroll
          for (int jj = 0; jj < 3; ++jj)
            if (comp_weight(c, jj) != 0.f)
              u += G[d * 3 + jj] * T(comp_weight(c, jj)) * sq[(comp_field(c, jj) * Np + m) * kES + e];
          b[i] = u;
        }
      } else {
        const int jf = min(4 * (s - 3 * NB) + g, NF4 - 1);
#pragma unroll
        for (int i = 0; i < NC; ++i) b[i] = sF[(wave_comp(W, i) * NF4 + jf) * kES + e];
      }
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int i = 0; i < NC; ++i) acc[i][t] = mma_f(fc[t][j], b[i], acc[i][t]);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) fc[t] = fn[t];
  }
}

// The raw right-hand side R q (volume terms and LIFT, before the mass
// inverse) of wave W's components from its phase-C accumulators, rows
// 16 t + 4 g + j of element column e, to r_out (FP32 only)
template <int N, int W>
__device__ __forceinline__ void store_raw(const BxArgs& A, int64_t e0, int ne, int lane,
                                          const f32x4 (&acc)[3][BOrd<N>::RT]) {
  using O = BOrd<N>;
  constexpr int Np = O::Np, RT = O::RT, NC = wave_ncomp(W);
  const int e = lane & 15, g = lane >> 4;
  if (e >= ne) return;
  const int64_t KNp = A.K * Np;
  float* out = A.r_out + (e0 + e) * Np;
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = 16 * t + 4 * g + j;
        if (n < Np) out[wave_comp(W, i) * KNp + n] = acc[i][t][j];
      }
}

// Phase D of the FP32 kernel for wave W: per chunk of two quadrature tiles,
// V_q with the node accumulators as the B operand (K step (t, j) is row
// 16 t + 4 g + j), the pointwise weight-adjusted material operator, and
// P_q with the weighted values as the B operand (K step (u, j) is point
// 16 u + 4 g + j); the nodal result goes to sr.
template <int N, int W, typename T>
__device__ __forceinline__ void quad_proj_f(const BxArgsT<T>& A, const FragsF<N, T>& F, int64_t tile, int lane,
                                            const v4_t<T> (&acc)[3][BOrd<N>::RT],
                                            const v4_t<T> (&m0)[3][2], T* sr) {
  using O = FOrd<N>;
  using V4 = v4_t<T>;
  constexpr int Np = O::Np, RT = O::RT, QT = O::QT, QC = O::QC;
  constexpr int NC = wave_ncomp(W);
  const int e = lane & 15, g = lane >> 4;
  V4 out[NC][RT];
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t) out[i][t] = V4{0, 0, 0, 0};
  V4 m[3][2];
#pragma unroll
  for (int f = 0; f < 3; ++f) m[f][0] = m0[f][0], m[f][1] = m0[f][1];
#pragma unroll
  for (int ch = 0; ch < QC; ++ch) {
    V4 fv[2][RT], fp[RT][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int qt = 2 * ch + u < QT ? 2 * ch + u : QT - 1;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        fv[u][t] = F.load(O::OFF_Q / 64, qt * RT + t);
        fp[t][u] = F.load(O::OFF_P / 64, t * QT + qt);
      }
    }
    V4 mn[3][2];
    if (ch + 1 < QC) mat_chunk<N, W, T>(A, tile, lane, ch + 1, mn);
    __builtin_amdgcn_sched_barrier(0);
    V4 w[NC][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        w[i][u] = V4{0, 0, 0, 0};
        if (2 * ch + u < QT) {
#pragma unroll
          for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int j = 0; j < 4; ++j) w[i][u] = mma_f(fv[u][t][j], acc[i][t][j], w[i][u]);
        }
      }
    }
    const V4* mi = m[0];
    const V4* ml = m[1];
    const V4* mm = m[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if constexpr (W == 0) {
        w[0][u] *= mi[u];
        w[1][u] *= mi[u];
      } else if constexpr (W == 1) {
        w[0][u] *= mi[u];
        w[1][u] *= T(2) * mm[u];
      } else if constexpr (W == 2) {
        const V4 tr = w[0][u] + w[1][u] + w[2][u];
        const V4 m2 = T(2) * mm[u];
#pragma unroll
        for (int i = 0; i < 3; ++i) w[i][u] = ml[u] * tr + m2 * w[i][u];
      } else {
        w[0][u] *= T(2) * mm[u];
        w[1][u] *= T(2) * mm[u];
      }
    }
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (2 * ch + u < QT) {
#pragma unroll
          for (int i = 0; i < NC; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) out[i][t] = mma_f(fp[t][u][j], w[i][u][j], out[i][t]);
        }
      }
    if (ch + 1 < QC) {
#pragma unroll
      for (int f = 0; f < 3; ++f) m[f][0] = mn[f][0], m[f][1] = mn[f][1];
    }
  }
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int n = 16 * t + acc_row(sizeof(T) == 8, g, j);
        if (n < Np) sr[(wave_comp(W, i) * Np + n) * kES + e] = out[i][t][j];
      }
}

// Item map of the tile's state, shared by the staging loads and the final
// update: field f of the tile is TS = 16 Np consecutive floats.  Main items
// r = tid + 256 it (it < MI) cover rows below 256 MI of every field; the TT
// rows left per field form 9 TT tail items t = tid + 256 j, clamped to the
// last one (duplicates repeat its load and store).  Rows are clamped to the
// tile's last valid row.
template <int N>
struct TileMap {
  static constexpr int Np = BOrd<N>::Np;
  static constexpr int TS = kTile * Np;
  static constexpr int MI = TS / kThreads;
  static constexpr int TT = TS - MI * kThreads;
  static constexpr int IT = (9 * TT + kThreads - 1) / kThreads;
  static_assert(TT > 0, "tail items assume 16 Np is not a multiple of 256");
  int rmax;   // last valid row: ne Np - 1
  __device__ explicit TileMap(int ne) : rmax(ne * Np - 1) {}
  __device__ unsigned main_row(int tid, int it) const {
    return min(unsigned(tid + it * kThreads), unsigned(rmax));
  }
  __device__ int tail_item(int tid, int j) const { return min(tid + j * kThreads, 9 * TT - 1); }
  __device__ int tail_field(int tid, int j) const { return tail_item(tid, j) / TT; }
  __device__ unsigned tail_row(int tid, int j) const {
    const int t = tail_item(tid, j);
    return min(unsigned(MI * kThreads + t - (t / TT) * TT), unsigned(rmax));
  }
  // LDS offset of row r (element r / Np, node r % Np) in a [Np][17] field block
  __device__ static int lds_row(unsigned r) {
    const unsigned e = r / Np;
    return int((r - e * Np) * kES + e);
  }
};

// FP32 products: three bf16 parts at orders 3 and 4, where they are 1.3 times
// faster a stage; at orders 1 and 2 the contractions are short and the splits
// cost more than the FP32 products they replace (3,072 elements: order 1 5.0 us
// against 5.8, order 2 7.8 against 8.3)
constexpr bool bx_three_parts(int N) { return N >= 3; }

// Phase C of wave W on split products, with the material of chunk 0 loaded before
// the products, or after them (LATE)
template <int N, int W, int P, bool LATE>
__device__ __forceinline__ void split_c(const BxArgs& A, const FragsS<N>& F, int64_t tile,
                                        const float* sq, const float* sg, const float* sF, int lane,
                                        f32x4 (&m0)[3][2], f32x4 (&acc)[3][BOrd<N>::RT]) {
  if constexpr (!LATE) mat_chunk<N, W>(A, tile, lane, 0, m0);
  vol_lift<N, W, P>(A, F, sq, sg, sF, lane, acc);
  if constexpr (LATE) mat_chunk<N, W>(A, tile, lane, 0, m0);
}

// The stage of one tile: launch position bid of a grid of G positions over
// the context's tiles (G = ceil(K / 16)); the kernels below call it for a
// single context or for one slot of a batch.
template <int N, bool F32, typename T = float, bool RST = false, bool FP = false>
__device__ __forceinline__ void stage_bx_run(const BxArgsT<T>& A, int64_t G, int64_t bid) {
  static_assert(F32 || sizeof(T) == 4, "BF16x3 products work on FP32 data");
  static_assert(!RST || (F32 && sizeof(T) == 4), "R q is stored by the FP32 kernel");
  using O = BOrd<N>;
  using L = BLds<N, T>;
  using V4 = v4_t<T>;
  constexpr int Np = O::Np, Nfp = O::Nfp, NF4 = O::NF4, RT = O::RT;
  constexpr bool plain = sizeof(T) == 8 || FP || (F32 && !bx_three_parts(N));   // FOrd fragments
  constexpr int NP = F32 ? 3 : 2;                   // else split products of NP bf16 parts
  constexpr bool alternate = !plain && NP == 3;     // odd elements negated (see kProd)
  __shared__ __align__(16) T smem[L::BYTES / sizeof(T)];
  T* sq = smem;                   // [9][Np][17]
  T* sg = sq + L::SQ;             // [16][9]
  T* sz = sg + L::SG;             // [2][Np][17]: Z_p, Z_s of the tile's nodes
  T* sF = smem + L::OFF_U;        // [9][NF4][17]  (phases B, C)
  T* sr = sF;                     // [9][Np][17]   (phases D, E)
  bf16x8* srl = reinterpret_cast<bf16x8*>(sF + L::RO);   // wave 2, phase D

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // XCD-aware tile order: consecutive workgroups go round-robin to the eight
  // XCDs, so give each XCD one contiguous range of launch positions; the
  // host's tile order sweeps each range so that face neighbours run close
  // together (neighbour traces then mostly hit that XCD's L2)
  const int64_t xcd = bid & 7, per = G >> 3, rem8 = G & 7;
  const int64_t tile = A.torder[xcd * per + (xcd < rem8 ? xcd : rem8) + (bid >> 3)];
  const int64_t K = A.K;
  const int64_t KNp = K * Np;
  const int64_t e0 = tile * kTile;
  const int ne = int((K - e0) < kTile ? (K - e0) : kTile);
  // component group of this wave, rotated with the tile: the waves of a
  // workgroup go to the CU's four SIMDs in order, so the three-component
  // group of two workgroups sharing a CU then mostly runs on different SIMDs
  const int grp = (wave + int(bid >> 3)) & 3;

  // A: stage q and the metric terms; every thread issues all its loads
  // before the first LDS store (the phase is latency bound otherwise).  The
  // tile's values of field f are the TS = 16 Np consecutive floats at
  // f K Np + e0 Np.  Rows r < 256 MI of every field are read as
  // r = tid + 256 it from a per-field uniform base (no per-item index
  // arithmetic); the TT values left per field are spread over the threads
  // (item t: field t / TT).  Rows past the last element of a ragged tile are
  // clamped to its last value: their columns never reach memory.
  const TileMap<N> tm(ne);
  // Face-node tasks of phase B: one thread per (element, face node),
  // consecutive threads on consecutive face nodes of one element (so that a
  // wave's neighbour gathers fall in a few neighbour elements' lines).  Their
  // loads (neighbour node, face geometry, impedances) are issued here, behind
  // the state loads, and the neighbour gathers right after the state is
  // stored, so that phase B waits for data already in flight.  Slots past
  // the tile (ragged last tile, idx beyond the count) read a valid element
  // and face node and store zero.
  constexpr int TF = kTile * NF4;
  constexpr int IF = (TF + kThreads - 1) / kThreads;
  int vM[IF];
  bool ok[IF];
  T fg[IF][4], qP[IF][9], zpP[IF], zsP[IF];
  unsigned nbi[IF];
  {
    // level 1: the face-node task tables (the gathers depend on nbn), the
    // state, the impedances and the metric terms; level 2: the neighbour
    // gathers.  Issue order matters: the load counter is in order, so the
    // gathers wait for nbn but not for the state loads.
    const int32_t* nbt = A.nbn + e0 * NF4;
    const V4* fgt = reinterpret_cast<const V4*>(A.fgeo) + e0 * 4;
    unsigned ecs[IF];
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = tid + it * kThreads;
      const unsigned ic = min(unsigned(idx), unsigned(TF - 1));
      const unsigned e = ic / NF4, jf = ic - e * NF4;
      ok[it] = idx < TF && int(e) < ne;
      ecs[it] = min(e, unsigned(ne - 1));   // a valid element of the tile
      nbi[it] = unsigned(nbt[ecs[it] * NF4 + jf]);
      vM[it] = A.fmask[jf];
      const V4 g4 = fgt[ecs[it] * 4 + jf / Nfp];
#pragma unroll
      for (int j = 0; j < 4; ++j) fg[it][j] = g4[j];
    }
    __builtin_amdgcn_sched_barrier(0);
    const T* qt = A.q_in + e0 * Np;
    T vm[TileMap<N>::MI > 0 ? TileMap<N>::MI : 1][9], vt[TileMap<N>::IT];
#pragma unroll
    for (int it = 0; it < TileMap<N>::MI; ++it)
#pragma unroll
      for (int f = 0; f < 9; ++f) vm[it][f] = (qt + f * KNp)[tm.main_row(tid, it)];
#pragma unroll
    for (int j = 0; j < TileMap<N>::IT; ++j) vt[j] = qt[tm.tail_field(tid, j) * KNp + tm.tail_row(tid, j)];
    T gv = tid < kTile * 9 && tid / 9 < ne ? A.geo[e0 * 9 + tid] : T(0);
    if (alternate && tid / 9 % 2) gv = -gv;
    constexpr int IZ = (kTile * Np + kThreads - 1) / kThreads;
    T zv[2][IZ];
#pragma unroll
    for (int it = 0; it < IZ; ++it) {
      const unsigned r = min(unsigned(tid + it * kThreads), unsigned(tm.rmax));
      zv[0][it] = (A.zp + e0 * Np)[r];
      zv[1][it] = (A.zs + e0 * Np)[r];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      // a neighbour inside the tile is read from LDS in phase B; its lanes
      // load the tile's first row instead (one hot line for all of them)
      const unsigned lr = unsigned(nbi[it] - unsigned(e0 * Np)) < unsigned(kTile * Np)
                              ? unsigned(e0 * Np) : nbi[it];
#pragma unroll
      for (int f = 0; f < 9; ++f) qP[it][f] = (A.q_in + f * KNp)[lr];
      zpP[it] = A.zp[lr];
      zsP[it] = A.zs[lr];
    }
#pragma unroll
    for (int it = 0; it < TileMap<N>::MI; ++it) {
      const int li = tm.lds_row(tm.main_row(tid, it));
#pragma unroll
      for (int f = 0; f < 9; ++f) sq[f * Np * kES + li] = vm[it][f];
    }
#pragma unroll
    for (int j = 0; j < TileMap<N>::IT; ++j)   // clamped duplicates store equal values
      sq[tm.tail_field(tid, j) * Np * kES + tm.lds_row(tm.tail_row(tid, j))] = vt[j];
    if (tid < kTile * 9) sg[tid] = gv;
#pragma unroll
    for (int it = 0; it < IZ; ++it) {
      const int r = tid + it * kThreads;
      if (r < kTile * Np) {
        const int li = tm.lds_row(unsigned(r));
        sz[li] = zv[0][it];
        sz[Np * kES + li] = zv[1][it];
      }
    }
  }
  __syncthreads();

  // B: face fluxes
  {
#pragma unroll
    for (int it = 0; it < IF; ++it) {
      const int idx = tid + it * kThreads;
      const int e = min(idx / NF4, kTile - 1);
      const int jf = idx - (idx / NF4) * NF4;
      T qM[9];
#pragma unroll
      for (int f = 0; f < 9; ++f) qM[f] = sq[(f * Np + vM[it]) * kES + e];
      const T nx = fg[it][0], ny = fg[it][1], nz = fg[it][2], fs = fg[it][3];
      // neighbour trace: from LDS when the neighbour is in the tile
      const unsigned rl = nbi[it] - unsigned(e0 * Np);
      const bool inT = rl < unsigned(kTile * Np);
      {
        const unsigned rc = inT ? rl : 0u;
        const unsigned en = rc / Np;
        const int ln = int((rc - en * Np) * kES + en);
#pragma unroll
        for (int f = 0; f < 9; ++f) {
          const T x = sq[f * Np * kES + ln];
          qP[it][f] = inT ? x : qP[it][f];
        }
        const T zpl = sz[ln], zsl = sz[Np * kES + ln];
        zpP[it] = inT ? zpl : zpP[it];
        zsP[it] = inT ? zsl : zsP[it];
      }
      const T* P = qP[it];
      const T jtx = (P[3] - qM[3]) * nx + (P[8] - qM[8]) * ny + (P[7] - qM[7]) * nz;
      const T jty = (P[8] - qM[8]) * nx + (P[4] - qM[4]) * ny + (P[6] - qM[6]) * nz;
      const T jtz = (P[7] - qM[7]) * nx + (P[6] - qM[6]) * ny + (P[5] - qM[5]) * nz;
      const T jvx = P[0] - qM[0], jvy = P[1] - qM[1], jvz = P[2] - qM[2];
      if constexpr (RST) {
        // the jumps the adjoint's impedance gradient reads (jt = t(P) - t(M),
        // t = sigma n, the same expressions as the flux's)
        if (A.j_out && ok[it]) {
          V4* jo = reinterpret_cast<V4*>(A.j_out + ((e0 + e) * NF4 + jf) * 8);
          jo[0] = V4{jvx, jvy, jvz, jtx};
          jo[1] = V4{jty, jtz, T(0), T(0)};
        }
      }
      T dvx, dvy, dvz, dtx, dty, dtz;
      if (A.upwind) {
        const int lm = vM[it] * kES + e;
        const T ZpM = sz[lm], ZsM = sz[Np * kES + lm], ZpP = zpP[it], ZsP = zsP[it];
        const T jvn = jvx * nx + jvy * ny + jvz * nz;
        const T jtn = jtx * nx + jty * ny + jtz * nz;
        // reciprocals of the (positive) impedance sums: 1 ulp in FP32
        const T dvn = (ZpP * jvn + jtn) * rcp_t(ZpM + ZpP);
        const T ivs = rcp_t(ZsM + ZsP);
        const T dvtx = (ZsP * (jvx - jvn * nx) + (jtx - jtn * nx)) * ivs;
        const T dvty = (ZsP * (jvy - jvn * ny) + (jty - jtn * ny)) * ivs;
        const T dvtz = (ZsP * (jvz - jvn * nz) + (jtz - jtn * nz)) * ivs;
        dvx = dvn * nx + dvtx;
        dvy = dvn * ny + dvty;
        dvz = dvn * nz + dvtz;
        const T dtn = ZpM * dvn;
        dtx = dtn * nx + ZsM * dvtx;
        dty = dtn * ny + ZsM * dvty;
        dtz = dtn * nz + ZsM * dvtz;
      } else {
        dvx = T(0.5) * jvx; dvy = T(0.5) * jvy; dvz = T(0.5) * jvz;
        dtx = T(0.5) * jtx; dty = T(0.5) * jty; dtz = T(0.5) * jtz;
      }
      T z = ok[it] ? fs : T(0);   // zero flux outside the tile
      if (alternate && e % 2) z = -z;
      T fl[9];
      fl[0] = z * dtx;
      fl[1] = z * dty;
      fl[2] = z * dtz;
      fl[3] = z * dvx * nx;
      fl[4] = z * dvy * ny;
      fl[5] = z * dvz * nz;
      fl[6] = z * T(0.5) * (dvy * nz + dvz * ny);
      fl[7] = z * T(0.5) * (dvx * nz + dvz * nx);
      fl[8] = z * T(0.5) * (dvx * ny + dvy * nx);
      if (idx < TF) {
#pragma unroll
        for (int c = 0; c < 9; ++c) sF[(c * NF4 + jf) * kES + e] = fl[c];
      }
    }
  }
  __syncthreads();

  // C: volume + LIFT per wave (BF16x3 in two bf16 parts, FP32 in three or on the
  // FP32 products, FP64 on the FP64 products)
  V4 acc[3][RT];
  V4 m0[3][2];   // chunk-0 material, in flight during phase C
  const FragsS<N> F(A.frags, O::NFRAG * NP, lane);   // split products
  const FragsF<N, T> FF(A.frags, FOrd<N>::NF4S / 64, lane);
  if constexpr (plain) {
    switch (grp) {
      case 0: mat_chunk<N, 0, T>(A, tile, lane, 0, m0); vol_lift_f<N, 0, T>(FF, sq, sg, sF, lane, acc); break;
      case 1: mat_chunk<N, 1, T>(A, tile, lane, 0, m0); vol_lift_f<N, 1, T>(FF, sq, sg, sF, lane, acc); break;
      case 2: mat_chunk<N, 2, T>(A, tile, lane, 0, m0); vol_lift_f<N, 2, T>(FF, sq, sg, sF, lane, acc); break;
      default: mat_chunk<N, 3, T>(A, tile, lane, 0, m0); vol_lift_f<N, 3, T>(FF, sq, sg, sF, lane, acc); break;
    }
    if constexpr (RST) {
      switch (grp) {
        case 0: store_raw<N, 0>(A, e0, ne, lane, acc); break;
        case 1: store_raw<N, 1>(A, e0, ne, lane, acc); break;
        case 2: store_raw<N, 2>(A, e0, ne, lane, acc); break;
        default: store_raw<N, 3>(A, e0, ne, lane, acc); break;
      }
    }
  } else {
    constexpr bool late = NP == 3;   // the material after the products (registers)
    switch (grp) {
      case 0: split_c<N, 0, NP, late>(A, F, tile, sq, sg, sF, lane, m0, acc); break;
      case 1: split_c<N, 1, NP, late>(A, F, tile, sq, sg, sF, lane, m0, acc); break;
      case 2: split_c<N, 2, NP, late>(A, F, tile, sq, sg, sF, lane, m0, acc); break;
      default: split_c<N, 3, NP, late>(A, F, tile, sq, sg, sF, lane, m0, acc); break;
    }
  }
  __syncthreads();   // fluxes consumed: sr may overwrite them

  // D: quadrature and projection per wave
  if constexpr (plain) {
    switch (grp) {
      case 0: quad_proj_f<N, 0, T>(A, FF, tile, lane, acc, m0, sr); break;
      case 1: quad_proj_f<N, 1, T>(A, FF, tile, lane, acc, m0, sr); break;
      case 2: quad_proj_f<N, 2, T>(A, FF, tile, lane, acc, m0, sr); break;
      default: quad_proj_f<N, 3, T>(A, FF, tile, lane, acc, m0, sr); break;
    }
  } else {
    switch (grp) {
      case 0: quad_proj<N, 0, NP>(A, F, tile, lane, acc, m0, sr, srl); break;
      case 1: quad_proj<N, 1, NP>(A, F, tile, lane, acc, m0, sr, srl); break;
      case 2: quad_proj<N, 2, NP>(A, F, tile, lane, acc, m0, sr, srl); break;
      default: quad_proj<N, 3, NP>(A, F, tile, lane, acc, m0, sr, srl); break;
    }
  }

  // E: right-hand side store or fused stage update, coalesced, done by the
  // three waves other than the three-component one (whose phase D is the
  // longest).  Updater thread u (0..191) owns rows u + 192 it of every
  // field; rows past the tile's last valid row are clamped to it (a
  // duplicate writes the value the row's owner writes).  The residual loads
  // are issued before the barrier, so that they overlap the end of phase D.
  // The thread index is rebuilt from the lane count, which the compiler
  // cannot match with phase A's index arithmetic: otherwise it keeps phase
  // A's addresses alive through the whole kernel to reuse them.
  constexpr int EP = 3 * 64, EI = (kTile * Np + EP - 1) / EP;
  const int64_t t0 = e0 * Np;
  unsigned er[EI];
  T rs[9][EI];
  if (grp != 2) {
    const int u = (grp > 2 ? grp - 1 : grp) * 64 +
                  int(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
#pragma unroll
    for (int it = 0; it < EI; ++it) er[it] = min(unsigned(u + it * EP), unsigned(tm.rmax));
    if (A.lsrk) {
#pragma unroll
      for (int f = 0; f < 9; ++f)
#pragma unroll
        for (int it = 0; it < EI; ++it) rs[f][it] = (A.res + t0 + f * KNp)[er[it]];
    }
  }
  __syncthreads();
  if (grp != 2) {
#pragma unroll
    for (int it = 0; it < EI; ++it) {
      const int li = tm.lds_row(er[it]);
#pragma unroll
      for (int f = 0; f < 9; ++f) {
        const int64_t fb = t0 + f * KNp;
        const T rv = sr[f * Np * kES + li];
        if (A.lsrk) {
          const T rr = A.a * rs[f][it] + A.dt * rv;
          (A.res + fb)[er[it]] = rr;
          (A.q_out + fb)[er[it]] = sq[f * Np * kES + li] + A.b * rr;
        } else {
          (A.rhs_out + fb)[er[it]] = rv;
        }
      }
    }
  }
}

// waves per SIMD that registers have to allow: LDS holds two workgroups per CU at
// order 4, three at orders 1-3 (order 3 would take 171 registers, three more than
// three workgroups leave)
constexpr int bx_waves(int N) { return N == 3 ? 3 : 2; }

template <int N, bool F32>
__global__ __launch_bounds__(kThreads, bx_waves(N)) void stage_bx(BxArgs A) {
  stage_bx_run<N, F32>(A, gridDim.x, blockIdx.x);
}

// The FP32 stage on FP32 products at orders 3 and 4 (FOrd fragments), as stage_bx
// takes them at orders 1 and 2: the forward run of the discrete adjoint.  The face-node jumps that its
// gradients are made of cancel to 1e-5 of the state, so that another rounding of
// the states changes an FP32 gradient by 1e-5 to 1e-3 of its norm, as much as its
// own error; the adjoint therefore keeps these products in all of its parts.
template <int N>
__global__ __launch_bounds__(kThreads, 2) void stage_bx_p(BxArgs A) {
  stage_bx_run<N, true, float, false, true>(A, gridDim.x, blockIdx.x);
}

// The same stage that also stores the raw right-hand side R q of its input
// (r_out) and, for the upwind flux, the jumps at its face nodes (j_out): the
// replay of a checkpoint interval, whose reverse stage needs R y of every stage
// input and, for the impedance gradient, its face-node jumps
template <int N>
__global__ __launch_bounds__(kThreads, 2) void stage_bx_r(BxArgs A) {
  stage_bx_run<N, true, float, true, true>(A, gridDim.x, blockIdx.x);
}

// FP64 stage on the matrix cores (v_mfma_f64_16x16x4f64): the FP32 kernel's
// tiling in double precision.  At order 4 its LDS (124 KiB) holds one
// workgroup per CU, whose waves may then use all 512 registers of a lane.
template <int N>
__global__ __launch_bounds__(kThreads, 1) void stage_bx_d(BxArgsT<double> A) {
  stage_bx_run<N, true, double>(A, gridDim.x, blockIdx.x);
}

}  // namespace dgb

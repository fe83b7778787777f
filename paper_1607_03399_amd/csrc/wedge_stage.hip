// Fused wedge stage kernel of libwdg for CDNA4 (gfx950): volume term,
// surface fluxes and lifts, L^{tri,k} application and the low-storage
// Runge-Kutta update of one stage (Sec. 4.2-4.3).
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>
#include <utility>

#include "device_common.hpp"
#include "ref_tables.inc"
#include "wedge_node.hpp"

namespace wdg {
namespace {

// Highest order whose element triangular mass is factored in the block
// (above: its stored inverse is read), and the LDS a block may take.
#ifndef WDG_CHOL_MAX_N
#define WDG_CHOL_MAX_N 3
#endif
#ifndef WDG_STAGE_LDS
#define WDG_STAGE_LDS 81920
#endif

// Wavefronts per SIMD that the register allocation aims at, one per resident
// block: as many blocks as the LDS of a CU holds where the registers suffice.
#ifndef WDG_W32
#define WDG_W32 {0, 8, 8, 6, 4, 3}
#endif
#ifndef WDG_W64
#define WDG_W64 {0, 5, 4, 3, 2, 2}
#endif
#ifndef WDG_A32
#define WDG_A32 {0, 8, 6, 5, 3, 2}
#endif
#ifndef WDG_A64
#define WDG_A64 {0, 4, 4, 2, 1, 1}
#endif
template <int N, typename T, int MODE>
constexpr int stage_waves() {
  constexpr int w32[6] = WDG_W32, w64[6] = WDG_W64;
  constexpr int a32[6] = WDG_A32, a64[6] = WDG_A64;  // adjoint
  if (MODE == 4) return sizeof(T) == 4 ? a32[N] : a64[N];
  return sizeof(T) == 4 ? w32[N] : w64[N];
}

// Launch shape: four wavefronts per block, one per equation, all over the same
// chunk of EPB = 64 / Nq elements (fewer where the LDS would exceed the cap);
// lane = (element, level j).  (One wavefront with all four equations in its
// registers ran one or two wavefronts per SIMD, and a stage of a small mesh
// lasted its 3480 VALU instructions: with a wavefront per equation, which does
// 1000, two (orders 4 and 5 in FP64) to eight run per SIMD.  us per stage before
// and after: 128 wedges at N = 3 in FP32 11.6 -> 6.8 (with the host's part of
// calls of 20 steps 12.1 -> 7.2), 262 144 wedges 146 -> 142 (HBM: 688 MB at
// 4.9 TB/s); N = 4 / 5 in FP32 on 73 728 wedges 117 / 265 -> 78 / 155; in FP64
// N = 3 on 110 592 160 -> 134, N = 4 on 24 576 264 -> 69.)  LDS holds the staged
// state as four planes and a second region that first holds the triangular operators, geometry records
// and face fluxes, and afterwards the right-hand side, again four planes, on
// its way to the coalesced update.
template <int N, typename T>
struct Cfg {
  static constexpr int NT = Dim<N>::NT, Nq = Dim<N>::Nq, NP = Dim<N>::NP;
  static constexpr int BS = 256;
  // the element's triangular mass M^{tri,k} = sum_v w_v M_v is factored
  // (Cholesky) in the block from the vertex weights of the geometry record;
  // else the stored inverse (lower triangle) is read
  static constexpr bool CHOL = N <= WDG_CHOL_MAX_N;
  static constexpr int VL = Dim<N>::LS / 4, VLS = VL | 1;      // 4-vectors of the triangular operator, LDS stride
  static constexpr int VG = kGeoStride / 4, VGS = VG | 1;      // of the geometry record (odd strides: banks)
  static constexpr int XT = 4 * NT;                            // triangular-face fluxes per element
  static constexpr int NQF = 3 * Nq * Nq;                      // quadrilateral-face nodes per element
  static constexpr int per_elem = (4 * (VLS + VGS) + XT + 2 * NQF + 4 * NP) * int(sizeof(T));
  // N = 2: 20 instead of 21 elements, so that chunks start on whole 128-byte
  // lines (442 368 wedges in FP32: 123.3 -> 119.4 us per stage; at N = 4 and 5
  // whole lines would idle a quarter of the lanes and more)
  static constexpr int EPB_FULL = N == 2 ? 20 : 64 / Nq, EPB_CAP = WDG_STAGE_LDS / per_elem;
  static constexpr int EPB = EPB_FULL < EPB_CAP ? EPB_FULL : EPB_CAP;
  // 4-vectors of the chunk each lane stages and carries through the coalesced update
  static constexpr int UPD = (EPB * NP + BS - 1) / BS;
  // A plane holds NP values per element without padding: at every order the
  // lanes' NT-strided reads then fall on different banks but for pairs.  One
  // spare value takes the lanes past the chunk.
  static constexpr int PL = EPB * NP + 1;
  // 4-vectors of the second region, the last one spare
  static constexpr int XV_ = EPB * (VLS + VGS) + (EPB * (XT + 2 * NQF) + 3) / 4;
  static constexpr int XV = (XV_ > PL ? XV_ : PL) + 1;
  // the adjoint stage: a third set of planes, which later takes the jumps of
  // its faces, behind the right-hand side's (over operators no longer needed)
  static constexpr int JV = (EPB * (6 * Nq * Nq + 4 * NT) + 3) / 4;
  static constexpr int XVG_ = PL + (JV > PL ? JV : PL);
  static constexpr int XVG = XV > XVG_ ? XV : XVG_;
  // Triangular faces: the first Nq / 2 lanes of an element share out the
  // bottom's NT nodes, the others the top's, TPL each (surplus slots redo the
  // last node).  NG: neighbour nodes a lane gathers.
  static constexpr int TPL = (NT + Nq / 2 - 1) / (Nq / 2);
  static constexpr int NG = Nq > TPL ? Nq : TPL;
};

// acc1 += c x1; acc2 += c x2 for a reference-operator entry c known at
// compile time; exact zeros of the operator cost nothing
template <typename T>
__device__ __forceinline__ void constexpr_or_skip(double c, T& acc, T x) {
  if (c != 0.0) acc += T(c) * x;
}

// Entries of the 1D operators that depend on the lane's level, as sums of
// compile-time entries times 0/1 masks of the level (exact: one term is
// non-zero; the masks are hidden from the compiler by an empty asm
// statement, or it makes the selection a load at a selected address, whose
// wait, late in a kernel, waits for every load in flight).  A table in memory
// read with the first loads saves the sums but is one address that all
// wavefronts read: 210 against 155 us per stage on 262 144 wedges at N = 3.
template <int Nq, typename T>
struct LevelMask {
  T m[Nq];
  __device__ __forceinline__ explicit LevelMask(int j) {
#pragma unroll
    for (int jj = 0; jj < Nq; ++jj) {
      m[jj] = j == jj ? T(1) : T(0);
      asm volatile("" : "+v"(m[jj]));
    }
  }
  // sum over the levels jj of f(jj) m[jj]; f maps an integral constant to a constant
  template <typename F, int... J>
  __device__ __forceinline__ T sum(F f, std::integer_sequence<int, J...>) const {
    T v = T(0);
    ((v += m[J] * f(std::integral_constant<int, J>{})), ...);
    return v;
  }
  template <typename F>
  __device__ __forceinline__ T pick(F f) const {
    return sum(f, std::make_integer_sequence<int, Nq>{});
  }
  // rows of a (Nq x Nq) operator: out[m] = f(j, m)
  template <typename F, int... M>
  __device__ __forceinline__ void rows(F f, T* out, std::integer_sequence<int, M...>) const {
    ((out[M] = pick([f](auto jj) { return f(jj, std::integral_constant<int, M>{}); })), ...);
  }
  template <typename F>
  __device__ __forceinline__ void row(F f, T* out) const {
    rows(f, out, std::make_integer_sequence<int, Nq>{});
  }
};

// Sums of products with the rounding spelled out: left to the compiler, which
// product is rounded before the sum may differ between the kernel's modes,
// whose results are the same bit for bit.
template <typename T>
__device__ __forceinline__ T dot2(T a, T x, T b, T y) {
  return std::fma(b, y, a * x);
}
template <typename T>
__device__ __forceinline__ T dot3(T a, T x, T b, T y, T c, T z) {
  return std::fma(c, z, dot2(a, x, b, y));
}

// Factor (a power of two) of an element's mass M^{tri,k} by its first weight, see
// kTinyWeight: the factored mass takes it back in its entries; what the stored
// inverse is applied to is multiplied by it, in the few factors that the
// pre-lift sums and the moments are linear in (a branch around a scaling of the
// sums themselves cost a stage of 1024 wedges at N = 4 0.3 us of 8.7).
template <typename T>
__device__ __forceinline__ T mass_unit(T w0) {
  return sizeof(T) == 4 && w0 < T(kTinyWeight) ? T(kTinyUp) : T(1);
}

// 1 / x and 1 / sqrt(x) of positive normal numbers (sums of impedances, whose
// reciprocals the records hold as normal numbers too; a factor's pivots, see
// tiny) to about one unit in the last place: the hardware approximation refined by Newton steps (in place of
// the division and square root sequences, which also cover the special
// values: 250 of the 604 instructions of the factor below at N = 3)
__device__ __forceinline__ float inv(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return std::fma(r, std::fma(-x, r, 1.0f), r);
}
__device__ __forceinline__ double inv(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = std::fma(r, std::fma(-x, r, 1.0), r);
  return std::fma(r, std::fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float inv_sqrt(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return std::fma(0.5f * r, std::fma(-x * r, r, 1.0f), r);
}
__device__ __forceinline__ double inv_sqrt(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = std::fma(0.5 * r, std::fma(-x * r, r, 1.0), r);
  return std::fma(0.5 * r, std::fma(-x * r, r, 1.0), r);
}

// A wedge's accumulators across the reverse sweep: FP64 sums; FP32 Kahan
// (compensated) sums, the record holding the sums, then their compensations.
// Read early (grad_record_load), then one stage's terms x[kGradStride] added
// and written back (grad_record_add).
template <typename T>
struct GradRecord {
  T v[kGradRecord<T>];
};
template <typename T>
__device__ __forceinline__ void grad_record_load(const void* gacc, int64_t e, GradRecord<T>& r) {
  const T* ga = static_cast<const T*>(gacc) + e * kGradRecord<T>;
#pragma unroll
  for (int k = 0; k < kGradRecord<T>; ++k) r.v[k] = ga[k];
}
template <typename T>
__device__ __forceinline__ void grad_record_add(void* gacc, int64_t e, const GradRecord<T>& r, const T* x) {
  T* ga = static_cast<T*>(gacc) + e * kGradRecord<T>;
  if constexpr (sizeof(T) == 8) {
#pragma unroll
    for (int k = 0; k < kGradStride; ++k) ga[k] = r.v[k] + x[k];
  } else {
#pragma unroll
    for (int k = 0; k < kGradStride; ++k) {
      const T y = x[k] - r.v[kGradStride + k];
      const T t = r.v[k] + y;
      ga[kGradStride + k] = (t - r.v[k]) - y;
      ga[k] = t;
    }
  }
}

// Gradient terms of one reverse stage of the adjoint sweep (MODE 4), run by
// the stage kernel after its update.  Per wedge it accumulates the mass terms
// b_s U~_p^T M res_p, b_s U~_u^T M res_u (their sum over a step's stages is
// that of dt sig_p^T M R_p, dt sig_u^T M R_u with R_s the stage's right-hand
// side; as dJ/dc = 2/(c kappa) m_p, dJ/drho = m_p/(rho kappa) + m_u) and per
// face dt times the face integrals 1/2 int sig_p [p], 1/2 int sig_un [u_n] of
// Us weighted by the penalties' derivatives (gacc slots 2..6), which the
// combine kernel adds up over both sides of every face.  sig is the stage
// input (the adjoint stage vector), U~ the incoming adjoint state, res_s the
// forward residual after stage s, Us the forward stage input.
// M^k = (sum_v w_v M_v) (x) M^1D and the face masses are literals (reference
// triangle, 1D, edge masses).  The wavefronts share the work as the stage
// does: each the mass term of its field; p, u_x, u_y one quadrilateral face
// each, u_z the triangular faces, whose nodes and fields its lanes share out.
// Bound by HBM and by the loads that the blocks of a CU keep in flight: sig
// stays in LDS beside U~, a third set of planes (res_s, then the jumps of Us)
// and the geometry values it reads; res_s and the gathers are loaded before
// the update's stores, which a later load would wait for, and Us over the mass
// terms, so that registers hold loads in flight only: at N = 3 in FP32 96 of
// them and 32 KB, five blocks per CU.  us per reverse stage with sig, geometry
// and all loads in registers (158, three blocks) and as it is: N = 3 in FP32 on
// 524 288 wedges 560 -> 506 (4.3 TB/s), N = 5 on 73 728 592 -> 328, N = 3 in FP64
// on 110 592 403 -> 290.
template <int N, typename T>
struct EpiData {
  using C = Cfg<N, T>;
  V4<T> b[C::UPD];  // the chunk's res_s, coalesced
  V4<T> gn[C::NG];  // neighbour nodes of Us on the lane's faces
  bool inner;       // a neighbour across the lane's face
};
// what it reads of the geometry records: values kEpi0 .. kGeoStride - 1
constexpr int kEpi0 = 9, kEpiStride = kGeoStride - kEpi0;
template <int N, typename T>
__device__ __forceinline__ void grad_load(const StageLaunch& A, int64_t e0, int nE, int tid, int f, int j, int64_t e,
                                          int nbr, int code, const T* sG, T* sE, EpiData<N, T>& L) {
  using C = Cfg<N, T>;
  constexpr int NT = C::NT, Nq = C::Nq, NP = C::NP, NG = C::NG, V4B = 4 * int(sizeof(T));
  const auto bb = chunk_rsrc(static_cast<const V4<T>*>(A.gRs) + e0 * NP, int64_t(nE) * NP * V4B);
#pragma unroll
  for (int k = 0; k < C::UPD; ++k) L.b[k] = bload<T, kStream>(bb, tid + C::BS * k);
  // the neighbour nodes of the stage's gathers (own element on the boundary):
  // the branches choose the nodes, the loads are common
  const int face = j < Nq / 2 ? 0 : 1, ti0 = (face ? j - Nq / 2 : j) * C::TPL;
  const V4<T>* nb = static_cast<const V4<T>*>(A.gUs) + (nbr >= 0 ? int64_t(nbr) : e) * NP;
  int off[NG];
  if (f != 1) {
    const int ned = (code >> (8 + 2 * (f == 0 ? 0 : f - 1))) & 3;
    nb += j * NT;
#pragma unroll
    for (int q = 0; q < NG; ++q)
      off[q] = q >= Nq ? 0
                       : (ned == 0 ? edge_node(N, 0, N - q) : (ned == 1 ? edge_node(N, 1, N - q) : edge_node(N, 2, N - q)));
  } else {
    const int pc = (code >> (3 * face)) & 7;
    nb += (((code >> (6 + face)) & 1) ? N : 0) * NT;
#pragma unroll
    for (int t = 0; t < NG; ++t) off[t] = face_perm<N>(pc, t < C::TPL && ti0 + t < NT ? ti0 + t : NT - 1);
  }
#pragma unroll
  for (int t = 0; t < Nq; ++t) L.gn[t] = nb[off[t]];
  if (f == 1) {
#pragma unroll
    for (int t = Nq; t < NG; ++t) L.gn[t] = nb[off[t]];
  }
  L.inner = nbr >= 0;
  // the records' copy, before the right-hand side replaces them
  for (int i = tid; i < C::EPB * kEpiStride; i += C::BS) {
    const int el = i / kEpiStride;
    sE[i] = sG[el * 4 * C::VGS + kEpi0 + i - el * kEpiStride];
  }
}

template <int N, typename T>
__device__ __forceinline__ void grad_epilogue(const StageLaunch& A, int tid, int f, int le, int j, bool active,
                                              int64_t e0, int nE, const T* sU, T* sX, T* sV, const T* sE,
                                              const EpiData<N, T>& L) {
  using C = Cfg<N, T>;
  using RT = gen::RefTables<N>;
  constexpr int NT = C::NT, Nq = C::Nq, NP = C::NP, EPB = C::EPB, PL = C::PL;
  constexpr int GS = 3;  // partial sums per lane: mass term, face p, face u_n
  static_assert(4 * EPB * Nq * GS <= 4 * PL, "partial sums fit the second region");
  const T bsign = (A.flags & kDirichlet) ? T(-1) : T(1);
  const int ed = f == 0 ? 0 : f - 1;
  const int le0 = active ? le : 0;
  const int lb = le0 * NP + j * NT;  // the lane's level in a plane
  const T* const g = sE + le0 * kEpiStride - kEpi0;  // the element's geometry record from kEpi0 on
  // quadrilateral face: J_f at its vertices, n_x, n_y; triangular face (level j < Nq / 2: bottom): J_f, n
  const int face = j < Nq / 2 ? 0 : 1, ti0 = (face ? j - Nq / 2 : j) * C::TPL;
  const T* const fg = g + (f != 1 ? 20 + 4 * ed : 12 + 4 * face);
  auto put = [&](T* s, int k, const V4<T>& v) {
    const int l = tid + C::BS * k < EPB * NP ? tid + C::BS * k : EPB * NP;
    s[l] = v.p;
    s[PL + l] = v.uz;
    s[2 * PL + l] = v.ux;
    s[3 * PL + l] = v.uy;
  };
  // own node of the wavefront's quadrilateral face
  auto qnode = [&](int q) {
    return lb + (ed == 0 ? edge_node(N, 0, q) : (ed == 1 ? edge_node(N, 1, q) : edge_node(N, 2, q)));
  };
#pragma unroll
  for (int k = 0; k < C::UPD; ++k) put(sV, k, L.b[k]);  // res_s
  V4<T> a[C::UPD];  // the chunk's Us, in flight over the mass terms
  {
    const auto ba = chunk_rsrc(static_cast<const V4<T>*>(A.gUs) + e0 * NP, int64_t(nE) * NP * 4 * int(sizeof(T)));
#pragma unroll
    for (int k = 0; k < C::UPD; ++k) a[k] = bload<T>(ba, tid + C::BS * k);
  }
  __syncthreads();  // the update is done; U~, res_s complete

  // Mass terms.  The stage's right-hand side R_s enters as sig_s^T M R_s; with
  // dt R_s = res_s - a_s res_{s-1} (a_1 = 0) the sum over a step's stages equals
  // the sum of (sig_s - a_{s+1} sig_{s+1})^T M res_s / dt, and the reverse sweep
  // has sig_s - a_{s+1} sig_{s+1} = b_s U~, U~ the adjoint state this stage
  // reads (left in the second LDS region by the update).  So the forward
  // keeps its residuals instead of writing every right-hand side.
  // On this level: U~^T (M^{tri,k} (x) M^1D) res_s, M^{tri,k} = sum_v w_v M_v.
  T m1[Nq];
  {
    const LevelMask<Nq, T> lm(j);
    lm.row([](auto jj, auto m) { constexpr T v = T(RT::M1[jj * Nq + m]); return v; }, m1);
  }
  T mass = 0;
  {
    const T w0 = g[37], w1 = g[38], w2 = g[39];
    const T* const rs = sV + f * PL + le0 * NP;
    const T* const ua = sX + f * PL + lb;
    T y[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      T s = 0;
#pragma unroll
      for (int m = 0; m < Nq; ++m) s += m1[m] * rs[m * NT + i];
      y[i] = s;
    }
    // M^{tri,k} is symmetric: each entry is formed once and used for both
    // rows (left to the compiler, all of them stay in registers)
    T z[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) z[i] = T(0);
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      if (i % 2 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int k = 0; k <= i; ++k) {
        T m = 0;
        constexpr_or_skip(RT::Mv[i * NT + k], m, w0);
        constexpr_or_skip(RT::Mv[NT * NT + i * NT + k], m, w1);
        constexpr_or_skip(RT::Mv[2 * NT * NT + i * NT + k], m, w2);
        z[i] += m * y[k];
        if (k < i) z[k] += m * y[i];
      }
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) mass += ua[i] * z[i];
  }
  // (left alone, the sum moves below the barriers with its operands in registers)
  asm volatile("" : "+v"(mass));
  __syncthreads();  // U~ and res_s in LDS are consumed
#pragma unroll
  for (int k = 0; k < C::UPD; ++k) put(sX, k, a[k]);  // Us
  __syncthreads();

  // jumps of Us (over res_s): quadrilateral faces [edge][wedge][level][p, u_n][node],
  // then triangular ones [wedge][face][p, u_n][node]; boundary faces see the mirror state
  T* const sT = sV + EPB * 6 * Nq * Nq;
  if (f != 1) {
    T* const o = sV + ((ed * EPB + le0) * Nq + j) * Nq * 2;
#pragma unroll
    for (int q = 0; q < Nq; ++q) {
      const int i = qnode(q);
      const T pm = sX[i], unm = fg[2] * sX[2 * PL + i] + fg[3] * sX[3 * PL + i];
      const T pp = L.inner ? L.gn[q].p : bsign * pm;
      const T unp = L.inner ? fg[2] * L.gn[q].ux + fg[3] * L.gn[q].uy : -bsign * unm;
      if (active) {
        o[q] = pp - pm;
        o[Nq + q] = unp - unm;
      }
    }
  } else {
    T* const o = sT + (le0 * 2 + face) * 2 * NT;
#pragma unroll
    for (int t = 0; t < C::TPL; ++t) {
      const int i = ti0 + t < NT ? ti0 + t : NT - 1;
      const int l = le0 * NP + face * N * NT + i;
      const T pm = sX[l];
      const T unm = fg[1] * sX[2 * PL + l] + fg[2] * sX[3 * PL + l] + fg[3] * sX[PL + l];
      const T pp = L.inner ? L.gn[t].p : bsign * pm;
      const T unp =
          L.inner ? fg[1] * L.gn[t].ux + fg[2] * L.gn[t].uy + fg[3] * L.gn[t].uz : -bsign * unm;
      if (active) {
        o[i] = pp - pm;
        o[NT + i] = unp - unm;
      }
    }
  }
  __syncthreads();  // jumps complete; Us in LDS is consumed

  // against the trace of sig times the face mass
  T fp = 0, fn = 0;
  if (f != 1) {
    T sp[Nq], sn[Nq], ap[Nq], an[Nq];
#pragma unroll
    for (int q = 0; q < Nq; ++q) {
      const int i = qnode(q);
      sp[q] = sU[i];
      sn[q] = fg[2] * sU[2 * PL + i] + fg[3] * sU[3 * PL + i];
    }
#pragma unroll
    for (int qq = 0; qq < Nq; ++qq) {
      T vpa = 0, vna = 0, vpb = 0, vnb = 0;
#pragma unroll
      for (int q = 0; q < Nq; ++q) {
        constexpr_or_skip(RT::Ma[q * Nq + qq], vpa, sp[q]);
        constexpr_or_skip(RT::Ma[q * Nq + qq], vna, sn[q]);
        constexpr_or_skip(RT::Mb[q * Nq + qq], vpb, sp[q]);
        constexpr_or_skip(RT::Mb[q * Nq + qq], vnb, sn[q]);
      }
      ap[qq] = fg[0] * vpa + fg[1] * vpb;
      an[qq] = fg[0] * vna + fg[1] * vnb;
    }
    // quadrilateral faces: couple the levels through M^1D
    const T* const sj = sV + (ed * EPB + le0) * Nq * Nq * 2;
#pragma unroll
    for (int m = 0; m < Nq; ++m) {
      T tp = 0, tn = 0;
#pragma unroll
      for (int qq = 0; qq < Nq; ++qq) {
        tp += ap[qq] * sj[m * 2 * Nq + qq];
        tn += an[qq] * sj[m * 2 * Nq + Nq + qq];
      }
      fp += m1[m] * tp;
      fn += m1[m] * tn;
    }
    fp *= T(0.5);
    fn *= T(0.5);
  } else {
    // sum_i sig_i sum_k Mtri[i][k] jump_k of one field; where a face has two
    // lanes, the first takes p and the others u_n
    auto contract = [&](bool un) {
      const T* const jmp = sT + (le0 * 2 + face) * 2 * NT + (un ? NT : 0);
      const T* const sg = sU + le0 * NP + face * N * NT;
      T x[NT], s = 0;
#pragma unroll
      for (int k = 0; k < NT; ++k) x[k] = jmp[k];
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        T v = 0;
#pragma unroll
        for (int k = 0; k < NT; ++k) constexpr_or_skip(RT::Mtri[i * NT + k], v, x[k]);
        const T t = un ? fg[1] * sg[2 * PL + i] + fg[2] * sg[3 * PL + i] + fg[3] * sg[PL + i] : sg[i];
        s += t * v;
      }
      return s * (T(0.5) * fg[0]);
    };
    if constexpr (Nq / 2 > 1) {
      fp = fn = contract(ti0 > 0);
    } else {
      fp = contract(false);
      fn = contract(true);
    }
  }
  // the wedge's accumulators, read after the contractions (14 registers that
  // would be held through them)
  const bool last = f == 0 && active && j == 0;
  GradRecord<T> rec;
  if (last) grad_record_load<T>(A.gacc, e0 + le, rec);
  if (active) {
    T* const o = sX + ((f * EPB + le) * Nq + j) * GS;
    o[0] = mass;
    o[1] = fp;
    o[2] = fn;
  }
  __syncthreads();
  if (last) {
    auto part = [&](int w, int l, int k) { return sX[((w * EPB + le) * Nq + l) * GS + k]; };
    T mp = 0, mu = 0, tp[5], tn[5];
#pragma unroll
    for (int l = 0; l < Nq; ++l) {
      mp += part(0, l, 0);
      mu += part(1, l, 0) + part(2, l, 0) + part(3, l, 0);
    }
    constexpr int top = Nq / 2, un = Nq / 2 > 1 ? 1 : 0;  // lanes of the top face; of u_n beside p
    tp[0] = part(1, 0, 1);
    tn[0] = part(1, un, 2);
    tp[1] = part(1, top, 1);
    tn[1] = part(1, top + un, 2);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int w = d == 0 ? 0 : d + 1;
      tp[2 + d] = tn[2 + d] = T(0);
#pragma unroll
      for (int l = 0; l < Nq; ++l) {
        tp[2 + d] += part(w, l, 1);
        tn[2 + d] += part(w, l, 2);
      }
    }
    const T kap = g[9], irho = g[10];
    const T c = std::sqrt(kap * irho);
    const T dt = T(A.dt);
    T x[kGradStride];
    const T gb = T(A.gb);  // dt times the mass terms' factor b_s / dt
    x[0] = gb * T(2) / (c * kap) * mp;
    x[1] = gb * (mp * irho / kap + mu);
    // per face dtau_p/dZ = -tau_p^2 / 2, dtau_u/dZ = 1/2 (upwind, tau_p = 2 / (Z- + Z+);
    // the central flux has no penalties)
    const bool upwind = !(A.flags & kCentral);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const T t = T(2) / g[32 + k];  // Z- + Z+
      x[2 + k] = upwind ? dt * (-T(0.5) * t * t * tp[k] - T(0.5) * tn[k]) : T(0);
    }
    grad_record_add<T>(A.gacc, e0 + le, rec, x);
  }
}

// ---------------------------------------------------------------------------
// Fused stage kernel
//
// Lane (element, level j) of wavefront f owns the triangular slice j of its
// element for equation f.  The reference triangle and 1D operators are
// compile-time constants (instruction literals).  The chunk's state, geometry
// and connectivity are staged in LDS with coalesced loads; the vertical
// derivative and the triangle-face lifts couple the levels of one element
// through it.
//   phase 1: face fluxes (p, u_x, u_y: one quadrilateral face each; u_z: the
//            triangular faces and the factor of M^{tri,k}) to LDS;
//            B = -W (vertical part of D_x, D_y, D_z, before L^{tri,k})
//   phase 2: B += triangular-face lifts; R = (M^{tri,k})^-1 (M^tri B +
//            quadrilateral-face moments) + H (horizontal part); scale by
//            kappa, 1/rho; sources
//   update:  R goes through LDS so that the low-storage Runge-Kutta update
//            reads and writes res and U with fully coalesced accesses
// MODE 0: wedges only; 1: tetrahedra across triangular faces; 2: also mortars;
// 3: wedges only, vertical neighbours inside the chunk read from LDS (layer marching);
// 4: wedges only, adjoint stage with its gradient terms (grad_epilogue);
// 5: as 3 for one chunk of a column marched from the bottom (wedge_column_stage):
//    the wedge below the chunk's first one is the previous chunk's last, whose
//    top level the previous call left in carry (when has_carry); this call
//    leaves its own last wedge's top level there.
// The chunk holds wedges e0 .. e0 + nE - 1 (nE <= EPB).
template <int N, typename T, int MODE>
__device__ __forceinline__ void wedge_stage_chunk(const StageLaunch& A, int64_t e0, int nE, V4<T>* carry = nullptr,
                                                  bool has_carry = false) {
  constexpr bool HYB = MODE == 1 || MODE == 2;
  constexpr bool MARCH = MODE == 3 || MODE == 5;
  using C = Cfg<N, T>;
  using RT = gen::RefTables<N>;
  constexpr int NT = C::NT, Nq = C::Nq, NP = C::NP, EPB = C::EPB, BS = C::BS, PL = C::PL;
  constexpr int VL = C::VL, VG = C::VG, VLS = C::VLS, GS = 4 * C::VGS, UPD = C::UPD;
  constexpr int V4B = 4 * int(sizeof(T));
  __shared__ T sU[4 * PL];  // planes p, u_z, u_x, u_y (the spare value of each takes the lanes past the chunk)
  __shared__ V4<T> sX[MODE == 4 ? C::XVG : C::XV];
  [[maybe_unused]] __shared__ T sE[MODE == 4 ? EPB * kEpiStride : 1];
  V4<T>* const sL = sX;
  T* const sG = reinterpret_cast<T*>(sX + EPB * VLS);
  T* const sF = sG + EPB * GS;       // triangular-face fluxes [F_p, F_u][element][face][node]
  T* const sQ = sF + EPB * C::XT;    // quadrilateral-face fluxes [F_p, F_u][element][edge][level][node]
  T* const sR = reinterpret_cast<T*>(sX);  // right-hand side, planes as sU

  const V4<T>* __restrict__ Uin = static_cast<const V4<T>*>(A.Uin);
  const T* __restrict__ geo = static_cast<const T*>(A.geo);
  const int* __restrict__ conn = A.conn;

  int tid = threadIdx.x;
  // marching a column, each chunk derives its lane constants anew: hoisted
  // out of the column loop they would stay live across chunks and spill
  if constexpr (MODE == 5) asm volatile("" : "+v"(tid));
  // the equation of this wavefront, in plane order: 0 p, 1 u_z, 2 u_x, 3 u_y
  const int f = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int ed = f == 0 ? 0 : f - 1;  // its quadrilateral face (not for u_z)
  const int le = lane / Nq;
  const int j = lane - le * Nq;
  const bool active = lane < EPB * Nq && le < nE;
  const int64_t e = e0 + (active ? le : 0);  // idle lanes shadow a valid element
  const T bsign = (A.flags & kDirichlet) ? T(-1) : T(1);
  const T tau_on = (A.flags & kCentral) ? T(0) : T(1);
  // triangular faces: see Cfg::TPL
  constexpr int per = C::TPL;
  const int face = j < Nq / 2 ? 0 : 1;
  const int ti0 = (face ? j - Nq / 2 : j) * per;

  // The lane's own connectivity is read first and the neighbour gathers are
  // issued as soon as it arrives, while the chunk's coalesced staging loads
  // are still in flight: both memory latencies overlap.
  // (Named values, not an array: a lane-dependent selection from a private
  // array becomes a scratch load.)
  const int4* cp = reinterpret_cast<const int4*>(conn + e * kConnStride);
  const int4 c0 = cp[0], c1 = cp[1];
  const int nb0 = c0.x, nb1 = c0.y, code = c1.y;            // across the bottom and top triangles
  const int nbq[3] = {c0.z, c0.w, c1.x};                    // across the quadrilaterals
  const int qnbr = ed == 0 ? nbq[0] : (ed == 1 ? nbq[1] : nbq[2]);
  constexpr int SL = C::CHOL ? 0 : (EPB * VL + BS - 1) / BS, SG = (EPB * VG + BS - 1) / BS;
  V4<T> rU[UPD], rL[SL > 0 ? SL : 1], rG[SG];
  {
    const auto bu = chunk_rsrc(Uin + e0 * NP, int64_t(nE) * NP * V4B);
    const auto bg = chunk_rsrc(geo + e0 * kGeoStride, int64_t(nE) * VG * V4B);
#pragma unroll
    for (int k = 0; k < UPD; ++k) rU[k] = bload<T>(bu, tid + BS * k);
    if constexpr (!C::CHOL) {
      const auto bl = chunk_rsrc(static_cast<const T*>(A.L) + e0 * Dim<N>::LS, int64_t(nE) * VL * V4B);
#pragma unroll
      for (int k = 0; k < SL; ++k) rL[k] = bload<T>(bl, tid + BS * k);
    }
#pragma unroll
    for (int k = 0; k < SG; ++k) rG[k] = bload<T>(bg, tid + BS * k);
  }
  const int tnbr = face ? nb1 : nb0;
  const int tpc = (code >> (3 * face)) & 7, tlev = ((code >> (6 + face)) & 1) ? N : 0;
  // the neighbours' face vertices in the own order (vertex permutation 0) all
  // over the wavefront: as on meshes layered column by column
  const bool plain = __builtin_amdgcn_ballot_w64(tpc != 0) == 0;
  // The branches below only choose the nodes (element base and offsets); the
  // loads are common to all wavefronts, but for the ones that the triangular
  // faces need beyond Nq.  (Loads of both branches into one array are merged
  // by the compiler component by component, and two arrays cost 16 registers
  // at N = 3: on 262 144 wedges 215 and 149 us per stage.)
  constexpr int NG = C::NG;
  const V4<T>* nb;
  int off[NG];
  bool skip = false;  // layer marching: read from the staged chunk instead
  if (f != 1) {
    // neighbour nodes of the wavefront's quadrilateral face on this level
    // (boundary faces read the own element, a valid address; the mirror state
    // is blended in later)
    const int ned = (code >> (8 + 2 * ed)) & 3;
    nb = Uin + (qnbr >= 0 ? int64_t(qnbr) : e) * NP + j * NT;
#pragma unroll
    for (int q = 0; q < NG; ++q)
      off[q] = q >= Nq ? 0
                       : (ned == 0 ? edge_node(N, 0, N - q) : (ned == 1 ? edge_node(N, 1, N - q) : edge_node(N, 2, N - q)));
  } else {
    // triangular-face neighbour nodes
    // Layer marching (MODE 3): a chunk is a run of consecutive layers of one
    // column, so the wedge below or above usually sits in the same chunk; its
    // face nodes are then read from the staged chunk after the barrier instead
    // of being gathered from memory.
    const int64_t src = tnbr >= 0 ? int64_t(tnbr) : e;
    nb = Uin + src * NP + tlev * NT;
    bool tet = false;
    if constexpr (HYB) {
      // a tetrahedron neighbour: its nodes follow all wedge nodes
      tet = src >= A.Kw;
      if (tet) nb = Uin + A.Kw * NP + (src - A.Kw) * TDim<N>::NP;
    }
    if constexpr (MARCH) {
      skip = (tnbr >= 0 && src >= e0 && src < e0 + nE) ||
             (MODE == 5 && has_carry && tnbr >= 0 && src == e0 - 1 && tlev == N);
    }
#pragma unroll
    for (int t = 0; t < NG; ++t) off[t] = t < per && ti0 + t < NT ? ti0 + t : NT - 1;
    if (!plain) {
#pragma unroll
      for (int t = 0; t < per; ++t) off[t] = face_perm<N>(tpc, off[t]);
    }
    if constexpr (HYB) {
#pragma unroll
      for (int t = 0; t < per; ++t)
        off[t] = tet ? tet_face_node<N>((code >> (14 + 2 * face)) & 3, off[t]) : off[t];
    }
  }
  V4<T> gn[NG];
#pragma unroll
  for (int t = 0; t < Nq; ++t) {
    if constexpr (MARCH) gn[t] = V4<T>{T(0), T(0), T(0), T(0)};
    if (!MARCH || !skip) gn[t] = nb[off[t]];
  }
  if (f == 1) {
#pragma unroll
    for (int t = Nq; t < NG; ++t) {
      if constexpr (MARCH) gn[t] = V4<T>{T(0), T(0), T(0), T(0)};
      if (!MARCH || !skip) gn[t] = nb[off[t]];
    }
  }
#pragma unroll
  for (int k = 0; k < UPD; ++k) {
    const int idx = tid + BS * k < EPB * NP ? tid + BS * k : EPB * NP;
    sU[idx] = rU[k].p;
    sU[PL + idx] = rU[k].uz;
    sU[2 * PL + idx] = rU[k].ux;
    sU[3 * PL + idx] = rU[k].uy;
  }
#pragma unroll
  for (int k = 0; k < SL; ++k) {
    const int idx = tid + BS * k;
    sX[idx < EPB * VL ? idx + (idx / VL) * (VLS - VL) : C::XV - 1] = rL[k];
  }
#pragma unroll
  for (int k = 0; k < SG; ++k) {
    const int idx = tid + BS * k;
    sX[idx < EPB * VG ? EPB * VLS + idx + (idx / VG) * (C::VGS - VG) : C::XV - 1] = rG[k];
  }
  __syncthreads();

  const T* const elp = sU + (active ? le : 0) * NP;  // the element's planes
  const T* const elz = elp + PL;
  const T* const elx = elp + 2 * PL;
  const T* const ely = elp + 3 * PL;
  const T* g = sG + (active ? le : 0) * GS;
  // what the stored inverse is applied to is multiplied by this
  const T up = C::CHOL ? T(1) : mass_unit(g[37]);

  // face fluxes
  if (f != 1) {
    const T w_in = qnbr >= 0 ? T(1) : T(0);
    const T nx = g[22 + 4 * ed], ny = g[23 + 4 * ed];
    const T zs = g[34 + ed];  // Z- + Z+ (= 2 Z- on the boundary)
    const T taup = tau_on * T(2) * inv(zs);
    const T tauu = tau_on * zs * T(0.5);
    T fp[Nq], fu[Nq];
#pragma unroll
    for (int q = 0; q < Nq; ++q) {
      const int i = j * NT + (ed == 0 ? edge_node(N, 0, q) : (ed == 1 ? edge_node(N, 1, q) : edge_node(N, 2, q)));
      const V4<T> v = gn[q];
      const T pm = elp[i];
      const T unm = dot2(nx, elx[i], ny, ely[i]);
      // mirror state: p+ = s p-, u_n+ = -s u_n- (s = -1 Dirichlet, +1 rigid)
      const T pb = bsign * pm, ub = -bsign * unm;
      const T pp = pb + w_in * (v.p - pb);
      // (u_z enters with weight zero, which keeps the gather one 16-byte load)
      const T unp = ub + w_in * (dot3(nx, v.ux, ny, v.uy, T(0), v.uz) - ub);
      const T jp = pp - pm, jun = unp - unm;
      fp[q] = T(0.5) * (taup * jp - jun);
      fu[q] = T(0.5) * (tauu * jun - jp);
    }
    if (active) {
      T* const o = sQ + ((le * 3 + ed) * Nq + j) * Nq;
#pragma unroll
      for (int q = 0; q < Nq; ++q) o[q] = fp[q];
#pragma unroll
      for (int q = 0; q < Nq; ++q) o[EPB * C::NQF + q] = fu[q];
    }
  } else {
    if constexpr (MARCH) {
      const int64_t ln = int64_t(tnbr) - e0;
#pragma unroll
      for (int t = 0; t < per; ++t) {
        const int i = ti0 + t < NT ? ti0 + t : NT - 1;
        const int fn = face_perm<N>(tpc, i);
        if (tnbr >= 0 && ln >= 0 && ln < nE) {
          const T* s = sU + int(ln) * NP + tlev * NT + fn;
          gn[t] = V4<T>{s[0], s[PL], s[2 * PL], s[3 * PL]};
        } else if (MODE == 5 && has_carry && tnbr >= 0 && ln == -1 && tlev == N) {
          gn[t] = carry[fn];
        }
      }
    }
    // triangular-face fluxes (premultiplied by J_f) go to LDS for every level
    const T w_in = tnbr >= 0 ? T(1) : T(0);
    const T* gf = g + 12 + 4 * face;
    const T Jf = T(0.5) * gf[0], nx = gf[1], ny = gf[2], nz = gf[3];
    const T zs = g[32 + face];
    const T taup = tau_on * T(2) * inv(zs);
    const T tauu = tau_on * zs * T(0.5);
    const int own = face * N * NT;
#pragma unroll
    for (int t = 0; t < per; ++t) {
      const int i = ti0 + t < NT ? ti0 + t : NT - 1;
      const V4<T> v = gn[t];
      const T pm = elp[own + i];
      const T unm = dot3(nx, elx[own + i], ny, ely[own + i], nz, elz[own + i]);
      const T pb = bsign * pm, ub = -bsign * unm;
      const T pp = pb + w_in * (v.p - pb);
      const T unp = ub + w_in * (dot3(nx, v.ux, ny, v.uy, nz, v.uz) - ub);
      const T jp = pp - pm, jun = unp - unm;
      if (active) {
        sF[(le * 2 + face) * NT + i] = Jf * (taup * jp - jun);
        sF[EPB * 2 * NT + (le * 2 + face) * NT + i] = Jf * (tauu * jun - jp);
      }
    }
    if constexpr (C::CHOL) {
      // M^{tri,k} = L L^T, row by row into the element's triangular-operator
      // slots (entry (i, m) at i (i + 1) / 2 + m, the diagonal holding 1 / L_ii)
      if (active && j == 0) {
        constexpr int NK = Dim<N>::NPK;
        T w0 = g[37], w1 = g[38], w2 = g[39];
        const T unit = mass_unit(w0);
        const bool small = unit != T(1);
        if (__builtin_amdgcn_ballot_w64(small)) {
          w0 *= unit;
          w1 *= unit;
          w2 *= unit;
        }
        T a[4 * VL];
#pragma unroll
        for (int q = 0; q < NK; ++q) {
          const int i = tri_row(q), m = q - i * (i + 1) / 2;
          T v = 0;
          constexpr_or_skip(RT::Mv[i * NT + m], v, w0);
          constexpr_or_skip(RT::Mv[NT * NT + i * NT + m], v, w1);
          constexpr_or_skip(RT::Mv[2 * NT * NT + i * NT + m], v, w2);
          a[q] = v;
        }
#pragma unroll
        for (int q = 0; q < NK; ++q) {
          const int i = tri_row(q), m = q - i * (i + 1) / 2;
          T sm = a[q];
#pragma unroll
          for (int k = 0; k < m; ++k) sm -= a[i * (i + 1) / 2 + k] * a[m * (m + 1) / 2 + k];
          a[q] = m < i ? sm * a[m * (m + 1) / 2 + m] : inv_sqrt(sm);
        }
        if (__builtin_amdgcn_ballot_w64(small)) {
          // the factor itself: 2^96 = (2^48)^2
          const T d = small ? T(0x1p48) : T(1), o = small ? T(0x1p-48) : T(1);
#pragma unroll
          for (int q = 0; q < NK; ++q) a[q] *= q == tri_row(q) * (tri_row(q) + 3) / 2 ? d : o;
        }
#pragma unroll
        for (int q = NK; q < 4 * VL; ++q) a[q] = T(0);
#pragma unroll
        for (int q = 0; q < VL; ++q) sL[le * VLS + q] = V4<T>{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
      }
    }
  }
  // pre-lift sums of the wavefront's equation on this level: vertical part
  // W = t_dJ(t_j) (D_t U)(level j)
  T B[NT];
  {
    const LevelMask<Nq, T> lm(j);
    T dtr[Nq];
    lm.row([](auto jj, auto m) { constexpr T v = T(RT::Dt[jj * Nq + m]); return v; }, dtr);
    if (f == 0) {
      const T tl = lm.pick([](auto jj) { constexpr T v = T(0.5 * (1.0 - RT::t[jj])); return v; }), th = T(1) - tl;
      const T tzJ = up * g[4];
      const T txJ = up * dot2(g[5], tl, g[6], th);
      const T tyJ = up * dot2(g[7], tl, g[8], th);
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        T dX = 0, dY = 0, dZ = 0;
#pragma unroll
        for (int m = 0; m < Nq; ++m) {
          dX += dtr[m] * elx[m * NT + i];
          dY += dtr[m] * ely[m * NT + i];
          dZ += dtr[m] * elz[m * NT + i];
        }
        B[i] = -dot3(txJ, dX, tyJ, dY, tzJ, dZ);
      }
    } else {
      const T tl = lm.pick([](auto jj) { constexpr T v = T(0.5 * (1.0 - RT::t[jj])); return v; }), th = T(1) - tl;
      const T tdJ = up * (f == 1 ? g[4] : dot2(g[2 * f + 1], tl, g[2 * f + 2], th));
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        T dP = 0;
#pragma unroll
        for (int m = 0; m < Nq; ++m) dP += dtr[m] * elp[m * NT + i];
        B[i] = -(tdJ * dP);
      }
    }
  }

  __syncthreads();

  // residual of the previous stage, in the coalesced layout of the update.
  // The first stage reads none: its resource has an empty range, so the
  // loads return zeros without touching memory and need no branch.
  const bool rd = (A.flags & kReadRes) != 0, wu = (A.flags & kWriteU) != 0;
  const bool stream = (A.flags & kStreamRes) != 0, stream_u = (A.flags & kStreamU) != 0;
  V4<T>* const res_chunk = static_cast<V4<T>*>(A.res) + e0 * NP;
  const auto bres_in = chunk_rsrc(res_chunk, rd ? int64_t(nE) * NP * V4B : 0);
  V4<T> rprev[UPD];
#pragma unroll
  for (int k = 0; k < UPD; ++k)
    rprev[k] = stream ? bload<T, kStream>(bres_in, tid + BS * k) : bload<T>(bres_in, tid + BS * k);

  // ---- phase 2, the same code for all equations: the flux (F_p or F_u) and
  // the factors it is lifted with (1, or the normal's component) differ
  T R[NT];
  {
    // triangular-face lifts: flux spread over all levels by (M^1D)^-1 e_{0,N}
    // (exact mass) or, lumped (Gauss-Lobatto weights w), e_{0,N} / w_{0,N}
    const T wend = T(0.5 * N * (N + 1));  // 1 / w_0 = 1 / w_N
    const bool lumped = (A.flags & kLumped) != 0;
    const LevelMask<Nq, T> lm(j);
    T cb = lm.pick([](auto jj) { constexpr T v = T(RT::g0[jj]); return v; });
    T ct = lm.pick([](auto jj) { constexpr T v = T(RT::gN[jj]); return v; });
    if (lumped) {
      cb = lm.m[0] * wend;
      ct = lm.m[N] * wend;
    }
    cb *= up;
    ct *= up;
    if (f != 0) {
      const int c = f == 1 ? 2 : f - 2;  // n_x, n_y, n_z
      cb *= g[13 + c];
      ct *= g[17 + c];
    }
    const T* ft = sF + (f == 0 ? 0 : EPB * 2 * NT) + (active ? le : 0) * 2 * NT;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      B[i] += cb * ft[i];
      B[i] += ct * ft[NT + i];
    }

    if constexpr (MODE == 2) {
      // mortar faces: pre-lift contributions of the common refinement; the
      // buffer's range check returns zeros for the other faces
      if (f != 1) {
        constexpr int NTP = (NT + 3) / 4 * 4;
        const auto rb = chunk_rsrc(A.mortB, A.nmort * 2 * Nq * NTP * int64_t(sizeof(T)));
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const T sc = f == 0 ? up : up * g[22 + 4 * d + f - 2];
          const int64_t mo = nbq[d] <= -2 ? int64_t(-2 - nbq[d]) : int64_t(A.nmort);
          const int idx0 = int((mo * 2 * Nq + (f == 0 ? 0 : Nq) + j) * NTP / 4);
#pragma unroll
          for (int c = 0; c < NTP / 4; ++c) {
            const V4<T> s = bload<T>(rb, idx0 + c);
            const T v[4] = {s.p, s.uz, s.ux, s.uy};
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (4 * c + k < NT) B[4 * c + k] += sc * v[k];
          }
        }
      }
    }

    // R = L^{tri,k} B with L^{tri,k} = (M^{tri,k})^-1 M^tri (Sec. 4.2): the
    // reference mass as literals, then the quadrilateral-face moments (the
    // lift E_e before M^tri becomes the Nq x Nq edge mass on the edge's own
    // nodes after it: M^tri E_e = int_edge l l_q (1 -+ xi) / 2), then the
    // element's inverse mass
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      T s = 0;
#pragma unroll
      for (int m = 0; m < NT; ++m) constexpr_or_skip(RT::Mtri[i * NT + m], s, B[m]);
      R[i] = s;
    }
    if (f != 1) {
      const T* const fq = sQ + (f == 0 ? 0 : EPB * C::NQF) + ((active ? le : 0) * 3 * Nq + j) * Nq;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        T Ja = g[20 + 4 * d], Jb = g[21 + 4 * d];
        // a mortar face (-2 - m) takes its flux from the mortar kernel instead
        if (MODE == 2 && nbq[d] <= -2) Ja = Jb = T(0);
        const T nd = f == 0 ? up : up * g[22 + 4 * d + f - 2];
        Ja *= nd;
        Jb *= nd;
        T fl[Nq];
#pragma unroll
        for (int q = 0; q < Nq; ++q) fl[q] = fq[d * Nq * Nq + q];
        // the edge mass J^a M^a + J^b M^b is symmetric
#pragma unroll
        for (int qq = 0; qq < Nq; ++qq) {
#pragma unroll
          for (int q = 0; q <= qq; ++q) {
            const T m = dot2(Ja, T(RT::Ma[qq * Nq + q]), Jb, T(RT::Mb[qq * Nq + q]));
            R[edge_node(N, d, qq)] += m * fl[q];
            if (q < qq) R[edge_node(N, d, q)] += m * fl[qq];
          }
        }
      }
    }
    const V4<T>* Lv = sL + (active ? le : 0) * VLS;
    if constexpr (C::CHOL) {
      // R = L^-T L^-1 R: forward substitution row by row, then the
      // transposed solve column by column (the factor's entries in reverse)
      // (no more than four 4-vectors of the operator ahead: hoisted all at
      // once they set the kernel's register count, 99 against 82 at N = 3 and
      // 299 against 157 at N = 4 in FP64)
#pragma unroll
      for (int c = 0; c < VL; ++c) {
        if (c % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const V4<T> l4 = Lv[c];
        const T lv[4] = {l4.p, l4.uz, l4.ux, l4.uy};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int q = 4 * c + k;
          if (q < Dim<N>::NPK) {
            const int i = tri_row(q), m = q - i * (i + 1) / 2;
            if (m < i) R[i] -= lv[k] * R[m];
            else R[i] *= lv[k];
          }
        }
      }
#pragma unroll
      for (int c = VL - 1; c >= 0; --c) {
        if (c % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        const V4<T> l4 = Lv[c];
        const T lv[4] = {l4.p, l4.uz, l4.ux, l4.uy};
#pragma unroll
        for (int k = 3; k >= 0; --k) {
          const int q = 4 * c + k;
          if (q < Dim<N>::NPK) {
            const int i = tri_row(q), m = q - i * (i + 1) / 2;
            if (m < i) R[m] -= lv[k] * R[i];
            else R[i] *= lv[k];
          }
        }
      }
    } else {
      // the stored lower triangle of the symmetric inverse: each off-diagonal entry serves two rows
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        B[i] = R[i];
        R[i] = T(0);
      }
#pragma unroll
      for (int c = 0; c < VL; ++c) {
        if (c % 4 == 0) __builtin_amdgcn_sched_barrier(0);
        const V4<T> l4 = Lv[c];
        const T lv[4] = {l4.p, l4.uz, l4.ux, l4.uy};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int q = 4 * c + k;
          if (q < Dim<N>::NPK) {
            const int i = tri_row(q), m = q - i * (i + 1) / 2;
            R[i] += lv[k] * B[m];
            if (m < i) R[m] += lv[k] * B[i];
          }
        }
      }
    }

    // horizontal part on the own slice:
    //   R_p -= D_r (r_x u_x + r_y u_y) + D_s (s_x u_x + s_y u_y)
    //   R_x -= D_r (r_x p) + D_s (s_x p) ;  R_y -= D_r (r_y p) + D_s (s_y p)
    if (f != 1) {
      T Ar[NT], As[NT];
      if (f == 0) {
        const T rx = g[0], ry = g[1], sx = g[2], sy = g[3];
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          const T x = elx[j * NT + m], y = ely[j * NT + m];
          Ar[m] = dot2(rx, x, ry, y);
          As[m] = dot2(sx, x, sy, y);
        }
      } else {
        const T rd_ = g[f - 2], sd = g[f];
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          const T p = elp[j * NT + m];
          Ar[m] = rd_ * p;
          As[m] = sd * p;
        }
      }
#pragma unroll
      for (int i = 0; i < NT; ++i) {
#pragma unroll
        for (int m = 0; m < NT; ++m) {
          constexpr_or_skip(-RT::Dr[i * NT + m], R[i], Ar[m]);
          constexpr_or_skip(-RT::Ds[i * NT + m], R[i], As[m]);
        }
      }
    }

    const T scale = f == 0 ? g[9] : g[10];
#pragma unroll
    for (int i = 0; i < NT; ++i) R[i] *= scale;
    if (f == 0) {
      for (int s = 0; s < A.nsrc; ++s) {
        if (active && A.src_elem[s] == e) {
          const T* sv = static_cast<const T*>(A.srcvec) + s * NP + j * NT;
          const T amp = T(A.src_amp[s]);
#pragma unroll
          for (int i = 0; i < NT; ++i) R[i] += amp * sv[i];
        }
      }
    }
  }
  // the gradient epilogue's loads and geometry, before the right-hand side
  // replaces the geometry records
  [[maybe_unused]] EpiData<N, T> ep;
  [[maybe_unused]] int eg = active ? le : 0;  // (the element anew, not held from the start: two registers)
  if constexpr (MODE == 4) {
    asm volatile("" : "+v"(eg));
    grad_load<N, T>(A, e0, nE, tid, f, j, e0 + eg, f != 1 ? qnbr : tnbr, code, sG, sE, ep);
  }
  // the right-hand side replaces factors, geometry and fluxes in LDS
  __syncthreads();
  if (active) {
    T* const o = sR + f * PL + le * NP + j * NT;
#pragma unroll
    for (int i = 0; i < NT; ++i) o[i] = R[i];
  }
  __syncthreads();

  // low-storage Runge-Kutta update, coalesced over the chunk
  const T ca = T(A.a), cb = T(A.b), dt = T(A.dt), cg = (A.flags & kGamma) ? T(A.g) : T(1);
  const auto bres = chunk_rsrc((A.flags & kResOut) ? static_cast<V4<T>*>(A.rout) + e0 * NP : res_chunk,
                               int64_t(nE) * NP * V4B);
  const auto bout = chunk_rsrc(static_cast<V4<T>*>(A.Uout) + e0 * NP, int64_t(nE) * NP * V4B);
#pragma unroll
  for (int k = 0; k < UPD; ++k) {
    const int idx = tid + BS * k;
    const int l = idx < EPB * NP ? idx : EPB * NP;
    const V4<T> q = rprev[k];
    const V4<T> r{dot2(ca, q.p, dt, sR[l]), dot2(ca, q.uz, dt, sR[PL + l]), dot2(ca, q.ux, dt, sR[2 * PL + l]),
                  dot2(ca, q.uy, dt, sR[3 * PL + l])};
    if (stream) bstore<T>(bres, idx, r);
    else bstore<T, 0>(bres, idx, r);
    // the adjoint sweep's mass terms take the incoming adjoint state from
    // here (each slot is read above by the lane that writes it; the lanes
    // past the chunk write the spare slot)
    if constexpr (MODE == 4) {
      sR[l] = q.p;
      sR[PL + l] = q.uz;
      sR[2 * PL + l] = q.ux;
      sR[3 * PL + l] = q.uy;
    }
    if (wu) {
      const V4<T> u{dot2(cg, sU[l], cb, r.p), dot2(cg, sU[PL + l], cb, r.uz), dot2(cg, sU[2 * PL + l], cb, r.ux),
                    dot2(cg, sU[3 * PL + l], cb, r.uy)};
      if (stream_u) bstore<T>(bout, idx, u);
      else bstore<T, 0>(bout, idx, u);
    }
  }
  if constexpr (MODE == 4) grad_epilogue<N, T>(A, tid, f, le, j, active, e0, nE, sU, sR, sR + 4 * PL, sE, ep);
  if constexpr (MODE == 5) {
    __syncthreads();  // the update's reads of the staged state are done
    if (tid < NT) {
      const T* s = sU + (nE - 1) * NP + N * NT + tid;
      carry[tid] = V4<T>{s[0], s[PL], s[2 * PL], s[3 * PL]};
    }
    __syncthreads();  // the next chunk may restage
  }
}

// chunk c of a mesh: wedges c EPB .. min((c + 1) EPB, Kw) - 1
template <int N, typename T, int MODE>
__device__ __forceinline__ void wedge_stage_chunk_at(const StageLaunch& A, int chunk) {
  constexpr int EPB = Cfg<N, T>::EPB;
  const int64_t e0 = int64_t(chunk) * EPB;
  const int64_t left = A.Kw - e0;
  wedge_stage_chunk<N, T, MODE>(A, e0, left < EPB ? int(left) : EPB);
}

// XCD-aware mapping: consecutive workgroups go to different XCDs, so give
// every XCD one contiguous range of chunks (face neighbours share its L2).
__device__ __forceinline__ int xcd_chunk(int bid, int nb) {
  const int qd = nb / 8, rm = nb % 8, xcd = bid % 8, kk = bid / 8;
  return xcd < rm ? xcd * (qd + 1) + kk : rm * (qd + 1) + (xcd - rm) * qd + kk;
}

template <int N, typename T, int MODE>
__global__ void __launch_bounds__(256, (stage_waves<N, T, MODE>())) wedge_stage(StageLaunch A) {
  wedge_stage_chunk_at<N, T, MODE>(A, xcd_chunk(blockIdx.x, gridDim.x));
}

// Column marching (the layer-by-layer reuse the paper proposes as future
// work, Sec. 7): block b walks the wedges of column segment b (a run of at
// most 2 EPB consecutive elements stacked bottom to top, from A.cols; the
// host splits taller columns) in two chunks of EPB layers from the bottom;
// vertical neighbours inside a chunk come from its staged state, the wedge
// below the second chunk's first one from the first chunk's top level kept
// in LDS, so no triangular face inside the segment is gathered from memory.
// (Straight-line code for the two chunks: a loop over chunks keeps values
// live across its back edge and spills.)
template <int N, typename T>
__global__ void __launch_bounds__(256, (stage_waves<N, T, 5>())) wedge_column_stage(StageLaunch A) {
  constexpr int EPB = Cfg<N, T>::EPB;
  __shared__ V4<T> carry[Dim<N>::NT];
  const int2 col = A.cols[xcd_chunk(blockIdx.x, gridDim.x)];
  wedge_stage_chunk<N, T, 5>(A, int64_t(col.x), col.y < EPB ? col.y : EPB, carry, false);
  if (col.y > EPB) {
    const int left = col.y - EPB;
    wedge_stage_chunk<N, T, 5>(A, int64_t(col.x) + EPB, left < EPB ? left : EPB, carry, true);
  }
}

// Many independent meshes of one order in one launch: block b takes chunk
// w = (problem, chunk) of a problem-major list, every XCD one contiguous range
// of it (face neighbours share an L2).  The stage record of each problem
// (buffers, coefficients, time step, source amplitudes) is in device memory,
// written by the batch preparation kernel of the stage.  WPE is the
// occupancy the register allocation aims at, chosen per order by the batch
// autotuner.
template <int N, typename T, int WPE>
__global__ void __launch_bounds__(256, WPE)
    wedge_batch_stage(const StageLaunch* __restrict__ probs, const int2* __restrict__ work, int nwork) {
  const int w = xcd_chunk(blockIdx.x, gridDim.x);
  if (w >= nwork) return;
  const int2 it = work[w];
  wedge_stage_chunk_at<N, T, 0>(probs[it.x], it.y);  // the record is wave-uniform: scalar loads
}

// Problems of one order on both wedge kernels (orders 4 and 5 in FP32) in one
// launch: a work item with a negative chunk is a chunk ~it.y of the node-lane
// kernel.  For batches whose blocks are few: a second launch, on a stream of its
// own or not, costs a stage 10 us (8 meshes of 24 and 8 of 128 wedges at order
// 4: 25 us per stage in two launches, 15 in one).  The node-lane chunks are small,
// so that both kernels' LDS leaves three blocks per CU at order 4, two at order 5.
template <int N>
constexpr int kBothEpb = N == 4 ? 4 : 3;  // elements per node-lane chunk
template <int N>
__global__ void __launch_bounds__(256, N == 4 ? 3 : 2)
    wedge_batch_both(const StageLaunch* __restrict__ probs, const int2* __restrict__ work, int nwork) {
  const int w = xcd_chunk(blockIdx.x, gridDim.x);
  if (w >= nwork) return;
  const int2 it = work[w];
  if (it.y >= 0) wedge_stage_chunk_at<N, float, 0>(probs[it.x], it.y);
  else wedge_node_chunk<N, float, 0, kBothEpb<N>, 256>(probs[it.x], ~it.y);
}

template <int N, typename T>
hipError_t launch_wedge_batch_t(const StageLaunch* probs, const int2* work, int nwork, int wpe, hipStream_t st) {
  if (nwork <= 0) return hipSuccess;
  constexpr int W = stage_waves<N, T, 0>();
  if (wpe == W)
    hipLaunchKernelGGL((wedge_batch_stage<N, T, W>), dim3(unsigned(nwork)), dim3(Cfg<N, T>::BS), 0, st, probs, work,
                       nwork);
  else
    hipLaunchKernelGGL((wedge_batch_stage<N, T, W - 1>), dim3(unsigned(nwork)), dim3(Cfg<N, T>::BS), 0, st, probs,
                       work, nwork);
  return hipGetLastError();
}

template <int N, typename T>
hipError_t launch_wedge_stage_t(const StageLaunch& a, hipStream_t st) {
  using C = Cfg<N, T>;
  const int64_t nchunks = (a.Kw + C::EPB - 1) / C::EPB;
  if (nchunks <= 0) return hipSuccess;
  if (a.nmort > 0)
    hipLaunchKernelGGL((wedge_stage<N, T, 2>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else if (a.Kt == 0 && (a.flags & kGrad))
    hipLaunchKernelGGL((wedge_stage<N, T, 4>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else if (a.Kt == 0 && (a.flags & kColumnMarch) && a.cols && a.ncols > 0)
    hipLaunchKernelGGL((wedge_column_stage<N, T>), dim3(unsigned(a.ncols)), dim3(C::BS), 0, st, a);
  else if (a.Kt == 0 && (a.flags & kLayerMarch))
    hipLaunchKernelGGL((wedge_stage<N, T, 3>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else if (a.Kt > 0)
    hipLaunchKernelGGL((wedge_stage<N, T, 1>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  else
    hipLaunchKernelGGL((wedge_stage<N, T, 0>), dim3(unsigned(nchunks)), dim3(C::BS), 0, st, a);
  return hipGetLastError();
}

}  // namespace

int wedge_chunk_elems(int N, int bits) {
  int epb = 0;
#define WDG_EPB(n, T) epb = Cfg<n, T>::EPB
  WDG_DISPATCH_N(N, bits, WDG_EPB)
#undef WDG_EPB
  return epb;
}

int wedge_waves(int N, int bits, int idx) {
  int w = 0;
#define WDG_WAVES(n, T) w = stage_waves<n, T, 0>()
  WDG_DISPATCH_N(N, bits, WDG_WAVES)
#undef WDG_WAVES
  return w - (idx ? 1 : 0);
}

int wedge_both_epb(int N) { return N == 4 ? kBothEpb<4> : kBothEpb<5>; }

hipError_t launch_wedge_batch_both(int N, const StageLaunch* probs, const int2* work, int nwork, hipStream_t st) {
  if (nwork <= 0) return hipSuccess;
  if (N == 4)
    hipLaunchKernelGGL(wedge_batch_both<4>, dim3(unsigned(nwork)), dim3(256), 0, st, probs, work, nwork);
  else if (N == 5)
    hipLaunchKernelGGL(wedge_batch_both<5>, dim3(unsigned(nwork)), dim3(256), 0, st, probs, work, nwork);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_wedge_batch(int N, int bits, const StageLaunch* probs, const int2* work, int nwork, int wpe,
                              hipStream_t st) {
  hipError_t err = hipErrorInvalidValue;
#define WDG_STAGE(n, T) err = launch_wedge_batch_t<n, T>(probs, work, nwork, wpe, st)
  WDG_DISPATCH_N(N, bits, WDG_STAGE)
#undef WDG_STAGE
  return err;
}

hipError_t launch_wedge_stage(int N, int bits, const StageLaunch& a, hipStream_t st) {
  hipError_t err = hipErrorInvalidValue;
#define WDG_STAGE(n, T) err = launch_wedge_stage_t<n, T>(a, st)
  WDG_DISPATCH_N(N, bits, WDG_STAGE)
#undef WDG_STAGE
  return err;
}

}  // namespace wdg

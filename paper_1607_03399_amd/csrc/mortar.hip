// Mortar kernel of libwdg: wedge quadrilateral faces covered by two
// tetrahedron triangles, coupled on the common refinement.
#include <hip/hip_runtime.h>

#include "device_common.hpp"

namespace wdg {
namespace {

// ---------------------------------------------------------------------------
// Only the pressure and the normal velocity enter the flux, so both traces of
// a mortar are carried as (p, u.n) with the wedge's outward normal: z_w on the
// wedge face nodes (level-major, Nq x Nq; negated, so that sums are jumps:
// tetrahedron trace minus wedge trace), z_s on the tetrahedron face nodes of
// side s of the diagonal.  The jump's moments on side s are
//   wedge basis        WW_s z_w + WT_s z_s
//   tetrahedron basis  WT_s^T z_w + TT_s z_s
// with blocks that depend on the geometry only: the host integrates them once
// per mesh in FP64 (mort_nx(N) Gauss points along the edge times Nq in t on
// each side of the diagonal, exact in t).  Three of the six are stored: TT_s
// is (area / 2) M^tri, which the output's (M^tri)^-1 / (area / 2) takes back
// to the identity, and WW_0 + WW_1 is the mass of the whole face, (edge mass
// weighted by the face's height) x M^1D, whose M^1D the output's (M^1D)^-1
// takes back: with flux factors a_s of the sides
//   sum_s a_s WW_s z_w = (a_0 - a_1) WW_0 z_w + a_1 (WW_0 + WW_1) z_w.
// The upwind / central flux combinations follow, then
//   wedge:       pre-lift contributions, (M^1D)^-1 in t and (M^tri)^-1
//                restricted to the edge nodes, applied to the wedge moments
//   tetrahedra:  equivalent nodal face flux (M^tri)^-1 (moments) / (area / 2)
// Bound by the blocks' bytes: at N = 4 in FP32 a mortar reads 4.3 KB of them
// (6.6 KB with all six) of 6.0 KB in all.  us per stage of hybrid meshes with
// all six and with three: 39 312 wedges, 29 520 tetrahedra and 23 232 mortars
// at N = 4 in FP32 137.8 -> 130.3 (the kernel itself 48 -> 38); 25 792 elements
// at N = 5 in FP32 115.8 -> 107.9, at N = 4 in FP64 131.6 -> 121.0; 154 800 at
// N = 3 in FP32 166 -> 151.
// One wavefront per mortar.
// ---------------------------------------------------------------------------
template <int N>
struct MortTab {
  static constexpr int NT = (N + 1) * (N + 2) / 2, Nq = N + 1;
  static constexpr int MI1 = 0, ME = Nq * Nq, MTI = ME + 3 * NT * Nq, HE = MTI + NT * NT,
                       SIZE = HE + 2 * 3 * NT * Nq;
};

// Cache policy of the coupling-matrix loads: each value is read once per
// stage, so they stream (non-temporal) instead of evicting the state vectors
// that the wedge and tetrahedron kernels read next (on the 39 312-wedge +
// 29 520-tetrahedron N = 4 hybrid mesh the default
// policy cost those kernels 14 and 4 us per stage)
#ifndef WDG_MORT_CORE_AUX
#define WDG_MORT_CORE_AUX 2
#endif
// 4-vector idx of a buffer resource; past its end the hardware returns zeros
template <typename T>
__device__ __forceinline__ V4<T> core_load(__amdgpu_buffer_rsrc_t r, int idx) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(V4<T>, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 16, 0, WDG_MORT_CORE_AUX));
  } else {
    struct H2 {
      u32x4 lo, hi;
    } h{__builtin_amdgcn_raw_buffer_load_b128(r, idx * 32, 0, WDG_MORT_CORE_AUX),
        __builtin_amdgcn_raw_buffer_load_b128(r, idx * 32 + 16, 0, WDG_MORT_CORE_AUX)};
    return __builtin_bit_cast(V4<T>, h);
  }
}

template <int N, typename T>
__global__ void __launch_bounds__(64) mortar_kernel(StageLaunch A) {
  using TB = MortTab<N>;
  constexpr int NT = TB::NT, Nq = TB::Nq;
  constexpr int NPW = Dim<N>::NP, NPT = TDim<N>::NP;
  constexpr int NW = Nq * Nq, CS = mort_dev_stride(N), WT = NW * (NW + 1) / 2;
  constexpr int CV = CS / 4, CVL = (CV + 63) / 64;  // 4-vectors of the coupling blocks, per lane
  constexpr int NST = NW + 2 * NT, NSL = (NST + 63) / 64;
  constexpr int NTP = (NT + 3) / 4 * 4;
  static_assert(2 * NTP <= 64, "one lane per wedge output column");
  struct alignas(2 * sizeof(T)) P2 {
    T p, u;
  };
  __shared__ V4<T> sC[CV];    // the mortar's coupling blocks
  __shared__ P2 sZ[NST];      // z_w, z_0, z_1
  __shared__ P2 sJ[NST];      // WW_0 z_w, WT_0^T z_w, WT_1^T z_w
  __shared__ P2 sK[2 * NW];   // WT_0 z_0, WT_1 z_1
  __shared__ T sMW[2 * NW];   // wedge flux moments [field][level * Nq + edge node]
  __shared__ T sMT[4 * NT];   // tetrahedron flux moments [side][field][face node], without TT_s z_s

  const T* __restrict__ tab = static_cast<const T*>(A.mortTab);
  const V4<T>* __restrict__ Uin = static_cast<const V4<T>*>(A.Uin);
  const int tid = threadIdx.x;
  const int64_t mo = blockIdx.x;
  const int* mi = A.mortI + mo * kMortIntStride;
  const double* mg = static_cast<const double*>(A.mortG) + mo * kMortGeoStride;
  // Loads in the order their results are needed, each issued before any
  // wait: the mortar's record, its coupling matrices (which do not depend on
  // the record), then the node gathers addressed from the record.  The
  // vector-memory counter completes in order, so waiting for the record does
  // not wait for the matrices.
  const int wel = mi[0], e = mi[1], t0 = mi[3], f0 = mi[4], t1 = mi[5], f1 = mi[6];
  const double mgx = mg[5], mgy = mg[6], mz0 = mg[27], mz1 = mg[28], ms0 = mg[25], ms1 = mg[26];
  const double ma = 0.25 * mg[4] * (mg[2] - mg[0]), mb = 0.25 * mg[4] * (mg[3] - mg[1]);
  V4<T> cv[CVL];
  {
    const auto rc = chunk_rsrc(static_cast<const V4<T>*>(A.mortC) + mo * CV, int64_t(CV) * 4 * int64_t(sizeof(T)));
#pragma unroll
    for (int l = 0; l < CVL; ++l) cv[l] = core_load<T>(rc, tid + 64 * l);
  }

  // node values: the wedge face (Nq x Nq, level-major), then both tetrahedron
  // faces; lanes past them read node 0 (a valid address, never used)
  V4<T> nv[NSL];
#pragma unroll
  for (int l = 0; l < NSL; ++l) {
    const int idx = tid + 64 * l;
    const int lev = idx / Nq, q = idx - lev * Nq;
    const int r = idx - NW, side = r >= NT ? 1 : 0, i = r - side * NT;
    const int64_t aw = int64_t(wel) * NPW + lev * NT + edge_node(N, e, q < Nq ? q : 0);
    const int64_t at = A.Kw * NPW + (int64_t(side ? t1 : t0) - A.Kw) * NPT +
                       tet_face_node<N>(side ? f1 : f0, i >= 0 && i < NT ? i : 0);
    nv[l] = Uin[idx < NW ? aw : (idx < NST ? at : 0)];
  }
  const T nx = T(mgx), ny = T(mgy);
#pragma unroll
  for (int l = 0; l < NSL; ++l) {
    const int idx = tid + 64 * l;
    const T vp = nv[l].p, vn = nx * nv[l].ux + ny * nv[l].uy;
    if (idx < NW) sZ[idx] = P2{-vp, -vn};
    else if (idx < NST) sZ[idx] = P2{vp, vn};
  }
#pragma unroll
  for (int l = 0; l < CVL; ++l)
    if (tid + 64 * l < CV) sC[tid + 64 * l] = cv[l];
  __syncthreads();

  const T* C = reinterpret_cast<const T*>(sC);
  // products with z_w: lane r < NW the row r of WW_0, lanes from NW on a
  // column of WT_0 or WT_1
#pragma unroll
  for (int l = 0; l < NSL; ++l) {
    const int o = tid + 64 * l;
    if (o < NST) {
      const int row = o < NW ? o : -1;
      const int base = o < NW ? o * NW - o * (o - 1) / 2 - o : WT + (o - NW) * NW;
      P2 acc{T(0), T(0)};
#pragma unroll
      for (int c = 0; c < NW; ++c) {
        const T cc = C[c <= row ? c * NW - c * (c - 1) / 2 - c + row : base + c];
        acc.p += cc * sZ[c].p;
        acc.u += cc * sZ[c].u;
      }
      sJ[o] = acc;
    }
  }
  // products of WT_s with z_s
#pragma unroll
  for (int l = 0; l < (2 * NW + 63) / 64; ++l) {
    const int o = tid + 64 * l;
    if (o < 2 * NW) {
      const int s = o >= NW ? 1 : 0;
      const T* Cs = C + WT + s * NT * NW + (o - s * NW);
      const P2* z = sZ + NW + s * NT;
      P2 acc{T(0), T(0)};
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const T cc = Cs[c * NW];
        acc.p += cc * z[c].p;
        acc.u += cc * z[c].u;
      }
      sK[o] = acc;
    }
  }
  __syncthreads();

  // fluxes of the jump's halves J:
  //   wedge        F_p = taup J_p - J_u,   F_u = tauu J_u - J_p
  //   tetrahedron  F_p = -taup J_p - J_u,  F_u = tauu J_u + J_p  (the jump seen from its side)
  const T tau_on = (A.flags & kCentral) ? T(0) : T(1);
  const T z0 = T(mz0), z1 = T(mz1);
  const T taup[2] = {tau_on * T(2) / z0, tau_on * T(2) / z1}, tauu[2] = {tau_on * z0 * T(0.5), tau_on * z1 * T(0.5)};
  if (tid < NW) {
    const P2 ww = sJ[tid], k0 = sK[tid], k1 = sK[NW + tid];
    sMW[tid] = T(0.5) * ((taup[0] - taup[1]) * ww.p + (taup[0] * k0.p + taup[1] * k1.p) - (k0.u + k1.u));
    sMW[NW + tid] = T(0.5) * ((tauu[0] - tauu[1]) * ww.u + (tauu[0] * k0.u + tauu[1] * k1.u) - (k0.p + k1.p));
  }
  if (tid < 2 * NT) {
    const int s = tid >= NT ? 1 : 0, i = tid - s * NT;
    const P2 d = sJ[NW + tid];
    const T tp = s ? taup[1] : taup[0], tu = s ? tauu[1] : tauu[0];
    sMT[(2 * s + 0) * NT + i] = T(0.5) * (-tp * d.p - d.u);
    sMT[(2 * s + 1) * NT + i] = T(0.5) * (tu * d.u + d.p);
  }
  __syncthreads();

  // wedge pre-lift contributions [field][level j][node i] (i padded to NTP):
  //   sum_m (M^1D)^-1[j][m] sum_q (M^tri)^-1[i][node q of edge e] moments[m][q],
  // and of the whole face's mass, the same with its M^1D taken back
  if (tid < 2 * NTP) {
    const int f = tid / NTP, i = tid - f * NTP;
    T H[Nq], mine[Nq];
#pragma unroll
    for (int q = 0; q < Nq; ++q) {
      const int o = (e * NT + (i < NT ? i : 0)) * Nq + q;
      mine[q] = tab[TB::ME + o];
      H[q] = T(0.5) * (T(ma) * tab[TB::HE + o] + T(mb) * tab[TB::HE + 3 * NT * Nq + o]);
    }
    const T t1 = f ? tauu[1] : taup[1];
    T G[Nq];
#pragma unroll
    for (int m = 0; m < Nq; ++m) {
      T acc = 0;
#pragma unroll
      for (int q = 0; q < Nq; ++q) acc += mine[q] * sMW[f * NW + m * Nq + q];
      G[m] = acc;
    }
    T* outB = static_cast<T*>(A.mortB) + mo * (2 * Nq * NTP) + f * Nq * NTP + i;
#pragma unroll
    for (int j = 0; j < Nq; ++j) {
      T acc = 0;
#pragma unroll
      for (int m = 0; m < Nq; ++m) acc += tab[TB::MI1 + j * Nq + m] * G[m];
#pragma unroll
      for (int q = 0; q < Nq; ++q) {
        const P2 z = sZ[j * Nq + q];
        acc += H[q] * (f ? t1 * z.u - z.p : t1 * z.p - z.u);
      }
      outB[j * NTP] = i < NT ? acc : T(0);
    }
  }
  // equivalent nodal flux of both tetrahedron faces [side][field][node]
  for (int o = tid; o < 4 * NT; o += 64) {
    const int side = o / (2 * NT), r = o - side * 2 * NT, f = r / NT, i = r - f * NT;
    const P2 z = sZ[NW + side * NT + i];
    const T own = T(0.5) * (f ? (side ? tauu[1] : tauu[0]) * z.u + z.p : -(side ? taup[1] : taup[0]) * z.p - z.u);
    T acc = 0;
    // (M^tri)^-1 is symmetric: read so that consecutive lanes read consecutive values
#pragma unroll
    for (int k = 0; k < NT; ++k) acc += tab[TB::MTI + k * NT + i] * sMT[(2 * side + f) * NT + k];
    static_cast<T*>(A.mortF)[(mo * 2 + side) * 2 * NT + f * NT + i] = own + acc * T(side ? ms1 : ms0);
  }
}

template <int N, typename T>
hipError_t launch_mortar_stage_t(const StageLaunch& a, hipStream_t st) {
  if (a.nmort <= 0) return hipSuccess;
  if (a.nmort > int64_t(0x7fffffff) || !a.mortC) return hipErrorInvalidValue;
  hipLaunchKernelGGL((mortar_kernel<N, T>), dim3(unsigned(a.nmort)), dim3(64), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_mortar_stage(int N, int bits, const StageLaunch& a, hipStream_t st) {
  hipError_t err = hipErrorInvalidValue;
#define WDG_STAGE(n, T) err = launch_mortar_stage_t<n, T>(a, st)
  WDG_DISPATCH_N(N, bits, WDG_STAGE)
#undef WDG_STAGE
  return err;
}

int mortar_table_size(int N) {
  switch (N) {
    case 1: return MortTab<1>::SIZE;
    case 2: return MortTab<2>::SIZE;
    case 3: return MortTab<3>::SIZE;
    case 4: return MortTab<4>::SIZE;
    case 5: return MortTab<5>::SIZE;
    default: return 0;
  }
}

}  // namespace wdg

// Adjoint element kernel: g_e = - sum_c lambda_{c,e}^T (K_e / E_e) u_{c,e}.
//
// K_e is linear in E_e at fixed Poisson ratio, so dK_e/dE_e is the element
// operator rebuilt with (lambda/E, mu/E).  Each element forms that operator on
// the fly (as the EBE product does, Section 2) for every case, contracts it
// with the adjoint state and writes its own entry: no scatter, no atomics.
//
// One work-item per (fan, case): the chain of up to three tetrahedra around
// an edge that the products use (patches.cpp), so 18 nodes' u and lambda
// values are read for three tetrahedra instead of 30, and each tetrahedron
// after the first needs the coordinates of one more corner only.  The cases of
// a fan are adjacent lanes and are summed with a cross-lane reduction.
// Consecutive fans (which share nodes) stay on one XCD.  The kernel waits for
// its loads (bytes at 64x64x32 hexahedra x 6, FP64, 4 cases: 0.26 GB); one
// work-item per (element, case) with the elements dealt to the XCDs in turn
// took 240 us there.  The element-by-element kernels below serve meshes
// without fans (2^25 nodes or more) and small ones.
#include <hip/hip_runtime.h>

#include "patch_common.h"

namespace ebe {
namespace {

constexpr int kBlock = 256;

// wavefronts per SIMD the register allocation aims at: FP32 three (168
// registers) and FP64 two (256); the kernel waits for its loads, and both fit
// the fan's u and lambda values
template <typename T, int NR>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3))) void k_adjoint_fan(
    const uint32_t* __restrict__ fanw, const int32_t* __restrict__ felem, const double4* __restrict__ xv,
    const double* __restrict__ young, const typename Pair<T>::type* __restrict__ lame, const T* __restrict__ u,
    const T* __restrict__ lam, T* __restrict__ g,
    int64_t nfan) {
  constexpr int G = 64 / NR;  // fans per wavefront
  constexpr int HALF = NR > 8 ? 8 : (NR > 4 ? 4 : (NR > 2 ? 2 : 1));
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane / NR, r = lane - j * NR;
  const int64_t f = (int64_t(xcd_patch(blockIdx.x, gridDim.x)) * (kBlock / 64) + wave) * G + j;
  const bool live = j < G && f < nfan;
  const uint32_t* w = fanw + (live ? f : 0) * kFanStride;
  const int len = live ? int(w[kFanWords] & 3u) : 0;
  const uint32_t flags[2] = {w[kFanWords], w[kFanWords + 1]};
  auto ld = [&](const T* v, int a, int c) -> T {
    const uint32_t bit = a < 10 ? flags[0] >> (2 + 3 * a + c) : flags[1] >> (3 * (a - 10) + c);
    const T x = v[size_t(w[a] & kPtabIdMask) * (3 * NR) + c * NR + r];
    return (bit & 1u) ? T(0) : x;
  };
  // u and lambda of the spine (p, q, pq) and of the current spoke
  T ud[3][3], us[3][3], ld_[3][3], ls[3][3];
  // corner p, and the edge vectors from it to q and to the current spoke's corner
  double4 xp{};
  T ea[3], eb[3];
  auto edge = [&](int a, T e[3]) {
    const double4 v = xv[w[a] & kPtabIdMask];
    e[0] = T(v.x - xp.x);
    e[1] = T(v.y - xp.y);
    e[2] = T(v.z - xp.z);
  };
  if (live) {
    xp = xv[w[0] & kPtabIdMask];
    edge(1, ea);
    edge(3, eb);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        ud[a][c] = ld(u, a, c);
        us[a][c] = ld(u, 3 + a, c);
        ld_[a][c] = ld(lam, a, c);
        ls[a][c] = ld(lam, 3 + a, c);
      }
  }
#pragma unroll
  for (int i = 0; i < kFanLen; ++i) {
    T acc = T(0);
    if (i < len) {
      const int s1 = 6 + 4 * i;  // spoke i + 1, then the rim
      T un[3][3], ur[3], ln[3][3], lr[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          un[a][c] = ld(u, s1 + a, c);
          ln[a][c] = ld(lam, s1 + a, c);
        }
        ur[c] = ld(u, s1 + 3, c);
        lr[c] = ld(lam, s1 + 3, c);
      }
      T Gm[4][3], ec[3];
      edge(s1, ec);
      const int32_t e = felem[f * kFanLen + i];
      const auto lm = lame[e];
      const T s = tet_geometry<T>(ea, eb, ec, Gm) * T(0.05) / T(young[e]);
      const T cl = T(lm.x) * s, cm = T(lm.y) * s;
#pragma unroll
      for (int c = 0; c < 3; ++c) eb[c] = ec[c];
      // value of local node a (p, q, spoke i, spoke i + 1, then the edges)
      auto pick = [&](const T (&d)[3][3], const T (&s)[3][3], const T (&n)[3][3], const T (&m)[3], int a, int c) -> T {
        return a == 0 ? d[0][c] : a == 1 ? d[1][c] : a == 2 ? s[0][c] : a == 3 ? n[0][c] : a == 4 ? d[2][c]
             : a == 5 ? s[2][c] : a == 6 ? s[1][c] : a == 7 ? n[1][c] : a == 8 ? n[2][c] : m[c];
      };
      T unused = T(0);
      p2_apply(
          Gm, cl, cm, [&](int a, int c) -> T { return pick(ud, us, un, ur, a, c); },
          [&](int a, const T fv[3]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) acc += pick(ld_, ls, ln, lr, a, c) * fv[c];
          },
          false, unused);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          us[a][c] = un[a][c];
          ls[a][c] = ln[a][c];
        }
    }
    if constexpr (NR > 1) {  // the fan's cases
#pragma unroll
      for (int off = HALF; off > 0; off >>= 1) {
        const T o = __shfl_down(acc, off, 64);
        if (r < off && r + off < NR) acc += o;
      }
    }
    if (i < len && r == 0) g[felem[f * kFanLen + i]] = -acc;
  }
}

template <typename T, int NR>
void launch_adjoint_fan(const ebe_mesh* m, const typename Pair<T>::type* lame, const T* u, const T* lam, T* g,
                        hipStream_t s) {
  constexpr int per_block = (kBlock / 64) * (64 / NR);
  hipLaunchKernelGGL((k_adjoint_fan<T, NR>), dim3(unsigned((m->nfan + per_block - 1) / per_block)), dim3(kBlock), 0,
                     s, m->fanw.as<uint32_t>(), m->felem.as<int32_t>(), m->xv.as<double4>(), m->young.as<double>(),
                     lame, u, lam, g, m->nfan);
}

// one work-item per (element, case), NR a power of two: an element's cases are
// adjacent lanes of one wavefront
template <typename T, int NR>
__global__ __launch_bounds__(kBlock) void k_adjoint(const int32_t* __restrict__ conn, const double4* __restrict__ xv,
                                                    const double* __restrict__ young,
                                                    const typename Pair<T>::type* __restrict__ lame,
                                                    const T* __restrict__ u, const T* __restrict__ lam,
                                                    T* __restrict__ g, int64_t nelem) {
  const int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int64_t e = t / NR;
  const int r = int(t - e * NR);
  const bool live = e < nelem;
  T acc = T(0);
  if (live) {
    int32_t cw[10];
#pragma unroll
    for (int a = 0; a < 10; ++a) cw[a] = conn[e * 10 + a];
    T G[4][3];
    const T V = tet_geometry<T>(xv[cw[0] & kIdxMask], xv[cw[1] & kIdxMask], xv[cw[2] & kIdxMask],
                                xv[cw[3] & kIdxMask], G);
    const auto lm = lame[e];
    const T s = V * T(0.05) / T(young[e]);
    // nodal values read as needed, each nodal force contracted with the
    // adjoint state as soon as it is known
    T unused = T(0);
    p2_apply(
        G, T(lm.x) * s, T(lm.y) * s,
        [&](int a, int c) -> T {
          return ((cw[a] >> (kIdxBits + c)) & 1) ? T(0) : u[size_t(cw[a] & kIdxMask) * (3 * NR) + c * NR + r];
        },
        [&](int a, const T f[3]) {
          const T* p = lam + size_t(cw[a] & kIdxMask) * (3 * NR) + r;
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (!((cw[a] >> (kIdxBits + c)) & 1)) acc += p[c * NR] * f[c];
        },
        false, unused);
  }
#pragma unroll
  for (int off = 1; off < NR; off <<= 1) acc += __shfl_xor(acc, off, NR);
  if (live && r == 0) g[e] = -acc;
}

// other numbers of cases: one work-item per element, looping over them
template <typename T>
__global__ __launch_bounds__(kBlock) void k_adjoint_loop(const int32_t* __restrict__ conn,
                                                         const double4* __restrict__ xv,
                                                         const double* __restrict__ young,
                                                         const typename Pair<T>::type* __restrict__ lame,
                                                         const T* __restrict__ u, const T* __restrict__ lam,
                                                         T* __restrict__ g, int64_t nelem, int nrhs) {
  const int64_t e = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (e >= nelem) return;
  int32_t cw[10];
#pragma unroll
  for (int a = 0; a < 10; ++a) cw[a] = conn[e * 10 + a];
  T G[4][3];
  const T V = tet_geometry<T>(xv[cw[0] & kIdxMask], xv[cw[1] & kIdxMask], xv[cw[2] & kIdxMask],
                              xv[cw[3] & kIdxMask], G);
  const auto lm = lame[e];
  const T s = V * T(0.05) / T(young[e]);
  T acc = T(0);
  for (int r = 0; r < nrhs; ++r) {
    T unused = T(0);
    p2_apply(
        G, T(lm.x) * s, T(lm.y) * s,
        [&](int a, int c) -> T {
          return ((cw[a] >> (kIdxBits + c)) & 1) ? T(0) : u[size_t(cw[a] & kIdxMask) * 3 * nrhs + c * nrhs + r];
        },
        [&](int a, const T f[3]) {
          const T* p = lam + size_t(cw[a] & kIdxMask) * 3 * nrhs + r;
#pragma unroll
          for (int c = 0; c < 3; ++c)
            if (!((cw[a] >> (kIdxBits + c)) & 1)) acc += p[c * nrhs] * f[c];
        },
        false, unused);
  }
  g[e] = -acc;
}

template <typename T>
hipError_t adjoint_elements_t(const ebe_mesh* m, int nrhs, const typename Pair<T>::type* lame, const T* u,
                              const T* lam, T* g, hipStream_t s) {
  auto grid = [](int64_t work) { return dim3(unsigned((work + kBlock - 1) / kBlock)); };
  switch (nrhs) {
#define EBE_CASE(n)                                                                                             \
  case n:                                                                                                       \
    hipLaunchKernelGGL((k_adjoint<T, n>), grid(m->n_elem * n), dim3(kBlock), 0, s, m->conn.as<int32_t>(),       \
                       m->xv.as<double4>(), m->young.as<double>(), lame, u, lam, g, m->n_elem);                 \
    break;
    EBE_CASE(1) EBE_CASE(2) EBE_CASE(4) EBE_CASE(8) EBE_CASE(16)
#undef EBE_CASE
    default:
      hipLaunchKernelGGL(k_adjoint_loop<T>, grid(m->n_elem), dim3(kBlock), 0, s, m->conn.as<int32_t>(),
                         m->xv.as<double4>(), m->young.as<double>(), lame, u, lam, g, m->n_elem, nrhs);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t adjoint_t(const ebe_mesh* m, int nrhs, const void* u, const void* lam, void* g, hipStream_t s,
                     bool by_element) {
  using P = typename Pair<T>::type;
  const T* uu = static_cast<const T*>(u);
  const T* ll = static_cast<const T*>(lam);
  T* gg = static_cast<T*>(g);
  const P* lame = (sizeof(T) == 8) ? reinterpret_cast<const P*>(m->lame64.as<void>())
                                   : reinterpret_cast<const P*>(m->lame32.as<void>());
  if (by_element) return adjoint_elements_t<T>(m, nrhs, lame, uu, ll, gg, s);
  switch (nrhs) {
#define EBE_CASE(n) \
  case n: launch_adjoint_fan<T, n>(m, lame, uu, ll, gg, s); break;
    EBE_CASE(1) EBE_CASE(2) EBE_CASE(3) EBE_CASE(4) EBE_CASE(5) EBE_CASE(6) EBE_CASE(7) EBE_CASE(8)
    EBE_CASE(9) EBE_CASE(10) EBE_CASE(11) EBE_CASE(12) EBE_CASE(13) EBE_CASE(14) EBE_CASE(15) EBE_CASE(16)
#undef EBE_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* u, const void* lam,
                          void* g, hipStream_t s, bool by_element) {
  // A fan is three tetrahedra long: where every (element, case) can be resident at
  // once and a wavefront holds an element's cases, those end sooner (by fans / by
  // elements: 4^3 cube FP64 1 case 7.0 / 5.3 us, 18x18x12 lattice, 23328 elements,
  // 1 case 8.8 / 6.0, 4 cases 8.4 / 8.6, 8 cases 8.7 / 10.9; FP32 4 cases 7.2 / 6.5, 8
  // 6.9 / 8.2; 67,000 elements 1 case 9.0 / 8.9, FP32 7.4 / 7.6).
  const int64_t resident = dt == EBE_F64 ? 80000 : 96000;
  by_element |= m->nfan == 0 || ((nrhs & (nrhs - 1)) == 0 && m->n_elem * nrhs < resident);
  return dt == EBE_F64 ? adjoint_t<double>(m, nrhs, u, lam, g, s, by_element)
                       : adjoint_t<float>(m, nrhs, u, lam, g, s, by_element);
}

}  // namespace ebe

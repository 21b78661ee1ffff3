// Quadratic EBE product for few cases (pipelined form, at most kWideCases
// cases, straight-sided elements).
//
// At one to four cases a patch of 48 elements is a chain of latencies (its
// tables, x, LDS additions, write-back) with little work in it, and 78% of its
// nodes are shared with other patches.  A wide patch is a run of consecutive
// patches, 4x4x4 hexahedra (or 2x4x4) on a Morton-ordered mesh: half the shared
// rows to stage and add (0.75 a node instead of 1.5), and an accumulator that
// still leaves the CU its wavefronts.  One workgroup per wide patch, one
// work-item per (fan, case): the fans of fan_kernel.h (a chain of up to three
// tetrahedra around an edge), read from patch-local ids of two bytes.  The
// element geometry is formed from the corner coordinates, kept in LDS: each
// tetrahedron of a fan after the first needs one more corner, where a row of
// the geometry cache is 64 or 128 bytes of memory traffic.
//
// 64^3 cube, gather form before: FP64 1 / 2 / 4 cases 150 / 275 / 417 -> 119 /
// 194 / 332 us, FP32 104 / 166 / 235 -> 72 / 119 / 208 us, with the tables in the
// last-level cache; when other meshes' products run in between, FP64 1 case
// takes 148 -> 139 us (90 MB of tables come from memory then).  What bounds it
// is the load unit (at one case every lane of an x gather touches a line of its
// own), LDS additions and two to three wavefronts a SIMD.  Staging the patch's x
// rows in LDS with whole-line loads was slower (FP64 1 case 168 us, FP32 102 us);
// loading the moduli and first x rows ahead of the corners gained nothing.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "patch_common.h"

namespace ebe {
namespace {

template <typename T>
constexpr int wide_threads(int nr) {
  const int g = 64 / nr;
  const int want = ((kWideElems[wide_size(int(sizeof(T)), nr)] / kFanLen + g - 1) / g * g * nr + 63) / 64 * 64;
  return want > 256 ? 256 : want;
}

template <typename T, int NR, bool MASK, bool GAMMA>
__global__ __launch_bounds__(wide_threads<T>(NR)) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3))) void
k_ebe_wide(const uint16_t* __restrict__ fanl, const int32_t* __restrict__ felem, const int32_t* __restrict__ pfan,
           const int32_t* __restrict__ pcorner, const int32_t* __restrict__ poff, const int32_t* __restrict__ pnode,
           const int32_t* __restrict__ pslot, const double4* __restrict__ xv,
           const typename Pair<T>::type* __restrict__ lame, const T* __restrict__ x,
           T* __restrict__ y, T* __restrict__ stage, int stream, int bc, int add, double* __restrict__ gamma,
           double* __restrict__ gslot, unsigned* __restrict__ gcount, const int* __restrict__ gate) {
  constexpr int W = 3 * NR;
  constexpr int TPB = wide_threads<T>(NR);
  constexpr int VEC = pass_vec(NR, NR, int(sizeof(T)));
  constexpr int NV = W / VEC;
  constexpr int G = 64 / NR;
  using V = VecT<T, VEC>;
  constexpr int SIZE = wide_size(int(sizeof(T)), NR);
  __shared__ double F[kWideNodes[SIZE] * W];
  __shared__ double C[kWideCorners[SIZE]][3];
  __shared__ int32_t words[kWideNodes[SIZE]];
  __shared__ double gsum[NR];
  if (gate && *gate == 0) return;
  const int tid = threadIdx.x;
  const int p = xcd_patch(blockIdx.x, gridDim.x);
  const int f0 = pfan[p], nf = pfan[p + 1] - f0;
  const int o0 = poff[p], nn = poff[p + 1] - o0;
  const int nc = pcorner[p];
  // a patch is a chain of memory latencies: its bounds; the node words and this
  // work-item's fan row and elements; corners and x
  const int K = (nf + G - 1) / G;  // a wavefront's fans lie K apart (neighbouring fans share nodes)
  int w = tid, r = 0, len = 0;
  uint4 l0{}, l1{}, l2{};
  int32_t fe[kFanLen];
  auto lid = [&](int a) -> uint32_t {  // patch-local id of the fan's node a
    const uint4& q = a < 8 ? l0 : (a < 16 ? l1 : l2);
    const int k = (a >> 1) & 3;
    const uint32_t v = k == 0 ? q.x : (k == 1 ? q.y : (k == 2 ? q.z : q.w));
    return (a & 1) ? v >> 16 : v & 0xffffu;
  };
  auto fetch = [&]() {  // work-item w's fan: ids and elements; len = 0 without one
    const int j = w / NR;
    r = w - j * NR;
    const int fl = (j % G) * K + j / G;
    len = 0;
    if (w >= K * G * NR || fl >= nf) return;
    const int64_t f = int64_t(f0) + fl;
    const uint4* fr = reinterpret_cast<const uint4*>(fanl + f * kWideStride);
    l0 = fr[0];
    l1 = fr[1];
    l2 = fr[2];
#pragma unroll
    for (int i = 0; i < kFanLen; ++i) fe[i] = felem[f * kFanLen + i];
    len = 1;  // (the number of tetrahedra is in the row, read after the barrier)
  };
  auto ld = [&](uint32_t l, T v[3]) {  // the node's values in this case
    const int32_t wd = words[l];
    const T* xr = x + size_t(wd & kIdxMask) * W + r;
    if constexpr (NR == 1) {  // the row in one load (FP32) or two (FP64)
      struct __attribute__((packed, aligned(4))) Row {
        T v[3];
      };
      const Row q = *reinterpret_cast<const Row*>(xr);
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = q.v[c];
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = xr[c * NR];
    }
    if constexpr (MASK) {
#pragma unroll
      for (int c = 0; c < 3; ++c) v[c] = ((wd >> (kIdxBits + c)) & 1) ? T(0) : v[c];
    }
  };
  fetch();
  for (int i = tid; i < nn; i += TPB) words[i] = pnode[o0 + i];
  for (int i = tid; i < nn * W; i += TPB) F[i] = 0.0;
  if (GAMMA && tid < NR) gsum[tid] = 0.0;
  __syncthreads();
  {
    constexpr int KC = (kWideCorners[SIZE] + TPB - 1) / TPB;
    double4 cv[KC];
#pragma unroll
    for (int k = 0; k < KC; ++k)
      if (tid + k * TPB < nc) cv[k] = xv[words[tid + k * TPB] & kIdxMask];
#pragma unroll
    for (int k = 0; k < KC; ++k) {
      const int i = tid + k * TPB;
      if (i < nc) {
        C[i][0] = cv[k].x;
        C[i][1] = cv[k].y;
        C[i][2] = cv[k].z;
      }
    }
  }
  __syncthreads();
  constexpr bool kLaneCase = (64 % NR) == 0 && (TPB % NR) == 0;
  double en_acc = 0.0;
  auto put = [&](uint32_t l, int c, double v) { atomicAdd(&F[l * W + c * NR + r], v); };
#pragma unroll 1
  while (w < K * G * NR) {
    T us[3][3], ud[3][3];
    if (len > 0) {
      len = int(lid(kFanWords));
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        ld(lid(a), ud[a]);
        ld(lid(3 + a), us[a]);
      }
    }
    double fd[3][3], fs[3][3];  // forces of the spine (p, q, pq) and of the current spoke
    double xp[3];
    T ea[3], eb[3];
    auto edge = [&](uint32_t l, T e[3]) {
#pragma unroll
      for (int c = 0; c < 3; ++c) e[c] = T(C[l][c] - xp[c]);
    };
#pragma unroll
    for (int c = 0; c < 3; ++c) xp[c] = C[lid(0)][c];
    edge(lid(1), ea);
    edge(lid(3), eb);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int c = 0; c < 3; ++c) fd[a][c] = fs[a][c] = 0.0;
#pragma unroll
    for (int i = 0; i < kFanLen; ++i) {
      if (i >= len) continue;
      const int s0 = i == 0 ? 3 : 2 + 4 * i, s1 = 6 + 4 * i;  // spokes i and i + 1; the rim is s1 + 3
      T un[3][3], ur[3], ec[3];
      edge(lid(s1), ec);
#pragma unroll
      for (int a = 0; a < 3; ++a) ld(lid(s1 + a), un[a]);
      ld(lid(s1 + 3), ur);
      const auto lm = lame[fe[i]];
      T Gm[4][3];
      const T s = tet_geometry<T>(ea, eb, ec, Gm) * T(0.05);
      const T cl = T(lm.x) * s, cm = T(lm.y) * s;
#pragma unroll
      for (int c = 0; c < 3; ++c) eb[c] = ec[c];
      auto u = [&](int a, int c) -> T {
        return a == 0 ? ud[0][c] : a == 1 ? ud[1][c] : a == 2 ? us[0][c] : a == 3 ? un[0][c] : a == 4 ? ud[2][c]
             : a == 5 ? us[2][c] : a == 6 ? us[1][c] : a == 7 ? un[1][c] : a == 8 ? un[2][c] : ur[c];
      };
      double nx[3][3];
      T en = T(0);
      auto emit = [&](int a, const T fv[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if constexpr (GAMMA) {  // as in fan_kernel.h
            if (a == 0) asm volatile("" : "+v"(ud[0][c]));
            else en += fv[c] * (u(a, c) - ud[0][c]);
          }
          const double d = double(fv[c]);
          if (a == 0 || a == 1 || a == 4) {
            fd[a == 4 ? 2 : a][c] += d;
          } else if (a == 2 || a == 5 || a == 6) {  // spoke i is complete
            const int k = a == 2 ? 0 : (a == 6 ? 1 : 2);
            put(lid(s0 + k), c, fs[k][c] + d);
          } else if (a == 9) {
            put(lid(s1 + 3), c, d);
          } else {
            nx[a == 3 ? 0 : a - 6][c] = d;
          }
        }
      };
      T unused = T(0);
      p2_apply(Gm, cl, cm, u, emit, false, unused);
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          fs[a][c] = nx[a][c];
          us[a][c] = un[a][c];
        }
      if constexpr (GAMMA) {
        if constexpr (kLaneCase) en_acc += double(en);
        else atomicAdd(&gsum[r], double(en));
      }
    }
    // the last spoke (its place depends on the fan's length) and the spine
    if (len > 0) {
      const uint32_t l3[3] = {len == 1 ? lid(6) : (len == 2 ? lid(10) : lid(14)),
                              len == 1 ? lid(7) : (len == 2 ? lid(11) : lid(15)),
                              len == 1 ? lid(8) : (len == 2 ? lid(12) : lid(16))};
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          put(l3[a], c, fs[a][c]);
          put(lid(a), c, fd[a][c]);
        }
    }
    w += TPB;  // (a full patch of full fans takes one trip, two in FP64 at 3 and 4 cases)
    fetch();
  }
  if constexpr (GAMMA && kLaneCase) {
#pragma unroll
    for (int off = 32; off >= NR; off >>= 1) en_acc += __shfl_xor(en_acc, off, 64);
    if ((tid & 63) < NR) atomicAdd(&gsum[tid & 63], en_acc);
  }
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < nn * NV; i += TPB) {
    const int ent = i / NV, sv = i - ent * NV, sq = sv * VEC, sc = sq / NR;
    const int32_t wd = words[ent];
    V v;
#pragma unroll
    for (int t = 0; t < VEC; ++t) v.v[t] = T(F[ent * W + sq + t]);
    const bool fixed = bc && ((wd >> (kIdxBits + sc)) & 1);
    if (wd < 0) {  // shared node: partial sum to its staging slot
      T* sp = stage + size_t(pslot[o0 + ent]) * W + sq;
      if (stream) store_stream<T, VEC>(sp, v);
      else *reinterpret_cast<V*>(sp) = v;
    } else {
      V* yp = reinterpret_cast<V*>(y + size_t(wd & kIdxMask) * W + sq);
      if (!GAMMA && add) {
        if (!fixed) {
          V o = *yp;
#pragma unroll
          for (int t = 0; t < VEC; ++t) o.v[t] += v.v[t];
          *yp = o;
        }
      } else {
        if (fixed) {
#pragma unroll
          for (int t = 0; t < VEC; ++t) v.v[t] = T(0);
        }
        *yp = v;
      }
    }
  }
  if constexpr (GAMMA) fold_gamma<NR, TPB>(gsum, gamma, gslot, gcount);
}

template <typename T, int NR, bool MASK, bool GAMMA>
void launch_wide_k(const ebe_mesh* m, const void* x, void* y, bool stream, bool bc, bool add, const int* gate,
                   hipStream_t s, double* gamma) {
  using P = typename Pair<T>::type;
  const ebe_mesh::Wide& D = m->wide[wide_size(int(sizeof(T)), NR)];
  const PatchLevel& L = D.pl;
  const P* lame = (sizeof(T) == 8) ? reinterpret_cast<const P*>(m->lame64.as<void>())
                                   : reinterpret_cast<const P*>(m->lame32.as<void>());
  hipLaunchKernelGGL((k_ebe_wide<T, NR, MASK, GAMMA>), dim3(unsigned(L.npatch)), dim3(wide_threads<T>(NR)), 0, s,
                     D.fanl.as<uint16_t>(), m->felem.as<int32_t>(), D.pfan.as<int32_t>(), D.pcorner.as<int32_t>(),
                     L.poff.as<int32_t>(), L.pnode.as<int32_t>(), L.pslot.as<int32_t>(), m->xv.as<double4>(), lame,
                     static_cast<const T*>(x), static_cast<T*>(y), m->pl[0].stage.as<T>(), int(stream), int(bc),
                     int(add), gamma, m->gacc.as<double>(),
                     reinterpret_cast<unsigned*>(m->gacc.as<char>() + kGammaBytes - 64), gate);
}

}  // namespace

template <typename T, int NR>
hipError_t launch_wide(const ebe_mesh* m, const void* x, void* y, bool mask_in, bool bc, bool add, const int* gate,
                       hipStream_t s, double* gamma) {
  const PatchLevel& L = m->wide[wide_size(int(sizeof(T)), NR)].pl;
  if (gamma && (mask_in || add)) return hipErrorInvalidValue;  // no caller needs both
  const bool st = int64_t(L.nslots) * 3 * NR * int64_t(sizeof(T)) > kStreamStageBytes;
  if (mask_in) launch_wide_k<T, NR, true, false>(m, x, y, st, bc, add, gate, s, nullptr);
  else if (gamma) launch_wide_k<T, NR, false, true>(m, x, y, st, bc, add, gate, s, gamma);
  else launch_wide_k<T, NR, false, false>(m, x, y, st, bc, add, gate, s, nullptr);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || L.nshared == 0) return e;
  const int64_t work = L.nshared * (3 * NR / reduce_width<T, NR>());
  hipLaunchKernelGGL((k_reduce_shared<T, NR>), dim3(unsigned((work + 255) / 256)), dim3(256), 0, s,
                     L.snode.as<int32_t>(), L.soff.as<int32_t>(), m->pl[0].stage.as<T>(), int(st),
                     static_cast<T*>(y), int32_t(L.nshared), int(bc), int(add), gate);
  return hipGetLastError();
}

#define EBE_INST(T, n)                                                                                       \
  template hipError_t launch_wide<T, n>(const ebe_mesh*, const void*, void*, bool, bool, bool, const int*, \
                                        hipStream_t, double*);
EBE_INST(float, 1) EBE_INST(float, 2) EBE_INST(float, 3) EBE_INST(float, 4)
EBE_INST(double, 1) EBE_INST(double, 2) EBE_INST(double, 3) EBE_INST(double, 4)
#undef EBE_INST

}  // namespace ebe

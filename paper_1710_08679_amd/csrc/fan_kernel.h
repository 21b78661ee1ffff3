// Pipelined and coloured forms of the quadratic EBE product (Section 2,
// Eq. (3)) on straight-sided elements, at more than kWideCases cases on meshes
// of enough patches (kFanFrom).
//
// Fans.  The tetrahedra of a patch are grouped on the host into fans: chains
// of at most three tetrahedra around a common edge (the spine p-q), each
// sharing a face with the next (patches.cpp).  A work-item takes one fan of
// one case.  It reads each of the fan's nodes once and adds each node's force
// into the patch accumulator once: 18 nodes for three tetrahedra instead of
// 30, so x gathers and LDS additions fall by 40%.  The forces of the spine and
// of the spoke nodes two tetrahedra share are summed in FP64 registers, as
// they were in the FP64 accumulator.
//
// A persistent workgroup works through a sequence of chains of patches (those
// of its XCD's contiguous range, in steps of the number of workgroups on that
// XCD) and keeps the next patch's metadata in flight while it computes the
// current one.  Within a chain the accumulator rows that the next patch shares
// stay in F, so they are written once, when their last patch of the chain ends:
// on a mesh of 2x2x2-hexahedron patches 1.13 rows a node are staged and added
// instead of 1.53 (64^3 cube: FP32 16 cases 638 -> 595 us, FP64 16 cases 1200 ->
// 1104 us, FP32 8 cases 376 -> 357 us).  Per patch:
//   A. commit the prefetched node words, staging slots and fan words to LDS
//      (fan words as byte offsets of the node rows in x and in the FP64
//      accumulator F, so the element phase adds only its case offset);
//   B. issue the next patch's loads;
//   C. element phase: one work-item per (fan, case);
//   D. write back the finished nodes, zeroing F behind it: exclusive nodes
//      straight into y, shared nodes as partial sums into their staging slots
//      (a node-centric pass adds them after).
//
// Coloured form: the patches are coloured so that no two patches of a colour
// share a node, and the colours run one launch after another.  A patch writes
// every one of its nodes straight into y: the first patch (in colour order) to
// touch a node stores its sum, the later ones add theirs to what y holds.  No
// staging buffer, no second pass and no atomics in global memory, at the price
// of one launch per colour and a read of y for the nodes shared between
// colours.  The patches' sums reach a node in colour order; inside a patch
// they are LDS atomics as in the other forms (so not bitwise reproducible).
#pragma once

#include "patch_common.h"

namespace ebe {
namespace {

// positions of a fan's node words (kFanWords of them, kFanStride per fan)
constexpr int fan_spoke(int i) { return i == 0 ? 3 : 2 + 4 * i; }  // spoke i: corner, edge to p, edge to q
constexpr int fan_rim(int i) { return 9 + 4 * i; }                 // edge between spokes i and i + 1
// Fans whose node tables are in LDS at once: a full patch of full fans has 16;
// 20 leaves room for some shorter ones while three workgroups of 16 cases
// still fit in a CU's LDS.  Patches of more fans take several rounds.
constexpr int kFanCap = 20;

// Whether a work-item takes one tetrahedron of a fan instead of the whole fan:
// where the 16 fans of a patch would leave many lanes of their wavefronts idle
// (16 n work-items on ceil(n / 4) wavefronts, two of which fit a SIMD in FP64;
// 48 n tetrahedra fill theirs, and their 160 registers leave room for three).
// Fans / tetrahedra, FP64, 64x64x40 lattice: 5 cases 367 / 343 us, 9 631 / 536,
// 10 593 / 557, 11 720 / 649, 12 633 / 639 (but 35.1 / 32.6 at 15x17x26), 13 761
// / 724; 6 360 / 381, 8 374 / 473, 16 666 / 795.  FP32: 9 495 / 448, 10 441 / 421;
// 5 234 / 262, 8 223 / 260, 12 341 / 405, 16 370 / 418.
template <typename T>
constexpr bool fan_singles(int nr) {
  return nr == 9 || nr == 10 || (sizeof(T) == 8 && (nr == 5 || (nr >= 11 && nr <= 13)));
}
// one work-item per (fan or tetrahedron, case) of a full patch of full fans
template <typename T>
constexpr int fan_threads(int nr) {
  if (fan_singles<T>(nr)) return threads_for(nr, 2, int(sizeof(T)), false);
  const int g = 64 / nr;  // fans per wavefront
  const int fans = kPatchElems / kFanLen;
  // 4, 8, 12, 16 cases fill whole wavefronts in any case
  const int want = nr % 4 == 0 ? fans * nr : ((fans + g - 1) / g * g * nr + 63) / 64 * 64;
  return want > 256 ? 256 : want;
}
constexpr int fan_lds_bytes(int nr) {
  return kPatchNodes * 3 * nr * 8 + kFanCap * kFanStride * 8 + 9 * kPatchNodes + 8 * nr + 16;
}
// Wavefronts per SIMD that the LDS of a workgroup leaves room for, at most
// three in FP32 (168 registers: three tetrahedra's shared sums stay in
// registers) and two in FP64 (256; by tetrahedra with (x, K x) three, which
// left to itself takes as many registers as two allow).
template <typename T>
constexpr int fan_waves_per_simd(int nr, bool gamma) {
  const int wg = 163840 / ((fan_lds_bytes(nr) + 1279) / 1280 * 1280);
  const int w = (wg * (fan_threads<T>(nr) / 64) + 3) / 4;
  const int most = sizeof(T) == 8 ? (gamma && fan_singles<T>(nr) ? 3 : 2) : (fan_singles<T>(nr) ? 4 : 3);
  return w > most ? most : (w < 1 ? 1 : w);
}

// lane L's value of each 16 lanes (row_newbcast)
template <int L>
__device__ __forceinline__ float row_value(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + L, 0xf, 0xf, true));
}
template <int L>
__device__ __forceinline__ double row_value(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + L, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + L, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// GAMMA: also form gamma[r] += (x_r, K x_r), what CG needs from q = K p (never
// with add, nor coloured), free of the rounding that a translation common to a tetrahedron's
// nodes would bring in: from the nodes' differences from corner p (in FP32 the
// error of the plain sum of force times nodal value was twice to eight times
// that of the gather form's strains).  By tetrahedra: strains and stresses of the
// differences (force times value read x twice: 64x64x40 lattice, FP64 12 cases
// 1168 us, FP32 9 cases 514; now 646 and 455).  By fans, where that took more
// instructions and registers that made the FP64 kernel spill: forces times
// differences, which FP64 takes as it reads x (kShift: p's own terms fall away,
// 670 us at 16 cases against 732) and FP32 as it sums (376 us against 386;
// without (x, K x) 367).
// MASK: zero the fixed DOFs of x while reading it.  COLOUR: the coloured form.
// plist lists this launch's patches: all of them in chain order, the node
// entries being by place in it, or one colour, the entries being by patch.
template <typename T, int NR, bool MASK, bool GAMMA, bool COLOUR>
__global__ __launch_bounds__(fan_threads<T>(NR)) __attribute__((amdgpu_waves_per_eu(fan_waves_per_simd<T>(NR, GAMMA)))) void
k_ebe_fan(const T* __restrict__ gfan, const uint32_t* __restrict__ fanw, const int32_t* __restrict__ pfan,
          const int32_t* __restrict__ poff, const int32_t* __restrict__ pnode, const int32_t* __restrict__ pslot,
          const uint8_t* __restrict__ prow, const int32_t* __restrict__ plist, const T* __restrict__ x,
          T* __restrict__ y, T* __restrict__ stage,
          int stream, int npatch, int bc, int add, double* __restrict__ gamma, double* __restrict__ gslot,
          unsigned* __restrict__ gcount, const int* __restrict__ gate) {
  constexpr int W = 3 * NR;                         // values of a node row
  constexpr uint32_t RB = uint32_t(W * sizeof(T));  // bytes of a node row in x and y
  constexpr uint32_t FB = uint32_t(W * 8);          // bytes of a node row in F
  constexpr int TPB = fan_threads<T>(NR);
  constexpr int MAXN = kPatchNodes;
  constexpr int KW = (MAXN + TPB - 1) / TPB;              // node entries per work-item
  constexpr int NT = kFanCap * kFanStride;                // fan words in LDS
  constexpr int KF = (NT + TPB - 1) / TPB;                // fan words per work-item
  constexpr int VEC = pass_vec(NR, NR, int(sizeof(T)));
  constexpr int NV = W / VEC;                             // vectors of a node row
  constexpr int EPK = TPB / NV;
  constexpr int KIT = (MAXN + EPK - 1) / EPK;
  constexpr int G = 64 / NR;                              // fans per wavefront
  constexpr int GV = 16 / int(sizeof(T));
  constexpr bool kTouch = !COLOUR && (sizeof(T) == 8 || fan_singles<T>(NR));
  constexpr bool kRowLane = NR == 16 && sizeof(T) == 8;
  constexpr bool kShift = GAMMA && sizeof(T) == 8;
  using V = VecT<T, VEC>;
  using GR = VecT<T, GV>;
  __shared__ double F[MAXN * W];
  __shared__ __align__(16) uint32_t xtab[kFanCap][kFanStride];  // x-row byte offsets, then the two flag words
  __shared__ __align__(16) uint32_t ftab[kFanCap][kFanStride];  // F-row byte offsets
  __shared__ int32_t words[MAXN];
  __shared__ int32_t slots[COLOUR ? 1 : MAXN];
  __shared__ uint8_t rows[COLOUR ? 1 : MAXN];  // the entries' rows of F (coloured: entry i has row i)
  __shared__ double gsum[NR];
  if (gate && *gate == 0) return;
  const int tid = threadIdx.x;
  // this workgroup's patches: XCD x owns [start, stop), in units of one chain
  // and, after those, of one patch; its g-th workgroup takes units g, g + wx, ...
  const int Gd = gridDim.x, xcd = blockIdx.x % kXcds;
  const int wx = (Gd - xcd + kXcds - 1) / kXcds;  // workgroups on this XCD
  const int q = npatch / kXcds, rr = npatch % kXcds;
  const int start = xcd * q + (xcd < rr ? xcd : rr), stop = start + q + (xcd < rr ? 1 : 0);
  const int nchain = COLOUR ? 0 : int(fan_chained(stop - start)) / kChain;
  int unit = int(blockIdx.x) / kXcds;
  auto unit_place = [&](int u) { return start + u + (kChain - 1) * min(u, nchain); };
  auto step = [&](int pp) {  // the place after pp; advances to the next unit at the end of one
    if (unit < nchain && (pp + 1 - start) % kChain != 0) return pp + 1;
    unit += wx;
    return unit_place(unit);
  };
  int p = unit_place(unit);
  if (GAMMA && tid < NR) gsum[tid] = 0.0;
  // F starts at zero; every write-back zeroes what it read, so it stays zero between patches
  for (int i = tid; i < MAXN * W; i += TPB) F[i] = 0.0;
  // prefetched state of the next patch
  int f0 = 0, nf = 0, o0 = 0, nn = 0;
  int pw[KW], ps[KW], pr[KW];
  uint32_t pt[KF];
  uint32_t touched = 0;
  auto fetch = [&](int pp) {
    const bool chained = unit < nchain;  // (a single patch takes its place in the order, its entries their own rows)
    const int id = COLOUR || chained ? plist[pp] : pp, en = COLOUR ? id : pp;
    f0 = pfan[id];
    nf = pfan[id + 1] - f0;
    o0 = poff[en];
    nn = poff[en + 1] - o0;
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int i = tid + k * TPB;
      pw[k] = i < nn ? pnode[o0 + i] : 0;
      if constexpr (!COLOUR) pr[k] = chained && i < nn ? prow[o0 + i] : i;
      if constexpr (!COLOUR) ps[k] = i < nn ? pslot[o0 + i] : 0;
    }
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int i = tid + k * TPB;
      pt[k] = (i < NT && i < nf * kFanStride) ? fanw[size_t(f0) * kFanStride + i] : 0u;
    }
    // one word of each 128-byte line of the patch's geometry, so that the
    // element phase finds it in L2 (FP64 2-3% faster, FP32 by fans 0-1% slower)
    if constexpr (kTouch)
      if (tid * 128 < nf * kFanLen * 16 * int(sizeof(T)))
        touched = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(gfan) +
                                                     size_t(f0) * (kFanLen * 16 * sizeof(T)) + tid * 128);
  };
  auto put_word = [&](int i, uint32_t w) {  // word i of the LDS tables
    const int f = i / kFanStride, a = i - f * kFanStride;
    xtab[f][a] = a < kFanWords ? (w & kPtabIdMask) * RB : w;
    ftab[f][a] = (w >> kPtabLocalShift) * FB;
  };
  if (p < stop) fetch(p);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the first commit, as every later one, finds its loads done
  // (x, K x): a work-item keeps one case when n divides 64, so it sums in a
  // register and the lanes of a case are combined across the wavefront at the end
  constexpr bool kLaneCase = (64 % NR) == 0 && (TPB % NR) == 0;
  double en_acc = 0.0;
#pragma unroll 1
  while (p < stop) {
    // A. commit this patch
#pragma unroll
    for (int k = 0; k < KW; ++k) {
      const int i = tid + k * TPB;
      if (i < nn) {
        words[i] = pw[k];
        if constexpr (!COLOUR) {
          slots[i] = ps[k];
          rows[i] = uint8_t(pr[k]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < KF; ++k) {
      const int i = tid + k * TPB;
      if (i < NT && i < nf * kFanStride) put_word(i, pt[k]);
    }
    const int cf0 = f0, cnf = nf, cnn = nn;
    __syncthreads();
    // B. the next patch's metadata
    p = step(p);
    if (p < stop) fetch(p);
    const char* xb = reinterpret_cast<const char*>(x);
    char* fbase = reinterpret_cast<char*>(F);
    // C. element phase
#pragma unroll 1
    for (int c0 = 0; c0 < cnf; c0 += kFanCap) {
      if (c0 > 0) {  // a patch of more fans than the tables hold: the next ones, read now
        __syncthreads();
        for (int i = tid; i < NT && i < (cnf - c0) * kFanStride; i += TPB)
          put_word(i, fanw[(size_t(cf0) + c0) * kFanStride + i]);
        __syncthreads();
      }
      const int cf = min(cnf - c0, kFanCap);
      if constexpr (fan_singles<T>(NR)) {  // one work-item per (tetrahedron, case)
        const int ce = cf * kFanLen;
        const int K = (ce + G - 1) / G, GP = (ce + K - 1) / K;
#pragma unroll 1
        for (int w = tid; w < K * GP * NR; w += TPB) {
          const int j = w / NR, r = w - j * NR;
          const int e = (j % GP) * K + j / GP;
          const int f = e / kFanLen, i = e - f * kFanLen;
          if (e >= ce) continue;
          const uint32_t rx = uint32_t(r) * uint32_t(sizeof(T)), rf = uint32_t(r) * 8u;
          const uint32_t* xt = xtab[f];
          const uint32_t* ft = ftab[f];
          const uint32_t flags0 = xt[kFanWords], flags1 = MASK ? xt[kFanWords + 1] : 0u;
          if (i >= int(flags0 & 3u)) continue;
          // the ten words by pairs: p, q; pq; words 2 + 4 i .. (spoke i, after pq
          // where i = 0); words 6 + 4 i .. (spoke i + 1 and the rim)
          auto offsets = [&](const uint32_t* t, uint32_t r0, uint32_t o[10]) {
            const uint2* q = reinterpret_cast<const uint2*>(t);
            const uint2 pq = q[0], a0 = q[1 + 2 * i], a1 = q[2 + 2 * i], b0 = q[3 + 2 * i], b1 = q[4 + 2 * i];
            const bool z = i == 0;
            o[0] = pq.x + r0;
            o[1] = pq.y + r0;
            o[2] = (z ? a0.y : a0.x) + r0;
            o[3] = b0.x + r0;
            o[4] = t[2] + r0;
            o[5] = (z ? a1.y : a1.x) + r0;
            o[6] = (z ? a1.x : a0.y) + r0;
            o[7] = b0.y + r0;
            o[8] = b1.x + r0;
            o[9] = b1.y + r0;
          };
          uint32_t xo[10], fo[10];
          offsets(xt, rx, xo);
          offsets(ft, rf, fo);
          T Gm[4][3], cl = T(0), cm = T(0);
          const T* row = gfan + ((size_t(cf0) + c0 + f) * kFanLen + i) * 16;
#pragma unroll
          for (int v = 0; v < 16 / GV; ++v) {
            const GR gv = *reinterpret_cast<const GR*>(row + v * GV);
#pragma unroll
            for (int t = 0; t < GV; ++t) {
              const int k = (v * GV + t) / 4, d = (v * GV + t) % 4;
              if (d < 3) Gm[k][d] = gv.v[t];
              else if (k == 0) cl = gv.v[t];
              else if (k == 1) cm = gv.v[t];
            }
          }
          auto value = [&](int a, int c) -> T {
            return *reinterpret_cast<const T*>(xb + size_t(xo[a]) + size_t(c) * NR * sizeof(T));
          };
          T up[3];
          if constexpr (GAMMA) {
#pragma unroll
            for (int c = 0; c < 3; ++c) up[c] = value(0, c);
          }
          auto u = [&](int a, int c) -> T {
            const T v = value(a, c);
            if constexpr (GAMMA) {
              return v - up[c];
            } else if constexpr (MASK) {
              const int wa = a == 0 ? 0 : a == 1 ? 1 : a == 4 ? 2 : a == 2 ? (i == 0 ? 3 : 2 + 4 * i)
                           : a == 6 ? (i == 0 ? 4 : 3 + 4 * i) : a == 5 ? (i == 0 ? 5 : 4 + 4 * i)
                           : a == 3 ? 6 + 4 * i : a == 9 ? 9 + 4 * i : a + 4 * i;  // (7, 8)
              const uint32_t bit = wa < 10 ? flags0 >> (2 + 3 * wa + c) : flags1 >> (3 * (wa - 10) + c);
              return (bit & 1u) ? T(0) : v;
            } else {
              return v;
            }
          };
          T en = T(0);
          auto emit = [&](int a, const T fv[3]) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
              atomicAdd(reinterpret_cast<double*>(fbase + fo[a]) + c * NR, double(fv[c]));
          };
          p2_apply<GAMMA>(Gm, cl, cm, u, emit, GAMMA, en);
          if constexpr (GAMMA) {
            if constexpr (kLaneCase) en_acc += double(en);
            else atomicAdd(&gsum[r], double(en));
          }
        }
        continue;
      }
      // a wavefront's fans lie K apart (neighbouring fans share nodes)
      const int K = (cf + G - 1) / G, GP = NR % 4 == 0 ? (cf + K - 1) / K : G;
#pragma unroll 1
      for (int w = tid; w < K * GP * NR; w += TPB) {
        const int j = w / NR, r = w - j * NR;
        const int f = (j % GP) * K + j / GP;
        if (f >= cf) continue;
        const uint32_t rx = uint32_t(r) * uint32_t(sizeof(T)), rf = uint32_t(r) * 8u;
        const uint32_t* xt = xtab[f];
        const uint32_t* ft = ftab[f];
        const uint32_t flags0 = xt[kFanWords], flags1 = MASK ? xt[kFanWords + 1] : 0u;
        const int len = int(flags0 & 3u);
        auto ld = [&](int a, int c) -> T {
          const T v = *reinterpret_cast<const T*>(xb + size_t(xt[a] + rx) + size_t(c) * NR * sizeof(T));
          if constexpr (MASK) {
            const uint32_t bit = a < 10 ? flags0 >> (2 + 3 * a + c) : flags1 >> (3 * (a - 10) + c);
            return (bit & 1u) ? T(0) : v;
          } else {
            return v;
          }
        };
        auto put = [&](int a, int c, double v) {
          atomicAdd(reinterpret_cast<double*>(fbase + ft[a] + rf) + c * NR, v);
        };
        T us[3][3], ud[3][3];
        double fd[3][3], fs[3][3];  // forces of the spine (p, q, pq) and of the current spoke
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            ud[a][c] = ld(a, c);
            us[a][c] = ld(3 + a, c);
            fd[a][c] = fs[a][c] = 0.0;
          }
        T up[3] = {T(0), T(0), T(0)};
        if constexpr (kShift) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            up[c] = ud[0][c];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
              if (a > 0) ud[a][c] -= up[c];
              us[a][c] -= up[c];
            }
          }
        }
        auto shift = [&](T v, int c) -> T {
          if constexpr (kShift) return v - up[c];
          else return v;
        };
        const T* grow = gfan + (size_t(cf0 + c0 + f) * kFanLen) * 16;
#pragma unroll
        for (int i = 0; i < kFanLen; ++i) {
          // tetrahedron i: corners p, q, spoke i, spoke i + 1
          if (i >= len) continue;
          T un[3][3], ur[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int a = 0; a < 3; ++a) un[a][c] = shift(ld(fan_spoke(i + 1) + a, c), c);
            ur[c] = shift(ld(fan_rim(i), c), c);
          }
          auto u = [&](int a, int c) -> T {
            return a == 0 ? ud[0][c] : a == 1 ? ud[1][c] : a == 2 ? us[0][c] : a == 3 ? un[0][c] : a == 4 ? ud[2][c]
                 : a == 5 ? us[2][c] : a == 6 ? us[1][c] : a == 7 ? un[1][c] : a == 8 ? un[2][c] : ur[c];
          };
          // component c of local node a's force: 0, 1, 4 the spine; 2, 6, 5
          // spoke i, now complete; 3, 7, 8 spoke i + 1, which starts the
          // next sum; 9 the rim
          auto add_force = [&](int a, int c, double d) {
            if (a == 0 || a == 1 || a == 4) {
              fd[a == 4 ? 2 : a][c] += d;
            } else if (a == 2 || a == 5 || a == 6) {
              const int k = a == 2 ? 0 : (a == 6 ? 1 : 2);
              put(fan_spoke(i) + k, c, fs[k][c] + d);
            } else if (a == 9) {
              put(fan_rim(i), c, d);
            }
          };
          const T* row = grow + 16 * i;
          T Gm[4][3], cl = T(0), cm = T(0);
          if constexpr (kRowLane) {  // value t in lane t of the 16
            const T g = row[r];
#define EBE_ROW(t) row_value<t>(g)
            Gm[0][0] = EBE_ROW(0); Gm[0][1] = EBE_ROW(1); Gm[0][2] = EBE_ROW(2); cl = EBE_ROW(3);
            Gm[1][0] = EBE_ROW(4); Gm[1][1] = EBE_ROW(5); Gm[1][2] = EBE_ROW(6); cm = EBE_ROW(7);
            Gm[2][0] = EBE_ROW(8); Gm[2][1] = EBE_ROW(9); Gm[2][2] = EBE_ROW(10);
            Gm[3][0] = EBE_ROW(12); Gm[3][1] = EBE_ROW(13); Gm[3][2] = EBE_ROW(14);
#undef EBE_ROW
          } else {
#pragma unroll
            for (int v = 0; v < 16 / GV; ++v) {
              const GR gv = *reinterpret_cast<const GR*>(row + v * GV);
#pragma unroll
              for (int t = 0; t < GV; ++t) {
                const int k = (v * GV + t) / 4, d = (v * GV + t) % 4;
                if (d < 3) Gm[k][d] = gv.v[t];
                else if (k == 0) cl = gv.v[t];
                else if (k == 1) cm = gv.v[t];
              }
            }
          }
          double nx[3][3];
          T en = T(0);
          auto emit = [&](int a, const T fv[3]) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              if constexpr (kShift) {
                if (a > 0) en += fv[c] * u(a, c);
              } else if constexpr (GAMMA) {  // (not before the forces: the differences would occupy registers)
                if (a == 0) asm volatile("" : "+v"(ud[0][c]));
                else en += fv[c] * (u(a, c) - ud[0][c]);
              }
              if (a == 3 || a == 7 || a == 8) nx[a == 3 ? 0 : a - 6][c] = double(fv[c]);
              else add_force(a, c, double(fv[c]));
            }
          };
          T unused = T(0);
          p2_apply<kShift>(Gm, cl, cm, u, emit, false, unused);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            fs[0][c] = nx[0][c];
            fs[1][c] = nx[1][c];
            fs[2][c] = nx[2][c];
          }
#pragma unroll
          for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int c = 0; c < 3; ++c) us[a][c] = un[a][c];
          if constexpr (GAMMA) {
            if constexpr (kLaneCase) en_acc += double(en);
            else atomicAdd(&gsum[r], double(en));
          }
        }
        const int last = 2 + 4 * len;  // fan_spoke(len)
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            put(last + a, c, fs[a][c]);
            put(a, c, fd[a][c]);
          }
      }
    }
    // the next patch's metadata has arrived before this patch's write-back
    // stores are issued, so the next commit waits for no store
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    if constexpr (kTouch) asm volatile("" ::"v"(touched));
    __syncthreads();
    // D. write back, zeroing F behind it.  Coloured form at 8 or more cases
    // (at 4, FP64, it measured 15% slower): the rows that are read, added to
    // and written back are all read before the first store, so the reads do
    // not wait for this patch's stores (64^3 cube, 16 cases: 1.385 ->
    // 1.321 ms FP64).  The pipelined form reads y only for y += K x and
    // keeps one read per row piece.  y is written with streaming
    // (non-temporal) stores: a product's y is larger than the last-level
    // cache at 16 cases, and keeping x there instead measured faster.
    constexpr bool kReadFirst = COLOUR && NR >= 8;
    // this work-item's vector of a node row: value sq of the row, component sc
    // (formed anew at each write-back: kept, they would cost the element
    // phase registers)
    int wtid = tid;
    asm volatile("" : "+v"(wtid));
    const int sv = wtid % NV, sent = wtid < EPK * NV ? wtid / NV : MAXN, sq = sv * VEC, sc = sq / NR;
    V* const yv = reinterpret_cast<V*>(y);
    V old[kReadFirst ? KIT : 1];
#pragma unroll
    for (int k = 0; k < (kReadFirst ? KIT : 0); ++k) {
      const int ent = sent + k * EPK;
      if (ent < cnn) {
        const int32_t wd = words[ent];  
        const bool fixed = bc && ((wd >> (kIdxBits + sc)) & 1);
        if (((!GAMMA && add && wd != kNoEntry) || wd < 0) && !fixed)
          old[k] = yv[uint32_t(wd & kIdxMask) * uint32_t(NV) + uint32_t(sv)];
      }
    }
#pragma unroll
    for (int k = 0; k < KIT; ++k) {
      const int ent = sent + k * EPK;
      if (ent < cnn) {
        const int32_t wd = words[ent];
        if (COLOUR && wd == kNoEntry) continue;
        double* const fr = F + (COLOUR ? ent : int(rows[ent])) * W + sq;
        V v;
#pragma unroll
        for (int t = 0; t < VEC; ++t) {
          v.v[t] = T(fr[t]);
          fr[t] = 0.0;
        }
        const bool fixed = bc && ((wd >> (kIdxBits + sc)) & 1);
        if (!COLOUR && wd < 0) {  // shared node: partial sum to its staging slot
          V* sp = reinterpret_cast<V*>(stage) + (uint32_t(slots[ent]) * uint32_t(NV) + uint32_t(sv));
          if (stream) store_stream<T, VEC>(reinterpret_cast<T*>(sp), v);
          else *sp = v;
        } else {
          V* yp = yv + (uint32_t(wd & kIdxMask) * uint32_t(NV) + uint32_t(sv));
          if ((!GAMMA && add) || (COLOUR && wd < 0)) {  // y += (the caller, or an earlier colour, wrote y)
            if (!fixed) {  // (a fixed DOF keeps what y holds: the caller's value, or the first colour's zero)
              V o;
              if constexpr (kReadFirst) o = old[k];
              else o = *yp;
#pragma unroll
              for (int t = 0; t < VEC; ++t) o.v[t] += v.v[t];
              store_stream<T, VEC>(reinterpret_cast<T*>(yp), o);
            }
          } else {
            if (fixed) {
#pragma unroll
              for (int t = 0; t < VEC; ++t) v.v[t] = T(0);
            }
            store_stream<T, VEC>(reinterpret_cast<T*>(yp), v);
          }
        }
      }
    }
    __syncthreads();  // F, words, slots and fan tables (next patch)
  }
  if constexpr (GAMMA) {
    if constexpr (kLaneCase) {
      double v = en_acc;
#pragma unroll
      for (int off = 32; off >= NR; off >>= 1) v += __shfl_xor(v, off, 64);
      if ((tid & 63) < NR) atomicAdd(&gsum[tid & 63], v);
    }
    __syncthreads();
    fold_gamma<NR, TPB>(gsum, gamma, gslot, gcount);
  }
}

// as many persistent workgroups as fit on the device at once (measured
// occupancy x CUs), at most one per patch
template <typename T, int NR, bool MASK, bool GAMMA, bool COLOUR>
hipError_t launch_fan_k(const ebe_mesh* m, const int32_t* plist, int64_t npatch, const void* x, void* y, bool stream,
                        bool bc, bool add, const int* gate, hipStream_t s, double* gamma) {
  constexpr int TPB = fan_threads<T>(NR);
  static const int per_cu = [] {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ebe_fan<T, NR, MASK, GAMMA, COLOUR>, TPB, 0) !=
            hipSuccess ||
        n < 1)
      n = 1;
    return n;
  }();
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device) != hipSuccess || cus < 1)
    cus = 256;
  const int64_t grid = std::min<int64_t>(npatch, int64_t(per_cu) * cus);
  if (grid < 1) return hipSuccess;
  const PatchLevel& L = m->chain;
  hipLaunchKernelGGL((k_ebe_fan<T, NR, MASK, GAMMA, COLOUR>), dim3(unsigned(grid)), dim3(TPB), 0, s,
                     m->gfan[sizeof(T) == 8 ? 0 : 1].as<T>(), m->fanw.as<uint32_t>(), m->pfan.as<int32_t>(),
                     (COLOUR ? m->croff : L.poff).as<int32_t>(), (COLOUR ? m->crow : L.pnode).as<int32_t>(),
                     L.pslot.as<int32_t>(), m->cslot.as<uint8_t>(), plist,
                     static_cast<const T*>(x), static_cast<T*>(y), m->pl[0].stage.as<T>(),
                     int(stream), int(npatch), int(bc), int(add), gamma, m->gacc.as<double>(),
                     reinterpret_cast<unsigned*>(m->gacc.as<char>() + kGammaBytes - 64), gate);
  return hipGetLastError();
}

template <typename T, int NR, bool COLOUR>
hipError_t launch_fan_c(const ebe_mesh* m, const int32_t* plist, int64_t npatch, const void* x, void* y, bool stream,
                        bool mask_in, bool bc, bool add, const int* gate, hipStream_t s, double* gamma) {
  if (mask_in && gamma) return hipErrorInvalidValue;  // no caller needs both
  if (mask_in)
    return launch_fan_k<T, NR, true, false, COLOUR>(m, plist, npatch, x, y, stream, bc, add, gate, s, nullptr);
  if (gamma && add) return hipErrorInvalidValue;
  if constexpr (COLOUR) {
    if (gamma) return hipErrorInvalidValue;  // quad_kernel names another
  } else {
    if (gamma)
      return launch_fan_k<T, NR, false, true, COLOUR>(m, plist, npatch, x, y, stream, bc, add, gate, s, gamma);
  }
  return launch_fan_k<T, NR, false, false, COLOUR>(m, plist, npatch, x, y, stream, bc, add, gate, s, nullptr);
}

}  // namespace

template <typename T, int NR>
hipError_t launch_fan(const ebe_mesh* m, const void* x, void* y, bool mask_in, bool bc, bool add, const int* gate,
                      hipStream_t s, double* gamma, bool colour) {
  if (colour) {
    if constexpr (kFanFrom[1][sizeof(T) == 8 ? 0 : 1][NR] != kNever) {
      const PatchLevel& L = m->pl[0];
      const int32_t* cp = L.cperm.as<int32_t>();
      for (size_t c = 0; c + 1 < L.coff.size(); ++c) {
        const hipError_t e = launch_fan_c<T, NR, true>(m, cp + L.coff[c], L.coff[c + 1] - L.coff[c], x, y, false,
                                                       mask_in, bc, add, gate, s, gamma);
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    } else {
      return hipErrorInvalidValue;  // quad_kernel names another
    }
  }
  // stream the staged partials past the caches when they cannot stay in the
  // last-level cache until the shared-node pass reads them back
  const PatchLevel& L = m->chain;
  const bool st = int64_t(L.nslots) * 3 * NR * int64_t(sizeof(T)) > kStreamStageBytes;
  hipError_t e = launch_fan_c<T, NR, false>(m, m->cseq.as<int32_t>(), L.npatch, x, y, st, mask_in, bc, add, gate, s,
                                            gamma);
  if (e != hipSuccess || L.nshared == 0) return e;
  const int64_t work = L.nshared * (3 * NR / reduce_width<T, NR>());
  hipLaunchKernelGGL((k_reduce_shared<T, NR>), dim3(unsigned((work + 255) / 256)), dim3(256), 0, s,
                     L.snode.as<int32_t>(), L.soff.as<int32_t>(), m->pl[0].stage.as<T>(), int(st), static_cast<T*>(y),
                     int32_t(L.nshared), int(bc), int(add), gate);
  return hipGetLastError();
}

}  // namespace ebe

// Internal declarations of the EBE library: the mesh handle, device buffers,
// error reporting and the kernel launchers shared between translation units.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "ebe.h"

namespace ebe {

// Connectivity words carry the node id in the low 28 bits and the node's
// Dirichlet flags (x, y, z) in bits 28..30, so that a kernel that gathers a
// node also knows which of its DOFs are fixed without a second load.
constexpr int32_t kIdxBits = 28;
constexpr int32_t kIdxMask = (1 << kIdxBits) - 1;

void set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));

// Kernels move node rows of vectors in 16-byte pieces.
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

#define EBE_TRY_HIP(call)                                                        \
  do {                                                                           \
    hipError_t e_ = (call);                                                      \
    if (e_ != hipSuccess) {                                                      \
      ::ebe::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),    \
                       __FILE__, __LINE__);                                      \
      return EBE_ERR_HIP;                                                        \
    }                                                                            \
  } while (0)

// Owned device allocation.
class DBuf {
 public:
  DBuf() = default;
  DBuf(const DBuf&) = delete;
  DBuf& operator=(const DBuf&) = delete;
  ~DBuf() { release(); }
  ebe_status alloc(size_t bytes);        // no-op when already at least this large
  void view(void* p, size_t bytes);      // bytes of another buffer's memory, which outlives this one
  void release();
  template <class T> T* as() const { return static_cast<T*>(p_); }
  size_t bytes() const { return n_; }
 private:
  void* p_ = nullptr;
  size_t n_ = 0;
  bool owned_ = false;
};

// Uploads of a mesh's tables: those of at most kSmall bytes are gathered and
// go into one allocation with one copy when finish() is called, the others at
// once into allocations of their own.  A 4^3 cube has about 60 tables, and an
// allocation and a copy for each were most of its creation (0.55 -> 0.18 ms).
class Uploads {
 public:
  explicit Uploads(hipStream_t s) : s_(s) {}
  ebe_status add(DBuf& b, const void* host, size_t bytes);
  ebe_status finish(DBuf& owner);
 private:
  static constexpr size_t kSmall = 64 << 10;
  struct Item {
    DBuf* b;
    size_t at, bytes;
  };
  hipStream_t s_;
  std::vector<Item> items_;
  std::vector<char> host_;
};

// An operator assembled into 3x3 blocks, in slices of kSliceRows rows: slice
// s has soff[s+1] - soff[s] slots (its longest row), slot j of row r is entry
// j * kSliceRows + r; short rows are padded with zero blocks whose column is
// the row itself.  Values value-major within a slot, so the rows of a
// wavefront read each value from one contiguous run.
struct AsmOp {
  DBuf soff;    // int32 [nslices+1]
  DBuf col;     // int32 [slots][kSliceRows] column id | fix bits
  DBuf val[2];  // [slots][9][kSliceRows] block values (row-major 3x3), per dtype (F64, F32)
  int64_t rows = 0, slots = 0;
  bool ready[2] = {false, false};
  // FP16 copy of the values divided by half_scale (the largest magnitude
  // over 2^14), for the coarse levels of a mixed solve with coarse_half set
  DBuf val16;
  double half_scale = 1.0;
  bool ready16 = false;
};

// Solver workspace; grown to the largest nrhs seen.
struct Workspace {
  int nrhs_cap = 0;
  // FP64 outer vectors [N][3][nrhs]
  DBuf r, p, q;
  // preconditioner vectors (FP32 or FP64) on levels 0, 1 and 2
  DBuf rb, ub, e0, p0, q0;
  DBuf r1, u1, e1, p1, q1;
  DBuf r2, u2, e2, p2, q2;
  // per-column scalars and reduction partials
  DBuf scal;      // double scalars (see solver.cpp for the slots)
  DBuf partials;  // block partial sums
  DBuf flags;     // int32 device flags
  DBuf counter;   // int32/uint32 arrival counters for last-block reductions
  int* host_flags = nullptr;  // pinned host mirror
  // Instantiated graphs of fixed runs of solver steps, keyed by everything
  // baked into their kernel arguments (buffer addresses, nrhs, step count).
  struct Graph {
    std::vector<uintptr_t> key;
    hipGraphExec_t exec = nullptr;
  };
  std::vector<Graph> graphs;
  int64_t captures = 0;  // graphs captured so far (ebe_pcg_stats reports the count per solve)
};

// Element patches (patches.cpp): consecutive element ranges whose node sums
// fit in LDS.  Quadratic level: at most kPatchElems elements touching at most
// kPatchNodes nodes; 48 elements and 128 nodes fit a block of 2x2x2
// hexahedra of 6 tetrahedra (5^3 = 125 nodes) exactly, so on meshes in
// Morton order patches are compact blocks and fewer of their nodes are shared
// than with 64-element ranges that cut hexahedra apart.  Linear level: at most
// kLinPatchElems elements touching at most kLinPatchCorners corners (a linear
// element carries far less work, so its patches are larger).
#ifndef EBE_PATCH_ELEMS
#define EBE_PATCH_ELEMS 48
#endif
#ifndef EBE_PATCH_NODES
#define EBE_PATCH_NODES 128
#endif
#ifndef EBE_LIN_PATCH_ELEMS
#define EBE_LIN_PATCH_ELEMS 256
#endif
#ifndef EBE_LIN_PATCH_CORNERS
#define EBE_LIN_PATCH_CORNERS 128
#endif
#ifndef EBE_PATCH_THREADS
#define EBE_PATCH_THREADS 512
#endif
#ifndef EBE_PATCH_THREADS_F64
#define EBE_PATCH_THREADS_F64 256
#endif
// Fans of the quadratic patches (pipelined and coloured forms, fan_kernel.h):
// chains of at most kFanLen tetrahedra around a common edge.  A fan has
// kFanWords node words (node id | patch-local id << kPtabLocalShift): the
// spine's ends and mid node, then the spokes and rims; then two flag words
// (tetrahedra in bits 0-1, the nodes' fix bits, three per node, ten nodes from
// bit 2 of the first word, eight in the second).
constexpr int kFanLen = 3;
constexpr int kFanWords = 6 + 4 * kFanLen;
constexpr int kFanStride = kFanWords + 2;
// Wide patches (ebe_wide.hip): runs of consecutive patches for products of at
// most kWideCases cases, in two sizes (blocks of 2x4x4 and 4x4x4 hexahedra of a
// Morton-ordered mesh): at most so many elements, nodes and corners.  Rows of
// kWideStride patch-local ids per fan: the kFanWords nodes, then the number of
// tetrahedra.
constexpr int kWideSizes = 2;
constexpr int kWideElems[kWideSizes] = {192, 384};
constexpr int kWideNodes[kWideSizes] = {408, 736};
constexpr int kWideCorners[kWideSizes] = {128, 160};
constexpr int kWideCases = 4;
constexpr int kWideStride = 24;
// the size a product takes: FP32 at three or four cases the smaller (its
// accumulator leaves room for three workgroups of four wavefronts; 64^3 cube,
// 4 cases 207 us against 229), the others the larger (FP64 1 case 131 -> 116
// us, FP64 4 cases 376 -> 335 us, FP32 1 case 87 -> 71 us)
constexpr int wide_size(int value_bytes, int nr) { return value_bytes == 4 && nr >= 3 ? 0 : 1; }
constexpr int kSliceRows = 64;  // rows per slice of an assembled operator (AsmOp)
constexpr int kA2MaxRow = 800;  // longest level-2 row (blocks) whose sums fit 64 KB of LDS
constexpr int kPatchElems = EBE_PATCH_ELEMS;
constexpr int kPatchNodes = EBE_PATCH_NODES;
constexpr int kLinPatchElems = EBE_LIN_PATCH_ELEMS;
constexpr int kLinPatchCorners = EBE_LIN_PATCH_CORNERS;  // local ids are bytes: at most 256
constexpr int kPatchThreads = EBE_PATCH_THREADS;  // workgroup size cap of the patch kernels
// FP64 quadratic patches: smaller workgroups, so two fit per CU within the
// registers the FP64 element operator needs (two wavefronts per SIMD)
constexpr int kPatchThreadsF64 = EBE_PATCH_THREADS_F64;
static_assert(kPatchNodes <= 256 && kLinPatchCorners <= 256, "patch-local node ids are bytes");
// (x, K x) sums of the patch kernels: workgroup w adds its per-case sums to
// slot w % kGammaSlots (one 128-byte line each), and the last workgroup to
// finish folds the slots into the caller's result.
constexpr int kGammaSlots = 64;
constexpr size_t kGammaBytes = size_t(kGammaSlots) * EBE_MAX_RHS * sizeof(double) + 64;  // slots + counter

// Patch tables of one level (0: all nodes of the quadratic mesh, 1: corners).
struct PatchLevel {
  DBuf pelem;   // int32 [npatch+1] element offsets (patches are element ranges)
  int64_t npatch = 0;
  DBuf poff;    // int32 [npatch+1] entry offsets
  DBuf pnode;   // int32 [entries] node id | fix bits << 28 | shared << 31
  DBuf pslot;   // int32 [entries] staging slot of a shared entry, -1 otherwise
  DBuf snode;   // int32 [nshared] shared node id | fix bits << 28, increasing id
  DBuf soff;    // int32 [nshared+1] first staging slot of each shared node (its slots are consecutive)
  DBuf stage;   // staging buffer [nslots][3][nrhs] of the product's dtype
  int64_t nslots = 0, nshared = 0, entries = 0;
  int max_nodes = 0;
  // element node words [E][10] (quadratic, straight meshes) or [E][4] (linear): node id |
  // patch-local id << kPtabLocalShift; empty on meshes of 2^25 nodes or more
  DBuf ptab;
  // colouring of the patches (quadratic level): no two patches of a colour
  // share a node; cperm lists the patches colour by colour (increasing id
  // within a colour), colour c is cperm[coff[c] .. coff[c+1]); cword is
  // pnode with bit 31 meaning "an earlier colour wrote this node"
  DBuf cperm;
  DBuf cword;
  std::vector<int64_t> coff;
  // node-centric incidence lists of the quadratic patches (deterministic
  // form): pinc [E][10] element slots (element - patch's first) * 10 + a,
  // grouped by patch entry in element order; pistart [entries] the start of
  // an entry's list relative to its patch's first slot
  DBuf pinc;
  DBuf pistart;
};
// element node words: 25 bits of node id, 7 bits of patch-local id
constexpr int kPtabLocalShift = 25;
constexpr uint32_t kPtabIdMask = (1u << kPtabLocalShift) - 1;
static_assert(kPatchNodes <= 128 && kLinPatchCorners <= 128, "patch-local ids must fit 7 bits");

// Kernels of the pipelined and coloured forms on the quadratic level: by fans
// of tetrahedra (fan_kernel.h; pipelined at up to kWideCases cases by wide
// patches, ebe_wide.hip) or by single elements (pipe_kernel.h), the geometry
// read per work-item or kept in LDS.
enum class QuadKernel { fans, elements, elements_lds };

// Patches of 48 elements from which fans are the faster, by [pipelined,
// coloured, pipelined with (x, K x)][FP64, FP32][cases].  A fan's work-item is three tetrahedra long, so
// it needs several patches per workgroup to hide that; below, one element a
// work-item ends sooner (pipelined, 29x23x17 lattice, 1417 patches, elements / fans:
// FP64 8 cases 32.5 / 35.5 us, 16 53.4 / 51.8; FP32 8 24.7 / 27.0, 16 33.4 / 33.8;
// 64x64x40 lattice, 20480 patches: 478 / 376, 866 / 660; 267 / 224, 443 / 367).  At
// FP64 5 and FP32 9 and 10 cases only the chains of larger meshes repay fans
// (40x40x20: FP64 5 cases 59.8 / 64.2, FP32 9 82.0 / 87.8).  A colour is an eighth of
// the mesh, and its launch ends with its slowest workgroup (coloured, 1417
// patches: FP64 1 case 102 / 151 us, FP32 8 87 / 148, 16 115 / 153; 20480: FP32 8 285
// / 264, 12 426 / 348, 16 424 / 396): never by fans at up to 5 cases and at most
// numbers of cases in FP64.  (x, K x) costs each workgroup an addition to one of a
// few places in memory, so wide patches, of which there are fewer, repay
// themselves earlier with it (1417 patches, FP32 1 case 30.0 / 20.4 us; without
// 12.8 / 15.8) and fans later (FP32 7 cases 34.8 / 40.9; without 31.8 / 29.5);
// coloured it goes by elements, whose registers have room for it (6912 patches,
// FP32 8 cases 144 against 223).  Measured on twelve lattices of 144 to 32768 patches
// at 1 to 16 cases; each number lies between the sizes where the order changes.
constexpr int32_t kNever = 0x7fffffff;
constexpr int32_t kFanFrom[3][2][EBE_MAX_RHS + 1] = {
    {{0, 5000, 1200, 3500, 3500, 6144, 2200, 1200, 2200, 1200, 1200, 1200, 1200, 1200, 2200, 0, 0},
     {0, 5000, 3500, 5000, 2200, 2200, 1200, 1200, 2200, 6144, 6144, 2200, 1200, 3500, 1200, 3500, 2200}},
    {{0, kNever, kNever, kNever, kNever, kNever, 6144, 32000, kNever, kNever, kNever, kNever, kNever, kNever, 3500,
      kNever, 20000},
     {0, kNever, kNever, kNever, kNever, kNever, 6144, 14000, 6500, kNever, kNever, 9000, 6144, 14000, 9000, 20000,
      9000}},
    {{0, 1200, 1200, 3500, 3500, 2200, 2200, 2200, 4500, 4500, 1200, 1200, 1200, 1200, 0, 0, 0},
     {0, 1200, 1200, 1200, 1200, 5000, 2200, 2200, 6144, 10000, 6144, 2200, 2200, 2200, 1200, 2200, 3500}}};

// Elements with the geometry in LDS are instantiated where they measured 1 to 7%
// faster than the other two: coloured, FP64, 6 and 7 cases on smaller meshes
// (40x40x20 lattice 104 us against 113, 135 against 143; 5952 patches 223 against
// 231, but 290 against 251), pipelined, FP64, 9 to 11 and FP32, 9 and 10 cases on
// meshes without chains (40x40x20: FP64 9 cases 109 against 113, 10 110 against
// 112, FP32 10 76.2 against 77.1).
constexpr bool lds_elements(bool colour, int value_bytes, int nr) {
  return colour ? value_bytes == 8 && (nr == 6 || nr == 7) : (nr == 9 || nr == 10 || (value_bytes == 8 && nr == 11));
}
constexpr bool lds_patches(bool colour, int nr, int64_t npatch) {
  return colour ? npatch < (nr == 6 ? 6144 : 5000) : npatch >= 2200 && npatch < 6144;
}

constexpr int kXcds = 8;  // dies of the GPU, each with an L2 of its own

// Chains of the pipelined quadratic form: kChain consecutive patches in an
// order in which neighbours share many nodes.  The workgroup that works through
// a chain keeps the accumulator rows that the next patch shares, so a face
// between two patches costs no partial sums of its own.  Of an XCD's cnt
// patches the first fan_chained(cnt) are in chains and the others single, which
// evens out the workgroups' shares: whole rounds of 64 or 96 workgroups an XCD
// (two or three per CU, FP64 and FP32 at 16 cases).
constexpr int kChain = 4;
constexpr int64_t kChainRound = 192 * kChain;
constexpr int32_t kNoEntry = kIdxMask;
constexpr int64_t fan_chained(int64_t cnt) { return cnt / kChainRound * kChainRound; }

}  // namespace ebe

struct ebe_mesh {
  ebe::DBuf small_tables;  // owns the memory of the tables that Uploads gathered
  int64_t n_nodes = 0, n_vertices = 0, n_elem = 0;
  bool has_bc = false;
  // isoparametric (curved) quadratic elements: the quadratic level uses the
  // curved element kernel (gather form), xv holds every node
  bool curved = false;
  int device = 0;
  ebe::DBuf conn;       // int32 [E][10], packed (see kIdxBits)
  ebe::DBuf xv;         // double4 [Nv] corner coordinates (curved: [N], corners first; w unused)
  ebe::DBuf lame64;     // double2 [E] (lambda, mu)
  ebe::DBuf lame32;     // float2  [E]
  ebe::DBuf young;      // double [E]
  ebe::DBuf poisson;    // double [E]
  ebe::DBuf fix;        // uint8  [N] bit c = DOF c fixed
  ebe::DBuf edge_ends;  // int32 [N-Nv][2]
  ebe::DBuf v2e_off;    // int32 [Nv+1] corner -> incident edge nodes (CSR)
  ebe::DBuf v2e_idx;    // int32 [2 (N-Nv)]
  ebe::DBuf v2el_off;   // int32 [Nv+1] corner -> incident elements (CSR)
  ebe::DBuf v2el;       // int32 [4E] element * 4 + the corner's local index, by element
  // element patches of the two levels
  ebe::DBuf lconn;      // uint8 [E][16] quadratic-patch-local ids of the 10 nodes (padded to 16 bytes)
  ebe::DBuf lconn1;     // uint8 [E][4]  linear-patch-local ids of the 4 corners
  ebe::PatchLevel pl[2];
  // fans of the quadratic patches; empty on meshes of 2^25 nodes or more and on curved ones
  ebe::DBuf pfan;       // int32 [npatch+1] fan offsets
  ebe::DBuf fanw;       // uint32 [nfan][kFanStride]
  ebe::DBuf felem;      // int32 [nfan][kFanLen] element, -1: none
  int64_t nfan = 0;
  // pipelined form: the patches in the order it takes them, and the nodes each
  // one finishes (see fan_chained); staged in pl[0].stage
  ebe::PatchLevel chain;
  ebe::DBuf cseq;       // int32 [npatch] patch at a place of the order
  ebe::DBuf cslot;      // uint8 [chain.entries] accumulator row of a finished node
  // coloured form: by patch, pl[0].cword at each node's accumulator row, kNoEntry in between
  ebe::DBuf croff;      // int32 [npatch+1]
  ebe::DBuf crow;       // int32
  // wide patches of each size
  struct Wide {
    ebe::PatchLevel pl;   // node tables (corners first) and staging slots; staged in pl[0].stage
    ebe::DBuf pfan;       // int32 [pl.npatch+1] fan offsets
    ebe::DBuf pcorner;    // int32 [pl.npatch] corners
    ebe::DBuf fanl;       // uint16 [nfan][kWideStride] the fans' patch-local ids
  } wide[ebe::kWideSizes];
  ebe::DBuf gacc;       // kGammaBytes: (x, K x) slots, then the arrival counter; zero between products
  // EBE product form per [level][dtype F64, F32][nrhs]: one of the forms, or
  // EBE_FORM_AUTO (untuned: a fixed default)
  int8_t form[2][2][EBE_MAX_RHS + 1];
  // kernel variant of the form per [level][dtype][nrhs], set by the tuner
  int8_t fvar[2][2][EBE_MAX_RHS + 1];
  ebe_mesh() {
    std::memset(form, EBE_FORM_AUTO, sizeof(form));
    std::memset(fvar, 0, sizeof(fvar));
  }
  // 3x3 block Jacobi: inverted symmetric blocks (xx yy zz yz zx xy), per level
  // (levels 0 and 1 with the material; level 2 with its operator)
  ebe::DBuf minv64[3], minv32[3];
  bool minv_ready = false;
  // geometry cache [E][16] per dtype (F64, F32): G, V, lambda, mu; filled on
  // first use by an entry point, dropped when the material changes
  ebe::DBuf geo[2];
  bool geo_ready[2] = {false, false};
  // the same by fan tetrahedra, corners in fan order [nfan][kFanLen][16] (G_m[d] at 4 m + d,
  // lambda V / 20 at 3, mu V / 20 at 7), for the pipelined and coloured forms of the quadratic level
  ebe::DBuf gfan[2];
  bool gfan_ready[2] = {false, false};
  // by dtype: a product has been prepared; it read geo, gfan (filled again after
  // a change of material whichever form is next: captured graphs may read them)
  bool prepared[2] = {false, false}, geo_used[2] = {false, false}, gfan_used[2] = {false, false};
  hipEvent_t material = nullptr;  // recorded when a change of material has been enqueued
  // assembled linear-level operator K1 over the corner graph (its edges are
  // the quadratic mesh's edge nodes); structure at creation, values on demand
  ebe::AsmOp k1;
  // level 2 (smoothed aggregation of the corner graph): aggregate of each
  // corner, coarse fix bits (a component is fixed when it is fixed at every
  // member), the smoothed prolongator P2 by fine rows (p2_width slots: the
  // aggregates of the corner and its neighbours, increasing, -1 padding; 3x3
  // blocks per slot, values with A2), its transpose as lists of P2 entries
  // per aggregate, and A2 = P2^T K1p P2 with its rows' lengths
  int64_t n_agg = 0;
  int32_t p2_width = 0;
  int32_t a2_maxlen = 0;  // longest row of A2 (blocks)
  ebe::DBuf agg;        // int32 [Nv]
  ebe::DBuf cfix;       // uint8 [Na]
  ebe::DBuf p2_col;     // int32 [Nv][p2_width]
  ebe::DBuf p2_val[2];  // [Nv][p2_width][9] per dtype (F64, F32)
  ebe::DBuf p2t_off;    // int32 [Na+1]
  ebe::DBuf p2t_idx;    // int32 [entries]: v * p2_width + slot
  ebe::DBuf a2_len;     // int32 [Na]
  ebe::AsmOp a2;
  ebe::Workspace ws;
};

namespace ebe {

// rows (nodes) of level 0 (quadratic mesh), 1 (corners) or 2 (aggregates)
inline int64_t level_rows(const ebe_mesh* m, int level) {
  return level == 0 ? m->n_nodes : (level == 1 ? m->n_vertices : m->n_agg);
}

// ---- kernel launchers (ebe_kernels.hip) -----------------------------------
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_ebe_p2(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y,
                         bool bc, hipStream_t s);
hipError_t launch_ebe_p1(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y,
                         bool bc, hipStream_t s);
// general form: order 2 (quadratic) or 1 (linear); mask_in: zero x's fixed
// DOFs while gathering; bc: zero y's fixed DOFs; add: y += K x instead of
// y = K x; the kernels do nothing when gate is non-null and *gate == 0 on the
// device.  gamma (optional, device [nrhs] FP64): gamma[r] += (x_r, K x_r)
// formed element by element.  The staging buffers must have been sized by
// ensure_stage.
// y = A2 x at level 2 (its values must be prepared: ensure_level2)
hipError_t launch_level2(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y, bool mask_in, bool bc,
                         bool add, const int* gate, hipStream_t s, double* gamma = nullptr);
// y = A x in FP32 from the FP16 values of an assembled operator (level 1: K1,
// level 2: A2; ensure_half first)
hipError_t launch_asm_half(const ebe_mesh* m, int level, int nrhs, const float* x, float* y, bool mask_in, bool bc,
                           bool add, const int* gate, hipStream_t s, double* gamma = nullptr);
// FP16 values of an assembled operator from its FP64 values (allocates; synchronous)
ebe_status ensure_half(ebe_mesh* m, int level, hipStream_t s);
// out = bit pattern of max |a_i| (device, one 64-bit word); b = FP16(a * inv_scale)
hipError_t launch_absmax(const double* a, int64_t n, unsigned long long* out, hipStream_t s);
hipError_t launch_to_f16(const double* a, void* b, int64_t n, double inv_scale, hipStream_t s);
hipError_t launch_ebe(const ebe_mesh* m, int order, ebe_dtype dt, int nrhs, const void* x, void* y, bool mask_in,
                      bool bc, bool add, const int* gate, hipStream_t s, double* gamma = nullptr);
// the same with the product form given (0 <= form < EBE_NUM_FORMS)
hipError_t launch_ebe_form(const ebe_mesh* m, int order, int form, ebe_dtype dt, int nrhs, const void* x, void* y,
                           bool mask_in, bool bc, bool add, const int* gate, hipStream_t s, double* gamma = nullptr);
// the form launch_ebe uses for (order, dtype, nrhs)
// form is one of the EBE_FORM_* values and exists at this order (assembled: linear only)
bool form_available(int order, int form);
// ... and it can run on this mesh for (dtype, nrhs): the pipelined and
// coloured forms need the element node words (meshes below 2^25 nodes) and
// node rows addressable with 32-bit byte offsets; the coloured form needs
// the patch colouring
bool form_usable(const ebe_mesh* m, int order, int form, ebe_dtype dt, int nrhs);
int product_form(const ebe_mesh* m, int order, ebe_dtype dt, int nrhs);
// the kernel that a pipelined or coloured product of the quadratic level runs in
// its variant; gamma: with (x, K x)
QuadKernel quad_kernel(const ebe_mesh* m, int form, ebe_dtype dt, int nrhs, bool gamma);
// the form and its kernel variant as one key (graph keys: a replay must run the same kernels)
inline uintptr_t product_key(const ebe_mesh* m, int order, ebe_dtype dt, int nrhs) {
  return uintptr_t(product_form(m, order, dt, nrhs)) |
         (uintptr_t(m->fvar[order == 2 ? 0 : 1][dt == EBE_F64 ? 0 : 1][nrhs]) << 8);
}
// time every form of y = K x on this mesh (x, y: device vectors of the
// level's size; y is overwritten) and record the fastest; synchronous.
ebe_status tune_product(ebe_mesh* m, int level, ebe_dtype dt, int nrhs, const void* x, void* y, hipStream_t s,
                        double ms[EBE_NUM_FORMS]);
hipError_t launch_diag_blocks(const ebe_mesh* m, int level, double* blk6, hipStream_t s);
hipError_t launch_invert_blocks(const ebe_mesh* m, int level, const double* blk6, double* inv64,
                                float* inv32, hipStream_t s);
hipError_t launch_expand_blocks(int64_t n, const double* blk6, double* out9, hipStream_t s);
hipError_t launch_lame(const ebe_mesh* m, hipStream_t s);
hipError_t launch_node_words(const ebe_mesh* m, hipStream_t s);  // pl[0].ptab
hipError_t launch_geometry(const ebe_mesh* m, ebe_dtype dt, void* out, hipStream_t s);
hipError_t launch_fan_geometry(const ebe_mesh* m, ebe_dtype dt, void* out, hipStream_t s);
// K1 of the linear (corner) mesh into k1.val[0] (FP64, atomics into zeroed
// blocks), and its FP32 copy into k1.val[1] when f32 is set
// assemble: form the FP64 values (zeroed first); f32: copy them to the FP32 values
hipError_t launch_assemble_p1(const ebe_mesh* m, bool assemble, bool f32, hipStream_t s);
// P2 (FP64 and FP32) from the FP64 K1 values and the level-1 block Jacobi,
// then A2 = P2^T K1p P2 (FP64 atomics into zeroed blocks) when assemble is
// set; the FP32 copy of A2 when f32 is set
hipError_t launch_assemble_a2(const ebe_mesh* m, bool assemble, bool f32, hipStream_t s);
// FP64 diagonal blocks of an assembled operator as 6 symmetric values per row
hipError_t launch_asm_diag(const AsmOp& op, double* blk6, hipStream_t s);
hipError_t launch_check_material(const double* young, const double* poisson, int64_t n, int* bad,
                                 hipStream_t s);

// ---- vector kernels (ebe_vec.hip) -----------------------------------------
hipError_t launch_prolong(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y,
                          bool bc, hipStream_t s);
hipError_t launch_restrict(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y,
                           bool bc, hipStream_t s);
// level 2: y[Nv] = P2 x[Na] (zero at fixed DOFs), y[Na] = P2^T x[Nv] (zero at fixed coarse DOFs)
hipError_t launch_prolong_p2(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y, hipStream_t s);
hipError_t launch_restrict_p2(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y, hipStream_t s);
hipError_t launch_bjacobi(const ebe_mesh* m, int level, ebe_dtype dt, int nrhs, const void* x,
                          void* y, hipStream_t s);

// ---- adjoint (ebe_adjoint.hip) ---------------------------------------------
// by_element: the kernels of small meshes and of those without fans, whichever the mesh
hipError_t launch_adjoint(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* u,
                          const void* lam, void* g, hipStream_t s, bool by_element = false);

ebe_status ensure_blocks(ebe_mesh* m, hipStream_t s);
// the geometry caches that products of (level, dtype, nrhs) read in their form
// and variant (gamma: with (x, K x)): geo, gfan
struct GeometryNeed {
  bool elements = false, fans = false;
};
GeometryNeed geometry_need(const ebe_mesh* m, int level, int form, ebe_dtype dt, int nrhs, bool gamma);
inline bool geometry_ready(const ebe_mesh* m, GeometryNeed n, ebe_dtype dt) {
  const int k = dt == EBE_F64 ? 0 : 1;
  return (!n.elements || m->geo_ready[k]) && (!n.fans || m->gfan_ready[k]);
}
// fill the geometry cache of dtype dt if it is not (allocates the first time)
ebe_status ensure_geometry(ebe_mesh* m, ebe_dtype dt, hipStream_t s);
// the same for the fan-ordered rows
ebe_status ensure_fan_geometry(ebe_mesh* m, ebe_dtype dt, hipStream_t s);
// A form or variant was chosen after products of this dtype: allocate and fill
// the cache that it reads now, so that its first product can be captured.  (Not
// an error when it cannot be: the product tries again.)
void prepare_chosen_form(ebe_mesh* m, int level, ebe_dtype dt, int nrhs);
// build the assembled linear-level operator of dtype dt if needed (allocates)
ebe_status ensure_assembled(ebe_mesh* m, ebe_dtype dt, hipStream_t s);
// everything products of (level, dtype, nrhs) in their current form need:
// staging, the geometry cache that it reads, assembled operator (allocates:
// before any capture); gamma: also products with (x, K x)
ebe_status prepare_products(ebe_mesh* m, int level, ebe_dtype dt, int nrhs, hipStream_t s, bool gamma = false);
ebe_status build_patches(ebe_mesh* m, const int32_t* conn10, const uint8_t* fix, Uploads& s);
// ---- assembled operators (assembled.cpp) ------------------------------------
// CSR rows (each increasing, non-empty) -> sliced layout with the columns' fix
// bits; false: too large for 32-bit block indices
bool slice_rows(const std::vector<int32_t>& ptr, const std::vector<int32_t>& col, const uint8_t* fix,
                      std::vector<int32_t>& soff, std::vector<int32_t>& scol);
ebe_status upload_asm(AsmOp& op, int64_t rows, const std::vector<int32_t>& soff, const std::vector<int32_t>& scol,
                      Uploads& s);
// aggregation, coarse fix bits, the structures of P2, P2^T and A2: on the host
// (no HIP call: may run beside other host work), then their upload
struct Level2Tables {
  std::vector<int32_t> agg, pcol, toff, tidx, alen, asoff, ascol;
  std::vector<uint8_t> cfix;
  int32_t width = 1;
  const char* error = nullptr;
};
void build_level2(const std::vector<int32_t>& bptr, const std::vector<int32_t>& bcol, const uint8_t* fix,
                  Level2Tables& t);
ebe_status upload_level2(ebe_mesh* m, const Level2Tables& t, Uploads& s);
// A2 values (FP64, and FP32 when asked) and the level-2 block Jacobi (allocates)
ebe_status ensure_level2(ebe_mesh* m, ebe_dtype dt, hipStream_t s);
// grow the staging buffers for products with up to nrhs cases of the given element size
ebe_status ensure_stage(ebe_mesh* m, int nrhs, size_t elem_bytes);

// ---- deterministic product form (ebe_det.hip) -------------------------------
// y = K x (quadratic level) with no atomics in the sums; needs the geometry
// cache of dtype dt and the staging buffer (prepare_products).  colour: the
// patches colour by colour with sums straight into y (else staging and the
// shared-node pass)
hipError_t launch_det(const ebe_mesh* m, ebe_dtype dt, int nrhs, bool colour, const void* x, void* y, bool mask_in,
                      bool bc, bool add, const int* gate, hipStream_t s, double* gamma);

// ---- allocation-free product (ebe_kernels.hip) ------------------------------
// Size of the fixed device array that stages shared-node partial sums for
// ebe_matvec_noalloc (nslots * 3 * nrhs values of the dtype must fit).
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
// device address of that array on `device` (looked up once per device)
ebe_status noalloc_scratch(int device, void** ptr);
// y = K x (or P K P x) in the gather form with the staging in `stage` (the
// scratch array's device address); geometry from the mesh's cache when it
// exists, else from the corner coordinates; allocates nothing
hipError_t launch_ebe_noalloc(const ebe_mesh* m, ebe_dtype dt, int nrhs, const void* x, void* y, bool bc,
                              void* stage, hipStream_t s);

}  // namespace ebe

// Element patches: the work decomposition of the EBE products.
//
// Elements are cut, in the order given, into patches of at most kPatchElems
// elements touching at most kPatchNodes distinct nodes.  A workgroup owns one
// patch: it accumulates the patch's element forces in LDS, then writes each
// patch node once.  A node touched by a single patch ("exclusive") is written
// straight to the output; a node touched by several patches ("shared") gets
// one partial sum per patch in a staging buffer, and a second, node-centric
// pass adds those partials in patch order.  No atomics reach global memory
// and the result does not depend on scheduling.
//
// The linear level (corner nodes only) has patches of its own, larger in
// elements: a linear element's product is a fraction of a quadratic one's,
// so its workgroups need more elements to carry the fixed cost of a patch.
#include <algorithm>
#include <cstring>
#include <thread>
#include <vector>

#include "ebe_internal.h"
#include "host_threads.h"

namespace ebe {

namespace {

struct LevelTables {
  std::vector<int32_t> poff, pnode, pslot;      // per patch entries
  std::vector<int32_t> snode, soff;             // reduction of shared nodes
  int64_t nslots = 0;
  int max_nodes = 0;
};

// Staging slots and the shared nodes' lists from a level's patch entries
// (pnode: plain node ids; count: patches touching each node).  The partial
// sums of one shared node sit in consecutive slots, nodes in increasing id, a
// node's partials in patch order.
void stage_level(int64_t n_nodes, const uint8_t* fix, const std::vector<int32_t>& count, LevelTables& t) {
  // start[] is cumulative over shared nodes only, so it doubles as the offset list
  std::vector<int64_t> start(n_nodes + 1, 0);
  for (int64_t v = 0; v < n_nodes; ++v) start[v + 1] = start[v] + (count[v] > 1 ? count[v] : 0);
  t.nslots = start[n_nodes];
  t.pslot.assign(t.pnode.size(), -1);
  std::vector<int64_t> fill(start.begin(), start.end() - 1);
  for (size_t i = 0; i < t.pnode.size(); ++i) {
    const int32_t v = t.pnode[i];
    if (count[v] > 1) t.pslot[i] = int32_t(fill[v]++);
  }
  t.snode.clear();
  t.soff.assign(1, 0);
  for (int64_t v = 0; v < n_nodes; ++v)
    if (count[v] > 1) {
      t.snode.push_back(int32_t(v) | (int32_t(fix[v]) << kIdxBits));
      t.soff.push_back(int32_t(start[v + 1]));
    }
  // pack node words: id | fix bits | shared flag
  for (size_t i = 0; i < t.pnode.size(); ++i) {
    const int32_t v = t.pnode[i];
    t.pnode[i] = v | (int32_t(fix[v]) << kIdxBits) | (count[v] > 1 ? int32_t(1u << 31) : 0);
  }
}

// Entries of one level: nodes_of(e, a) for local slot a < nloc.
template <class NodeOf>
void build_level(const std::vector<int32_t>& pelem, int nloc, int64_t n_nodes, const uint8_t* fix,
                 NodeOf node_of, std::vector<uint8_t>& lconn, int lstride, LevelTables& t) {
  const int64_t npatch = int64_t(pelem.size()) - 1;
  std::vector<int32_t> stamp(n_nodes, -1), local(n_nodes, 0), count(n_nodes, 0);
  t.poff.assign(npatch + 1, 0);
  t.pnode.clear();
  for (int64_t p = 0; p < npatch; ++p) {
    const int32_t base = int32_t(t.pnode.size());
    for (int32_t e = pelem[p]; e < pelem[p + 1]; ++e) {
      for (int a = 0; a < nloc; ++a) {
        const int32_t v = node_of(e, a);
        if (stamp[v] != int32_t(p)) {
          stamp[v] = int32_t(p);
          local[v] = int32_t(t.pnode.size()) - base;
          t.pnode.push_back(v);
          count[v]++;
        }
        lconn[size_t(e) * lstride + a] = uint8_t(local[v]);
      }
    }
    t.poff[p + 1] = int32_t(t.pnode.size());
    t.max_nodes = std::max(t.max_nodes, t.poff[p + 1] - base);
  }
  stage_level(n_nodes, fix, count, t);
}

// Cut elements, in order, into ranges of at most max_elems elements touching
// at most max_nodes distinct nodes (the nloc nodes of element e are
// node_of(e, 0..nloc-1), distinct within an element).
template <class NodeOf>
std::vector<int32_t> cut_patches(int64_t E, int nloc, int64_t n_nodes, int max_elems, int max_nodes,
                                 NodeOf node_of) {
  std::vector<int32_t> pelem(1, 0), stamp(n_nodes, -1);
  int32_t pid = 0, ne = 0, nn = 0;
  for (int64_t e = 0; e < E; ++e) {
    int fresh = 0;
    for (int a = 0; a < nloc; ++a) fresh += stamp[node_of(e, a)] != pid;
    if (ne == max_elems || nn + fresh > max_nodes) {
      pelem.push_back(int32_t(e));
      ++pid;
      ne = 0;
      nn = 0;
    }
    for (int a = 0; a < nloc; ++a) {
      const int32_t v = node_of(e, a);
      if (stamp[v] != pid) {
        stamp[v] = pid;
        ++nn;
      }
    }
    ++ne;
  }
  pelem.push_back(int32_t(E));
  return pelem;
}

// Element node words: node id | patch-local id << kPtabLocalShift, [E][nloc].
template <class NodeOf>
std::vector<uint32_t> node_words(int64_t E, int nloc, NodeOf node_of, const std::vector<uint8_t>& lconn,
                                 int lstride) {
  std::vector<uint32_t> w(size_t(E) * nloc);
  for (int64_t e = 0; e < E; ++e)
    for (int a = 0; a < nloc; ++a)
      w[size_t(e) * nloc + a] =
          uint32_t(node_of(e, a)) | (uint32_t(lconn[size_t(e) * lstride + a]) << kPtabLocalShift);
  return w;
}

// A fan: a chain of at most kFanLen tetrahedra of a patch around a common edge
// (p, q), each sharing a face with the next.  corner[i]: element-local corners
// (p, q, spoke i, spoke i + 1), an even permutation of the element's own order,
// so the orientation stays positive.
struct Fan {
  int32_t len = 0;
  int32_t elem[kFanLen];
  uint8_t corner[kFanLen][4];
};

// element-local corners of the ends of each edge and of the other two, as even permutations
const uint8_t kEdgePerm[6][4] = {{0, 1, 2, 3}, {1, 2, 0, 3}, {0, 2, 3, 1}, {0, 3, 1, 2}, {1, 3, 2, 0}, {2, 3, 0, 1}};
// edge node between two local corners
const int kEdgeNode[4][4] = {{-1, 4, 6, 7}, {4, -1, 5, 8}, {6, 5, -1, 9}, {7, 8, 9, -1}};

// Groups elements [e0, e0 + ne) into fans: each element not yet in one, in
// order, seeds the longest fan any of its six edges allows (ties: the lowest
// element numbers, which in a Kuhn lattice keeps a hexahedron's six
// tetrahedra, a ring around its diagonal, in two fans of three).
void fans_of_patch(int32_t e0, int32_t ne, const int32_t* conn10, std::vector<Fan>& out) {
  struct Face {
    int32_t v[3];  // corners, increasing
    int32_t el;
    uint8_t opposite;  // the element's local corner off the face
  };
  std::vector<Face> faces;
  faces.reserve(size_t(ne) * 4);
  for (int32_t el = 0; el < ne; ++el) {
    const int32_t* c = conn10 + size_t(e0 + el) * 10;
    for (int o = 0; o < 4; ++o) {
      Face f{};
      int n = 0;
      for (int k = 0; k < 4; ++k)
        if (k != o) f.v[n++] = c[k];
      std::sort(f.v, f.v + 3);
      f.el = el;
      f.opposite = uint8_t(o);
      faces.push_back(f);
    }
  }
  std::sort(faces.begin(), faces.end(), [](const Face& a, const Face& b) {
    for (int k = 0; k < 3; ++k)
      if (a.v[k] != b.v[k]) return a.v[k] < b.v[k];
    return a.el < b.el;
  });
  // across[el * 4 + o]: neighbour over the face opposite local corner o, as element * 4 + its opposite corner
  std::vector<int32_t> across(size_t(ne) * 4, -1);
  for (size_t i = 0; i + 1 < faces.size(); ++i) {
    const Face &a = faces[i], &b = faces[i + 1];
    if (std::equal(a.v, a.v + 3, b.v)) {
      across[size_t(a.el) * 4 + a.opposite] = b.el * 4 + b.opposite;
      across[size_t(b.el) * 4 + b.opposite] = a.el * 4 + a.opposite;
    }
  }
  struct Link {
    int32_t el;
    uint8_t c[4];
  };
  // the neighbour n (element * 4 + opposite corner) of t over the face of p, q
  // and t's spoke t.c[keep], as a link; false if its corners would not be an even permutation
  auto link = [&](const Link& t, int keep, int32_t n, Link& l) {
    const int32_t* ct = conn10 + size_t(e0 + t.el) * 10;
    const int32_t* cn = conn10 + size_t(e0 + n / 4) * 10;
    l.el = n / 4;
    const int from[3] = {0, 1, keep}, to[3] = {0, 1, keep == 3 ? 2 : 3};
    l.c[keep == 3 ? 3 : 2] = uint8_t(n % 4);
    for (int i = 0; i < 3; ++i)
      l.c[to[i]] = uint8_t(std::find(cn, cn + 4, ct[t.c[from[i]]]) - cn);
    int inv = 0;
    for (int i = 0; i < 4; ++i)
      for (int j = i + 1; j < 4; ++j) inv += l.c[i] > l.c[j];
    return (inv & 1) == 0;
  };
  std::vector<uint8_t> used(ne, 0);
  for (int32_t el = 0; el < ne; ++el) {
    if (used[el]) continue;
    Fan best;
    int64_t best_sum = 0;
    for (const auto& perm : kEdgePerm) {
      Link chain[2 * kFanLen];
      int lo = kFanLen, hi = kFanLen;
      chain[lo] = Link{el, {perm[0], perm[1], perm[2], perm[3]}};
      auto extend = [&](const Link& t, int keep, Link& l) {
        const int32_t n = across[size_t(t.el) * 4 + t.c[keep == 3 ? 2 : 3]];
        if (n < 0 || used[n / 4]) return false;
        for (int i = lo; i <= hi; ++i)
          if (chain[i].el == n / 4) return false;
        return link(t, keep, n, l);
      };
      while (hi - lo + 1 < kFanLen && extend(chain[hi], 3, chain[hi + 1])) ++hi;
      while (hi - lo + 1 < kFanLen && extend(chain[lo], 2, chain[lo - 1])) --lo;
      const int len = hi - lo + 1;
      int64_t sum = 0;
      for (int i = lo; i <= hi; ++i) sum += chain[i].el;
      if (len > best.len || (len == best.len && sum < best_sum)) {
        best.len = len;
        best_sum = sum;
        for (int i = 0; i < len; ++i) {
          best.elem[i] = e0 + chain[lo + i].el;
          std::copy(chain[lo + i].c, chain[lo + i].c + 4, best.corner[i]);
        }
      }
    }
    for (int i = 0; i < best.len; ++i) used[best.elem[i] - e0] = 1;
    out.push_back(best);
  }
}

// Fan tables of all patches (long fans first within a patch, so a wavefront's
// fans have like lengths), patches spread over a few host threads.
void build_fans(const std::vector<int32_t>& pelem, const int32_t* conn10, const std::vector<uint8_t>& lconn,
                const uint8_t* fix, std::vector<int32_t>& pfan, std::vector<uint32_t>& fanw,
                std::vector<int32_t>& felem) {
  const int64_t npatch = int64_t(pelem.size()) - 1;
  const int nthread = int(std::max<int64_t>(1, std::min<int64_t>({8, int64_t(std::thread::hardware_concurrency()),
                                                                   npatch / 256})));
  std::vector<std::vector<Fan>> part(nthread);
  pfan.assign(npatch + 1, 0);
  auto first = [&](int t) { return npatch * t / nthread; };
  parallel(nthread, [&](int t) {
    // a patch's fans depend only on which corners its elements share: on a
    // lattice most patches repeat one of a few patterns
    struct Pattern {
      std::vector<uint8_t> key;  // the elements' corners, numbered by first appearance
      std::vector<Fan> fans;     // elements relative to the patch's first
    };
    std::vector<Pattern> seen;
    size_t oldest = 0;
    std::vector<uint8_t> key;
    for (int64_t p = first(t); p < first(t + 1); ++p) {
      const int32_t e0 = pelem[p], ne = pelem[p + 1] - e0;
      key.resize(size_t(ne) * 4);
      int16_t number[256];
      std::fill(number, number + 256, int16_t(-1));
      int16_t n = 0;
      for (int32_t el = 0; el < ne; ++el)
        for (int a = 0; a < 4; ++a) {
          int16_t& v = number[lconn[(size_t(e0) + el) * 16 + a]];
          if (v < 0) v = n++;
          key[size_t(el) * 4 + a] = uint8_t(v);
        }
      const Pattern* same = nullptr;
      for (const Pattern& q : seen)
        if (q.key == key) same = &q;
      if (!same) {
        if (seen.size() < 16) seen.emplace_back();
        Pattern& q = seen[oldest];
        oldest = (oldest + 1) % 16;
        q.key = key;
        q.fans.clear();
        fans_of_patch(e0, ne, conn10, q.fans);
        std::stable_sort(q.fans.begin(), q.fans.end(), [](const Fan& a, const Fan& b) { return a.len > b.len; });
        for (Fan& f : q.fans)
          for (int i = 0; i < f.len; ++i) f.elem[i] -= e0;
        same = &q;
      }
      for (Fan f : same->fans) {
        for (int i = 0; i < f.len; ++i) f.elem[i] += e0;
        part[t].push_back(f);
      }
      pfan[p + 1] = int32_t(same->fans.size());
    }
  });
  for (int64_t p = 0; p < npatch; ++p) pfan[p + 1] += pfan[p];
  fanw.assign(size_t(pfan[npatch]) * kFanStride, 0);
  felem.assign(size_t(pfan[npatch]) * kFanLen, -1);
  parallel(nthread, [&](int t) {
    size_t f = size_t(pfan[first(t)]);
    for (const Fan& fan : part[t]) {
      uint32_t* w = &fanw[f * kFanStride];
      auto put = [&](int a, int32_t e, int local) {
        const int32_t v = conn10[size_t(e) * 10 + local];
        w[a] = uint32_t(v) | (uint32_t(lconn[size_t(e) * 16 + local]) << kPtabLocalShift);
        if (a < 10) w[kFanWords] |= uint32_t(fix[v]) << (2 + 3 * a);
        else w[kFanWords + 1] |= uint32_t(fix[v]) << (3 * (a - 10));
      };
      w[kFanWords] = uint32_t(fan.len);
      for (int i = 0; i < fan.len; ++i) {
        const int32_t e = fan.elem[i];
        const uint8_t* c = fan.corner[i];
        felem[f * kFanLen + i] = e;
        if (i == 0) {
          put(0, e, c[0]);
          put(1, e, c[1]);
          put(2, e, kEdgeNode[c[0]][c[1]]);
          put(3, e, c[2]);
          put(4, e, kEdgeNode[c[0]][c[2]]);
          put(5, e, kEdgeNode[c[1]][c[2]]);
        }
        put(6 + 4 * i, e, c[3]);
        put(7 + 4 * i, e, kEdgeNode[c[0]][c[3]]);
        put(8 + 4 * i, e, kEdgeNode[c[1]][c[3]]);
        put(9 + 4 * i, e, kEdgeNode[c[2]][c[3]]);
      }
      ++f;
    }
  });
}

// Chains of patches (see fan_chained): the order of the patches, each one's
// finished nodes with their accumulator rows, and the rows of all patch nodes
// for the coloured form; the rows replace the patch-local ids in the fan words.
struct ChainTables {
  LevelTables t;               // by place in the order
  std::vector<int32_t> seq;    // [npatch] patch at each place
  std::vector<uint8_t> slot;   // [entries of t] accumulator row
  std::vector<int32_t> croff, crow;  // coloured form: by patch, cword by accumulator row
};
void build_chains(const LevelTables& t0, int64_t n_nodes, const uint8_t* fix, const std::vector<int32_t>& pfan,
                  const std::vector<int32_t>& cword, std::vector<uint32_t>& fanw, ChainTables& c) {
  const int64_t npatch = int64_t(t0.poff.size()) - 1;
  c.seq.resize(npatch);
  std::vector<uint8_t> rows(t0.pnode.size());  // accumulator rows of the patches' nodes
  struct Part {
    std::vector<int32_t> pnode, len;
    std::vector<uint8_t> slot;
  } part[kXcds];
  auto first = [&](int x) { return npatch / kXcds * x + std::min<int64_t>(x, npatch % kXcds); };
  auto range = [&](int x) {
    Part& out = part[x];
    const int64_t start = first(x), stop = first(x + 1), chained = start + fan_chained(stop - start);
    std::vector<int32_t> held, row;  // place whose patch finds the node in the accumulator already, and its row there
    if (chained > start) {
      held.assign(n_nodes, -1);
      row.resize(n_nodes);
    }
    std::vector<int32_t> stamp(chained > start ? n_nodes : 0, -1);
    auto nodes = [&](int64_t p, auto&& f) {
      for (int32_t i = t0.poff[p]; i < t0.poff[p + 1]; ++i) f(i, t0.pnode[i] & kIdxMask);
    };
    int32_t mark = 0;
    for (int64_t a = start; a < stop;) {
      const int n = a < chained ? kChain : 1;
      // the order with the most shared nodes between neighbours (the first of equal ones)
      int order[kChain] = {0, 1, 2, 3}, best[kChain] = {0, 1, 2, 3}, most = -1;
      int common[kChain][kChain] = {};
      for (int i = 0; i + 1 < n; ++i) {
        ++mark;
        nodes(a + i, [&](int32_t, int32_t v) { stamp[v] = mark; });
        for (int j = i + 1; j < n; ++j)
          nodes(a + j, [&](int32_t, int32_t v) { common[i][j] += stamp[v] == mark; });
        for (int j = i + 1; j < n; ++j) common[j][i] = common[i][j];
      }
      if (n > 1) do {
          int sum = 0;
          for (int i = 0; i + 1 < n; ++i) sum += common[order[i]][order[i + 1]];
          if (sum > most) {
            most = sum;
            std::copy(order, order + n, best);
          }
        } while (std::next_permutation(order, order + n));
      for (int k = 0; k < n; ++k) {
        const int64_t p = a + best[k], place = a + k;
        c.seq[place] = int32_t(p);
        bool taken[kPatchNodes] = {};
        if (k > 0)
          nodes(p, [&](int32_t, int32_t v) {
            if (held[v] == place) taken[row[v]] = true;
          });
        int free = 0;
        nodes(p, [&](int32_t i, int32_t v) {
          if (k > 0 && held[v] == place) {
            rows[i] = uint8_t(row[v]);
          } else {
            while (taken[free]) ++free;
            rows[i] = uint8_t(free++);
          }
        });
        const bool more = k + 1 < n;
        ++mark;
        if (more) nodes(a + best[k + 1], [&](int32_t, int32_t v) { stamp[v] = mark; });
        const size_t before = out.pnode.size();
        nodes(p, [&](int32_t i, int32_t v) {
          if (more && stamp[v] == mark) {
            held[v] = int32_t(place) + 1;
            row[v] = rows[i];
          } else {
            out.pnode.push_back(v);
            out.slot.push_back(rows[i]);
          }
        });
        out.len.push_back(int32_t(out.pnode.size() - before));
        for (int32_t f = pfan[p]; f < pfan[p + 1]; ++f)
          for (int i = 0; i < kFanWords; ++i) {
            uint32_t& w = fanw[size_t(f) * kFanStride + i];
            w = (w & kPtabIdMask) | uint32_t(rows[t0.poff[p] + int32_t(w >> kPtabLocalShift)]) << kPtabLocalShift;
          }
      }
      a += n;
    }
  };
  if (npatch < 2048)
    for (int x = 0; x < kXcds; ++x) range(x);
  else
    parallel(kXcds, range);
  std::vector<int32_t> count(n_nodes, 0);
  c.t.poff.assign(1, 0);
  for (const Part& q : part) {
    for (int32_t n : q.len) c.t.poff.push_back(c.t.poff.back() + n);
    for (int32_t v : q.pnode) ++count[v];
    c.t.pnode.insert(c.t.pnode.end(), q.pnode.begin(), q.pnode.end());
    c.slot.insert(c.slot.end(), q.slot.begin(), q.slot.end());
  }
  c.t.max_nodes = t0.max_nodes;
  stage_level(n_nodes, fix, count, c.t);
  c.croff.assign(1, 0);
  c.crow.reserve(cword.size());
  for (int64_t p = 0; p < npatch; ++p) {
    const size_t r0 = c.crow.size();
    for (int32_t i = t0.poff[p]; i < t0.poff[p + 1]; ++i) {
      if (r0 + rows[i] >= c.crow.size()) c.crow.resize(r0 + rows[i] + 1, kNoEntry);
      c.crow[r0 + rows[i]] = cword[i];
    }
    c.croff.push_back(int32_t(c.crow.size()));
  }
}

// Wide patches of a size: consecutive patches of level 0 put together while
// they have at most its elements, distinct nodes and corners (a single patch is
// always within them); corners first.
struct WideTables {
  LevelTables t;
  std::vector<int32_t> pfan;     // fan offsets
  std::vector<int32_t> pcorner;  // corners (the first nodes) of each
  std::vector<uint16_t> fanl;    // [nfan][kWideStride] patch-local ids
};
void build_wide(const std::vector<int32_t>& pelem, const LevelTables& t0, int64_t n_nodes, int64_t n_vertices,
                const uint8_t* fix, const std::vector<int32_t>& pfan, const std::vector<uint32_t>& fanw, int size,
                WideTables& w) {
  const int max_elems = kWideElems[size], max_nodes = kWideNodes[size], max_corners = kWideCorners[size];
  const int64_t npatch = int64_t(pelem.size()) - 1, nfan = pfan[npatch];
  std::vector<int32_t> stamp(n_nodes, -1), local(n_nodes, 0), count(n_nodes, 0);
  w.t.poff.assign(1, 0);
  w.pfan.assign(1, 0);
  w.pcorner.clear();
  w.fanl.assign(size_t(nfan) * kWideStride, 0);
  auto entries = [&](int64_t p, auto&& f) {
    for (int32_t i = t0.poff[p]; i < t0.poff[p + 1]; ++i) f(t0.pnode[i] & kIdxMask);
  };
  for (int64_t p0 = 0, p1 = 0; p0 < npatch; p0 = p1) {
    const int32_t id = int32_t(w.pcorner.size());
    int32_t nn = 0, nc = 0;
    for (p1 = p0; p1 < npatch; ++p1) {
      int32_t fresh = 0, corners = 0;
      entries(p1, [&](int32_t v) {
        fresh += stamp[v] != id;
        corners += stamp[v] != id && v < n_vertices;
      });
      if (p1 > p0 && (pelem[p1 + 1] - pelem[p0] > max_elems || nn + fresh > max_nodes || nc + corners > max_corners))
        break;
      entries(p1, [&](int32_t v) { stamp[v] = id; });
      nn += fresh;
      nc += corners;
    }
    // the nodes, corners first
    const size_t o0 = w.t.pnode.size();
    for (int pass = 0; pass < 2; ++pass)
      for (int64_t p = p0; p < p1; ++p)
        entries(p, [&](int32_t v) {
          if ((v < n_vertices) != (pass == 0) || stamp[v] != id) return;
          stamp[v] = -1;
          local[v] = int32_t(w.t.pnode.size() - o0);
          w.t.pnode.push_back(v);
          count[v]++;
        });
    for (int32_t f = pfan[p0]; f < pfan[p1]; ++f) {
      const uint32_t* fw = &fanw[size_t(f) * kFanStride];
      uint16_t* l = &w.fanl[size_t(f) * kWideStride];
      const int len = int(fw[kFanWords] & 3u);
      for (int a = 0; a < 6 + 4 * len; ++a) l[a] = uint16_t(local[fw[a] & kPtabIdMask]);
      l[kFanWords] = uint16_t(len);
    }
    w.t.poff.push_back(int32_t(w.t.pnode.size()));
    w.pfan.push_back(pfan[p1]);
    w.pcorner.push_back(nc);
  }
  for (size_t i = 0; i + 1 < w.t.poff.size(); ++i)
    w.t.max_nodes = std::max(w.t.max_nodes, w.t.poff[i + 1] - w.t.poff[i]);
  stage_level(n_nodes, fix, count, w.t);
}

// Greedy colouring of the patches (in patch order, each takes the smallest
// colour no patch sharing a node with it has), the patches listed colour by
// colour, and the node words with bit 31 set where an earlier patch in that
// order already wrote the node.
void colour_patches(int64_t n_nodes, const LevelTables& t, std::vector<int32_t>& cperm, std::vector<int64_t>& coff,
                    std::vector<int32_t>& cword) {
  const int64_t npatch = int64_t(t.poff.size()) - 1;
  // node -> patches (CSR)
  std::vector<int32_t> nstart(n_nodes + 1, 0);
  for (int32_t w : t.pnode) nstart[(w & kIdxMask) + 1]++;
  for (int64_t v = 0; v < n_nodes; ++v) nstart[v + 1] += nstart[v];
  std::vector<int32_t> npatches(t.pnode.size()), fillp(nstart.begin(), nstart.end() - 1);
  for (int64_t p = 0; p < npatch; ++p)
    for (int32_t i = t.poff[p]; i < t.poff[p + 1]; ++i) npatches[fillp[t.pnode[i] & kIdxMask]++] = int32_t(p);
  std::vector<int32_t> colour(npatch, -1);
  std::vector<int64_t> taken;  // taken[c] == p: colour c is used by a neighbour of patch p
  int ncol = 0;
  for (int64_t p = 0; p < npatch; ++p) {
    for (int32_t i = t.poff[p]; i < t.poff[p + 1]; ++i) {
      const int32_t v = t.pnode[i] & kIdxMask;
      for (int32_t k = nstart[v]; k < nstart[v + 1]; ++k) {
        const int32_t c = colour[npatches[k]];
        if (c >= 0) taken[c] = p;
      }
    }
    int c = 0;
    while (c < ncol && taken[c] == p) ++c;
    if (c == ncol) {
      ++ncol;
      taken.push_back(-1);
    }
    colour[p] = c;
  }
  coff.assign(ncol + 1, 0);
  for (int64_t p = 0; p < npatch; ++p) coff[colour[p] + 1]++;
  for (int c = 0; c < ncol; ++c) coff[c + 1] += coff[c];
  cperm.assign(npatch, 0);
  std::vector<int64_t> fillc(coff.begin(), coff.end() - 1);
  for (int64_t p = 0; p < npatch; ++p) cperm[fillc[colour[p]]++] = int32_t(p);
  cword.assign(t.pnode.size(), 0);
  std::vector<uint8_t> written(n_nodes, 0);
  for (int64_t k = 0; k < npatch; ++k) {
    const int32_t p = cperm[k];
    for (int32_t i = t.poff[p]; i < t.poff[p + 1]; ++i) {
      const int32_t w = t.pnode[i] & 0x7fffffff;  // id | fix bits
      const int32_t v = w & kIdxMask;
      cword[i] = w | (written[v] ? int32_t(1u << 31) : 0);
      written[v] = 1;
    }
  }
}

template <class T>
ebe_status up(DBuf& b, const std::vector<T>& h, Uploads& s) {
  return s.add(b, h.data(), h.size() * sizeof(T));
}

ebe_status up_level(PatchLevel& L, const LevelTables& t, int64_t npatch, Uploads& s) {
  ebe_status st = EBE_OK;
  if ((st = up(L.poff, t.poff, s)) != EBE_OK) return st;
  if ((st = up(L.pnode, t.pnode, s)) != EBE_OK) return st;
  if ((st = up(L.pslot, t.pslot, s)) != EBE_OK) return st;
  if ((st = up(L.snode, t.snode, s)) != EBE_OK) return st;
  if ((st = up(L.soff, t.soff, s)) != EBE_OK) return st;
  L.npatch = npatch;
  L.nslots = t.nslots;
  L.nshared = int64_t(t.snode.size());
  L.entries = int64_t(t.pnode.size());
  L.max_nodes = t.max_nodes;
  return EBE_OK;
}

}  // namespace

ebe_status build_patches(ebe_mesh* m, const int32_t* conn10, const uint8_t* fix, Uploads& s) {
  const int64_t E = m->n_elem;
  auto node_of = [&](int64_t e, int a) { return conn10[size_t(e) * 10 + a]; };
  // two independent halves of the work, side by side on meshes that repay a thread
  auto both = [&](auto&& f) {
    if (E >= 65536) {
      parallel(2, f);
    } else {
      f(0);
      f(1);
    }
  };
  // 1. cut elements into patches, separately for each level: 2. the quadratic
  // one (all 10 nodes) and the linear one (corners)
  std::vector<int32_t> pelem[2];
  std::vector<uint8_t> lconn(size_t(E) * 16, 0), lconn1(size_t(E) * 4, 0);
  LevelTables t[2];
  both([&](int l) {
    if (l == 0) {
      pelem[0] = cut_patches(E, 10, m->n_nodes, kPatchElems, kPatchNodes, node_of);
      build_level(pelem[0], 10, m->n_nodes, fix, node_of, lconn, 16, t[0]);
    } else {
      pelem[1] = cut_patches(E, 4, m->n_vertices, kLinPatchElems, kLinPatchCorners, node_of);
      build_level(pelem[1], 4, m->n_vertices, fix, node_of, lconn1, 4, t[1]);
    }
  });
  if (t[0].max_nodes > kPatchNodes || t[1].max_nodes > kLinPatchCorners) {
    set_error("build_patches: patch with %d nodes / %d corners exceeds %d / %d", t[0].max_nodes, t[1].max_nodes,
              kPatchNodes, kLinPatchCorners);
    return EBE_ERR_INDEX;
  }
  ebe_status st = EBE_OK;
  if ((st = up(m->lconn, lconn, s)) != EBE_OK) return st;
  if ((st = up(m->lconn1, lconn1, s)) != EBE_OK) return st;
  if (m->n_nodes <= int64_t(kPtabIdMask))  // element node words (pipelined form of the linear level)
    if ((st = up(m->pl[1].ptab, node_words(E, 4, node_of, lconn1, 4), s)) != EBE_OK) return st;
  std::vector<int32_t> cperm, cword, pistart, pfan, felem;
  std::vector<uint16_t> pinc;
  std::vector<uint32_t> fanw;
  WideTables w[kWideSizes];
  const bool fans = m->n_nodes <= int64_t(kPtabIdMask) && !m->curved;  // pipelined and coloured forms
  both([&](int k) {
    if (k == 0) {
      colour_patches(m->n_nodes, t[0], cperm, m->pl[0].coff, cword);
      // incidence lists of the quadratic patches: for each patch entry, the
      // element slots that touch it, in element order (deterministic form)
      const std::vector<int32_t>& pe = pelem[0];
      const LevelTables& t0 = t[0];
      pinc.resize(size_t(E) * 10);
      pistart.resize(t0.pnode.size());
      std::vector<int32_t> cnt;
      for (size_t p = 0; p + 1 < pe.size(); ++p) {
        const int32_t e0 = pe[p], ne = pe[p + 1] - e0, o0 = t0.poff[p], nn = t0.poff[p + 1] - o0;
        cnt.assign(size_t(nn) + 1, 0);
        for (int32_t el = 0; el < ne; ++el)
          for (int a = 0; a < 10; ++a) cnt[lconn[(size_t(e0) + el) * 16 + a] + 1]++;
        for (int32_t i = 0; i < nn; ++i) cnt[i + 1] += cnt[i];
        for (int32_t i = 0; i < nn; ++i) pistart[size_t(o0) + i] = cnt[i];
        for (int32_t el = 0; el < ne; ++el)
          for (int a = 0; a < 10; ++a) {
            const int lid = lconn[(size_t(e0) + el) * 16 + a];
            pinc[size_t(e0) * 10 + cnt[lid]++] = uint16_t(el * 10 + a);
          }
      }
    } else if (fans) {
      build_fans(pelem[0], conn10, lconn, fix, pfan, fanw, felem);
      static_assert(kWideSizes == 2, "");
      both([&](int i) { build_wide(pelem[0], t[0], m->n_nodes, m->n_vertices, fix, pfan, fanw, i, w[i]); });
    }
  });
  if ((st = up(m->pl[0].cperm, cperm, s)) != EBE_OK) return st;
  if ((st = up(m->pl[0].cword, cword, s)) != EBE_OK) return st;
  if ((st = up(m->pl[0].pinc, pinc, s)) != EBE_OK) return st;
  if ((st = up(m->pl[0].pistart, pistart, s)) != EBE_OK) return st;
  if (fans) {
    ChainTables c;
    build_chains(t[0], m->n_nodes, fix, pfan, cword, fanw, c);
    // (the chains and wide patches stage in pl[0].stage: a run of patches shares
    // no more rows with others than its parts do)
    if (std::max({c.t.nslots, w[0].t.nslots, w[1].t.nslots}) > t[0].nslots) {
      set_error("build_patches: %lld staged rows of chains or wide patches exceed %lld",
                (long long)std::max({c.t.nslots, w[0].t.nslots, w[1].t.nslots}), (long long)t[0].nslots);
      return EBE_ERR_INDEX;
    }
    m->nfan = int64_t(felem.size()) / kFanLen;
    if ((st = up(m->pfan, pfan, s)) != EBE_OK) return st;
    if ((st = up(m->fanw, fanw, s)) != EBE_OK) return st;
    if ((st = up(m->felem, felem, s)) != EBE_OK) return st;
    if ((st = up(m->cseq, c.seq, s)) != EBE_OK) return st;
    if ((st = up(m->cslot, c.slot, s)) != EBE_OK) return st;
    if ((st = up(m->croff, c.croff, s)) != EBE_OK) return st;
    if ((st = up(m->crow, c.crow, s)) != EBE_OK) return st;
    if ((st = up_level(m->chain, c.t, int64_t(c.seq.size()), s)) != EBE_OK) return st;
    for (int k = 0; k < kWideSizes; ++k) {
      ebe_mesh::Wide& d = m->wide[k];
      if ((st = up(d.pfan, w[k].pfan, s)) != EBE_OK) return st;
      if ((st = up(d.pcorner, w[k].pcorner, s)) != EBE_OK) return st;
      if ((st = up(d.fanl, w[k].fanl, s)) != EBE_OK) return st;
      if ((st = up_level(d.pl, w[k].t, int64_t(w[k].pcorner.size()), s)) != EBE_OK) return st;
    }
  }
  for (int l = 0; l < 2; ++l) {
    if ((st = up(m->pl[l].pelem, pelem[l], s)) != EBE_OK) return st;
    if ((st = up_level(m->pl[l], t[l], int64_t(pelem[l].size()) - 1, s)) != EBE_OK) return st;
  }
  return EBE_OK;
}

}  // namespace ebe

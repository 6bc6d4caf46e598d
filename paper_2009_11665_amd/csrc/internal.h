// Internal structures shared by the planner (plan.cpp) and the device
// runtime (runtime.hip).  Not part of the public interface.
#pragma once

#include <cstdint>
#include <map>
#include <mutex>
#include <tuple>
#include <string>
#include <vector>

#include "../../include/sg2v.h"

namespace sg2v {

void set_error(const char *fmt, ...);

// binomial coefficients C(a, b) for 0 <= a, b <= 64 (exact in int64 for the
// sizes used here: a <= SG2V_KMAX).
int64_t binom(int a, int b);

// colexicographic rank of a colour set given as a bit mask (bit c = colour c):
// rank = sum_i C(c_i, i) over the sorted elements c_1 < ... < c_m.
int64_t colex_rank(uint32_t mask);
// inverse: the mask of size m with the given rank among k colours.
uint32_t colex_unrank(int64_t rank, int m, int k);

// One distinct rooted sub-template.  Nodes are stored children first.
struct Node {
  int size = 1;
  int active = -1;   // node id of the active child (keeps the root)
  int passive = -1;  // node id of the passive child (cut-off subtree)
  int vertex = 0;    // template vertex rooting the first occurrence
  int n_kept = 0;    // number of that vertex's first children it keeps
  int64_t cols = 0;  // C(k, size)
  int n_active_uses = 0;   // splits using this node as active child
  int n_passive_uses = 0;  // splits using this node as passive child
  std::string canon;       // rooted canonical form
  // split tables (size > 1):
  int np = 0;                  // pairs per output column = C(size, size_a)
  std::vector<int32_t> pairs;  // [cols][np] x (ia, ip)
  std::vector<int32_t> drop;   // active child is one vertex: [k][cols] -> rank(C\{c}) or -1
  // adjoint tables (reverse-mode derivative of the multiply-add):
  int np_ta = 0;               // pairs per active column = C(k - size_a, size_p)
  std::vector<int32_t> tr_a;   // [cols_a][np_ta] x (I_s, I_p): output sets containing I_a
  int np_tp = 0;               // pairs per passive column = C(k - size_p, size_a)
  std::vector<int32_t> tr_p;   // [cols_p][np_tp] x (I_s, I_a): output sets containing I_p
  std::vector<int32_t> add;    // active child is one vertex: [k][cols_p] -> rank(P + {c}) or -1
  // colour-restricted multiply-add (general splits): a vertex of colour c has
  // M_s(i, C) = 0 unless c is in C, and only pairs whose active set holds c
  // contribute.  Per colour c (all sizes are equal across colours):
  //   ca[c][*]  active columns holding c      (Sa = C(k-1, |T_a|-1))
  //   cb[c][*]  passive columns not holding c (Sb = C(k-1, |T_p|))
  //   co[c][*]  output columns holding c      (U  = C(k-1, |T_s|-1))
  //   cz[c][*]  output columns not holding c  (Z  = C(k-1, |T_s|))
  //   cp[c][q][u] = position in ca | position in cb << 16, q < Q = C(|T_s|-1, |T_a|-1)
  int64_t c_sa = 0, c_sb = 0, c_u = 0, c_z = 0;
  int c_q = 0;
  std::vector<int32_t> ca, cb, co, cz;
  std::vector<uint32_t> cp;
};

enum RootKind {
  ROOT_SINGLE = 0,   // root split's active child is one vertex:  X = B_Q, no Y
  ROOT_FUSED = 1,    // active child is itself a one-vertex-active split used only
                     // here: X = B of its passive, Y = B_Q
  ROOT_GENERAL = 2,  // X = M of the active child, Y = B_Q
  ROOT_VERTEX = 3,   // the template is one vertex
};

// Root reduction of one template of a plan.
struct RootInfo {
  int node = -1;               // node id of the template itself
  int t = 0;                   // template vertices
  int kind = ROOT_VERTEX;
  int x_node = -1, y_node = -1;
  int64_t L = 0;
  std::vector<int32_t> list;   // [k][L] x (x, y)
  int64_t alpha = 1;           // |Aut(T)|
  double P = 1.0;              // colourful probability
  std::vector<int32_t> parent; // the template as given
};

constexpr size_t kRelLds = 64 * 1024;  // LDS of a vertex-relative multiply-add tile

struct Plan {
  // The first (or only) template: t, parent, root, alpha, P and the root_*
  // fields below describe it.  A plan of several templates (treelet
  // distributions) shares its sub-template nodes across them and keeps one
  // RootInfo per template in `roots`.
  int t = 0, k = 0;
  std::vector<int32_t> parent;
  std::vector<Node> nodes;
  int root = -1;
  int64_t alpha = 1;
  double P = 1.0;
  // root reduction: for every colour c, L entries (x, y): the sum over the
  // list of X(i, x) * Y(i, y) equals sum_C M_0(i, C) for a vertex of colour c.
  int root_kind = ROOT_VERTEX;
  int root_x_node = -1;  // node whose B (or M for ROOT_GENERAL) is X
  int root_y_node = -1;  // node whose B is Y (-1: Y = 1)
  int64_t root_L = 0;
  std::vector<int32_t> root_list;  // [k][L] x (x, y)
  // nodes whose tables are never materialised (fused into the root)
  std::vector<char> fused;
  std::vector<RootInfo> roots;   // one per template, roots[0] = the fields above
  std::vector<int> root_index;   // per node: index into roots, or -1
  // rel_ok for tables of 4-byte and of 8-byte elements with tiles of kRelLds, and
  // whether some aggregation goes in chunks: asked on every call
  bool rel32 = false, rel64 = false, any_wide = false;

  // device copies of the tables, uploaded on first use per device
  struct DeviceTables {
    int device = -1;
    std::vector<void *> owned;        // the allocations that hold the tables below
    std::vector<void *> pairs, drop;  // per node
    std::vector<void *> tr_a, tr_p, add;
    std::vector<void *> cpr;  // colour-restricted tables, one block per node
    std::vector<void *> root_list;    // per template
    std::vector<void *> root_list16;  // (x | y << 16), when every index fits 16 bits
    // vertex-relative tables: per node the split's pair list, the aggregation's
    // maps (colour maps followed by the output lists); per template the root list
    std::vector<void *> rel_pairs, rel_map, rel_root;
    // output columns where they are not the ranks (per node: multiply-adds,
    // aggregations); chunk tables of wide aggregations
    std::vector<void *> rel_mpos, rel_bpos, rel_hdr, rel_info, rel_tab;
    // adjoint in vertex-relative tables, uploaded on first use: maps, pairs of the
    // active and of the passive columns
    std::vector<void *> back_map, back_px, back_py;
    // SpMM colour-skip masks per (node, colourings per pass, chunk width)
    std::map<std::tuple<int, int, int>, void *> chunks;
  };
  mutable std::mutex mu;
  mutable std::vector<DeviceTables> dev;
};

// Vertex-relative tables: the q-sets of the k-1 colours other than a vertex's
// own, numbered in increasing order without it.
struct RelMap {
  int w_in = 0, w_out = 0;    // columns of a gathered and of an aggregated row
  int cw = 0, wout4 = 0;      // absolute sets and output columns, padded to 4
  int zero = 0;               // w_in padded to 4: position of a staged zero
  // [k][cw]: column of the absolute set without colour c in a row of colour c
  // (zero if it lacks c); then [k][wout4]: absolute set of each output position;
  // then [k][zero]: absolute set of each column plus c (cw: padding)
  std::vector<uint16_t> map;
};
// Aggregations too wide for one row per wave go in chunks.  The k colours are
// cut into the l = rel_low(k) lowest and the others; a chunk holds the sets P with
// one choice of high colours PH, its columns the choices of s = m - |PH| low
// ones.  In a gathered row of a vertex of colour c these are one run: the sets
// without c, of PH if c is low and of PH - {c} if it is high.
bool rel_wide(int k, int m);
// aggregations below those that may use their sorted entries (chunk tables are made)
bool rel_sorted(int k, int m);
int rel_low(int k);
// Columns of the q-sets: their ranks, or (tables gathered in chunks) each choice
// of high relative colours at a multiple of 32 columns.
struct RelLayout {
  int64_t width = 0;
  std::vector<int32_t> pos;  // by rank
};
RelLayout rel_layout(int k, int q, bool wide);
struct RelWide {
  int l = 0, nchunk = 0;
  // [nchunk][1 + 2k]: s, then per colour the first column of its run in a gathered
  // row (-1: none), then per colour the first output column (-1: none)
  std::vector<int32_t> hdr;
  // [l + 1][9], by s: columns padded to 4, offsets of inv and out in `tab`, run
  // lengths of low and high colours (with the gap inside), output columns of low
  // and high colours, and where and by how much the latter's have a gap
  std::vector<int32_t> info;
  // inv [l + 1][cw]: column within the run of each choice of low colours (row c: low
  // colour c, 0xFFFF if it lacks c; row l: any high colour); out [l + 1][cw]: choice
  // of each output column
  std::vector<uint16_t> tab;
};
// (also, with out_wide false, of an aggregation that is not wide: all colours low)
RelWide rel_wide_tables(int k, int m, bool out_wide);
// tables gathered in chunks, by node: its multiply-add's, its aggregation's
void rel_wide_nodes(const Plan &P, std::vector<char> &wide_m, std::vector<char> &wide_b);
// whether every table of the plan has a vertex-relative form, with elements of
// es bytes and multiply-add tiles of at most `lds` bytes
bool rel_ok(const Plan &P, int es, size_t lds);
inline bool rel_ok(const Plan &P, int es) { return es == 4 ? P.rel32 : P.rel64; }  // tiles of kRelLds
// maps of the aggregation of an m-vertex passive child, m >= 2, not wide
RelMap rel_map(int k, int m);
// pairs [np][ws] (x | y << 16) of a split (m vertices, ma of them active, 1 < ma < m)
std::vector<uint32_t> rel_pairs(int k, int m, int ma, const RelLayout &X, const RelLayout &Y);
// root list (x | y << 16) of a template of t vertices, ma in the active child
std::vector<uint32_t> rel_root_list(int k, int t, int ma, const RelLayout &X, const RelLayout &Y);

// Adjoint: maps of the aggregation (as rel_map's, but a gathered row is an
// aggregation's, an output row a passive table's), and the pairs (output set,
// other operand) of a split's active and passive columns
RelMap rel_map_back(int k, int m);
std::vector<uint32_t> rel_pairs_back(int k, int m, int ma, bool active);
// whether the adjoint of the plan runs in vertex-relative tables
bool rel_grad_ok(const Plan &P, int es);

sg2v_status plan_build(const int32_t *parent, int t, int k, Plan &out);
// Several templates over the same k, sharing isomorphic rooted sub-templates.
sg2v_status plan_build_multi(const int32_t *const *parents, const int32_t *ts, int n, int k,
                             Plan &out);
// Device workspace of one pass over one colouring, per vertex (runtime).
int64_t pass_bytes_per_vertex(const Plan &P, int fp32);
// Vertices of a registered graph (runtime).
int64_t graph_vertices(const sg2v_graph *g);

}  // namespace sg2v

struct sg2v_plan {
  sg2v::Plan p;
};

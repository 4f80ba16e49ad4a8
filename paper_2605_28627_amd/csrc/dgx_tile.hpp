// dgx_tile.hpp -- element-tile index helpers shared by the residual and FV
// kernels: work-items per element, node and line indexing, the basis copy,
// and the face-trace layout.
#pragma once

#include <hip/hip_runtime.h>

#include "dgx_internal.hpp"

namespace dgx {

template <int N>
struct Shape {
  static constexpr int n1 = N + 1;
  static constexpr int n2 = n1 * n1;
  static constexpr int n3 = n2 * n1;
  // Work-items per element: whole wavefronts, except at N = 1, whose 8 nodes
  // would leave 7/8 of one idle.  There a wavefront holds 4 elements of 16
  // work-items, each with its own LDS tile and numbering (Euler 60^3, 2 steps:
  // 4.55 -> 2.47 ms; 8 elements of 8 gain nothing more there and lose 5 % on
  // meshes that do not fill the chip, 2 of 32 lose 17 % at 60^3).  N = 2 packed
  // in pairs (27 of 32) gained 6 % at 40^3 and lost 9 % at 5x6x5.
  // What is uniform over the workgroup elsewhere (metric terms, element and
  // face flags) then differs between a wavefront's elements.  Returns and
  // barriers that depend on it are safe: the workgroup is that one wavefront,
  // whose LDS accesses stay in order and whose barriers wait for nobody.
  static constexpr int nth = N == 1 ? 16 : ((n3 + 63) / 64) * 64;
  static constexpr int epb = nth < 64 ? 64 / nth : 1;  // elements per workgroup
  static constexpr int block = nth * epb;
  __host__ __device__ static int grid(int nElems) { return (nElems + epb - 1) / epb; }
  static constexpr int nface = 6 * n2;                 // face nodes of one element
};

template <int N>
__device__ __forceinline__ int nidx(int i, int j, int k) { return (k * (N + 1) + j) * (N + 1) + i; }

// Volume node at position a along reference direction r, tangential face
// indices (pp, qq).  One stride per index, chosen by r: where r differs between
// lanes (face loops) that is three selects per line; a choice between three
// node formulas became two branches for every node of the line (the trace loop
// of an N = 3 Gauss element: 40 branches instead of 20 LDS reads in a row).
template <int N>
__device__ __forceinline__ int line_node(int r, int a, int pp, int qq) {
  constexpr int n1 = N + 1, n2 = n1 * n1;
  return pp * (r == 0 ? n1 : 1) + qq * (r == 2 ? n1 : n2) + a * (r == 0 ? 1 : (r == 1 ? n1 : n2));
}

// The entries of the basis the kernels read, at their exact size (the LDS
// footprint decides how many elements share a CU), in the order of
// DevBasis::packed.  (FVB: also the FV sub-cell operators Bs, Bs^-1.)
template <int N, bool FVB = false>
struct VolBasis {
  static constexpr int n1 = N + 1;
  static constexpr int nf = FVB ? n1 * n1 : 1;
  static constexpr int nd = 3 * n1 + 2 * n1 * n1 + (FVB ? 2 * n1 * n1 : 0);   // doubles copied
  double winv[n1], Lm[n1], Lp[n1], Dhat[n1 * n1], DS[n1 * n1], Bs[nf], Bsi[nf];
};

// The basis copy in two parts, so that its loads are in flight together with
// the element's own and nothing waits for them alone: load() at the start of a
// kernel, store() to LDS before the first barrier.  At most one value per
// work-item (FVB, N = 1 and 3: two); loaded array by array and stored at once it cost
// every workgroup two memory latencies before its first load of the state.
template <int N, bool FVB, int NTH>
struct BasisCopy {
  static constexpr int nd = VolBasis<N, FVB>::nd, k = (nd + NTH - 1) / NTH;
  double v[k];
  __device__ __forceinline__ void load(const DevBasis* src, int t) {
#pragma unroll
    for (int i = 0; i < k; ++i) v[i] = t + i * NTH < nd ? src->packed[t + i * NTH] : 0.0;
  }
  __device__ __forceinline__ void store(VolBasis<N, FVB>* dst, int t) const {
    double* d = reinterpret_cast<double*>(dst);
#pragma unroll
    for (int i = 0; i < k; ++i)
      if (t + i * NTH < nd) d[t + i * NTH] = v[i];
  }
};

// Where node t of element e finds its metric terms: component c (Ja^r_n at
// c = 3r+n, 1/J at c = 9) at base[off + c st].  Both stores are [10][...]:
// the node arrays (Ja, then sJ) and, for every element whose terms are the
// same at all of its nodes (affine), the per-element copy G.em, whose 1/J is
// positive exactly for those elements.  Such an element's nodes all read the
// copy and the node arrays are not touched (same values).
// Selects only, no branches; base and st are uniform over the element.
struct NodeMetric {
  const double* base;
  size_t off, st;
  __device__ __forceinline__ double ja(int c) const { return base[off + c * st]; }
  __device__ __forceinline__ double sj() const { return base[off + 9 * st]; }
};
// ELEM = false: always the node arrays (kernels whose register budget has no
// room for the selects).
template <bool ELEM = true>
__device__ __forceinline__ NodeMetric node_metric(const Geo& G, int e, int n3, int t) {
  const size_t nE = G.nElems;
  const bool el = ELEM && G.em[9 * nE + e] > 0.0;
  NodeMetric m;
  m.base = el ? G.em : G.Ja;
  m.off = el ? (size_t)e : (size_t)e * n3 + t;
  m.st = el ? nE : nE * n3;
  return m;
}

// Face f of face node ft.  With 64 face nodes (N = 7) a wavefront's lanes lie
// on one face: telling the compiler so moves the face table, the side's
// address arithmetic and constant normals to scalar registers.
template <int N>
__device__ __forceinline__ int face_of(int ft) {
  constexpr int n2 = (N + 1) * (N + 1);
  if constexpr (n2 == 64)
    return __builtin_amdgcn_readfirstlane(ft / n2);
  else
    return ft / n2;
}

// Normal (c = 0..2) and surface element (c = 3) of face node fi of a side: the
// side's own entry where its nodes share them (the faces of affine elements:
// 32 B per side instead of 32 B per face node, 24 B per node and evaluation at
// N = 7 and 48 B at N = 3), else the node's.  Both live in one array.
struct FaceGeom {
  const double* base;
  size_t st;
  __device__ __forceinline__ double operator()(int c) const { return base[c * st]; }
};
__device__ __forceinline__ FaceGeom face_geom(const Geo& G, int info, int n2, int fi) {
  const size_t nS = G.nSides, nf = nS * n2, side = efc_side(info);
  const bool cs = efc_const(info);
  FaceGeom g;
  g.base = G.face + (cs ? 4 * nf + side : side * n2 + fi);
  g.st = cs ? nS : nf;
  return g;
}

// Element of a one-element-per-workgroup launch.  Consecutive workgroups are
// dealt round-robin to the chip's 8 XCDs, each with its own L2.  With
// XCD-aware numbering (DGX_XCD_REMAP 1) XCD x walks a contiguous block of
// elements, so an element and its lexicographic neighbours (which read the
// same face data) run on the same XCD close in time.  XCD x then gets
// nE/8 (+1 for x < nE%8) elements starting at x (nE/8) + min(x, nE%8); the
// map is a bijection of [0, nE) for any nE (of one element per workgroup).  Measured, it gains nothing at
// N = 7 and costs 2-8 % at N = 3 (plausibly because in plain order the
// eight XCDs work on neighbouring elements at the same time and share the
// face data through the chip-wide last-level cache), so plain order (0) is
// the default.
#ifndef DGX_XCD_REMAP
#define DGX_XCD_REMAP 0
#endif
__device__ __forceinline__ int elem_of_block(int bid, int nE) {
  if constexpr (DGX_XCD_REMAP) {
    constexpr int kXcd = 8;
    const int q = nE / kXcd, r = nE - q * kXcd;
    int x, slot;
    if (bid < kXcd * q) { x = bid % kXcd; slot = bid / kXcd; }
    else { x = bid - kXcd * q; slot = q; }
    return x * q + (x < r ? x : r) + slot;
  } else {
    return bid;
  }
}

__device__ __forceinline__ size_t tr_index(int slot, int v, int nvar, int nSides, int side, int n2, int fi) {
  return (((size_t)slot * nvar + v) * nSides + side) * n2 + fi;
}

// Entropy-projected traces (split form on Gauss nodes): their ln rho and
// ln beta sit behind the trace values, at Utr + 2 tnv nSides n2 (tnv values
// per face node: 5, or 10 in FV contexts), layout [slot][2][side][(p,q)].
__device__ __forceinline__ double* trace_logs(double* Utr, int nS, int n2, int tnv = 5) {
  return Utr + (size_t)2 * tnv * nS * n2;
}
__device__ __forceinline__ const double* trace_logs(const double* Utr, int nS, int n2, int tnv = 5) {
  return Utr + (size_t)2 * tnv * nS * n2;
}

}  // namespace dgx

// Non-local PAW terms, node-wise recurrence kernels and column reductions,
// for gfx950.
//
// Non-local action (eq. "FE nonlocal contribution"): the projector
// coefficients c_a = C^a^T s X (s = 1 or M_D^{-1}) are a long-K skinny
// reduction over the support nodes of each atom (K <= 19^3 rows, M = nproj,
// N = columns): one workgroup per (atom, 128-row chunk, column tile),
// lane <-> column so every row read is one coalesced 512-byte segment and the
// C^a row is wave-uniform (scalar loads).  Partial sums go to a workspace and
// a second kernel adds the chunks of each atom in a fixed order (no atomics,
// deterministic).  The atom-block products (Delta x c, G^{ab} corrections)
// are small and run in two launches (k_atom_first, k_atom_second).  The add-back
// sum_a C^a q_a on the support rows is a pass of its own (k_nl_fixup) before or
// after the kernels that stream all rows.

#include <cstdint>
#include <initializer_list>
#include <type_traits>

#include "kernels.h"

namespace pawfe {

namespace {

constexpr int kRowsPerWaveGroup = 4;   // waves per 256-thread block in row-wise kernels

// (items, column tiles): a grid's y extent ends at 65,535, which the narrow tiles
// reach at a million columns; from there on z counts on
inline dim3 tile_grid(int64_t items, int64_t tiles) {
  constexpr int64_t kMaxY = 65535;
  return dim3((unsigned)items, (unsigned)std::min(tiles, kMaxY), (unsigned)((tiles + kMaxY - 1) / kMaxY));
}
__device__ __forceinline__ int tile_index() { return blockIdx.y + blockIdx.z * gridDim.y; }

// A workgroup of four waves takes an item's rows: SPLIT = 1, each wave owns 64
// of 256 columns and walks all rows; SPLIT = 4, the waves share one 64-column
// tile, a quarter of the rows each, and their sums meet in LDS, added in FP64.
// Rows are taken kUnroll at a time with all their loads issued before the
// FMAs (memory-level parallelism).  The walk over the rows is a chain of
// memory latencies (node list, then rows): it is the whole time of a small
// launch, which the split quarters (FP64, three 18-projector atoms x 40
// columns: 47.7 -> 17.1 us), while a launch that fills the chip without it
// only loses residency to the LDS (FP64, 128 atoms x 256 columns: 0.43 ->
// 0.60 ms; 27 atoms x 192 columns 107 -> 132 us; 16 complex atoms x 192
// real columns 86 -> 62 us).
constexpr int kUnroll = 8;

// sum of the four waves' partials of projector rows [0, npj) and 64 columns,
// written to the item's block
template <typename T, int NPJ>
__device__ __forceinline__ void store_partials(const T (&red)[kRowsPerWaveGroup][NPJ][64], int npj, int ncols,
                                               int n, int po, double* __restrict__ part) {
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (n >= ncols) return;
  for (int al = w; al < npj; al += kRowsPerWaveGroup)
    part[(int64_t)(po + al) * ncols + n] = (((double)red[0][al][lane] + (double)red[1][al][lane]) +
                                            ((double)red[2][al][lane] + (double)red[3][al][lane]));
}

// Complex operators (CPLX): the columns are (re, im) pairs of the complex
// columns and c = C^H x mixes them: c[n] = sum Cr x[n] + s' Ci x[n ^ 1],
// s' = +1 on real and -1 on imaginary columns; the partner value comes from
// the neighbouring lane.
template <typename T, int NPJ, bool SCALE, bool CPLX, int SPLIT>
__global__ void __launch_bounds__(256) k_nl_reduce(const T* __restrict__ X, int64_t ldx, int ncols,
                                                   const T* __restrict__ Minv,
                                                   const T* __restrict__ Cv, DeviceTables d,
                                                   double* __restrict__ part, const T* __restrict__ Cvi) {
  __shared__ T red[SPLIT == 4 ? kRowsPerWaveGroup : 1][SPLIT == 4 ? NPJ : 1][64];
  const int item = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = SPLIT == 4 ? tile_index() : tile_index() * kRowsPerWaveGroup + w;
  if (SPLIT == 1 && tile * 64 >= ncols) return;   // wave-uniform
  const int n = tile * 64 + lane;
  const bool valid = n < ncols;
  const int nc = valid ? n : 0;
  const int a = d.item_atom[item];
  const int npj = d.nproj[a];
  const int i0 = d.item_row0[item], i1 = d.item_row1[item];
  const int per = (i1 - i0 + SPLIT - 1) / SPLIT;
  const int r0 = SPLIT == 1 ? i0 : std::min(i0 + w * per, i1), r1 = std::min(r0 + per, i1);
  const int noff = d.atom_noff[a], coff = d.atom_coff[a];
  T acc[NPJ];
#pragma unroll
  for (int al = 0; al < NPJ; ++al) acc[al] = T(0);
  // every load is unconditional (indices clamped into range, padded entries
  // multiply zeros or land in accumulators that are never stored), so the
  // loads of a batch are all in flight together
  auto rows = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
    for (int rb = r0; rb < r1; rb += kUnroll) {
      // the node list is padded by kUnroll entries, so the batch of indices
      // is one contiguous read; rows past r1 are masked below
      int I[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) I[u] = d.atom_nodes[noff + rb + u];
      T x[kUnroll], m[kUnroll];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        x[u] = __builtin_nontemporal_load(X + (int64_t)I[u] * ldx + nc);
        if constexpr (SCALE) m[u] = Minv[I[u]];
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        if constexpr (SCALE) x[u] *= m[u];
        if (rb + u >= r1 || !valid) x[u] = T(0);
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int r = rb + u < r1 ? rb + u : r1 - 1;
        const T* cr = Cv + coff + (int64_t)r * npj;
#pragma unroll
        for (int al = 0; al < NPJ; ++al) acc[al] += cr[FULL ? al : (al < npj ? al : npj - 1)] * x[u];
        if constexpr (CPLX) {
          // the shuffle runs in every lane before the sign is chosen: a
          // lane-permute reads 0 from lanes that are switched off, so it
          // must not sit inside a branch on the column parity
          const T xs = __shfl_xor(x[u], 1);
          const T xp = (n & 1) ? -xs : xs;
          const T* ci = Cvi + coff + (int64_t)r * npj;
#pragma unroll
          for (int al = 0; al < NPJ; ++al) acc[al] += ci[FULL ? al : (al < npj ? al : npj - 1)] * xp;
        }
      }
    }
  };
  if (npj == NPJ) rows(std::true_type{}); else rows(std::false_type{});
  const int po = d.item_poff[item];
  if constexpr (SPLIT == 4) {
#pragma unroll
    for (int al = 0; al < NPJ; ++al) red[w][al][lane] = acc[al];
    __syncthreads();
    store_partials<T, NPJ>(red, npj, ncols, n, po, part);
  } else {
    if (!valid) return;
#pragma unroll
    for (int al = 0; al < NPJ; ++al)
      if (al < npj) part[(int64_t)(po + al) * ncols + n] = (double)acc[al];
  }
}

// The same reduction on the matrix cores (real operators, FP32 data), as
// the long-K skinny product  c[alpha][n] = sum_r C[r][alpha] x[r][n]:
// projectors alpha on the M side (two 16-blocks), support rows r on K,
// columns n on N.  Each wave owns 64 columns (four 16-column blocks), 16 rows
// at a time: their indices first, then all rows, then the products.
//   FP32:   v_mfma_f32_16x16x4f32, 4 rows per step; A[i][k] (lane i + 16k) =
//           C[r0 + k][16 b + i], B[k][j] (lane j + 16k) = x[r0 + k][n + j].
//   bf16x3: v_mfma_f32_16x16x16_bf16, 16 rows per step; lane (i, g) holds rows
//           r0 + 4g + e (e = 0..3) of its projector / column; both operands
//           split as hi = bf16(v), lo = bf16(v - hi), the product taken as
//           lo*hi + hi*lo + hi*hi with FP32 accumulation.
// D[i][j] sits in lane j + 16g, element e, i = 4g + e.
typedef float RF4 __attribute__((ext_vector_type(4)));
typedef short RB4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short nl_bf16(float x, float& back) {
  uint32_t u = __float_as_uint(x);
  u += 0x7FFFu + ((u >> 16) & 1u);
  back = __uint_as_float(u & 0xFFFF0000u);
  return (short)(u >> 16);
}

template <bool SCALE, bool BF3, int SPLIT>
__global__ void __launch_bounds__(256) k_nl_reduce_mfma(const float* __restrict__ X, int64_t ldx, int ncols,
                                                        const float* __restrict__ Minv,
                                                        const float* __restrict__ Cv, DeviceTables d,
                                                        double* __restrict__ part) {
  __shared__ float red[SPLIT == 4 ? kRowsPerWaveGroup : 1][SPLIT == 4 ? 32 : 1][64];
  const int item = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nbase = (SPLIT == 4 ? tile_index() : tile_index() * kRowsPerWaveGroup + w) * 64;
  if (SPLIT == 1 && nbase >= ncols) return;   // wave-uniform
  const int a = d.item_atom[item];
  const int npj = d.nproj[a];
  const int i0 = d.item_row0[item], i1 = d.item_row1[item];
  const int per = (i1 - i0 + SPLIT - 1) / SPLIT;
  const int r0 = SPLIT == 1 ? i0 : std::min(i0 + w * per, i1), r1 = std::min(r0 + per, i1);
  const int noff = d.atom_noff[a], coff = d.atom_coff[a];
  const int i = lane & 15, g = lane >> 4;
  RF4 acc[2][4];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[b][cb] = RF4{0.f, 0.f, 0.f, 0.f};
  for (int rb = r0; rb < r1; rb += 16) {
    // the lane's four rows of these sixteen: FP32 step q takes row 4 q + g,
    // bf16x3 takes rows 4 g + q in one step
    float xv[4][4], cv[2][4], m[4];
    int I[4], rr[4];
    bool rin[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = rb + (BF3 ? 4 * g + q : 4 * q + g);
      rin[q] = r < r1;
      rr[q] = rin[q] ? r : r1 - 1;
      I[q] = d.atom_nodes[noff + rr[q]];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      m[q] = SCALE ? Minv[I[q]] : 1.0f;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int n = nbase + 16 * cb + i;
        xv[cb][q] = X[(int64_t)I[q] * ldx + (n < ncols ? n : 0)];
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int al = 16 * b + i;
        cv[b][q] = Cv[coff + (int64_t)rr[q] * npj + (al < npj ? al : 0)];
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) xv[cb][q] = (rin[q] && nbase + 16 * cb + i < ncols) ? xv[cb][q] * m[q] : 0.0f;
#pragma unroll
      for (int b = 0; b < 2; ++b) cv[b][q] = 16 * b + i < npj ? cv[b][q] : 0.0f;
    }
    if constexpr (!BF3) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int cb = 0; cb < 4; ++cb)
            acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(cv[b][q], xv[cb][q], acc[b][cb], 0, 0, 0);
    } else {
      RB4 chi[2], clo[2], xhi[4], xlo[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          float h, dummy;
          chi[b][e] = nl_bf16(cv[b][e], h);
          clo[b][e] = nl_bf16(cv[b][e] - h, dummy);
        }
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          float h, dummy;
          xhi[cb][e] = nl_bf16(xv[cb][e], h);
          xlo[cb][e] = nl_bf16(xv[cb][e] - h, dummy);
        }
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(clo[b], xhi[cb], acc[b][cb], 0, 0, 0);
          acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(chi[b], xlo[cb], acc[b][cb], 0, 0, 0);
          acc[b][cb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(chi[b], xhi[cb], acc[b][cb], 0, 0, 0);
        }
    }
  }
  const int po = d.item_poff[item];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int al = 16 * b + 4 * g + e, n = nbase + 16 * cb + i;
        if constexpr (SPLIT == 4) red[w][al][16 * cb + i] = acc[b][cb][e];
        else if (al < npj && n < ncols) part[(int64_t)(po + al) * ncols + n] = (double)acc[b][cb][e];
      }
  if constexpr (SPLIT == 4) {
    __syncthreads();
    store_partials<float, 32>(red, npj, ncols, nbase + lane, po, part);
  }
}

// The atom-block algebra of a step, one workgroup per (atom, 16 columns), in
// two launches (every atom's d is needed before any t):
//   k_atom_first:   c = sum of the items' partials (- sum_b G^{ab} nw_b),
//                   d = (D1 - lam_n D2) c,  v = nw + d
//   k_atom_second:  t = c - sum_b G^{ab} d_b,  q = a Delta_H t,
//                   v = nw + d,  nw' = -q + ac d + zz d_prev  and the
//                   recurrence of Lambda_X
// The sum over the neighbours is one contraction (npj x about 150 rows at the
// paper's density x 16 columns) on the FP64 matrix cores
// (v_mfma_f64_16x16x4: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
// D[4 e + lane / 16][lane % 16] in element e); the four waves take every
// fourth step of four rows, whose loads are all in flight together, and add
// up in LDS.  The work is a few latencies long whatever the size, so a step
// has two such launches (128 atoms x 256 columns 71 + 35 us, 16 atoms x 192
// 18 + 11 us) in place of one per product, which read the neighbours' vectors
// once per projector (six launches, 182 us and 54 us).
// Complex operators: the columns are (re, im) pairs and an imaginary part
// mixes them: D c adds s Di c[n ^ 1], s = -1 on real, +1 on imaginary columns.
typedef double D4 __attribute__((ext_vector_type(4)));

struct AtomTile {
  double g[4][kNpjMax][17];   // the waves' sums of G x
  double c[kNpjMax][17];      // the atom's own vector
};

// the waves' parts of sum_b G^{ab} x_b, into L.g
__device__ __forceinline__ void gab_parts(const DeviceTables& d, int a, int npj, int n, int ncols,
                                          const double* __restrict__ x, AtomTile& L) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, k = lane >> 4;
  const int k0 = d.gq_ptr[a], K = d.gq_ptr[a + 1] - k0;
  const double* G = d.Gvals + d.gq_off[a];
  const double* Gi = d.Gvals_im ? d.Gvals_im + d.gq_off[a] : nullptr;
  const double sg = (n & 1) ? 1.0 : -1.0;
  D4 acc[2] = {D4{0, 0, 0, 0}, D4{0, 0, 0, 0}};
  constexpr int U = 5;   // steps in flight
  for (int j0 = 4 * w; j0 < K; j0 += 16 * U) {
    double b[U], a0[U], a1[U], i0[U], i1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 16 * u + k, jj = j < K ? j : K - 1;
      b[u] = x[(int64_t)d.gq_row[k0 + jj] * ncols + n];
      const bool in0 = j < K && i < npj, in1 = j < K && 16 + i < npj;
      a0[u] = G[in0 ? (int64_t)i * K + j : 0];
      a1[u] = G[in1 ? (int64_t)(16 + i) * K + j : 0];
      if (!in0) a0[u] = 0.0;
      if (!in1) a1[u] = 0.0;
      if (Gi) {
        i0[u] = in0 ? Gi[(int64_t)i * K + j] : 0.0;
        i1[u] = in1 ? Gi[(int64_t)(16 + i) * K + j] : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0[u], b[u], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1[u], b[u], acc[1], 0, 0, 0);
      if (Gi) {
        const double p = sg * __shfl_xor(b[u], 1);
        acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(i0[u], p, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(i1[u], p, acc[1], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int e = 0; e < 4; ++e) L.g[w][16 * m + 4 * e + k][i] = acc[m][e];
}

__device__ __forceinline__ double gab_sum(const AtomTile& L, int s, int j) {
  return (L.g[0][s][j] + L.g[1][s][j]) + (L.g[2][s][j] + L.g[3][s][j]);
}

// row s, column j of D c (c in L.c), with the imaginary part Di
__device__ __forceinline__ double block_row(const double* __restrict__ D, const double* __restrict__ Di, int s, int j,
                                            int npj, int n, const AtomTile& L) {
  double o = 0.0;
#pragma unroll 9
  for (int t = 0; t < npj; ++t) o += D[s * npj + t] * L.c[t][j];
  if (Di) {
    double oi = 0.0;
#pragma unroll 9
    for (int t = 0; t < npj; ++t) oi += Di[s * npj + t] * L.c[t][j ^ 1];
    o += (n & 1) ? oi : -oi;
  }
  return o;
}

// thread -> column j of the tile and rows s = tid / 16, + 16
__global__ void __launch_bounds__(256)
k_atom_first(const double* __restrict__ part, const double* __restrict__ nw, const double* __restrict__ D1,
             const double* __restrict__ D2, const double* __restrict__ lam, const double* __restrict__ D1i, int ncols,
             double* __restrict__ c, double* __restrict__ dv, double* __restrict__ v, DeviceTables d) {
  __shared__ AtomTile L;
  const int a = blockIdx.x;
  const int j = threadIdx.x & 15, s0 = threadIdx.x >> 4;
  const int n0 = tile_index() * 16 + j;
  const bool valid = n0 < ncols;
  const int n = valid ? n0 : (ncols > 1 ? n0 & 1 : 0);   // in range, of the column's parity
  const int npj = d.nproj[a], po = d.poff[a];
  const int i0 = d.item_ptr[a], ni = d.item_ptr[a + 1] - i0;
  if (nw) gab_parts(d, a, npj, n, ncols, nw, L);
  // the partials of all items are independent loads: up to 24 of both rows in
  // flight at a time, summed in item order
  constexpr int U = 24;
  const double* src = part + (int64_t)d.item_poff[i0] * ncols + n;
  const int64_t gs = (int64_t)npj * ncols;
  const int sa = s0 < npj ? s0 : 0, sb = s0 + 16 < npj ? s0 + 16 : sa;
  double acc[2] = {0.0, 0.0};
  for (int it = 0; it < ni; it += U) {
    double p[U], q[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double* g = src + (it + u < ni ? it + u : it) * gs;
      p[u] = g[(int64_t)sa * ncols];
      if (npj > 16) q[u] = g[(int64_t)sb * ncols];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (it + u < ni) {
        acc[0] += p[u];
        if (npj > 16) acc[1] += q[u];
      }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = s0 + 16 * h;
    if (s >= npj) break;
    if (nw) acc[h] -= gab_sum(L, s, j);
    L.c[s][j] = acc[h];
    if (c && valid) c[(int64_t)(po + s) * ncols + n] = acc[h];
  }
  if (!D1) return;
  __syncthreads();
  if (!valid) return;
  const double l = D2 ? lam[n] : 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = s0 + 16 * h;
    if (s >= npj) break;
    double o = block_row(D1 + d.poff2[a], D1i ? D1i + d.poff2[a] : nullptr, s, j, npj, n, L);
    if (D2) o -= l * block_row(D2 + d.poff2[a], nullptr, s, j, npj, n, L);
    const int64_t g = (int64_t)(po + s) * ncols + n;
    if (dv) dv[g] = o;
    if (v) v[g] = (nw ? nw[g] : 0.0) + o;
  }
}

// nw, dprev may be null (zero: the first step); qv gets q where it is wanted
// by itself (the step with an explicit T: v, nw' and lamX null).  natoms = 0:
// the recurrence of Lambda_X only.
__global__ void __launch_bounds__(256)
k_atom_second(int natoms, int ncols, const double* __restrict__ c, const double* __restrict__ dv,
              const double* __restrict__ dprev, const double* __restrict__ nwprev, const double* __restrict__ dH,
              double* __restrict__ qv, double* __restrict__ v, double* __restrict__ nw, double* __restrict__ lamX,
              const double* __restrict__ lamY, const double* __restrict__ lam_in, double a_, double ac, double zz,
              DeviceTables d) {
  __shared__ AtomTile L;
  const int a = blockIdx.x;
  const int j = threadIdx.x & 15, s0 = threadIdx.x >> 4;
  const int n0 = tile_index() * 16 + j;
  const bool valid = n0 < ncols;
  if (lamX && a == 0 && s0 == 0 && valid)
    lamX[n0] = a_ * lamY[n0] * lam_in[n0] - ac * lamY[n0] - zz * lamX[n0];
  if (a >= natoms) return;
  const int n = valid ? n0 : (ncols > 1 ? n0 & 1 : 0);
  const int npj = d.nproj[a], po = d.poff[a];
  gab_parts(d, a, npj, n, ncols, dv, L);
  double acc[2], dd[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = s0 + 16 * h;
    if (s >= npj) break;
    acc[h] = c[(int64_t)(po + s) * ncols + n];
    dd[h] = dv[(int64_t)(po + s) * ncols + n];
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (s0 + 16 * h < npj) L.c[s0 + 16 * h][j] = acc[h] - gab_sum(L, s0 + 16 * h, j);
  __syncthreads();
  if (!valid) return;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int s = s0 + 16 * h;
    if (s >= npj) break;
    const double q = a_ * block_row(dH + d.poff2[a], nullptr, s, j, npj, n, L);
    const int64_t g = (int64_t)(po + s) * ncols + n;
    if (qv) qv[g] = q;
    if (v) {
      v[g] = (nwprev ? nwprev[g] : 0.0) + dd[h];
      nw[g] = -q + ac * dd[h] + (dprev ? zz * dprev[g] : 0.0);
    }
  }
}

// Row-wise kernels.  A 256-thread block is 4 waves; a wave takes R
// consecutive DOF rows at a time, so the row index and its projector entries
// are wave-uniform (scalar loads).  Each lane owns V consecutive columns:
// with V = 16 / sizeof(element) every access of the streamed blocks is one
// 16-byte load or store per lane.  All loads of the R rows are issued before
// the first store, which keeps enough bytes in flight per CU to cover the HBM
// latency.  The grid is persistent (a fixed multiple of 8 workgroups): work
// item = (group of 4 R rows, column tile); XCD x takes the x-th contiguous
// eighth of the items (block w runs on XCD w % 8) and its workgroups stride
// through it, so each XCD streams one slab of rows and the projector
// coefficients of the atoms in that slab stay in its L2.  The host takes
// V = 1 when a leading dimension, a base pointer or the column count does
// not allow 16-byte accesses.
constexpr int kRowsPerWave = 4;
constexpr int kPersistBlocks = 2048;

template <typename T, int V>
struct Lanes {
  T v[V];
};

// The row kernels touch each streamed element once per launch: their loads
// and stores carry the non-temporal hint, so the stream does not displace
// cached data (the projector tables, the other stream's working set).
template <int V, typename T>
__device__ __forceinline__ Lanes<T, V> vld(const T* p) {
  Lanes<T, V> r;
  if constexpr (V == 1) {
    r.v[0] = __builtin_nontemporal_load(p);
  } else {
    typedef T VT __attribute__((ext_vector_type(V)));
    const VT x = __builtin_nontemporal_load(reinterpret_cast<const VT*>(p));
#pragma unroll
    for (int i = 0; i < V; ++i) r.v[i] = x[i];
  }
  return r;
}

template <int V, typename T>
__device__ __forceinline__ void vst(T* p, const Lanes<T, V>& r) {
  if constexpr (V == 1) {
    __builtin_nontemporal_store(r.v[0], p);
  } else {
    typedef T VT __attribute__((ext_vector_type(V)));
    VT x;
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = r.v[i];
    __builtin_nontemporal_store(x, reinterpret_cast<VT*>(p));
  }
}

// Persistent loop; inside, I0 is the wave's first row and n its first
// column (both valid), the rows are I0 + [0, R) below M.  Row groups of 4 R
// rows are split into 8 contiguous ranges, one per XCD; the workgroups of an
// XCD stride through its range and sweep the column tiles of each group.
#define ROWS_BEGIN(V, R)                                                                         \
  const int lane_ = threadIdx.x & 63;                                                            \
  const int wv_ = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);                              \
  const int xcd_ = blockIdx.x & 7;                                                               \
  const int ngroups_ = (int)((M + kRowsPerWaveGroup * (R) - 1) / (kRowsPerWaveGroup * (R)));     \
  const int ge_ = (int)((int64_t)ngroups_ * (xcd_ + 1) / 8);                                     \
  for (int grp_ = (int)((int64_t)ngroups_ * xcd_ / 8) + (blockIdx.x >> 3); grp_ < ge_;           \
       grp_ += (gridDim.x >> 3)) {                                                               \
    const int64_t I0 = ((int64_t)grp_ * kRowsPerWaveGroup + wv_) * (R);                          \
    for (int ct_ = 0; ct_ < ncoltiles; ++ct_) {                                                  \
      const int n = (ct_ * 64 + lane_) * (V);                                                    \
      if (n < ncols && I0 < M) {
#define ROWS_END \
  }              \
  }              \
  }

// row I0 + r clamped into range (loads only; its result is not stored)
#define ROW_CLAMP(r) ((I0 + (r) < M) ? I0 + (r) : M - 1)

// Streaming parts of the node-wise operations (local terms only); the
// projector terms sum_a C^a v_a at the support nodes are added afterwards by
// k_nl_fixup.

template <typename T, int V, int R>
__global__ void __launch_bounds__(256) k_node_zero(int64_t M, int ncols, int ncoltiles, T* __restrict__ Y,
                                                   int64_t ldy) {
  ROWS_BEGIN(V, R)
  Lanes<T, V> z;
#pragma unroll
  for (int i = 0; i < V; ++i) z.v[i] = T(0);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (I0 + r >= M) break;
    vst<V>(Y + (I0 + r) * ldy + n, z);
  }
  ROWS_END
}

// Y = M_D^{-1} X
template <typename T, int V, int R>
__global__ void __launch_bounds__(256) k_node_sinv(int64_t M, int ncols, int ncoltiles,
                                                   const T* __restrict__ X, int64_t ldx, T* __restrict__ Y,
                                                   int64_t ldy, const T* __restrict__ Minv) {
  ROWS_BEGIN(V, R)
  Lanes<T, V> x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = vld<V>(X + ROW_CLAMP(r) * ldx + n);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = I0 + r;
    if (I >= M) break;
    const T m = Minv[I];
    Lanes<T, V> y;
#pragma unroll
    for (int i = 0; i < V; ++i) y.v[i] = m * x[r].v[i];
    vst<V>(Y + I * ldy + n, y);
  }
  ROWS_END
}

// T = M_D^{-1} R_Y;  R_X <- -a c R_Y - zeta zeta' R_X + a Y Lambda_Y
template <typename TR, int V, int R>
__global__ void __launch_bounds__(256) k_node_cheb(int64_t M, int ncols, int ncoltiles,
                                                   const TR* __restrict__ RY,
                                                   TR* __restrict__ RX, TR* __restrict__ Tb, int64_t ld,
                                                   const double* __restrict__ Y, int64_t ldy,
                                                   const double* __restrict__ lamY, double* __restrict__ lamX,
                                                   const double* __restrict__ lam_in, double a, double ac,
                                                   double zz, const TR* __restrict__ Minv) {
  ROWS_BEGIN(V, R)
  Lanes<TR, V> ry[R], rx[R];
  Lanes<double, V> y[R];
  TR m[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = ROW_CLAMP(r);
    ry[r] = vld<V>(RY + I * ld + n);
    rx[r] = vld<V>(RX + I * ld + n);
    y[r] = vld<V>(Y + I * ldy + n);
    m[r] = Minv[I];
  }
  double ly[V];
#pragma unroll
  for (int i = 0; i < V; ++i) ly[i] = a * lamY[n + i];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = I0 + r;
    if (I >= M) break;
    Lanes<TR, V> t, o;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      t.v[i] = m[r] * ry[r].v[i];
      // recurrence part in TR arithmetic, residual correction a Y lamY in FP64
      const TR part = (TR)(-ac) * ry[r].v[i] - (TR)zz * rx[r].v[i];
      o.v[i] = (TR)((double)part + y[r].v[i] * ly[i]);
    }
    vst<V>(Tb + I * ld + n, t);
    vst<V>(RX + I * ld + n, o);
    if (I == 0) {
#pragma unroll
      for (int i = 0; i < V; ++i)
        lamX[n + i] = a * lamY[n + i] * lam_in[n + i] - ac * lamY[n + i] - zz * lamX[n + i];
    }
  }
  ROWS_END
}

// Xout = M_D^{-1} R_Y + X Lambda_Y
template <typename TR, int V, int R>
__global__ void __launch_bounds__(256) k_node_finalize(int64_t M, int ncols, int ncoltiles,
                                                       const TR* __restrict__ RY, int64_t ld,
                                                       const double* __restrict__ X, int64_t ldx,
                                                       const double* __restrict__ lamY, double* __restrict__ Xo,
                                                       int64_t ldo, const TR* __restrict__ Minv) {
  ROWS_BEGIN(V, R)
  Lanes<TR, V> ry[R];
  Lanes<double, V> x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = ROW_CLAMP(r);
    ry[r] = vld<V>(RY + I * ld + n);
    x[r] = vld<V>(X + I * ldx + n);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = I0 + r;
    if (I >= M) break;
    const TR m = Minv[I];
    Lanes<double, V> o;
#pragma unroll
    for (int i = 0; i < V; ++i) o.v[i] = (double)(m * ry[r].v[i]) + x[r].v[i] * lamY[n + i];
    vst<V>(Xo + I * ldo + n, o);
  }
  ROWS_END
}

// Projector add-back on the support nodes:
//   out1[I] += s1 * w_I * sum_a sum_alpha C^a[I][alpha] v1_a[alpha][n]
//   out2[I] +=            sum_a sum_alpha C^a[I][alpha] v2_a[alpha][n]   (if out2)
// with w_I = M_D^{-1}[I] if minv, else 1.  Every row is written by one item, so
// all atoms go in one launch: workgroups [0, nshared) take the rows shared by
// several atoms (items of up to kFixShared rows with the same atoms), the rest
// the rows of one atom alone (items of up to 16 consecutive rows of C^a).
// Thread <-> column: an atom's coefficient vector for that column sits in
// registers and serves all rows of the item, kFixUnroll rows at a time with
// all loads issued first.  Bound by the read-modify-write of scattered rows;
// one launch per atom colour (atoms of a colour share no row) waited out the
// latency chain of its items six to eight times (128 atoms x 256 columns FP32
// 471 -> 354 us, FP64 663 -> 652, 3.7 TB/s; 18 atoms x 200 columns FP32
// 106 -> 55; 12 atoms x 101 columns 67 -> 17).
constexpr int kFixUnroll = 8;
static_assert(kFixUnroll == kFixShared, "rows in flight of a shared item");

// Waves per SIMD that the kernel is held to: with the items of shared rows it
// would take more registers than the walk over one atom's rows needs.  128 atoms
// of 18 projectors x 256 columns, us a launch, left alone -> held: FP64 678 (at
// six) -> 652 at five, complex 1307 -> 1127 at four; FP32 complex 584 -> 575 at
// seven, into FP64 rows 804 -> 739 at six.
constexpr int fix_waves(size_t tr, size_t to, int npj, bool has2, bool cplx) {
  if (npj > 18 || has2) return 1;
  if (tr == 8) return cplx && npj > 8 ? 4 : 5;
  return cplx && npj > 8 && to == 8 ? 6 : 7;
}

// CPLX (complex operators): (re, im) column pairs, C v mixes them:
// + s Ci v[n ^ 1], s = -1 on real and +1 on imaginary columns (partner value
// from the neighbouring lane).
template <typename TR, typename TO1, int NPJ, bool MINV, bool HAS2, bool CPLX>
__global__ void __launch_bounds__(256)
    __attribute__((amdgpu_waves_per_eu((fix_waves(sizeof(TR), sizeof(TO1), NPJ, HAS2, CPLX)))))
k_nl_fixup(int nshared, int ncols, const double* __restrict__ v1, double s1,
                                                  TO1* __restrict__ out1, int64_t ld1,
                                                  const double* __restrict__ v2, TR* __restrict__ out2,
                                                  int64_t ld2, const TR* __restrict__ Minv,
                                                  const TR* __restrict__ Cv, DeviceTables d,
                                                  const TR* __restrict__ Cvi) {
  const int n = blockIdx.y * 256 + threadIdx.x;
  if (n >= ncols) return;
  // All loads are unconditional (indices clamped into range), so they are in
  // flight together; an atom with exactly NPJ projectors takes the path with
  // plain indices (wide scalar loads of its C rows).
  TR w1[NPJ], w2[HAS2 ? NPJ : 1], p1[CPLX ? NPJ : 1], p2[CPLX && HAS2 ? NPJ : 1];
  // the coefficients of one atom for this column
  auto coeffs = [&](auto full, int po, int npj) {
    constexpr bool FULL = decltype(full)::value;
    auto idx = [&](int al) { return FULL ? al : (al < npj ? al : npj - 1); };
#pragma unroll
    for (int al = 0; al < NPJ; ++al) {
      const double x1 = v1[(int64_t)(po + idx(al)) * ncols + n];
      w1[al] = (FULL || al < npj) ? (TR)(s1 * x1) : TR(0);
      if constexpr (HAS2) {
        const double x2 = v2[(int64_t)(po + idx(al)) * ncols + n];
        w2[al] = (FULL || al < npj) ? (TR)x2 : TR(0);
      }
    }
    if constexpr (CPLX) {
      const TR sg = (n & 1) ? TR(1) : TR(-1);
#pragma unroll
      for (int al = 0; al < NPJ; ++al) {
        p1[al] = sg * __shfl_xor(w1[al], 1);
        if constexpr (HAS2) p2[al] = sg * __shfl_xor(w2[al], 1);
      }
    }
  };
  // c1 += C row . v1 (c2 += C row . v2), the row at offset r of Cv
  auto dot = [&](auto full, int64_t r, int npj, TR& c1, TR& c2) {
    constexpr bool FULL = decltype(full)::value;
    auto idx = [&](int al) { return FULL ? al : (al < npj ? al : npj - 1); };
    const TR* cr = Cv + r;
#pragma unroll
    for (int al = 0; al < NPJ; ++al) {
      const TR cv = cr[idx(al)];
      c1 += cv * w1[al];
      if constexpr (HAS2) c2 += cv * w2[al];
    }
    if constexpr (CPLX) {
      const TR* ci = Cvi + r;
#pragma unroll
      for (int al = 0; al < NPJ; ++al) {
        const TR cv = ci[idx(al)];
        c1 += cv * p1[al];
        if constexpr (HAS2) c2 += cv * p2[al];
      }
    }
  };
  TO1 o1[kFixUnroll];
  TR o2[kFixUnroll], c1[kFixUnroll], c2[kFixUnroll];
  auto load_rows = [&](const int (&I)[kFixUnroll]) {
#pragma unroll
    for (int u = 0; u < kFixUnroll; ++u) {   // rows touched once: non-temporal
      o1[u] = __builtin_nontemporal_load(out1 + (int64_t)I[u] * ld1 + n);
      if constexpr (HAS2) o2[u] = __builtin_nontemporal_load(out2 + (int64_t)I[u] * ld2 + n);
      c1[u] = c2[u] = TR(0);
    }
  };
  auto store_rows = [&](const int (&I)[kFixUnroll], int nrow) {
#pragma unroll
    for (int u = 0; u < kFixUnroll; ++u) {
      if (u >= nrow) break;
      if constexpr (MINV) c1[u] *= Minv[I[u]];
      __builtin_nontemporal_store(o1[u] + (TO1)c1[u], out1 + (int64_t)I[u] * ld1 + n);
      if constexpr (HAS2) __builtin_nontemporal_store(o2[u] + c2[u], out2 + (int64_t)I[u] * ld2 + n);
    }
  };
  int I[kFixUnroll];
  if ((int)blockIdx.x < nshared) {
    const int32_t* it = d.fixs_data + d.fixs_ptr[blockIdx.x];
    const int nat = d.fixs_nat[blockIdx.x];
#pragma unroll
    for (int u = 0; u < kFixUnroll; ++u) I[u] = it[u];
    load_rows(I);
    for (int k = 0; k < nat; ++k) {
      const int32_t* e = it + kFixShared + k * (kFixShared + 1);
      const int a = e[0], npj = d.nproj[a];
      auto body = [&](auto full) {
        coeffs(full, d.poff[a], npj);
#pragma unroll
        for (int u = 0; u < kFixUnroll; ++u) {
          dot(full, e[1 + u], npj, c1[u], c2[u]);
          // FP64 rows of an FP32 filter: the atoms' terms are summed in FP64
          if constexpr (sizeof(TO1) > sizeof(TR)) {
            if constexpr (MINV) c1[u] *= Minv[I[u]];
            o1[u] += (TO1)c1[u];
            c1[u] = TR(0);
          }
        }
      };
      if (npj == NPJ) body(std::true_type{}); else body(std::false_type{});
    }
    store_rows(I, d.fixs_nrow[blockIdx.x]);   // (c1 is zero where the terms are in o1)
    return;
  }
  const int item = blockIdx.x - nshared;
  const int a = d.fix_atom[item];
  const int r0 = d.fix_row0[item], r1 = d.fix_row1[item];
  const int npj = d.nproj[a], noff = d.atom_noff[a];
  const int64_t coff = d.atom_coff[a];
  auto body = [&](auto full) {
    coeffs(full, d.poff[a], npj);
    for (int rb = r0; rb < r1; rb += kFixUnroll) {
#pragma unroll
      for (int u = 0; u < kFixUnroll; ++u) I[u] = d.atom_nodes[noff + rb + u];   // list padded
      load_rows(I);
#pragma unroll
      for (int u = 0; u < kFixUnroll; ++u)
        dot(full, coff + (int64_t)(rb + u < r1 ? rb + u : r1 - 1) * npj, npj, c1[u], c2[u]);
      store_rows(I, r1 - rb);
    }
  };
  if (npj == NPJ) body(std::true_type{}); else body(std::false_type{});
}

template <typename TR, int V, int R>
__global__ void __launch_bounds__(256) k_cheb_init(int64_t M, int ncols, int ncoltiles,
                                                   const double* __restrict__ Y,
                                                   int64_t ldy, TR* __restrict__ RY, TR* __restrict__ RX,
                                                   int64_t ld, double f, double c,
                                                   const double* __restrict__ lam_in, double* __restrict__ lamY,
                                                   double* __restrict__ lamX) {
  ROWS_BEGIN(V, R)
  Lanes<double, V> y[R];
#pragma unroll
  for (int r = 0; r < R; ++r) y[r] = vld<V>(Y + ROW_CLAMP(r) * ldy + n);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t I = I0 + r;
    if (I >= M) break;
    Lanes<TR, V> ry, z;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      ry.v[i] = (TR)(f * y[r].v[i]);
      z.v[i] = TR(0);
    }
    vst<V>(RY + I * ld + n, ry);
    vst<V>(RX + I * ld + n, z);
    if (I == 0) {
#pragma unroll
      for (int i = 0; i < V; ++i) {
        lamY[n + i] = f * (lam_in[n + i] - c);
        lamX[n + i] = 1.0;
      }
    }
  }
  ROWS_END
}

template <int V, int R>
__global__ void __launch_bounds__(256) k_copy_cols(int64_t M, int ncols, int ncoltiles,
                                                   const double* __restrict__ X, int64_t ldx,
                                                   double* __restrict__ Y, int64_t ldy) {
  ROWS_BEGIN(V, R)
  Lanes<double, V> x[R];
#pragma unroll
  for (int r = 0; r < R; ++r) x[r] = vld<V>(X + ROW_CLAMP(r) * ldx + n);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (I0 + r >= M) break;
    vst<V>(Y + (I0 + r) * ldy + n, x[r]);
  }
  ROWS_END
}

template <typename T>
__global__ void k_fill(T* __restrict__ Y, int64_t n, T v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    Y[i] = v;
}

// partial[chunk][n] = sum_{i in chunk} A[i][n] B[i][n].  Sixteen waves share a
// chunk's rows, four in flight each: with four waves of one row at a time 92
// chunks x 256 columns read at 2.9 TB/s (373,000 rows 0.53 -> 0.295 ms,
// 5.2 TB/s).
constexpr int kDotWaves = 16;
__global__ void __launch_bounds__(64 * kDotWaves) k_coldot(const double* __restrict__ A, int64_t lda,
                                                           const double* __restrict__ B, int64_t ldb, int64_t nrows,
                                                           int ncols, int64_t rows_per_chunk,
                                                           double* __restrict__ partial) {
  __shared__ double red[kDotWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = blockIdx.y * 64 + lane;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per_chunk;
  const int64_t r1 = (r0 + rows_per_chunk < nrows) ? r0 + rows_per_chunk : nrows;
  double acc = 0.0;
  if (n < ncols) {
    const bool same = A == B && lda == ldb;   // squares: each row once
    for (int64_t i = r0 + w; i < r1; i += 4 * kDotWaves) {
      double x[4], y[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t k = i + u * kDotWaves;
        x[u] = k < r1 ? A[k * lda + n] : 0.0;
        y[u] = same ? x[u] : (k < r1 ? B[k * ldb + n] : 0.0);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += x[u] * y[u];
    }
  }
  red[w][lane] = acc;
  __syncthreads();
  if (w == 0 && n < ncols) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < kDotWaves; ++k) s += red[k][lane];
    partial[(int64_t)blockIdx.x * ncols + n] = s;
  }
}

__global__ void __launch_bounds__(256) k_coldot_final(const double* __restrict__ partial, int nchunks, int ncols,
                                                      double* __restrict__ out, const double* __restrict__ w,
                                                      int sqrt_out, int scalar) {
  __shared__ double red[256];
  if (!scalar) {
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= ncols) return;
    double s = 0.0;
    for (int c = 0; c < nchunks; ++c) s += partial[(int64_t)c * ncols + n];
    out[n] = sqrt_out ? sqrt(s) : s;
    return;
  }
  double s = 0.0;
  for (int n = threadIdx.x; n < ncols; n += 256) {
    double t = 0.0;
    for (int c = 0; c < nchunks; ++c) t += partial[(int64_t)c * ncols + n];
    s += (w ? w[n] : 1.0) * t;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] += red[0];
}

__global__ void k_grad_dh(const double* __restrict__ c, int ncols, const double* __restrict__ occ,
                          const int32_t* __restrict__ ent_atom, const int32_t* __restrict__ ent_s,
                          const int32_t* __restrict__ ent_t, int nent, DeviceTables d, double* __restrict__ out) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nent) return;
  const int a = ent_atom[k], s = ent_s[k], t = ent_t[k];
  const int po = d.poff[a], npj = d.nproj[a];
  const double* ps = c + (int64_t)(po + s) * ncols;
  const double* pt = c + (int64_t)(po + t) * ncols;
  double acc = 0.0;
  for (int n = 0; n < ncols; ++n) acc += (occ ? occ[n] : 1.0) * ps[n] * pt[n];
  out[d.poff2[a] + s * npj + t] = acc;
}

struct RowGrid {
  int ncoltiles;
  dim3 grid;
};
// Persistent grid: the workgroups of kernel K that are resident at once
// (so none waits for a second round), a multiple of 8, capped by the work.
template <typename K>
inline int resident_blocks(K kernel) {
  int dev = 0, ncu = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
    ncu = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess || per_cu <= 0)
    per_cu = 1;
  return std::max(8, ncu * per_cu / 8 * 8);
}
template <auto K>
inline RowGrid row_grid(int64_t M, int ncols, int V, int R) {
  static const int resident = resident_blocks(K);
  RowGrid g;
  g.ncoltiles = (ncols + 64 * V - 1) / (64 * V);
  const int64_t ngroups = (M + kRowsPerWaveGroup * R - 1) / (kRowsPerWaveGroup * R);
  g.grid = dim3((unsigned)std::max<int64_t>(8, std::min<int64_t>(resident, (ngroups + 7) / 8 * 8)));
  return g;
}

// True when V columns per lane are allowed: ncols a multiple of V and every
// (base pointer, leading dimension) pair 16-byte aligned row by row.
struct Strided {
  const void* p;
  int64_t ld;
};
inline bool vec_ok(int V, int ncols, std::initializer_list<Strided> xs) {
  if (ncols % V) return false;
  for (const Strided& x : xs)
    if ((reinterpret_cast<uintptr_t>(x.p) & 15) || x.ld % V) return false;
  return true;
}

template <typename T>
const T* pick(const double* d64, const float* d32) {
  if constexpr (std::is_same<T, double>::value) return d64; else return d32;
}

}  // namespace

// ---------------------------------------------------------------------------

template <typename T>
pawfe_status launch_nl_reduce(const pawfe_op* op, const T* X, int64_t ldx, int ncols, bool scale_minv, double* part,
                              hipStream_t s, bool bf3, bool by_op) {
  if (op->natoms == 0 || ncols <= 0) return PAWFE_OK;
  const T* Cv = pick<T>(op->d.Cvals, op->d.Cvals_f);
  const T* Minv = pick<T>(op->d.Minv, op->d.Minv_f);
  const T* Cvi = pick<T>(op->d.Cvals_im, op->d.Cvals_im_f);
  // fewer than three waves per SIMD without the split: take it
  static_assert(kRowsPerWaveGroup == 4, "waves of a reduction workgroup");
  const bool split = (int64_t)op->nitems * (((by_op ? kResidualColsNl : ncols) + 63) / 64) < 3000;
  const dim3 grid = tile_grid(op->nitems, split ? (ncols + 63) / 64 : (ncols + 255) / 256), block(256);
  if constexpr (std::is_same<T, float>::value) {
    if (!op->cplx) {   // real operators in FP32: the matrix-core reduction
      auto go = [&](auto scale, auto b3) {
        constexpr bool SC = decltype(scale)::value, B3 = decltype(b3)::value;
        if (split)
          hipLaunchKernelGGL((k_nl_reduce_mfma<SC, B3, 4>), grid, block, 0, s, X, ldx, ncols, Minv, Cv, op->d, part);
        else
          hipLaunchKernelGGL((k_nl_reduce_mfma<SC, B3, 1>), grid, block, 0, s, X, ldx, ncols, Minv, Cv, op->d, part);
      };
      if (scale_minv) {
        if (bf3) go(std::true_type{}, std::true_type{}); else go(std::true_type{}, std::false_type{});
      } else {
        if (bf3) go(std::false_type{}, std::true_type{}); else go(std::false_type{}, std::false_type{});
      }
      PAWFE_HIP(hipGetLastError());
      return PAWFE_OK;
    }
  }
  auto go = [&](auto scale, auto cplx) {
    constexpr bool SC = decltype(scale)::value, CX = decltype(cplx)::value;
    auto by_npj = [&](auto npj) {
      constexpr int NPJ = decltype(npj)::value;
      if (split)
        hipLaunchKernelGGL((k_nl_reduce<T, NPJ, SC, CX, 4>), grid, block, 0, s, X, ldx, ncols, Minv, Cv, op->d, part,
                           Cvi);
      else
        hipLaunchKernelGGL((k_nl_reduce<T, NPJ, SC, CX, 1>), grid, block, 0, s, X, ldx, ncols, Minv, Cv, op->d, part,
                           Cvi);
    };
    if (op->npj_max <= 8) by_npj(std::integral_constant<int, 8>{});
    else if (op->npj_max <= 18) by_npj(std::integral_constant<int, 18>{});
    else by_npj(std::integral_constant<int, 32>{});
  };
  if (op->cplx) {
    if (scale_minv) go(std::true_type{}, std::true_type{}); else go(std::false_type{}, std::true_type{});
  } else {
    if (scale_minv) go(std::true_type{}, std::false_type{}); else go(std::false_type{}, std::false_type{});
  }
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}
template pawfe_status launch_nl_reduce<double>(const pawfe_op*, const double*, int64_t, int, bool, double*,
                                               hipStream_t, bool, bool);
template pawfe_status launch_nl_reduce<float>(const pawfe_op*, const float*, int64_t, int, bool, double*, hipStream_t,
                                              bool, bool);

pawfe_status launch_atom_first(const pawfe_op* op, const double* part, const double* nw, const double* D1,
                               const double* D2, const double* lam, const double* D1i, int ncols, double* c,
                               double* dv, double* v, hipStream_t s) {
  if (op->natoms == 0 || ncols <= 0) return PAWFE_OK;
  hipLaunchKernelGGL(k_atom_first, tile_grid(op->natoms, (ncols + 15) / 16), dim3(256), 0, s, part, nw, D1, D2, lam, D1i,
                     ncols, c, dv, v, op->d);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

pawfe_status launch_atom_second(const pawfe_op* op, const double* c, const double* dv, const double* dprev,
                                const double* nwprev, double* qv, double* v, double* nw, double* lamX,
                                const double* lamY, const double* lam_in, double a, double ac, double zz, int ncols,
                                hipStream_t s) {
  if (ncols <= 0 || (op->natoms == 0 && !lamX)) return PAWFE_OK;
  hipLaunchKernelGGL(k_atom_second, tile_grid(std::max(op->natoms, 1), (ncols + 15) / 16), dim3(256), 0, s, op->natoms,
                     ncols, c, dv, dprev, nwprev, op->d.dH, qv, v, nw, lamX, lamY, lam_in, a, ac, zz, op->d);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

__global__ void k_dup_pairs(const double* __restrict__ in, double* __restrict__ out, int n) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < n) {
    const double v = in[j];
    out[2 * j] = v;
    out[2 * j + 1] = v;
  }
}

pawfe_status launch_dup_pairs(const double* in, double* out, int n, hipStream_t s) {
  if (n <= 0) return PAWFE_OK;
  hipLaunchKernelGGL(k_dup_pairs, dim3((n + 255) / 256), dim3(256), 0, s, in, out, n);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

// out1 += s1 w C v1 (w = M_D^{-1} if MINV), out2 += C v2 (if HAS2)
template <typename TR, typename TO1, bool MINV, bool HAS2>
pawfe_status nl_fixup(const pawfe_op* op, int ncols, const double* v1, double s1, TO1* out1, int64_t ld1,
                      const double* v2, TR* out2, int64_t ld2, hipStream_t s) {
  if (op->natoms == 0 || ncols <= 0) return PAWFE_OK;
  const TR* Cv = pick<TR>(op->d.Cvals, op->d.Cvals_f);
  const TR* Cvi = pick<TR>(op->d.Cvals_im, op->d.Cvals_im_f);
  const TR* Minv = pick<TR>(op->d.Minv, op->d.Minv_f);
  const int nshared = (int)op->fixs_nat.size(), nitems = nshared + (int)op->fix_atom.size();
  if (nitems == 0) return PAWFE_OK;
  const dim3 grid(nitems, (ncols + 255) / 256), block(256);
  auto go = [&](auto npj, auto cplx) {
    constexpr int NPJ = decltype(npj)::value;
    constexpr bool CX = decltype(cplx)::value;
    hipLaunchKernelGGL((k_nl_fixup<TR, TO1, NPJ, MINV, HAS2, CX>), grid, block, 0, s, nshared, ncols, v1, s1, out1, ld1,
                       v2, out2, ld2, Minv, Cv, op->d, Cvi);
  };
  auto by_npj = [&](auto cplx) {
    if (op->npj_max <= 8) go(std::integral_constant<int, 8>{}, cplx);
    else if (op->npj_max <= 18) go(std::integral_constant<int, 18>{}, cplx);
    else go(std::integral_constant<int, 32>{}, cplx);
  };
  if (op->cplx) by_npj(std::true_type{});
  else if constexpr (!HAS2) by_npj(std::false_type{});
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

pawfe_status launch_node_nl_init(const pawfe_op* op, const double* q, int ncols, float* Y, int64_t ldy,
                                 hipStream_t s) {
  if (ncols <= 0) return PAWFE_OK;
  constexpr int V = 4;
  if (vec_ok(V, ncols, {{Y, ldy}})) {
    const RowGrid g = row_grid<k_node_zero<float, V, kRowsPerWave>>(op->M, ncols, V, kRowsPerWave);
    hipLaunchKernelGGL((k_node_zero<float, V, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, Y,
                       ldy);
  } else {
    const RowGrid g = row_grid<k_node_zero<float, 1, kRowsPerWave>>(op->M, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_node_zero<float, 1, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, Y,
                       ldy);
  }
  PAWFE_HIP(hipGetLastError());
  return nl_fixup<float, float, false, false>(op, ncols, q, 1.0, Y, ldy, nullptr, (float*)nullptr, 0, s);
}

template <typename T>
pawfe_status launch_node_fixup(const pawfe_op* op, const double* v1, double s1, int ncols, T* out1, int64_t ld1,
                               hipStream_t s) {
  return nl_fixup<T, T, false, false>(op, ncols, v1, s1, out1, ld1, nullptr, (T*)nullptr, 0, s);
}
template pawfe_status launch_node_fixup<double>(const pawfe_op*, const double*, double, int, double*, int64_t,
                                                hipStream_t);
template pawfe_status launch_node_fixup<float>(const pawfe_op*, const double*, double, int, float*, int64_t,
                                               hipStream_t);

template <typename T>
pawfe_status launch_node_sinv(const pawfe_op* op, const T* X, int64_t ldx, const double* dv, int ncols, T* Y,
                              int64_t ldy, hipStream_t s) {
  if (ncols <= 0) return PAWFE_OK;
  constexpr int V = 16 / sizeof(T);
  const T* Minv = pick<T>(op->d.Minv, op->d.Minv_f);
  if (vec_ok(V, ncols, {{X, ldx}, {Y, ldy}})) {
    const RowGrid g = row_grid<k_node_sinv<T, V, kRowsPerWave>>(op->M, ncols, V, kRowsPerWave);
    hipLaunchKernelGGL((k_node_sinv<T, V, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, X, ldx,
                       Y, ldy, Minv);
  } else {
    const RowGrid g = row_grid<k_node_sinv<T, 1, kRowsPerWave>>(op->M, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_node_sinv<T, 1, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, X, ldx,
                       Y, ldy, Minv);
  }
  PAWFE_HIP(hipGetLastError());
  return nl_fixup<T, T, true, false>(op, ncols, dv, -1.0, Y, ldy, nullptr, (T*)nullptr, 0, s);
}
template pawfe_status launch_node_sinv<double>(const pawfe_op*, const double*, int64_t, const double*, int, double*,
                                               int64_t, hipStream_t);
template pawfe_status launch_node_sinv<float>(const pawfe_op*, const float*, int64_t, const double*, int, float*,
                                              int64_t, hipStream_t);

template <typename TR>
pawfe_status launch_node_cheb(const pawfe_op* op, const TR* RY, TR* RX, TR* Tb, int64_t ld, const double* Y,
                              int64_t ldy, const double* dv, const double* qv, const double* lamY, double* lamX,
                              const double* lam_in, double a, double ac, double zz, int ncols, hipStream_t s) {
  if (ncols <= 0) return PAWFE_OK;
  constexpr int V = 16 / sizeof(TR);
  const TR* Minv = pick<TR>(op->d.Minv, op->d.Minv_f);
  if (vec_ok(V, ncols, {{RY, ld}, {RX, ld}, {Tb, ld}, {Y, ldy}})) {
    const RowGrid g = row_grid<k_node_cheb<TR, V, kRowsPerWave>>(op->M, ncols, V, kRowsPerWave);
    hipLaunchKernelGGL((k_node_cheb<TR, V, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, RY,
                       RX, Tb, ld, Y, ldy, lamY, lamX, lam_in, a, ac, zz, Minv);
  } else {
    const RowGrid g = row_grid<k_node_cheb<TR, 1, kRowsPerWave>>(op->M, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_node_cheb<TR, 1, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, RY,
                       RX, Tb, ld, Y, ldy, lamY, lamX, lam_in, a, ac, zz, Minv);
  }
  PAWFE_HIP(hipGetLastError());
  // T -= M_D^{-1} C d ; R_X += C q  (q already scaled by a).  Real operators: one
  // launch each, which leaves the registers for twice the waves (128 atoms x 256
  // columns FP32 797 -> 2 x 361 us, 64 atoms of 8 projectors 119 -> 2 x 55);
  // complex ones read the coefficients of both together (1058 us, else 2 x 575)
  if (op->cplx) return nl_fixup<TR, TR, true, true>(op, ncols, dv, -1.0, Tb, ld, qv, RX, ld, s);
  const pawfe_status st = nl_fixup<TR, TR, true, false>(op, ncols, dv, -1.0, Tb, ld, nullptr, (TR*)nullptr, 0, s);
  if (st != PAWFE_OK) return st;
  return nl_fixup<TR, TR, false, false>(op, ncols, qv, 1.0, RX, ld, nullptr, (TR*)nullptr, 0, s);
}
template pawfe_status launch_node_cheb<double>(const pawfe_op*, const double*, double*, double*, int64_t,
                                               const double*, int64_t, const double*, const double*, const double*,
                                               double*, const double*, double, double, double, int, hipStream_t);
template pawfe_status launch_node_cheb<float>(const pawfe_op*, const float*, float*, float*, int64_t, const double*,
                                              int64_t, const double*, const double*, const double*, double*,
                                              const double*, double, double, double, int, hipStream_t);

template <typename TR>
pawfe_status launch_node_finalize(const pawfe_op* op, const TR* RY, int64_t ld, const double* dv, const double* X,
                                  int64_t ldx, const double* lamY, double* Xo, int64_t ldo, int ncols, hipStream_t s) {
  if (ncols <= 0) return PAWFE_OK;
  constexpr int V = 16 / sizeof(TR);
  const TR* Minv = pick<TR>(op->d.Minv, op->d.Minv_f);
  if (vec_ok(V, ncols, {{RY, ld}, {X, ldx}, {Xo, ldo}})) {
    const RowGrid g = row_grid<k_node_finalize<TR, V, kRowsPerWave>>(op->M, ncols, V, kRowsPerWave);
    hipLaunchKernelGGL((k_node_finalize<TR, V, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles,
                       RY, ld, X, ldx, lamY, Xo, ldo, Minv);
  } else {
    const RowGrid g = row_grid<k_node_finalize<TR, 1, kRowsPerWave>>(op->M, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_node_finalize<TR, 1, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles,
                       RY, ld, X, ldx, lamY, Xo, ldo, Minv);
  }
  PAWFE_HIP(hipGetLastError());
  return nl_fixup<TR, double, true, false>(op, ncols, dv, -1.0, Xo, ldo, nullptr, (TR*)nullptr, 0, s);
}
template pawfe_status launch_node_finalize<double>(const pawfe_op*, const double*, int64_t, const double*,
                                                   const double*, int64_t, const double*, double*, int64_t, int,
                                                   hipStream_t);
template pawfe_status launch_node_finalize<float>(const pawfe_op*, const float*, int64_t, const double*, const double*,
                                                  int64_t, const double*, double*, int64_t, int, hipStream_t);

template <typename TR>
pawfe_status launch_cheb_init(const pawfe_op* op, const double* Y, int64_t ldy, TR* RY, TR* RX, int64_t ld, double f,
                              double c, const double* lam_in, double* lamY, double* lamX, int ncols, hipStream_t s) {
  if (ncols <= 0) return PAWFE_OK;
  constexpr int V = 16 / sizeof(TR);
  if (vec_ok(V, ncols, {{Y, ldy}, {RY, ld}, {RX, ld}})) {
    const RowGrid g = row_grid<k_cheb_init<TR, V, kRowsPerWave>>(op->M, ncols, V, kRowsPerWave);
    hipLaunchKernelGGL((k_cheb_init<TR, V, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, Y, ldy,
                       RY, RX, ld, f, c, lam_in, lamY, lamX);
  } else {
    const RowGrid g = row_grid<k_cheb_init<TR, 1, kRowsPerWave>>(op->M, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_cheb_init<TR, 1, kRowsPerWave>), g.grid, dim3(256), 0, s, op->M, ncols, g.ncoltiles, Y, ldy,
                       RY, RX, ld, f, c, lam_in, lamY, lamX);
  }
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}
template pawfe_status launch_cheb_init<double>(const pawfe_op*, const double*, int64_t, double*, double*, int64_t,
                                               double, double, const double*, double*, double*, int, hipStream_t);
template pawfe_status launch_cheb_init<float>(const pawfe_op*, const double*, int64_t, float*, float*, int64_t,
                                              double, double, const double*, double*, double*, int, hipStream_t);

pawfe_status launch_copy_cols(const double* X, int64_t ldx, double* Y, int64_t ldy, int64_t nrows, int ncols,
                              hipStream_t s) {
  if (ncols <= 0 || nrows <= 0) return PAWFE_OK;
  if (vec_ok(2, ncols, {{X, ldx}, {Y, ldy}})) {
    const RowGrid g = row_grid<k_copy_cols<2, kRowsPerWave>>(nrows, ncols, 2, kRowsPerWave);
    hipLaunchKernelGGL((k_copy_cols<2, kRowsPerWave>), g.grid, dim3(256), 0, s, nrows, ncols, g.ncoltiles, X, ldx, Y,
                       ldy);
  } else {
    const RowGrid g = row_grid<k_copy_cols<1, kRowsPerWave>>(nrows, ncols, 1, kRowsPerWave);
    hipLaunchKernelGGL((k_copy_cols<1, kRowsPerWave>), g.grid, dim3(256), 0, s, nrows, ncols, g.ncoltiles, X, ldx, Y,
                       ldy);
  }
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

template <typename T>
pawfe_status launch_fill(T* Y, int64_t n, T v, hipStream_t s) {
  if (n <= 0) return PAWFE_OK;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)blocks), dim3(256), 0, s, Y, n, v);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}
template pawfe_status launch_fill<double>(double*, int64_t, double, hipStream_t);
template pawfe_status launch_fill<float>(float*, int64_t, float, hipStream_t);

pawfe_status launch_coldot(const double* A, int64_t lda, const double* B, int64_t ldb, int64_t nrows, int ncols,
                           double* partial, double* out, const double* w, bool sqrt_out, bool scalar, hipStream_t s) {
  const int64_t rpc = 4096;
  const int nchunks = (int)((nrows + rpc - 1) / rpc);
  hipLaunchKernelGGL(k_coldot, dim3(nchunks, (ncols + 63) / 64), dim3(64 * kDotWaves), 0, s, A, lda, B, ldb, nrows, ncols, rpc,
                     partial);
  hipLaunchKernelGGL(k_coldot_final, dim3(scalar ? 1 : (ncols + 255) / 256), dim3(256), 0, s, partial, nchunks, ncols,
                     out, w, (int)sqrt_out, (int)scalar);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

pawfe_status launch_grad_dh(const pawfe_op* op, const double* c, int ncols, const double* occ, double* out,
                            hipStream_t s) {
  if (op->natoms == 0) return PAWFE_OK;
  const int nent = op->npj2_total;
  hipLaunchKernelGGL(k_grad_dh, dim3((nent + 255) / 256), dim3(256), 0, s, c, ncols, occ, op->d_g2_atom, op->d_g2_s,
                     op->d_g2_t, nent, op->d, out);
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

}  // namespace pawfe

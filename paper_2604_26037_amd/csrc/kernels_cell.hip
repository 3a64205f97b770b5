// Cell-level entry of the FE operators and the band-energy density.
//
// launch_cell sets up the arguments of the cell operator (kinetic + V(q)W_q,
// the residual variant with -lambda_n M, or the mass; the cell-level product
// of the operator-action subsection) and runs, one launch per cell colour,
// the vector-ALU kernel (cell_valu.h: kernels_cell_valu.hip for operators
// whose cells share one size, with the imaginary k term of complex
// operators in the same launch; kernels_cell_gen_*.hip for graded meshes and
// the GGA term) or, for bf16x3, the matrix-core kernel of
// kernels_cell_mfma.hip.
//
// k_cell_density is the adjoint contraction of the potential term: the
// band-energy density W_q sum_n occ_n |u_n(x_q)|^2 at the Gauss points of
// every cell (the dE/dV of the governing equations), with the columns
// interpolated to the points by the same three 1-D sweeps as the V term.

#include "cell_valu.h"

namespace pawfe {

// Band-energy density: dE/dV[e][q] = W_q sum_n occ_n |u_n(x_q)|^2, one
// workgroup per cell whose four waves share the column tiles.  A wave takes a
// tile as the cell operator does (cell_wave.h): planes interpolated in x and y
// in registers, z lines through its own LDS slab; the sum over its tiles stays
// in registers (every output has one lane per column of a tile), so the tiles
// need no barrier, and the waves add up in LDS once at the end.  Bound by the
// vector ALU and the latency of the gathers: 1728 cells of degree 6 x 256
// columns 0.32 ms; a workgroup per tile with a barrier per pass and two
// shuffles per point and tile took 1.80 ms.
template <int NP, int NQ>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) k_cell_density(DensArgs A) {
  using W = Wave<double, NP, NQ>;
  constexpr int H = W::H, CB = W::CB, G = W::G, RB = W::RB, QB = W::QB, NQX = W::NQX;
  constexpr int NQ2 = NQ * NQ, NQ3 = NQ2 * NQ, LS = NP * CB, ZR = (NQ2 + G - 1) / G;
  static_assert(W::slab >= NQ3, "the slab holds a wave's sums at the end");
  __shared__ double slabs[4][W::slab];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double* const sl = slabs[wave];
  const int col = lane % CB, slot = (lane / CB) % W::PS, g = lane / CB;
  const int h = H == 2 ? lane >> 5 : 0;
  const bool pl = slot < NP;
  const int c = pl ? slot : NP - 1;
  const int e = blockIdx.x;
  const int ci = e % A.n0, cj = (e / A.n0) % A.n1, ck = e / (A.n0 * A.n1);
  const int p = NP - 1;
  const int Gx = A.n0 * p, Gy = A.n1 * p, Gz = A.n2 * p;
  double* const pb = sl + W::plane_at(lane);
  double* const zb = sl + g * LS + col;
  double acc[ZR][NQ];
  sfor<ZR>([&](auto i) { sfor<NQ>([&](auto q) { acc[i][q] = 0.0; }); });
  for (int n0 = wave * CB; n0 < A.ncols; n0 += 4 * CB) {
    const int n = n0 + col;
    const bool valid = n < A.ncols;
    const double w = valid ? (A.occ ? A.occ[n] : 1.0) : 0.0;
    int gz = ck * p + c;
    gz = gz >= Gz ? gz - Gz : gz;
    double u[RB][NQX];
    sfor<RB>([&](auto r) {
      const int b = RB * h + r < NP ? RB * h + r : NP - 1;
      int gy = cj * p + b;
      gy = gy >= Gy ? gy - Gy : gy;
      const double* row = A.X + (valid ? n : 0) + (int64_t)(Gx * (gy + Gy * gz)) * A.ldx;
      double x[NP], y[NQ];
      sfor<NP>([&](auto a) {
        int gx = ci * p + a;
        gx = gx >= Gx ? gx - Gx : gx;
        x[a] = row[(int64_t)gx * A.ldx];
      });
      line_B<NP, NQ>(x, y);
      sfor<NQX>([&](auto q) { u[r][q] = q < NQ ? y[q < NQ ? (int)q : 0] : 0.0; });
      if constexpr (H == 2) sfor<QB>([&](auto j) { swap_halves(u[r][j], u[r][QB + j]); });
    });
    wave_lds_order();
    if (pl) {
      sfor<QB>([&](auto j) {   // qx = QB h + j
        double xc[NP], y[NQ];
        sfor<NP>([&](auto b) { xc[b] = u[b % RB][j + QB * (b / RB)]; });
        line_B<NP, NQ>(xc, y);
        if (H == 1 || NQX == NQ || QB * h + j < NQ) sfor<NQ>([&](auto q) { pb[(q * NQ + QB * h + j) * LS] = y[q]; });
      });
    }
    wave_lds_order();
    sfor<ZR>([&](auto i) {
      if (NQ2 % G == 0 || i < ZR - 1 || g + G * i < NQ2) {
        double m[NP], y[NQ];
        sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
        line_B<NP, NQ>(m, y);
        sfor<NQ>([&](auto q) { acc[i][q] = fma(w * y[q], y[q], acc[i][q]); });
      }
    });
  }
  // over the columns of a tile (neighbouring lanes), then over the waves
  wave_lds_order();
  sfor<ZR>([&](auto i) {
    sfor<NQ>([&](auto q) {
      double v = acc[i][q];
#pragma unroll
      for (int o = CB / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, CB);
      if (col == 0 && g + G * i < NQ2) sl[g + G * i + NQ2 * q] = v;
    });
  });
  __syncthreads();
  const double cs = A.cscale ? A.cscale[e] : 1.0;
  for (int q = threadIdx.x; q < NQ3; q += 256)
    A.out[(int64_t)e * NQ3 + q] = A.W3[q] * cs * ((slabs[0][q] + slabs[1][q]) + (slabs[2][q] + slabs[3][q]));
}

bool cell_step_available(const pawfe_op* op) {
  return op->nq == op->p + 2 && op->p >= 2 && op->p <= 6 && op->d.cell_own != nullptr &&
         (!op->general || (op->d.frho != nullptr && !op->cplx));
}

template <typename T>
pawfe_status launch_cell(const pawfe_op* op, int mode, const T* X, int64_t ldx, T* Y, int64_t ldy,
                         int ncols, const double* lam, double alpha, hipStream_t s, bool bf3, bool overwrite,
                         void* cellbuf) {
  if (ncols <= 0) return PAWFE_OK;
  if (bf3 && overwrite) return fail(PAWFE_EUNSUPPORTED, "internal: the matrix-core cell kernel adds to Y");
  if (bf3 && sizeof(T) != 4) return fail(PAWFE_EINVAL, "bf16x3 needs FP32 data");
  CellArgs<T> a{};
  a.bf3 = bf3 ? 1 : 0;
  a.X = X;
  a.ldx = ldx;
  a.Y = Y;
  a.ldy = ldy;
  a.ncols = ncols;
  a.Vw = std::is_same<T, double>::value ? (const T*)op->d.Vw : (const T*)op->d.Vw_f;
  a.W3 = std::is_same<T, double>::value ? (const T*)op->d.W3 : (const T*)op->d.W3_f;
  a.lam = lam;
  a.alpha = (T)alpha;
  a.n0 = op->n[0];
  a.n1 = op->n[1];
  a.n2 = op->n[2];
  a.own = overwrite ? op->d.cell_own : nullptr;
  a.cellbuf = bf3 ? nullptr : (T*)cellbuf;
  a.gathers = overwrite;
  a.by_op = mode == kModeHRes;
  if (op->general) {   // graded mesh / GGA term: every local term on the vector-ALU variants
    if (bf3) return fail(PAWFE_EUNSUPPORTED, "bf16x3 is not built for graded meshes or the GGA term");
    return launch_cell_gen<T>(op, mode, a, s);
  }
  pawfe_status st = PAWFE_OK;
  bool done = false;
  // K + V, the residual K + V - lambda M and the mass term in FP32 or FP64:
  // vector-ALU kernel (the matrix-core kernel keeps bf16x3)
  if ((mode == kModeH || mode == kModeHRes || mode == kModeMass) && !bf3) st = launch_cell_valu(op, mode, a, s, &done);
  if (st == PAWFE_OK && !done && overwrite) return fail(PAWFE_EUNSUPPORTED, "internal: no cell variant that overwrites Y");
  if (st == PAWFE_OK && !done) st = launch_cell_mfma<T>(op, mode, a, s);
  if (done) return st;   // the vector-ALU variants include the imaginary k term
  // complex operators on the matrix cores: the imaginary local term, on the
  // (re, im) column pairs, as a second launch
  if (st != PAWFE_OK || !op->cplx || (mode != kModeH && mode != kModeHRes)) return st;
  return launch_cell_mfma<T>(op, kModeImg, a, s);
}

// One launch per colour is latency (4-10 us each, 8 to 27 of them) until a
// colour holds several thousand cell columns; below that one launch of all
// cells and a gather pay.  K + V, launches per colour against launch and
// gather: degree 6, 64 cells in 8 colours, FP64 76 -> 27 us at 500 cell columns
// per colour, 118 -> 88 at 3,000; 512 cells 159 -> 149 at 4,500 and 197 -> 210
// at 7,000 (FP32 114 -> 94 and 129 -> 118); 125 cells in 27 colours FP32
// 235 -> 55 at 1,000; degree 2, 512 cells, FP64 41 -> 33 at 4,500 and 41 -> 45
// at 7,000.  The bytes bound the scratch (142 MB: 296 -> 208 us).
constexpr int64_t kCellBufCols = 4500, kCellBufBytes = int64_t(192) << 20;

// Y[I][n] = sum over the (up to eight) cells sharing DOF I of their results
// times their factors (CellFactor F), added one after another in the order of
// the cells' colours to 0 (KIND 0) or to Y (KIND 1): product by product what the
// launches per colour do, so applies and residuals have the same bits with and
// without room for this.  KIND 2, the filter's step: the cells' sum is added to
// the node part -a c X - zeta zeta' Y + a lamY_n Yres (the last product and sum
// in FP64, rounded once) at the end; one after another to the node part, as
// the launches per colour have to, FP32 filters are up to a tenth less accurate.
// CW lanes share a row (its cells are found once per lane and serve all of its
// columns); all loads are issued before the sum.
template <typename T, int KIND, int F, int P>
__global__ void __launch_bounds__(256) k_cell_gather(CellArgs<T> A, int cw_log, int M) {
  constexpr int NP = P + 1, NL = NP * NP * NP;
  const int CW = 1 << cw_log;
  const int I = (int)blockIdx.x * (256 >> cw_log) + (int)(threadIdx.x >> cw_log);
  if (I >= M) return;
  const int Gx = A.n0 * P, Gy = A.n1 * P;
  const int g[3] = {I % Gx, (I / Gx) % Gy, I / (Gx * Gy)}, nc[3] = {A.n0, A.n1, A.n2};
  const int cs[3] = {1, A.n0, A.n0 * A.n1}, qs[3] = {1, NP, NP * NP};
  // per axis the cells' shares of the cell index and of the row of the results
  int ce[3][2], row[3][2];
  bool two[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int c0 = g[d] / P, q0 = g[d] - c0 * P, c1 = c0 == 0 ? nc[d] - 1 : c0 - 1;
    two[d] = q0 == 0;                                     // also the last node of the cell before
    // the cell of the lower colour (i mod 2; the last of an odd direction 2)
    // first: the one before an odd cell and before the last of an odd direction
    const bool turn = two[d] && ((c0 & 1) || ((nc[d] & 1) && c0 == nc[d] - 1));
    const int e0 = cs[d] * c0, e1 = cs[d] * c1, r0 = e0 * NL + qs[d] * q0, r1 = e1 * NL + qs[d] * P;
    ce[d][0] = turn ? e1 : e0;
    ce[d][1] = turn ? e0 : e1;
    row[d][0] = turn ? r1 : r0;
    row[d][1] = turn ? r0 : r1;
  }
  uint32_t off[8];   // (kCellBufBytes: well inside 32 bits)
  bool on[8];
  T f[F == kByAlpha ? 1 : 8];
  if constexpr (F == kByAlpha) f[0] = A.alpha;
#pragma unroll
  for (int k = 0; k < 8; ++k) {   // ascending colours: z most significant
    const int i = k & 1, j = (k >> 1) & 1, l = k >> 2;
    on[k] = (!i || two[0]) && (!j || two[1]) && (!l || two[2]);
    off[k] = (uint32_t)(row[0][i] + row[1][j] + row[2][l]) * (uint32_t)A.ncols;
    if constexpr (F != kByAlpha) {
      const T dj = A.geo[4 * (ce[0][i] + ce[1][j] + ce[2][l]) + 3];
      f[k] = F == kByDetJ ? A.alpha / dj : A.alpha * dj;
    }
  }
  for (int n = threadIdx.x & (CW - 1); n < A.ncols; n += CW) {
    T v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = on[k] ? A.cellbuf[off[k] + n] : T(0);
    T* y = A.Y + (int64_t)I * A.ldy + n;
    T s = T(0), node = T(0);
    if constexpr (KIND == 1) s = *y;
    if constexpr (KIND == 2) {
      const T part = fma_t((T)(-A.sac), A.X[(int64_t)I * A.ldx + n], -((T)A.szz * *y));
      node = (T)fma(A.y64[(int64_t)I * A.ldy64 + n], A.sa * A.lamY[n], (double)part);
    }
    const T w = F == kByMass && A.lam ? (T)(-A.lam[n]) : T(1);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const T fk = F == kByAlpha ? f[0] : (F == kByMass ? f[k] * w : f[k]);
      s = fma_t(fk, v[k], s);   // (a cell that is not there adds zero)
    }
    *y = KIND == 2 ? node + s : s;
  }
}

size_t cell_buf_bytes(const pawfe_op* op, int64_t ncols, size_t elem) {
  if (op->nq != op->p + 2 || op->p < 2 || op->p > 6 || ncols <= 0) return 0;
  const int64_t bytes = (int64_t)op->E * op->nloc * ncols * (int64_t)elem;
  return (int64_t)op->E * ncols <= kCellBufCols * op->ncolour && bytes <= kCellBufBytes ? (size_t)bytes : 0;
}

size_t cell_buf_limit() { return (size_t)kCellBufBytes; }

// With another block's launches beside them the launches per colour wait for less,
// so the gather stops paying earlier.  Time of a filter of two blocks of degree
// 10 with the gather over that without (512 and 840 cells in 8 colours), by cell
// columns per colour:
//   degree 6, FP64 graded or GGA  0.98 at 1,500, 1.20 at 2,400; one size 1.01 at
//   2,400, 1.05 at 2,800; FP32 0.96 to 1.02 at 3,000, 1.20 at 4,000; complex FP32
//   0.94 at 3,400, 1.08 at 4,000, FP64 0.98 at 4,490
//   degree 5, FP64 graded 1.04 at 2,800, 1.18 at 3,600; the others 0.99 to 1.06 at
//   3,600, complex FP64 0.88 there and 1.21 at 4,490
//   degree 4 at most 0.98 at 4,490
// Meshes odd along two axes or three (18 or 27 colours) add small colours, launches
// that the gather saves besides: 504 cells in 18 colours degree 6 FP32 0.93 at
// 4,490, FP64 graded 0.94 at 3,000 and 1.02 at 4,000; 891 cells in 27 colours GGA
// FP32 9.2 -> 7.9 ms at 3,300.  Odd along one axis is not enough (924 cells in 12
// colours GGA FP32 9.4 -> 11.2 ms at 3,700).
bool cell_buf_pays_beside(const pawfe_op* op, int64_t ncols, size_t elem) {
  const bool f64 = elem == 8;
  int64_t cols = kCellBufCols;
  if (op->p == 6) cols = !f64 || op->cplx ? 3000 : (op->general ? 1800 : 2400);
  else if (op->p == 5) cols = f64 && op->general ? 2600 : 3400;
  if (op->ncolour >= 18) cols = std::min(cols * 3 / 2, kCellBufCols);
  return (int64_t)op->E * ncols <= cols * op->ncolour;
}

template <typename T>
pawfe_status launch_cell_gather(const pawfe_op* op, const CellArgs<T>& a, bool step, CellFactor fk, hipStream_t s) {
  if (!step && fk != kByMass && !a.own) return fail(PAWFE_EUNSUPPORTED, "internal: no gather that adds to Y");
  if (fk != kByAlpha && !a.geo) return fail(PAWFE_EINVAL, "internal: gather without geometry");
  int cw = 2;   // lanes per row: the columns, at most a wave
  while (cw < 6 && (1 << cw) < a.ncols) ++cw;
  const int rows = 256 >> cw;
  const dim3 grid((unsigned)((op->M + rows - 1) / rows)), block(256);
  auto go = [&](auto p) {
    constexpr int P = decltype(p)::value;
    if (step && fk == kByDetJ) hipLaunchKernelGGL((k_cell_gather<T, 2, kByDetJ, P>), grid, block, 0, s, a, cw, (int)op->M);
    else if (step) hipLaunchKernelGGL((k_cell_gather<T, 2, kByAlpha, P>), grid, block, 0, s, a, cw, (int)op->M);
    else if (fk == kByMass && a.own) hipLaunchKernelGGL((k_cell_gather<T, 0, kByMass, P>), grid, block, 0, s, a, cw, (int)op->M);
    else if (fk == kByMass) hipLaunchKernelGGL((k_cell_gather<T, 1, kByMass, P>), grid, block, 0, s, a, cw, (int)op->M);
    else hipLaunchKernelGGL((k_cell_gather<T, 0, kByAlpha, P>), grid, block, 0, s, a, cw, (int)op->M);
  };
  switch (op->p) {
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    default: return fail(PAWFE_EUNSUPPORTED, "degree not compiled");
  }
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}
template pawfe_status launch_cell_gather<double>(const pawfe_op*, const CellArgs<double>&, bool, CellFactor,
                                                 hipStream_t);
template pawfe_status launch_cell_gather<float>(const pawfe_op*, const CellArgs<float>&, bool, CellFactor, hipStream_t);

template pawfe_status launch_cell<double>(const pawfe_op*, int, const double*, int64_t, double*, int64_t,
                                          int, const double*, double, hipStream_t, bool, bool, void*);
template pawfe_status launch_cell<float>(const pawfe_op*, int, const float*, int64_t, float*, int64_t,
                                         int, const double*, double, hipStream_t, bool, bool, void*);

pawfe_status launch_density(const pawfe_op* op, const double* X, int64_t ldx, int ncols,
                            const double* occ, double* out, hipStream_t s) {
  if (op->nq != op->p + 2) return fail(PAWFE_EUNSUPPORTED, "nq must be p + 2");
  DensArgs a{};
  a.X = X;
  a.ldx = ldx;
  a.ncols = ncols;
  a.occ = occ;
  a.out = out;
  a.W3 = op->d.W3;
  a.cscale = op->d.cscale;
  a.n0 = op->n[0];
  a.n1 = op->n[1];
  a.n2 = op->n[2];
  const dim3 grid(op->E), block(256);
  switch (op->p) {
    case 2: hipLaunchKernelGGL((k_cell_density<3, 4>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((k_cell_density<4, 5>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((k_cell_density<5, 6>), grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL((k_cell_density<6, 7>), grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL((k_cell_density<7, 8>), grid, block, 0, s, a); break;
    default: return fail(PAWFE_EUNSUPPORTED, "degree not compiled");
  }
  PAWFE_HIP(hipGetLastError());
  return PAWFE_OK;
}

}  // namespace pawfe

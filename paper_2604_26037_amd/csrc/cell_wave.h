// Cell operators with one wavefront per item (a cell and one column tile):
// the same contractions, modes and arguments as cell_valu.h, split over the
// lanes by node planes instead of over a workgroup by lines.
//
// Lane (col, c, h) owns column `col` of the tile and the z plane c of the
// cell (FP64 elements of degree 5 and 6: the half h of that plane), so the x
// and y contractions run in registers with no exchange at all (FP64 halves
// trade rows for columns with v_permlane32_swap) and only the z contraction
// goes through LDS, in a slab that belongs to the wave: no barrier anywhere,
// a wave waits for its own memory operations only, and the waves of a CU
// drift apart so that one's loads and stores run under another's arithmetic.
//   V:  planes By Bx -> slab, lines Bz, V(q) W_q, Bz^T in place, planes By^T Bx^T
//   M:  planes My Mx -> slab, lines fz Kz (residual: - lambda det J Mz too)
//   K:  planes fx My Kx + fy Ky Mx -> slab, lines Mz, added to M's lines
//   complex operators, before M and K: the same two rounds with G1 for the
//   imaginary k term, read back from the partner column's place in the slab
// and the sum is added to Y (first visits of the step as in cell_valu.h), or
// stored by itself where a small residual gathers its cells' results.
// The gathered rows are wave-uniform for x and y, so their addresses are
// scalar; the lanes only carry the offset of their plane and column.
//
// Bound by the memory system and the vector ALU about equally (degree 6,
// 1000 cells x 256 columns a launch): FP32 step 1.53e9 B of HBM traffic (1.02x
// its algorithmic bytes) and 144,000 vector instructions per SIMD.  Per launch,
// against the workgroup kernel: step FP32 0.538 -> 0.390 ms (3.9 TB/s), FP64
// 0.988 -> 0.722; K + V FP32 0.436 -> 0.298, FP64 0.852 -> 0.586; mass FP32
// 0.411 -> 0.267, FP64 0.798 -> 0.504.
//
// Slab: element (line L, plane c, col) at (L NP + c) CB + col.  A plane
// access (L fixed) is contiguous; a line access strides by NP CB elements,
// 56 words at degree 6, which spreads the eight lines of a 32-lane half over
// all banks.

#pragma once

#include "cell_valu.h"

namespace pawfe {

namespace {

// Modes with a one-wave variant that stores each cell's result by itself
// (CellArgs::cellbuf): those of the residual, which is FP64.
template <typename T>
constexpr bool is_wave_buf_mode(int mode) {
  return sizeof(T) == 8 && (mode == kValuHRes || mode == kValuHResC || mode == kValuGenH || mode == kValuGenMass);
}

template <typename T, int NP, int NQ>
struct Wave {
  static constexpr int H = (sizeof(T) == 8 && NP >= 6) ? 2 : 1;   // halves of a plane
  static constexpr int PS = NP <= 4 ? 4 : 8;                      // plane slots
  static constexpr int CB = 64 / (PS * H);                        // columns per item
  static constexpr int G = PS * H;                                // line groups of the z passes
  static constexpr int RB = (NP + H - 1) / H;                     // rows (or columns) of a half plane
  static constexpr int QB = (NQ + H - 1) / H;                     // Gauss columns of a half plane
  static constexpr int NPX = RB * H, NQX = QB * H;
  static constexpr int slab = NQ * NQ * NP * CB;
  // slab element of line 0 in a lane's plane (lanes past the last plane: the
  // last one, which they may read; line L adds L NP CB)
  static constexpr __host__ __device__ int plane_at(int lane) {
    const int s = (lane / CB) % PS;
    return (s < NP ? s : NP - 1) * CB + lane % CB;
  }
};
// Waves (neighbouring column tiles of one cell) per workgroup.  The mass term,
// which is all memory, takes four: they read the same 128-byte lines through
// one L1 (0.292 -> 0.264 ms FP32, 0.574 -> 0.507 FP64).  The others lose more
// by starting and ending together (K + V 0.299 -> 0.320, step 0.392 -> 0.438).
template <int MODE>
constexpr int kWaveTiles = (MODE == kValuMass || MODE == kValuGenMass) ? 4 : 1;

// order a wave's own LDS accesses (they execute in order; this keeps the
// compiler from moving them across)
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// a value the compiler cannot look through: what is computed from it is
// computed after this point
template <typename T>
__device__ __forceinline__ void opaque(T& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void opaque_s(uint64_t& v) { asm volatile("" : "+s"(v)); }

// upper 32 lanes of `lo` <-> lower 32 lanes of `hi`
template <typename T>
__device__ __forceinline__ void swap_halves(T& lo, T& hi) {
  constexpr int W = sizeof(T) / 4;
  unsigned a[W], b[W];
  __builtin_memcpy(a, &lo, sizeof(T));
  __builtin_memcpy(b, &hi, sizeof(T));
#pragma unroll
  for (int i = 0; i < W; ++i) {
    auto r = __builtin_amdgcn_permlane32_swap(a[i], b[i], false, false);
    a[i] = r[0];
    b[i] = r[1];
  }
  __builtin_memcpy(&lo, a, sizeof(T));
  __builtin_memcpy(&hi, b, sizeof(T));
}

}  // namespace

// BUF: each cell's result is stored in A.cellbuf (a variant of its own: as a
// test at run time it made the complex residual spill)
template <typename T, int NP, int NQ, int MODE, bool BUF>
__global__ void __launch_bounds__(64 * kWaveTiles<MODE>) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_cell_wave(CellArgs<T> A, int ncoltiles, int nitems, T fx, T fy, T fz) {
  using W = Wave<T, NP, NQ>;
  constexpr int H = W::H, CB = W::CB, G = W::G, RB = W::RB, QB = W::QB, NPX = W::NPX, NQX = W::NQX;
  constexpr bool GEN = is_general_mode(MODE);
  constexpr bool MASS = MODE == kValuGenMass || MODE == kValuMass;
  constexpr bool RES = MODE == kValuHRes || MODE == kValuHResC;
  constexpr bool STEP = MODE == kValuStep || MODE == kValuGenStep || MODE == kValuStepC;
  constexpr bool CPLX = MODE == kValuHC || MODE == kValuHResC || MODE == kValuStepC;
  constexpr bool SC = STEP;
  constexpr int NQ2 = NQ * NQ, NP2 = NP * NP, NQ3 = NQ * NQ * NQ;
  constexpr int WT = kWaveTiles<MODE>;
  static_assert(MASS || WT == 1, "V(q) W_q is staged by one wave");
  __shared__ T slabs[WT][W::slab];
  __shared__ T sv[MASS ? 1 : NQ3];
  const int lane = threadIdx.x & 63;
  const int wave = WT == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  T* const sl = slabs[wave];
  const int col = lane % CB;
  const int slot = (lane / CB) % W::PS;
  const int h = H == 2 ? lane >> 5 : 0;
  const int g = lane / CB;                     // line group
  const bool pl = slot < NP;                   // the lane's plane exists
  const int c = pl ? slot : NP - 1;
  const int p = NP - 1;
  const int Gx = A.n0 * p, Gy = A.n1 * p, Gz = A.n2 * p;
  const uint32_t ldxb = (uint32_t)(A.ldx * (int64_t)sizeof(T)), ldyb = (uint32_t)(A.ldy * (int64_t)sizeof(T));
  const uint64_t ld64b = STEP ? (uint64_t)A.ldy64 * 8 : 0;
  typedef const __attribute__((address_space(4))) int* ConstIntP;
  const ConstIntP cells = (ConstIntP)A.cells;
  const int xcd = blockIdx.x & 7;
  const int i_end = (int)((int64_t)nitems * (xcd + 1) / 8);
  const int item = (int)((int64_t)nitems * xcd / 8) + (int)(blockIdx.x >> 3);
  if (item >= i_end) return;
  const int cc = item / ncoltiles;
  const int packed = cells[cc];
  const int ci = packed & 1023, cj = (packed >> 10) & 1023, ck = (packed >> 20) & 1023;
  const int e = ci + A.n0 * (cj + A.n1 * ck);
  const int tile = (item - cc * ncoltiles) * WT + wave;
  if (WT > 1 && tile * CB >= A.ncols) return;   // wave-uniform
  const int n = tile * CB + col;
  const bool valid = n < A.ncols;
  const int nn = valid ? n : 0;
  const bool lastx = ci + 1 == A.n0;
  // rows of the lane's half plane: b = RB h + r (past the last: the last row)
  auto row_class = [&](int r) { const int b = RB * h + r; return b == 0 ? 0 : (b >= NP - 1 ? 6 : 3); };
  auto lrow = [&](int r) { const int b = RB * h + r; return b < NP ? b : NP - 1; };

  // byte offsets of the cell's node columns in an array (scalar; opaque, so
  // that they are not folded into a 64-bit vector multiply per access)
  auto xoffs = [&](uint64_t ldb, uint64_t(&o)[NP]) {
    sfor<NP>([&](auto a) {
      o[a] = (uint64_t)(a == NP - 1 && lastx ? 0 : ci * p + a) * ldb;
      opaque_s(o[a]);
    });
  };
  // the lane's plane of array `base` (`ldb` bytes per row): its pointer is
  // formed for each use rather than held in registers
  auto planeptr = [&](auto* base, uint64_t ldb) {
    using P = decltype(base);
    using C = typename std::conditional<std::is_const<typename std::remove_pointer<P>::type>::value, const char,
                                        char>::type;
    int gz = ck * p + c;
    opaque(gz);
    gz = gz >= Gz ? gz - Gz : gz;
    return reinterpret_cast<C*>(base + nn) + (uint64_t)(uint32_t)(gz * (Gx * Gy)) * (uint32_t)ldb;
  };
  // its row r, without the node column; scalar steps except where the halves
  // of a plane (rows r and RB + r) may wrap differently
  auto rowptr = [&](auto* plane, uint64_t ldb, int r) {
    if (H == 1 || r < NP - 1 - RB) {
      int gy = cj * p + r;
      gy = H == 1 && gy >= Gy ? gy - Gy : gy;
      plane += (uint64_t)(uint32_t)(gy * Gx) * (uint32_t)ldb;
      if (H == 2) plane += h ? (uint64_t)(uint32_t)(RB * Gx) * (uint32_t)ldb : 0;
      return plane;
    }
    int gy = cj * p + lrow(r);
    gy = gy >= Gy ? gy - Gy : gy;
    return plane + (uint64_t)(uint32_t)(gy * Gx) * (uint32_t)ldb;
  };

  T x[RB][NP];
  uint64_t xo[NP];
  xoffs(ldxb, xo);
  const char* xp = planeptr(A.X, ldxb);
  sfor<RB>([&](auto r) {
    const char* q = rowptr(xp, ldxb, r);
    sfor<NP>([&](auto a) { x[r][a] = *(const T*)(q + xo[a]); });
  });
  // the factor of the result goes into V(q) W_q and the kinetic factors
  T f = A.alpha, ifx = fx, ify = fy, ifz = fz, idet = A.detJ;
  if constexpr (GEN) {
    typedef const __attribute__((address_space(4))) T* ConstTP;
    const ConstTP gg = (ConstTP)A.geo + 4 * e;
    ifx = gg[0];
    ify = gg[1];
    ifz = gg[2];
    idet = gg[3];
  }
  if constexpr (STEP && GEN) f = f / idet;   // the cell's det J of M_D^{-1}
  if constexpr (MASS) f = f * idet * ((MODE == kValuGenMass && A.lam) ? (T)(-A.lam[nn]) : T(1));
  ifx *= f;
  ify *= f;
  ifz *= f;
  if constexpr (!MASS) {
    constexpr int NV = (NQ3 + 63) / 64;
    T v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (NQ3 % 64 == 0 || lane + 64 * i < NQ3) v[i] = A.Vw[(int64_t)e * NQ3 + lane + 64 * i];
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (NQ3 % 64 == 0 || lane + 64 * i < NQ3) sv[lane + 64 * i] = f * v[i];
  }
  // general step: face factors of the lumped mass (see cell_valu.h), applied
  // to a copy of each row on its way into the contractions
  T rf[STEP && GEN ? 4 : 1], rz = T(1);
  if constexpr (STEP && GEN) {
    typedef const __attribute__((address_space(4))) T* ConstTP;
    const ConstTP q = (ConstTP)A.frho + 6 * e;
#pragma unroll
    for (int k = 0; k < 4; ++k) rf[k] = q[k];
    const T z0 = q[4], z1 = q[5];
    rz = c == 0 ? z0 : (c == NP - 1 ? z1 : T(1));
  }
  auto row = [&](auto r, T(&o)[NP]) {
    sfor<NP>([&](auto a) { o[a] = x[r][a]; });
    if constexpr (STEP && GEN) {
      const int b = RB * h + r;
      const T f = rz * (b == 0 ? rf[2] : (b == NP - 1 ? rf[3] : T(1)));
      sfor<NP>([&](auto a) { o[a] *= a == 0 ? f * rf[0] : (a == NP - 1 ? f * rf[1] : f); });
    }
  };

  // slab addresses
  T* const pb = sl + W::plane_at(lane);                      // plane accesses: + line * NP CB
  T* const zb = sl + g * NP * CB + col;                      // line accesses: + round * G NP CB + plane * CB
  constexpr int LS = NP * CB;

  T acc[RB][NP];
  // ---- V term ------------------------------------------------------------
  if constexpr (!MASS) {
    T u[RB][NQX];
    sfor<RB>([&](auto r) {
      T xr[NP], y[NQ];
      row(r, xr);
      line_B<NP, NQ, SC>(xr, y);
      sfor<NQX>([&](auto q) { u[r][q] = q < NQ ? y[q < NQ ? (int)q : 0] : T(0); });
      if constexpr (H == 2) sfor<QB>([&](auto j) { swap_halves(u[r][j], u[r][QB + j]); });
    });
    wave_lds_order();
    if (pl) {
      sfor<QB>([&](auto j) {   // qx = QB h + j
        T xc[NP], y[NQ];
        sfor<NP>([&](auto b) { xc[b] = u[b % RB][j + QB * (b / RB)]; });
        line_B<NP, NQ, SC>(xc, y);
        if (H == 1 || NQX == NQ || QB * h + j < NQ)
          sfor<NQ>([&](auto q) { pb[(q * NQ + QB * h + j) * LS] = y[q]; });
      });
    }
    wave_lds_order();
    constexpr int ZR = (NQ2 + G - 1) / G;
    sfor<ZR>([&](auto i) {
      if (NQ2 % G == 0 || i < ZR - 1 || g + G * i < NQ2) {
        T m[NP], y[NQ], o[NP];
        sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
        line_B<NP, NQ, SC>(m, y);
        sfor<NQ>([&](auto q) { y[q] *= sv[g + G * i + NQ2 * q]; });
        line_Bt<NP, NQ>(y, o);
        sfor<NP>([&](auto k) { zb[(i * G * NP + k) * CB] = o[k]; });
      }
    });
    wave_lds_order();
    T w[NPX][QB];
    sfor<QB>([&](auto j) {
      T y[NQ], o[NP];
      const int qx = (H == 1 || NQX == NQ) ? QB * h + j : (QB * h + j < NQ ? QB * h + j : NQ - 1);
      sfor<NQ>([&](auto q) { y[q] = pb[(q * NQ + qx) * LS]; });
      line_Bt<NP, NQ>(y, o);
      sfor<NPX>([&](auto b) { w[b][j] = b < NP ? o[b < NP ? (int)b : 0] : T(0); });
    });
    sfor<RB>([&](auto r) {
      if constexpr (H == 2) sfor<QB>([&](auto j) { swap_halves(w[r][j], w[(int)r + RB < NPX ? (int)r + RB : 0][j]); });
      T y[NQ], o[NP];
      sfor<NQ>([&](auto q) { y[q] = w[r + RB * (q / QB)][q % QB]; });
      line_Bt<NP, NQ>(y, o);
      sfor<NP>([&](auto a) { acc[r][a] = o[a]; });
    });
  }
  // first visits of the lane's nodes, by their 9 (x, y) classes (none where
  // the result is added to what Y holds)
  unsigned cm = 0;
  if (STEP || A.own) {
    typedef const __attribute__((address_space(4))) unsigned* ConstUP;
    cm = ((ConstUP)A.own)[e] >> (c == 0 ? 0 : (c == NP - 1 ? 18 : 9));
  }
  // step: the rows' part of the node update, -a c R_Y' at first visits.  FP32
  // adds it to the whole local sum at the end: added here, between the V and
  // the K terms, it costs a filter of degree 20 up to 12 % in accuracy (degree 6
  // complex 4.79e-7 -> 5.38e-7 from the workgroup kernel's order, 4.50e-7 at
  // the end).  FP64 has no registers left to carry x that far (5.76 -> 6.44 ms
  // on 8000 cells x 256 columns) and shows no difference.
  constexpr bool kLateX = STEP && sizeof(T) == 4;
  auto add_x = [&](auto r) {
    const T mac = (T)(-A.sac);
    const unsigned cr = cm >> row_class(r);
    const T m0 = cr & 1u ? mac : T(0), m1 = cr & 2u ? mac : T(0), m2 = cr & 4u ? mac : T(0);
    sfor<NP>([&](auto a) {
      acc[r][a] = fma_t(a == 0 ? m0 : (a == NP - 1 ? m2 : m1), x[r][a], acc[r][a]);
      if constexpr (!kLateX) opaque(acc[r][a]);
    });
  };
  if constexpr (STEP) {
    sfor<RB>([&](auto r) {
      // opaque: products of x are formed here or at the end, not kept beside
      // it from the load on, and the sums not left until the end
      sfor<NP>([&](auto a) { opaque(x[r][a]); });
      if constexpr (kLateX) sfor<NP>([&](auto a) { opaque(acc[r][a]); });
      else add_x(r);
    });
  }
  constexpr int ZK = (NP2 + G - 1) / G;
  // ---- complex: the imaginary k term, added to the partner column ----------
  if constexpr (CPLX) {
    T gx[RB][NPX], mx[RB][NPX];
    sfor<RB>([&](auto r) {
      T xr[NP], y[NP];
      row(r, xr);
      const EOIn<NP, T> eo = split_eo<NP>(xr);
      line_sym<NP, NQ, false, SC>(eo, y);
      sfor<NPX>([&](auto a) { mx[r][a] = a < NP ? y[a < NP ? (int)a : 0] : T(0); });
      line_g1<NP, NQ, SC>(eo, y);
      sfor<NPX>([&](auto a) { gx[r][a] = a < NP ? y[a < NP ? (int)a : 0] : T(0); });
      if constexpr (H == 2) sfor<RB>([&](auto j) {
        swap_halves(mx[r][j], mx[r][RB + j]);
        swap_halves(gx[r][j], gx[r][RB + j]);
      });
    });
    const T g0 = f * A.gk[0], g1 = f * A.gk[1], g2 = f * A.gk[2];
    wave_lds_order();
    // columns: My Mx -> slab, gx My G1x + gy G1y Mx stays in gx
    if (pl) {
      sfor<RB>([&](auto j) {
        T mc[NP], gc[NP], y[NP], z[NP];
        sfor<NP>([&](auto b) {
          mc[b] = mx[b % RB][j + RB * (b / RB)];
          gc[b] = gx[b % RB][j + RB * (b / RB)];
        });
        const EOIn<NP, T> em = split_eo<NP>(mc);
        line_sym<NP, NQ, false, SC>(em, y);
        if (H == 1 || NPX == NP || RB * h + j < NP) sfor<NP>([&](auto b) { pb[(b * NP + RB * h + j) * LS] = y[b]; });
        line_sym<NP, NQ, false, SC>(split_eo<NP>(gc), z);
        line_g1<NP, NQ, SC>(em, y);
        sfor<NP>([&](auto b) { gx[b % RB][j + RB * (b / RB)] = fma_t(g0, z[b], g1 * y[b]); });
      });
    }
    wave_lds_order();
    T il[ZK][NP];
    sfor<ZK>([&](auto i) {
      if (NP2 % G == 0 || i < ZK - 1 || g + G * i < NP2) {
        T m[NP], y[NP];
        sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
        line_g1<NP, NQ, SC>(split_eo<NP>(m), y);
        sfor<NP>([&](auto k) { il[i][k] = g2 * y[k]; });
      }
    });
    wave_lds_order();
    if (pl) {
      sfor<RB>([&](auto j) {
        if (H == 1 || NPX == NP || RB * h + j < NP)
          sfor<NP>([&](auto b) { pb[(b * NP + RB * h + j) * LS] = gx[b % RB][j + RB * (b / RB)]; });
      });
    }
    wave_lds_order();
    sfor<ZK>([&](auto i) {
      if (NP2 % G == 0 || i < ZK - 1 || g + G * i < NP2) {
        T m[NP], y[NP];
        sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
        line_sym<NP, NQ, false, SC>(split_eo<NP>(m), y);
        sfor<NP>([&](auto k) { zb[(i * G * NP + k) * CB] = y[k] + il[i][k]; });
      }
    });
    wave_lds_order();
    // s_n = -1 on real, +1 on imaginary columns, of the partner column's term
    const T sg = (col & 1) ? T(1) : T(-1);
    const T* const pp = pb + ((col & 1) ? -1 : 1);
    sfor<RB>([&](auto r) {
      const int b = lrow(r);
      sfor<NP>([&](auto a) {
        acc[r][a] = fma_t(sg, pp[(b * NP + a) * LS], acc[r][a]);
        opaque(acc[r][a]);
        opaque(x[r][a]);
      });
    });
  }
  // ---- M and K terms -----------------------------------------------------
  T mx[RB][NPX], kx[MASS ? 1 : RB][NPX];
  sfor<RB>([&](auto r) {
    T xr[NP], y[NP];
    row(r, xr);
    const EOIn<NP, T> eo = split_eo<NP>(xr);
    line_sym<NP, NQ, false, SC>(eo, y);
    sfor<NPX>([&](auto a) { mx[r][a] = a < NP ? y[a < NP ? (int)a : 0] : T(0); });
    if constexpr (!MASS) {
      line_sym<NP, NQ, true, SC>(eo, y);
      sfor<NPX>([&](auto a) { kx[r][a] = a < NP ? y[a < NP ? (int)a : 0] : T(0); });
    }
    if constexpr (H == 2) sfor<RB>([&](auto j) {
      swap_halves(mx[r][j], mx[r][RB + j]);
      if constexpr (!MASS) swap_halves(kx[r][j], kx[r][RB + j]);
    });
  });
  wave_lds_order();
  // columns a = RB h + j: M -> slab, fx My K + fy Ky M stays in kx
  if (pl) {
    sfor<RB>([&](auto j) {
      T mc[NP], y[NP];
      sfor<NP>([&](auto b) { mc[b] = mx[b % RB][j + RB * (b / RB)]; });
      const EOIn<NP, T> em = split_eo<NP>(mc);
      line_sym<NP, NQ, false, SC>(em, y);
      const bool on = H == 1 || NPX == NP || RB * h + j < NP;
      if (on) sfor<NP>([&](auto b) { pb[(b * NP + RB * h + j) * LS] = y[b]; });
      if constexpr (!MASS) {
        T kc[NP], mk[NP];
        sfor<NP>([&](auto b) { kc[b] = kx[b % RB][j + RB * (b / RB)]; });
        line_sym<NP, NQ, false, SC>(split_eo<NP>(kc), mk);
        line_sym<NP, NQ, true, SC>(em, y);
        sfor<NP>([&](auto b) { kx[b % RB][j + RB * (b / RB)] = fma_t(ifx, mk[b], ify * y[b]); });
      }
    });
  }
  wave_lds_order();
  T zl[MASS ? 1 : ZK][NP];
  const T ml = RES ? -(T)A.lam[nn] * idet * f : T(0);
  sfor<ZK>([&](auto i) {
    if (NP2 % G == 0 || i < ZK - 1 || g + G * i < NP2) {
      T m[NP], y[NP];
      sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
      const EOIn<NP, T> em = split_eo<NP>(m);
      if constexpr (MASS) {
        line_sym<NP, NQ, false, SC>(em, y);
        sfor<NP>([&](auto k) { zb[(i * G * NP + k) * CB] = y[k]; });
      } else {
        line_sym<NP, NQ, true, SC>(em, y);
        sfor<NP>([&](auto k) { zl[i][k] = ifz * y[k]; });
        if constexpr (RES) {
          line_sym<NP, NQ, false, SC>(em, y);
          sfor<NP>([&](auto k) { zl[i][k] = fma_t(ml, y[k], zl[i][k]); });
        }
      }
    }
  });
  if constexpr (!MASS) {
    wave_lds_order();
    if (pl) {
      sfor<RB>([&](auto j) {
        if (H == 1 || NPX == NP || RB * h + j < NP)
          sfor<NP>([&](auto b) { pb[(b * NP + RB * h + j) * LS] = kx[b % RB][j + RB * (b / RB)]; });
      });
    }
    wave_lds_order();
  }
  // old rows (except at a first visit that overwrites them) and, of the step,
  // the first FP64 residual rows: requested here, used after the last z pass
  opaque(cm);
  T yo[RB][NP];
  xoffs(ldyb, xo);
  const char* yp = planeptr((const T*)A.Y, ldyb);
  sfor<RB>([&](auto r) {
    const char* q = rowptr(yp, ldyb, r);
    auto get = [&](auto a) { yo[r][a] = *(const T*)(q + xo[a]); };
    if constexpr (STEP) {
      sfor<NP>(get);
    } else {
      const unsigned cr = BUF ? ~0u : cm >> row_class(r);   // (BUF: nothing is added to)
      sfor<NP>([&](auto a) { yo[r][a] = T(0); });
      if (!(cr & 1u)) get(std::integral_constant<int, 0>{});
      if (!(cr & 2u)) sfor<NP - 2>([&](auto a) { get(std::integral_constant<int, a + 1>{}); });
      if (!(cr & 4u)) get(std::integral_constant<int, NP - 1>{});
    }
  });
  uint64_t x64[STEP ? NP : 1];
  if constexpr (STEP) xoffs(ld64b, x64);
  const char* y6 = STEP ? planeptr(A.y64, ld64b) : nullptr;
  double yr[STEP ? RB : 1][NP];   // set at first visits only
  // f(a) at the row's first visits, position class by position class
  auto first_visits = [&](auto r, auto&& f) {
    const unsigned cr = cm >> row_class(r);
    if (cr & 1u) f(std::integral_constant<int, 0>{});
    if (cr & 2u) sfor<NP - 2>([&](auto a) { f(std::integral_constant<int, a + 1>{}); });
    if (cr & 4u) f(std::integral_constant<int, NP - 1>{});
  };
  auto load_y = [&](auto r) {
    const char* q = rowptr(y6, ld64b, r);
    first_visits(r, [&](auto a) { yr[r][a] = *(const double*)(q + x64[a]); });
  };
  // rows ahead, as many as fit the registers (degree 6 FP32, 8000 cells x 256
  // columns: 3.10 ms with none, 3.12 with one, 3.43 and spills with two; complex
  // 1.91, 1.88 and 1.98 on 4096 cells; degree 5 1.12, 1.09 and 1.06 ms)
  constexpr int kAhead = sizeof(T) == 8 || (NP == 7 && CPLX) ? 1 : (NP == 7 ? 0 : 2);
  if constexpr (STEP) sfor<kAhead>([&](auto r) { load_y(r); });
  if constexpr (!MASS) {
    sfor<ZK>([&](auto i) {
      if (NP2 % G == 0 || i < ZK - 1 || g + G * i < NP2) {
        T m[NP], y[NP];
        sfor<NP>([&](auto k) { m[k] = zb[(i * G * NP + k) * CB]; });
        line_sym<NP, NQ, false, SC>(split_eo<NP>(m), y);
        sfor<NP>([&](auto k) { zb[(i * G * NP + k) * CB] = y[k] + zl[i][k]; });
      }
    });
  }
  wave_lds_order();
  sfor<RB>([&](auto r) {
    const int b = lrow(r);
    sfor<NP>([&](auto a) {
      const T k = pb[(b * NP + a) * LS];
      if constexpr (MASS) acc[r][a] = k; else acc[r][a] += k;
    });
    if constexpr (kLateX) add_x(r);
  });
  // ---- assembly ----------------------------------------------------------
  const double ly = STEP ? A.sa * A.lamY[nn] : 0.0;
  const T zz = STEP ? (T)A.szz : T(0);
  // every load before the first store: a load waits for the stores issued
  // before it (one counter, in order), which cost the step a round trip per row
  sfor<RB>([&](auto r) {
    if constexpr (STEP) {
      if constexpr (r + kAhead < RB) load_y(std::integral_constant<int, (r + kAhead < RB ? r + kAhead : 0)>{});
      first_visits(r, [&](auto a) { yo[r][a] = (T)((double)(-zz * yo[r][a]) + yr[r][a] * ly); });
    }
    if constexpr (BUF) sfor<NP>([&](auto a) { yo[r][a] = acc[r][a]; });
    else sfor<NP>([&](auto a) { yo[r][a] = MASS ? fma_t(f, acc[r][a], yo[r][a]) : yo[r][a] + acc[r][a]; });
  });
  if constexpr (BUF) {
    if (pl && valid) {
      T* out = A.cellbuf + (int64_t)e * (NP * NP * NP) * A.ncols + n;
      sfor<RB>([&](auto r) {
        const int b = RB * h + r;
        if (H == 1 || NPX == NP || b < NP)
          sfor<NP>([&](auto a) { out[(int64_t)(a + NP * (b + NP * c)) * A.ncols] = yo[r][a]; });
      });
    }
  } else if (pl && valid) {
    char* yw = planeptr(A.Y, ldyb);
    sfor<RB>([&](auto r) {
      if (H == 1 || NPX == NP || RB * h + r < NP) {
        char* q = rowptr(yw, ldyb, r);
        sfor<NP>([&](auto a) { *(T*)(q + xo[a]) = yo[r][a]; });
      }
    });
  }
}

namespace {

// Modes that have a one-wave variant.
constexpr bool is_wave_mode(int mode) {
  return mode == kValuH || mode == kValuHRes || mode == kValuMass || mode == kValuStep || mode == kValuGenH ||
         mode == kValuGenMass || mode == kValuGenStep || mode == kValuHC || mode == kValuHResC || mode == kValuStepC;
}

// Where the one-wave split pays.  An item takes one wave longer than it takes a
// workgroup, so a launch has to hold enough items to fill the chip: two waves on
// each of 1024 SIMDs run at once, and a last round of them that is nearly empty
// costs as much as a full one.  One-wave over workgroup time per launch, by the
// rounds of a launch (512 cells in 8 colours, step / K + V):
//   rounds             0.5       0.75      1.0       1.12      1.5       2.12      3.12
//   degree 6 FP32    1.11/1.15 0.97/0.89 0.92/0.88 1.22/1.12 0.96/0.95 1.00/1.00 0.94/0.92
//   degree 5 FP32    1.13/1.17 0.91/0.90 0.99/0.95 1.21/1.12 1.04/0.94 1.11/1.02 1.00/0.93
//   degree 4 FP32    1.12/1.16 0.86/0.87 0.91/0.88 1.09/1.09 0.93/0.92 1.10/0.99 1.00/0.89
//   6, complex FP32  1.20/1.23 1.03/0.94 0.97/0.89 1.30/1.25 1.02/1.05 1.07/1.05 0.95/0.94
//   5, complex FP32  1.13/1.17 0.90/0.91 0.84/0.85 1.23/1.18 0.97/0.94 1.02/1.01 0.93/0.92
//   4, complex FP32  1.07/1.11 0.84/0.87 0.78/0.79 1.12/1.12 0.87/0.88 0.99/0.93 0.90/0.85
//   6, complex FP64  1.04/1.01 0.99/1.01 0.91/0.89 1.12/1.09 0.91/0.96 0.96/1.00 0.90/0.94
// so there the rounds decide, as the share of them that is filled: from 0.72 on,
// from 0.9 on at degree 6 complex FP32 (1.05 at 0.88 rounds, 0.99 at 1.88), and
// always from three rounds on.  The others gain more than a round can cost and go
// by cell columns (cells x columns): degree 3 FP32 even at 8,000 (0.95), FP64
// at 4,000 (0.87); degree 2 FP32 at any size (0.82 at 4,000), FP64 at 4,000
// (0.74); degree 6 FP64 0.97/0.84 at 6,100 and at most 0.99 from there, degree 5
// 0.92/0.89 at 4,100, degree 4 0.89/0.92; complex FP64 degree 5 0.87/0.81 at
// 4,100, degree 4 0.96/0.90, degree 3 0.89/0.96.  The mass term is too short to
// lose: 5.2 -> 4.7 us at 128 cell columns.
constexpr double kWavesAtOnce = 2048.0;
// Decided launch by launch: an odd mesh has colours of very different sizes (11
// x 13 x 8 cells: 120, 24, 20 and 4).
template <typename T, int NP, int MODE>
bool wave_pays(double ncells, int ncols) {
  if (MODE == kValuMass || MODE == kValuGenMass) return true;
  constexpr bool kCplx = MODE == kValuHC || MODE == kValuHResC || MODE == kValuStepC;
  constexpr bool f32 = sizeof(T) == 4;
  if ((f32 && NP >= 5) || (kCplx && NP == 7)) {
    constexpr int CB = Wave<T, NP, NP + 1>::CB;
    const double rounds = ncells * ((ncols + CB - 1) / CB) / kWavesAtOnce;
    return rounds >= 3.0 || rounds >= (f32 && kCplx && NP == 7 ? 0.9 : 0.72) * std::ceil(rounds);
  }
  return ncells * ncols >= (f32 ? (NP == 3 ? 0 : 7000) : (NP == 3 ? 3000 : NP == 4 || kCplx ? 4000 : 8000));
}

template <typename T, int NP, int NQ, int MODE, bool BUF = false>
void launch_wave(const CellArgs<T>& a, int ncells, T fx, T fy, T fz, hipStream_t s) {
  constexpr int CB = Wave<T, NP, NQ>::CB;
  constexpr int WT = kWaveTiles<MODE>;
  const int ncoltiles = (a.ncols + CB * WT - 1) / (CB * WT);
  // one item per workgroup of one wave, XCD x takes the x-th eighth of the
  // items (workgroup w runs on XCD w % 8).  A resident set that strides over
  // the items was slower (degree-6 K + V of 1000 cells x 256 columns, FP32:
  // 0.39 against 0.30 ms)
  const int nitems = ncells * ncoltiles;
  hipLaunchKernelGGL((k_cell_wave<T, NP, NQ, MODE, BUF>), dim3((unsigned)((nitems + 7) / 8) * 8), dim3(64 * WT), 0, s, a,
                     ncoltiles, nitems, fx, fy, fz);
}

}  // namespace

}  // namespace pawfe

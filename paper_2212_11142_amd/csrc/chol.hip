// fp64 blocked Cholesky for the model fit, with triangular solves and L^-T carried as
// extra rows of the factorisation.
//
// Right-looking Cholesky on NB x NB blocks (NB = 32) with one launch per block column:
//   * chol_panel factors the first diagonal block;
//   * chol_trailing(k) computes the panel L_ik = A_ik D_k^T (D_k = L_kk^-1, so the
//     triangular solve is a GEMM), subtracts L_ik L_jk^T from every trailing block
//     (i >= j), and the workgroup owning block (k+1, k+1) factors it right away, so
//     the next launch already has L_{k+1,k+1} and D_{k+1}.
// Each diagonal factorisation also produces its inverse D_k, with which the panels are
// GEMMs. Optional extra rows E stored below A (rows n.., columns 0..n-1)
// are carried through the same right-looking updates; their final panels form
// L_E = E L^-T, i.e. L_E^T = L^-1 E^T, the forward solve of L against every column of
// E^T, at the cost of parallel workgroups beside the critical one. The last n_ident
// extra rows may be an identity block (L_E = L^-T there): its block row e stays zero
// until step e, so its workgroups start at that step.
// A device int `info` records the first failing pivot (1-based, global row); every
// kernel returns immediately once it is set.
#include <algorithm>

#include "common.h"

namespace bgp {
namespace {

constexpr int NB = kNB;      // factorisation block
constexpr int LP = NB + 1;   // LDS row stride (doubles)
constexpr int kPer = NB * NB / 256;  // elements of a block per thread
static_assert(NB * NB % 256 == 0, "block elements per thread");
static_assert(NB == 32, "the block factorisation works on 2 x 2 tiles of 16");

__device__ __forceinline__ void tri_index(int L, int &bi, int &bj) {
  int i = (int)((sqrt(8.0 * L + 1.0) - 1.0) * 0.5);
  while ((i + 1) * (i + 2) / 2 <= L) ++i;
  while (i * (i + 1) / 2 > L) --i;
  bi = i;
  bj = L - i * (i + 1) / 2;
}

// Block products on fp64 MFMA: each of the 4 wavefronts owns one 16 x 16 quadrant of a
// 32 x 32 result. v_mfma_f64_16x16x4f64 takes A[row l & 15][k l >> 4] and
// B[k l >> 4][col l & 15] from lane l and leaves element v of the quadrant's result at
// row (l >> 4) + 4 v, column l & 15 (the layout every "quad" array below follows).
typedef double doublex4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int quad_row(int v) {
  return 16 * ((int)threadIdx.x >> 7) + (((int)threadIdx.x & 63) >> 4) + 4 * v;
}
__device__ __forceinline__ int quad_col() {
  return 16 * (((int)threadIdx.x >> 6) & 1) + ((int)threadIdx.x & 15);
}

// acc (quadrant layout) += sum_q Aa[r][q] * Bb[c][q] over q < NB (LDS, stride LP); two
// accumulators split the k-chain
__device__ __forceinline__ void gemm_nt(const double *Aa, const double *Bb, doublex4 &acc) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double *ar = Aa + (16 * (w >> 1) + (lane & 15)) * LP + (lane >> 4);
  const double *br = Bb + (16 * (w & 1) + (lane & 15)) * LP + (lane >> 4);
  doublex4 acc2 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < NB; q += 8) {
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[q], br[q], acc, 0, 0, 0);
    acc2 = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[q + 4], br[q + 4], acc2, 0, 0, 0);
  }
  acc += acc2;
}

// 1/x and 1/sqrt(x) from the hardware estimates (relative error e below 2^-22) and one
// third-order step each, which leaves e^3: full fp64 accuracy to about 1 ulp, with a
// shorter dependency chain than IEEE divide / sqrt (it sits on the serial pivot chain).
__device__ __forceinline__ double rcp_nr(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsqrt_nr(double x) {
  const double r = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// Value of a double in one lane, the same for the whole wavefront.
__device__ __forceinline__ double lane_value(double x, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)lo | ((uint64_t)hi << 32));
}
// a, b, c or d for k = 0..3, without a branch (the asm keeps the four values computed)
__device__ __forceinline__ double sel4(double a, double b, double c, double d, int k) {
  asm("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
  const double ab = (k & 1) ? b : a, cd = (k & 1) ? d : c;
  return (k & 2) ? cd : ab;
}

// Cholesky of the nb x nb (nb <= 32) block in S (LDS, row stride LP, lower part read) and
// its inverse, by one wavefront, without LDS traffic or barriers; L's block at row and
// column g0 and D_k = L^-1 (zero padded) are stored as they are finished.
//
// The block and the identity rows below it (whose right-looking panels are L^-T) are held
// as 16 x 16 tiles, element M[l & 15][(l >> 4) + 4 v] in register v of lane l. Four
// consecutive columns of a tile are then one register, which is at once the operand
// [row l & 15][k l >> 4] of v_mfma_f64_16x16x4f64 (as A and as B), so a rank-4 update of a
// tile is one MFMA and nothing is moved between lanes. Per 4-column panel: the 4 x 4 pivot
// block is read into scalars and factored as U D U^T by every lane (the serial chain: one
// reciprocal per pivot), lane group k takes column k of U^-1, the panel X = P U^-T is one
// v_mfma_f64_4x4x4f64 per tile (its four blocks are the tile's four row groups), and the
// trailing tiles lose X D^-1 X^T. The scaled panels X D^-1/2 are L and L^-T.
//
// What bounds it is the chain of 32 pivots. Kernel times: chol_panel (one block's load,
// factorisation and stores) 5.9 us, a trailing launch of a single matrix 7.4; 9.2 and 11.3
// with the form it replaced, in which 256 threads shared the block through LDS with a
// barrier per panel. Every panel is unrolled: as a loop over register-shifted tiles, for a
// smaller instruction footprint, the block took 1.1 us longer.
#define BGP_MFMA16(A, B, C) __builtin_amdgcn_mfma_f64_16x16x4f64(A, B, C, 0, 0, 0)
#define BGP_MFMA4(A, B) __builtin_amdgcn_mfma_f64_4x4x4f64(A, B, 0.0, 0, 0, 0)
struct BlockPanel {
  double ui;   // U^-1, operand of the panel products
  double x;    // finished columns of the diagonal tile (unscaled), zero above the diagonal
  double qd;   // -X / piv of the rows below the panel, zero elsewhere
  double nip;  // -1 / piv of column l >> 4
  double rs;   // 1 / sqrt(piv) of column l >> 4
};
// Panel q of a diagonal tile, from the tile's register q; bits c0 + 4 q .. + 3 of `bad` are
// set for failing pivots (without a branch: one costs more than a pivot's arithmetic).
template <int q>
__device__ __forceinline__ BlockPanel block_panel(double d, int c0, uint32_t &bad, int fr, int fg) {
  double w[4][4], l[4][4], ip[4];
#pragma unroll
  for (int p = 0; p < 4; ++p)
#pragma unroll
    for (int s = p; s < 4; ++s) w[s][p] = lane_value(d, 4 * q + s + 16 * p);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    if (p < 3) ip[p] = rcp_nr(w[p][p]);
#pragma unroll
    for (int s = p + 1; s < 4; ++s) l[s][p] = w[s][p] * ip[p];
#pragma unroll
    for (int t = p + 1; t < 4; ++t)
#pragma unroll
      for (int s = t; s < 4; ++s) w[s][t] = fma(-l[s][p], w[t][p], w[s][t]);
  }
  // column fg of U^-1
  const double z0 = fg == 0 ? 1.0 : 0.0;
  const double z1 = fma(-l[1][0], z0, fg == 1 ? 1.0 : 0.0);
  const double z2 = fma(-l[2][1], z1, fma(-l[2][0], z0, fg == 2 ? 1.0 : 0.0));
  const double z3 = fma(-l[3][2], z2, fma(-l[3][1], z1, fma(-l[3][0], z0, fg == 3 ? 1.0 : 0.0)));
  BlockPanel o;
  o.ui = sel4(z0, z1, z2, z3, fr);
  const double x = BGP_MFMA4(o.ui, d);
  const double pv = sel4(w[0][0], w[1][1], w[2][2], w[3][3], fg);
  const uint64_t f = __ballot(!(pv > 0.0 && isfinite(pv)));  // column k: lanes 16 k .. 16 k + 15
  bad |= (uint32_t)((f & 1) | ((f >> 15) & 2) | ((f >> 30) & 4) | ((f >> 45) & 8)) << (c0 + 4 * q);
  o.rs = rsqrt_nr(pv);
  o.nip = -o.rs * o.rs;
  o.qd = fr >= 4 * q + 4 ? x * o.nip : 0.0;  // (the finished columns take no update)
  o.x = fr >= 4 * q + fg ? x : 0.0;
  return o;
}

struct BlockTiles {
  doublex4 a00, a10, a11, e00, e01, e11;
};
struct BlockOut {  // where and how much of the block is stored
  double *L, *Dk;
  int ldl, nb;
};
// One panel of columns 0..15: the tiles below it, the identity rows, and its stores.
template <int q>
__device__ __forceinline__ void block_left(BlockTiles &T, const BlockOut &s, uint32_t &bad, int fr,
                                           int fg) {
  const BlockPanel o = block_panel<q>(T.a00[q], 0, bad, fr, fg);
  if (q < 3) T.a00 = BGP_MFMA16(o.qd, o.x, T.a00);
  const double x1 = BGP_MFMA4(o.ui, T.a10[q]), xe = BGP_MFMA4(o.ui, T.e00[q]), q1 = x1 * o.nip;
  T.a11 = BGP_MFMA16(q1, x1, T.a11);
  if (q < 3) T.a10 = BGP_MFMA16(o.qd, x1, T.a10);
  if (q < 3) T.e00 = BGP_MFMA16(o.qd, xe, T.e00);
  T.e01 = BGP_MFMA16(q1, xe, T.e01);
  const int c = 4 * q + fg;
  if (c < s.nb && fr < s.nb) s.L[(int64_t)fr * s.ldl + c] = o.x * o.rs;
  if (c < s.nb && 16 + fr < s.nb) s.L[(int64_t)(16 + fr) * s.ldl + c] = x1 * o.rs;
  s.Dk[c * NB + fr] = (c < s.nb && fr < s.nb) ? xe * o.rs : 0.0;
}
// One panel of columns 16..31.
template <int q>
__device__ __forceinline__ void block_right(BlockTiles &T, const BlockOut &s, uint32_t &bad, int fr,
                                            int fg) {
  const BlockPanel o = block_panel<q>(T.a11[q], 16, bad, fr, fg);
  if (q < 3) T.a11 = BGP_MFMA16(o.qd, o.x, T.a11);
  const double x0 = BGP_MFMA4(o.ui, T.e01[q]), x1 = BGP_MFMA4(o.ui, T.e11[q]);
  if (q < 3) T.e01 = BGP_MFMA16(o.qd, x0, T.e01);
  if (q < 3) T.e11 = BGP_MFMA16(o.qd, x1, T.e11);
  const int c = 16 + 4 * q + fg;
  if (c < s.nb && 16 + fr < s.nb) s.L[(int64_t)(16 + fr) * s.ldl + c] = o.x * o.rs;
  s.Dk[c * NB + fr] = c < s.nb ? x0 * o.rs : 0.0;
  s.Dk[c * NB + 16 + fr] = (c < s.nb && 16 + fr < s.nb) ? x1 * o.rs : 0.0;
}

__device__ __forceinline__ void factor_store(const double *S, double *L, int ldl, double *Dk,
                                             int g0, int nb, int32_t *info) {
  const int lane = threadIdx.x & 63, fr = lane & 15, fg = lane >> 4;
  BlockTiles T;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int c = fg + 4 * v;
    const double id = fr == c ? 1.0 : 0.0;
    double s00 = S[fr * LP + c], s10 = S[(16 + fr) * LP + c], s11 = S[(16 + fr) * LP + 16 + c];
    asm("" : "+v"(s00), "+v"(s10), "+v"(s11));  // loaded by every lane, then selected
    T.a00[v] = (fr < nb && c <= fr) ? s00 : id;  // (rows and columns past nb: the identity)
    T.a10[v] = 16 + fr < nb ? s10 : 0.0;
    T.a11[v] = (16 + fr < nb && c <= fr) ? s11 : id;
    T.e00[v] = id;
    T.e01[v] = 0.0;
    T.e11[v] = id;
  }
  const BlockOut s{L + (int64_t)g0 * ldl + g0, Dk, ldl, nb};
#pragma unroll
  for (int v = 0; v < 4; ++v) {  // the zero tiles above the diagonal
    const int c = fg + 4 * v;
    if (16 + c < nb) s.L[(int64_t)fr * ldl + 16 + c] = 0.0;
    Dk[c * NB + 16 + fr] = 0.0;
  }
  uint32_t bad = 0;  // (a failed block's values are not used)
  block_left<0>(T, s, bad, fr, fg);
  block_left<1>(T, s, bad, fr, fg);
  block_left<2>(T, s, bad, fr, fg);
  block_left<3>(T, s, bad, fr, fg);
  if (nb > 16) {
    block_right<0>(T, s, bad, fr, fg);
    block_right<1>(T, s, bad, fr, fg);
    block_right<2>(T, s, bad, fr, fg);
    block_right<3>(T, s, bad, fr, fg);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 + fg + 4 * v;
      Dk[c * NB + fr] = 0.0;
      Dk[c * NB + 16 + fr] = 0.0;
    }
  }
  if (nb < 32) bad &= (1u << nb) - 1u;
  if (bad && lane == 0) *info = g0 + __ffs(bad);
}
#undef BGP_MFMA16
#undef BGP_MFMA4

__global__ __launch_bounds__(256) void chol_panel(const double *A, int32_t lda, double *L,
                                                   int32_t ldl, double *D, int32_t n,
                                                   int32_t *info, const int32_t *halt,
                                                   const CholBatch bt) {
  __shared__ double S[NB * LP];
  {
    const int64_t b = blockIdx.z;
    A += b * bt.sA;
    L += b * bt.sL;
    D += b * bt.sD;
    info += b;
  }
  if (*info || (halt && *halt)) return;
  const int nb = min(NB, n);
  double v[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {  // all loads in flight, then the LDS stores
    const int e = threadIdx.x + 256 * u, r = e / NB, c = e % NB;
    v[u] = (r < nb && c <= r) ? A[(int64_t)r * lda + c] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = threadIdx.x + 256 * u;
    S[(e / NB) * LP + e % NB] = v[u];
  }
  __syncthreads();
  if (threadIdx.x < 64) factor_store(S, L, ldl, D, 0, nb, info);
}

// Newton setup (see launch_newton_setup): workgroup 0 builds B's first diagonal block
// itself and factors it (dispatched first, it overlaps the rest); the next workgroups
// each write a tile of kSetupRows rows x 256 columns of the stacked matrix [B ; I]; the
// last ones form v = W^1/2 K b for kSetupVRows rows each. Probit terms are computed once
// per row and column of a tile (not per element: they are the costly part), the row
// terms into LDS; the tiles of row 0 also store the vectors.
constexpr int kSetupRows = 32;
constexpr int kSetupVRows = 8;
__global__ __launch_bounds__(256) void newton_setup_k(const double *K, const double *f,
                                                       const double *t, double *grad, double *W,
                                                       double *sw, double *b, double *v,
                                                       double *A, int32_t n, int64_t nfill,
                                                       double *L, double *D, int32_t *info,
                                                       const int32_t *halt) {
  __shared__ double S[NB * LP];
  __shared__ double swr[kSetupRows > NB ? kSetupRows : NB];
  if (*info || *halt) return;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    const int nb = min(NB, n);
    if (tid < nb) {
      double g, w;
      probit_terms(f[tid], t[tid], g, w);
      swr[tid] = sqrt(w);
    }
    __syncthreads();
    double kv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {  // all loads in flight, then the LDS stores
      const int e = tid + 256 * u, r = e / NB, c = e % NB;
      kv[u] = (r < nb && c <= r) ? K[(int64_t)r * n + c] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + 256 * u, r = e / NB, c = e % NB;
      S[r * LP + c] = (r < nb && c <= r) ? swr[r] * kv[u] * swr[c] + (r == c ? 1.0 : 0.0) : 0.0;
    }
    __syncthreads();
    if (tid < 64) factor_store(S, L, n, D, 0, nb, info);
    return;
  }
  if ((int64_t)blockIdx.x > nfill) {
    // v[r] = W_r^1/2 sum_c K[r][c] b[c] for kSetupVRows rows; each thread takes the
    // columns tid, tid + 256, ... (b from the probit terms at f) and every row's partial
    // sums are reduced over the workgroup in a fixed order
    const int r0 = (int)((int64_t)blockIdx.x - nfill - 1) * kSetupVRows;
    double acc[kSetupVRows];
#pragma unroll
    for (int q = 0; q < kSetupVRows; ++q) acc[q] = 0.0;
    for (int c = tid; c < n; c += 256) {
      double gc, wc;
      probit_terms(f[c], t[c], gc, wc);
      const double bc = fma(wc, f[c], gc);
#pragma unroll
      for (int q = 0; q < kSetupVRows; ++q)
        if (r0 + q < n) acc[q] = fma(K[(int64_t)(r0 + q) * n + c], bc, acc[q]);
    }
    const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
    for (int q = 0; q < kSetupVRows; ++q) {
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) acc[q] += __shfl_xor(acc[q], off);
      if (lane == 0) S[wv * kSetupVRows + q] = acc[q];
    }
    __syncthreads();
    if (tid < kSetupVRows && r0 + tid < n) {
      const int r = r0 + tid;
      double g, w;
      probit_terms(f[r], t[r], g, w);
      const double u = (S[tid] + S[kSetupVRows + tid]) + (S[2 * kSetupVRows + tid] + S[3 * kSetupVRows + tid]);
      v[r] = sqrt(w) * u;
    }
    return;
  }
  const int nct = (n + 255) / 256;
  const int tr = (int)(blockIdx.x - 1) / nct, tcol = (int)(blockIdx.x - 1) - tr * nct;
  const int r0 = tr * kSetupRows, rows = 2 * n;
  const int c = tcol * 256 + tid;
  if (r0 < n) {  // workgroup-uniform: the tile has rows of B
    if (tid < kSetupRows && r0 + tid < n) {
      double g, w;
      probit_terms(f[r0 + tid], t[r0 + tid], g, w);
      swr[tid] = sqrt(w);
    }
    __syncthreads();
  }
  if (c >= n) return;
  double gc, wc;
  probit_terms(f[c], t[c], gc, wc);
  const double swc = sqrt(wc);
  if (r0 == 0) {
    grad[c] = gc;
    W[c] = wc;
    sw[c] = swc;
    b[c] = fma(wc, f[c], gc);
  }
  const int rend = min(r0 + kSetupRows, rows);
  for (int r = r0; r < rend; ++r) {
    const double x = r < n ? swr[r - r0] * K[(int64_t)r * n + c] * swc + (r == c ? 1.0 : 0.0)
                           : (r - n == c ? 1.0 : 0.0);
    A[(int64_t)r * n + c] = x;
  }
}

// Global loads of the block steps are unconditional: a row or column index past the
// matrix is clamped to its last one (finite data), and whatever it feeds is either
// multiplied by the zero padding of D_k or never stored. All of a workgroup's loads are
// issued before its first barrier.

// Workgroup (e, bj) of the extra rows at block step k: rows n + e NB.. of A, trailing
// block column j0 = k0 + NB + bj NB. P_e = A_Ek D_k^T (final: L_E panel, stored by bj = 0,
// the only workgroup of block row e when there is no trailing column), P_j = A_jk D_k^T,
// A_Ej -= P_e P_j^T.
__device__ __forceinline__ void extra_rows_step(double *A, int32_t lda, const double *Dk,
                                                double *LE, int32_t ldle, int k, int e, int bj,
                                                int T, int n, int n_extra, bool le_t, double *Ds,
                                                double *Pi, double *Pj, double *Ts, double *Tj) {
  const int k0 = k * NB, ie = e * NB, j0 = k0 + NB + bj * NB;
  const int tid = threadIdx.x, qc = quad_col();
  const int rmax = n - 1, emax = n_extra - 1;
  doublex4 tile;
  double dv[kPer], tv[kPer], jv[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {  // all loads in flight, then the LDS stores
    const int q = tid + 256 * u, r = q / NB, c = q % NB;
    dv[u] = Dk[q];
    tv[u] = A[(int64_t)(n + min(ie + r, emax)) * lda + min(k0 + c, rmax)];
    jv[u] = T > 0 ? A[(int64_t)min(j0 + r, rmax) * lda + k0 + c] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int q = tid + 256 * u, r = q / NB, c = q % NB;
    Ds[r * LP + c] = dv[u];
    Ts[r * LP + c] = tv[u];
    if (T > 0) Tj[r * LP + c] = jv[u];
  }
  if (T > 0) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      tile[v] = A[(int64_t)(n + min(ie + quad_row(v), emax)) * lda + min(j0 + qc, rmax)];
  }
  __syncthreads();
  doublex4 acc = {0.0, 0.0, 0.0, 0.0}, acc2 = {0.0, 0.0, 0.0, 0.0};
  gemm_nt(Ts, Ds, acc);               // P_e = A_Ek D_k^T
  if (T > 0) gemm_nt(Tj, Ds, acc2);   // P_j = A_jk D_k^T
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    Pi[quad_row(v) * LP + qc] = acc[v];
    Pj[quad_row(v) * LP + qc] = acc2[v];
  }
  __syncthreads();
  if (bj == 0) {
    for (int q = tid; q < NB * NB; q += 256) {
      const int r = q / NB, c = q % NB;
      if (ie + r < n_extra && k0 + c < n) {
        if (le_t) LE[(int64_t)(k0 + c) * ldle + ie + r] = Pi[r * LP + c];  // L_E^T
        else LE[(int64_t)(ie + r) * ldle + k0 + c] = Pi[r * LP + c];
      }
    }
  }
  if (T == 0) return;
  doublex4 up = {0.0, 0.0, 0.0, 0.0};
  gemm_nt(Pi, Pj, up);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = ie + quad_row(v), c = j0 + qc;
    if (r < n_extra && c < n) A[(int64_t)(n + r) * lda + c] = tile[v] - up[v];
  }
}

__global__ __launch_bounds__(256) void chol_trailing(double *A, int32_t lda, double *L,
                                                      int32_t ldl, double *D, int32_t k,
                                                      int32_t n, int32_t n_extra, double *LE,
                                                      int32_t ldle, int32_t *info,
                                                      const int32_t *halt, const CholBatch bt,
                                                      int32_t le_t) {
  __shared__ double Ds[NB * LP], Pi[NB * LP], Pj[NB * LP], Ts[NB * LP], Tj[NB * LP];
  {
    const int64_t b = blockIdx.z;  // (a batched launch's extra rows are identity rows)
    A += b * bt.sA;
    L += b * bt.sL;
    D += b * bt.sD;
    if (LE) LE += b * bt.sX;
    info += b;
  }
  if (*info || (halt && *halt)) return;
  const int nbk = (n + NB - 1) / NB, T = nbk - 1 - k, nsq = T * (T + 1) / 2;
  if ((int)blockIdx.x >= nsq) {  // extra rows (identity blocks past step k are not launched)
    const int q = blockIdx.x - nsq, Tc = T > 0 ? T : 1;
    extra_rows_step(A, lda, D + (int64_t)k * NB * NB, LE, ldle, k, q / Tc, q % Tc, T, n, n_extra,
                    le_t != 0,
                    Ds, Pi, Pj, Ts, Tj);
    return;
  }
  int bi, bj;
  tri_index(blockIdx.x, bi, bj);
  const int k0 = k * NB;  // k < nbk - 1 here, so block column k is full
  const int i0 = k0 + NB + bi * NB, j0 = k0 + NB + bj * NB;
  const int tid = threadIdx.x, qc = quad_col();
  const int rmax = n - 1;
  const double *Dk = D + (int64_t)k * NB * NB;
  // A_ij (for bi = bj = 0 the next diagonal block), prefetched for the end
  doublex4 tile;
#pragma unroll
  for (int v = 0; v < 4; ++v)
    tile[v] = A[(int64_t)min(i0 + quad_row(v), rmax) * lda + min(j0 + qc, rmax)];
  double dv[kPer], tv[kPer], jv[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {  // all loads in flight, then the LDS stores
    const int e = tid + 256 * u, r = e / NB, c = e % NB;
    dv[u] = Dk[e];
    tv[u] = A[(int64_t)min(i0 + r, rmax) * lda + k0 + c];
    jv[u] = A[(int64_t)min(j0 + r, rmax) * lda + k0 + c];
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = tid + 256 * u, r = e / NB, c = e % NB;
    Ds[r * LP + c] = dv[u];
    Ts[r * LP + c] = tv[u];
    if (bi != bj) Tj[r * LP + c] = jv[u];
  }
  __syncthreads();
  {
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
    gemm_nt(Ts, Ds, acc);  // P_i = A_ik D_k^T = L_ik
#pragma unroll
    for (int v = 0; v < 4; ++v) Pi[quad_row(v) * LP + qc] = acc[v];
    if (bi != bj) {
      doublex4 acc2 = {0.0, 0.0, 0.0, 0.0};
      gemm_nt(Tj, Ds, acc2);  // P_j
#pragma unroll
      for (int v = 0; v < 4; ++v) Pj[quad_row(v) * LP + qc] = acc2[v];
    }
  }
  __syncthreads();
  const double *Pjj = (bi == bj) ? Pi : Pj;
  doublex4 up = {0.0, 0.0, 0.0, 0.0};
  gemm_nt(Pi, Pjj, up);
  if (bi == bj) {
    for (int e = tid; e < NB * NB; e += 256) {
      const int r = e / NB, c = e % NB;
      if (i0 + r < n) L[(int64_t)(i0 + r) * ldl + k0 + c] = Pi[r * LP + c];
    }
  }
  if (bi == 0 && bj == 0) {
    // block (k+1, k+1) has received all of its updates: factor it now
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = quad_row(v);
      Ts[r * LP + qc] = (i0 + r < n && i0 + qc < n) ? tile[v] - up[v] : 0.0;
    }
    __syncthreads();
    if (tid < 64)
      factor_store(Ts, L, ldl, D + (int64_t)(k + 1) * NB * NB, i0, min(NB, n - i0), info);
  } else {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = i0 + quad_row(v), c = j0 + qc;
      if (r < n && c < n) A[(int64_t)r * lda + c] = tile[v] - up[v];
    }
  }
}

// out = X^T X (both triangles) for lower-triangular X: the workgroup of output block
// (bi, bj), bi >= bj, sums X_{R,bi}^T X_{R,bj} over the block rows R >= bi (X is zero
// above them) on fp64 MFMA; the two column blocks go to LDS transposed so that the
// block product of gemm_nt contracts over the rows.
__global__ __launch_bounds__(256) void ata_mfma_k(const double *X, int32_t ld, double *out,
                                                   int32_t n, const int32_t *info,
                                                   const CholBatch bt) {
  __shared__ double Ta[NB * LP], Tb[NB * LP];
  {
    const int64_t b = blockIdx.z;
    if (info && info[b]) return;
    X += b * bt.sX;
    out += b * bt.sA;
  }
  int bi, bj;
  tri_index(blockIdx.x, bi, bj);
  const int nbk = (n + NB - 1) / NB, tid = threadIdx.x, qc = quad_col();
  const int ci = bi * NB, cj = bj * NB;
  doublex4 acc = {0.0, 0.0, 0.0, 0.0};
  // the next block row's values are loaded into registers while this one is multiplied
  double va[kPer], vb[kPer];
  auto load = [&](int Rb) {
    const int r0 = Rb * NB;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + 256 * u, r = e / NB, c = e % NB;
      const bool rin = r0 + r < n;
      const double *xr = X + (int64_t)(r0 + r) * ld;
      va[u] = (rin && ci + c < n) ? xr[ci + c] : 0.0;
      vb[u] = (rin && cj + c < n) ? xr[cj + c] : 0.0;
    }
  };
  load(bi);
  for (int Rb = bi; Rb < nbk; ++Rb) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = tid + 256 * u, r = e / NB, c = e % NB;
      Ta[c * LP + r] = va[u];
      Tb[c * LP + r] = vb[u];
    }
    __syncthreads();
    if (Rb + 1 < nbk) load(Rb + 1);
    gemm_nt(Ta, Tb, acc);  // acc[r][c] += sum_q X[q][ci + r] X[q][cj + c]
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int r = ci + quad_row(v), c = cj + qc;
    if (r < n && c < n) {
      out[(int64_t)r * ld + c] = acc[v];
      out[(int64_t)c * ld + r] = acc[v];
    }
  }
}

__global__ __launch_bounds__(256) void copy_lower_k(const double *src, int32_t lds, double *dst,
                                                     int32_t ldd, int32_t n) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (int64_t)n * n) return;
  const int r = (int)(idx / n), c = (int)(idx - (int64_t)r * n);
  dst[(int64_t)r * ldd + c] = src[(int64_t)r * lds + c];
}

// dst (2n rows, stride n) = [src; I]: the matrix, then identity rows whose factorisation
// panels give L^-T
__global__ __launch_bounds__(256) void copy_ident_k(const double *src, int32_t lds, double *dst,
                                                     int32_t n) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= 2 * (int64_t)n * n) return;
  const int r = (int)(idx / n), c = (int)(idx - (int64_t)r * n);
  dst[idx] = r < n ? src[(int64_t)r * lds + c] : (r - n == c ? 1.0 : 0.0);
}


}  // namespace

hipError_t launch_copy_ident(const double *src, int32_t lds, double *dst, int32_t n,
                             hipStream_t s) {
  const int64_t tot = 2 * (int64_t)n * n;
  if (tot <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_ident_k, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, src, lds,
                     dst, n);
  return hipGetLastError();
}

hipError_t chol_factor(double *A, int32_t lda, double *L, int32_t ldl, double *D, int32_t n,
                       int32_t *info, hipStream_t s, int32_t n_extra, double *LE, int32_t ldle,
                       const int32_t *halt, bool clear_upper, int32_t n_ident,
                       bool first_block_done) {
  if (n <= 0) return hipSuccess;
  if (n_extra < 0 || (n_extra > 0 && !LE)) return hipErrorInvalidValue;
  // identity rows: the last n extra rows, starting on a block boundary
  if (n_ident != 0 && (n_ident != n || n_extra < n_ident || (n_extra - n_ident) % NB))
    return hipErrorInvalidValue;
  const int nbk = (n + NB - 1) / NB, ne_dense = (n_extra - n_ident + NB - 1) / NB;
  const int ne_ident = (n_ident + NB - 1) / NB;
  if (clear_upper) {
    hipError_t e = hipMemsetAsync(L, 0, sizeof(double) * (size_t)ldl * n, s);
    if (e != hipSuccess) return e;
  }
  if (!first_block_done)
    hipLaunchKernelGGL(chol_panel, dim3(1), dim3(256), 0, s, A, lda, L, ldl, D, n, info, halt,
                       CholBatch{});
  for (int k = 0; k < nbk; ++k) {
    const int T = nbk - 1 - k;
    const int ne = ne_dense + std::min(k + 1, ne_ident);  // identity block e joins at step e
    const int grid = T * (T + 1) / 2 + ne * (T > 0 ? T : 1);
    if (grid == 0) break;  // last block column without extra rows
    hipLaunchKernelGGL(chol_trailing, dim3(grid), dim3(256), 0, s, A, lda, L, ldl, D, k, n,
                       n_extra, LE, ldle, info, halt, CholBatch{}, 0);
  }
  return hipGetLastError();
}

hipError_t chol_factor_batched(double *A, int32_t lda, double *L, int32_t ldl, double *D,
                               int32_t n, int32_t *info, const CholBatch &bt, hipStream_t s,
                               bool clear_upper, double *X, int32_t ldx) {
  if (n <= 0 || bt.count <= 0) return hipSuccess;
  if (bt.count > 65535 || bt.sL < (int64_t)ldl * n) return hipErrorInvalidValue;
  if (X && (bt.sA < 2 * (int64_t)lda * n || bt.sX < (int64_t)ldx * n)) return hipErrorInvalidValue;
  const int nbk = (n + NB - 1) / NB;
  if (clear_upper) {
    hipError_t e = hipMemsetAsync(L, 0, sizeof(double) * (size_t)bt.sL * bt.count, s);
    if (e != hipSuccess) return e;
  }
  if (X) {  // L^-1's blocks above the diagonal are never written
    hipError_t e = hipMemsetAsync(X, 0, sizeof(double) * (size_t)bt.sX * bt.count, s);
    if (e != hipSuccess) return e;
  }
  const unsigned z = (unsigned)bt.count;
  hipLaunchKernelGGL(chol_panel, dim3(1, 1, z), dim3(256), 0, s, A, lda, L, ldl, D, n, info,
                     nullptr, bt);
  for (int k = 0; k < nbk; ++k) {
    const int T = nbk - 1 - k;
    // with X: the identity rows' block e joins at step e; their panels, stored transposed,
    // are L^-1
    const int ne = X ? std::min(k + 1, nbk) : 0;
    const int grid = T * (T + 1) / 2 + ne * (T > 0 ? T : 1);
    if (grid == 0) break;
    hipLaunchKernelGGL(chol_trailing, dim3(grid, 1, z), dim3(256), 0, s, A, lda, L, ldl, D, k, n,
                       X ? n : 0, X, ldx, info, nullptr, bt, X ? 1 : 0);
  }
  return hipGetLastError();
}


hipError_t launch_newton_setup(const double *K, const double *f, const double *t, double *grad,
                               double *W, double *sw, double *b, double *v, double *A, int32_t n,
                               double *L, double *D, int32_t *info, const int32_t *halt,
                               hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t nfill = (int64_t)((2 * n + kSetupRows - 1) / kSetupRows) * ((n + 255) / 256);
  const int64_t nv = (n + kSetupVRows - 1) / kSetupVRows;
  hipLaunchKernelGGL(newton_setup_k, dim3((unsigned)(1 + nfill + nv)), dim3(256), 0, s, K, f, t,
                     grad, W, sw, b, v, A, n, nfill, L, D, info, halt);
  return hipGetLastError();
}


hipError_t launch_ata_batched(const double *X, int32_t ld, double *out, int32_t n,
                              const int32_t *info, const CholBatch &bt, hipStream_t s) {
  if (n <= 0 || bt.count <= 0) return hipSuccess;
  if (bt.count > 65535) return hipErrorInvalidValue;
  const int nbk = (n + NB - 1) / NB;
  hipLaunchKernelGGL(ata_mfma_k, dim3(nbk * (nbk + 1) / 2, 1, (unsigned)bt.count), dim3(256), 0, s,
                     X, ld, out, n, info, bt);
  return hipGetLastError();
}

hipError_t launch_ata_lower(const double *X, int32_t ld, double *out, int32_t n, hipStream_t s) {
  return launch_ata_batched(X, ld, out, n, nullptr, CholBatch{}, s);
}

hipError_t launch_copy_matrix(const double *src, int32_t lds, double *dst, int32_t ldd, int32_t n,
                              hipStream_t s) {
  const int64_t tot = (int64_t)n * n;
  if (tot <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_lower_k, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, src, lds,
                     dst, ldd, n);
  return hipGetLastError();
}

}  // namespace bgp

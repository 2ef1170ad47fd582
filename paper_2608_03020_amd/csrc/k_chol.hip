// k_chol.hip -- ridge solve (row a5 of the step).
//
// Eq. 7 / Theorem S6.1 in the linear-system form of Section S7:
//   (S + lam I) M = [S Lp | K]      (positive definite for lam > 0; no inverse)
// solved for every (block, lam) pair of a call in one batched pass:
//   1. Jacobi equilibration  A^ = D (S + lam I) D,  D = diag(S + lam I)^{-1/2};
//   2. right-looking blocked Cholesky A^ = U^T U (U upper, row-major) with
//      P-wide panels (P = 128 in fp32, 64 in fp64), four to a super-panel.  Per panel,
//      launches batched over all matrices: the diagonal block is factored and inverted
//      in LDS by one workgroup per matrix; the row panel takes the update by the
//      super-panel's earlier panels and U12 = U11^{-T} A12, matrix-core products; per
//      super-panel the trailing matrix takes the symmetric update A22 -= U12^T U12.  The right-hand sides ride
//      along as extra columns of the row panel and the update, so the forward
//      substitution costs nothing extra.  Products use MFMA (fp32 32x32x2, or
//      fp64 16x16x4 for fp64 statistics);
//   3. back substitution U M' = Y by row blocks, each a product with U11^{-1},
//      then M = D M'.
// The first non-positive pivot is reported in dev_info (1-based).
#include <mutex>

#include "loca_launch.h"
#include "loca_bf16.h"

#include <functional>
#include <utility>
#include <vector>

namespace loca {

namespace {

constexpr int kT = 256;       // threads

struct Lams {
  double v[8];
};
__global__ void k_set_lambdas(Lams l, double* out, int cnt) {
  if ((int)threadIdx.x < cnt) out[threadIdx.x] = l.v[threadIdx.x];
}

__global__ void k_fill_zero_i32(int32_t* p, int64_t cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cnt) p[i] = 0;
}

// D[mi][i] = 1 / sqrt(S_ii + lam_l) for matrix mi = b * nl + l.
template <typename T, typename ST>
__global__ void k_equil_diag(int64_t d, const ST* __restrict__ S, int64_t s_bstride, const double* __restrict__ lam,
                             int nl, T* __restrict__ D) {
  const int64_t mi = blockIdx.y;
  const int64_t b = mi / nl;
  const int l = (int)(mi % nl);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= d) return;
  const double v = (double)S[b * s_bstride + i * d + i] + lam[l];
  D[mi * d + i] = (T)(1.0 / sqrt(v));
}

// F[i][j] = D_i (S_ij + lam delta_ij) D_j for j >= i; RHS[i][c] = D_i [S Lp | K][i][c].
// One workgroup per (kEqRows rows, block): a row of S is read once for all nl lambdas.
constexpr int kEqRows = 16;
template <typename T, typename ST>
__global__ __launch_bounds__(256) void k_equil_setup(int64_t d, int64_t m, int64_t r_prev, const ST* __restrict__ S,
                                                     int64_t s_bstride, const ST* __restrict__ K, int64_t k_bstride,
                                                     const double* __restrict__ SLp, const double* __restrict__ lam,
                                                     int nl, const T* __restrict__ D, T* __restrict__ F,
                                                     T* __restrict__ R) {
  const int64_t b = blockIdx.y;
  const int64_t k = m - r_prev;
  for (int ii = 0; ii < kEqRows; ++ii) {
    const int64_t i = (int64_t)blockIdx.x * kEqRows + ii;
    if (i >= d) return;
    const ST* Si = S + b * s_bstride + i * d;
    for (int64_t j = i + threadIdx.x; j < d; j += blockDim.x) {
      const double sij = (double)Si[j];
      for (int l = 0; l < nl; ++l) {
        const int64_t mi = b * nl + l;
        const double v = sij + (j == i ? lam[l] : 0.0);
        F[mi * d * d + i * d + j] = (T)((double)D[mi * d + i] * v * (double)D[mi * d + j]);
      }
    }
    for (int64_t c = threadIdx.x; c < m; c += blockDim.x) {
      const double v = (c < r_prev) ? SLp[b * d * r_prev + i * r_prev + c] : (double)K[b * k_bstride + i * k + (c - r_prev)];
      for (int l = 0; l < nl; ++l) {
        const int64_t mi = b * nl + l;
        R[mi * d * m + i * m + c] = (T)((double)D[mi * d + i] * v);
      }
    }
  }
}

// RHS[i][c] = D_i [S Lp | K][i][c] only (the factor of an earlier call is reused).
template <typename T, typename ST>
__global__ void k_equil_rhs(int64_t d, int64_t m, int64_t r_prev, const ST* __restrict__ K, int64_t k_bstride,
                            const double* __restrict__ SLp, int nl, const T* __restrict__ D, T* __restrict__ R) {
  const int64_t mi = blockIdx.y, b = mi / nl;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d * m) return;
  const int64_t i = e / m, c = e % m, k = m - r_prev;
  const double v = (c < r_prev) ? SLp[b * d * r_prev + i * r_prev + c] : (double)K[b * k_bstride + i * k + (c - r_prev)];
  R[mi * d * m + e] = (T)((double)D[mi * d + i] * v);
}

// The same for float statistics and factors when d % 4 == 0 and the rows of S are 16-byte
// aligned, tiled so that every workgroup has the same amount of work: a workgroup takes
// kEqRows rows and one chunk of kEqCols columns (chunks wholly below the diagonal exit),
// each thread four consecutive columns (16-byte loads and stores of S, D and F, one load
// of S for all lambdas); the four-column group that holds the diagonal writes only its
// entries on or above it.  The right-hand sides are written by the workgroups of the last
// chunk (never wholly below the diagonal).
// The arithmetic is that of k_equil_setup, term for term.
constexpr int kEqCols = 1024;
__global__ __launch_bounds__(256) void k_equil_setup_v4(int64_t d, int64_t m, int64_t r_prev,
                                                        const float* __restrict__ S, int64_t s_bstride,
                                                        const float* __restrict__ K, int64_t k_bstride,
                                                        const double* __restrict__ SLp,
                                                        const double* __restrict__ lam, int nl,
                                                        const float* __restrict__ D, float* __restrict__ F,
                                                        float* __restrict__ R) {
  const int64_t b = blockIdx.z;
  const int64_t k = m - r_prev;
  const int64_t i0 = (int64_t)blockIdx.x * kEqRows;
  const int64_t c0 = (int64_t)blockIdx.y * kEqCols;
  if (c0 + kEqCols <= (i0 & ~(int64_t)3)) return;  // every row of the tile starts past this chunk
  const int64_t j = c0 + 4 * threadIdx.x;
  const bool jin = j < d;
  // every global load of the tile is issued before the first use: the rows of S at this
  // thread's four columns; per lambda, D at the columns and at the tile's rows
  float4 sv[kEqRows];
#pragma unroll
  for (int ii = 0; ii < kEqRows; ++ii) {
    const int64_t i = i0 + ii;
    const bool need = jin && i < d && j + 3 >= i;
    sv[ii] = *(const float4*)(S + b * s_bstride + (need ? i * d + j : 0));
  }
  for (int l = 0; l < nl; ++l) {
    const int64_t mi = b * nl + l;
    const float4 dj = *(const float4*)(D + mi * d + (jin ? j : 0));
    float di[kEqRows];
#pragma unroll
    for (int ii = 0; ii < kEqRows; ++ii) di[ii] = D[mi * d + (i0 + ii < d ? i0 + ii : d - 1)];
    const double li = lam[l];
#pragma unroll
    for (int ii = 0; ii < kEqRows; ++ii) {
      const int64_t i = i0 + ii;
      if (i < d && jin && j + 3 >= i) {
        const double dd = (double)di[ii];
        float o[4];
        o[0] = (float)(dd * ((double)sv[ii].x + (j == i ? li : 0.0)) * (double)dj.x);
        o[1] = (float)(dd * ((double)sv[ii].y + (j + 1 == i ? li : 0.0)) * (double)dj.y);
        o[2] = (float)(dd * ((double)sv[ii].z + (j + 2 == i ? li : 0.0)) * (double)dj.z);
        o[3] = (float)(dd * ((double)sv[ii].w + (j + 3 == i ? li : 0.0)) * (double)dj.w);
        float* dst = F + mi * d * d + i * d + j;
        if (j >= i) {
          *(float4*)dst = make_float4(o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
          for (int u = 1; u < 4; ++u)
            if (j + u >= i) dst[u] = o[u];
        }
      }
    }
  }
  if (blockIdx.y == gridDim.y - 1)  // the last chunk holds column d - 1 >= i of every row
    for (int ii = 0; ii < kEqRows; ++ii) {
      const int64_t i = i0 + ii;
      if (i >= d) break;
      for (int64_t c = threadIdx.x; c < m; c += blockDim.x) {
        const double v = (c < r_prev) ? SLp[b * d * r_prev + i * r_prev + c] : (double)K[b * k_bstride + i * k + (c - r_prev)];
        for (int l = 0; l < nl; ++l) {
          const int64_t mi = b * nl + l;
          R[mi * d * m + i * m + c] = (float)((double)D[mi * d + i] * v);
        }
      }
    }
}

// out[b] = S_sym L (d x r, fp64) from the upper triangle of S; L(j, c) = L[j l_sj + c l_sc].  A
// workgroup owns 64 rows and 16 NC columns of the product (grid: x over row tiles, y = block, z
// over column chunks) and walks the 64-wide column tiles of S in order: tiles on or above the
// diagonal are read row-major, tiles below it as the transpose of the stored tile above (both
// with coalesced rows), the diagonal tile mirrored from its upper half.  A wave forms 16 of the
// rows on the fp64 matrix cores, and the next tile's loads are in flight meanwhile: with one
// tile at a time and a thread per row on the vector unit, the load, the conversions of L and the
// sums followed one another (24 blocks of
// d = 896, r = 8: 135 -> 45 us; the projected form of one fp64 block of d = 896: 206 -> 35 us).
constexpr int kSM = 64;
template <typename ST, int NC>
__global__ __launch_bounds__(256) void k_sym_mul(int64_t d, int64_t r, const ST* __restrict__ S, int64_t s_bstride,
                                                 const float* __restrict__ Lall, int64_t l_bstride, int64_t l_sj,
                                                 int64_t l_sc, double* __restrict__ out) {
  constexpr int RC = 16 * NC, SU = kSM * kSM / 256, LU = kSM * RC / 256;
  __shared__ ST sS[kSM][kSM + 1];     // [row][column j]
  __shared__ float sL[RC][kSM + 1];   // [column c][j]
  const int64_t b = blockIdx.y;
  const int64_t i0 = (int64_t)blockIdx.x * kSM, c0 = (int64_t)blockIdx.z * RC;
  const ST* Sb = S + b * s_bstride;
  const float* L = Lall + b * l_bstride;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6, li = lane & 15, lk = lane >> 4;
  const bool jfast = l_sj == 1;  // L's contiguous direction: lanes along it
  f64x4_t acc[NC][2];
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int h = 0; h < 2; ++h) acc[q][h] = (f64x4_t){0.0, 0.0, 0.0, 0.0};
  ST vS[SU];
  float vL[LU];
  auto load = [&](int64_t j0) {  // the stored tile: rows r0.., columns q0.. (transposed left of the diagonal)
    const int64_t r0 = j0 < i0 ? j0 : i0, q0 = j0 < i0 ? i0 : j0;
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int e = t + 256 * u;
      const int64_t gi = r0 + e / kSM, gj = q0 + e % kSM;
      vS[u] = gi < d && gj < d ? Sb[gi * d + gj] : (ST)0;
    }
#pragma unroll
    for (int u = 0; u < LU; ++u) {
      const int e = t + 256 * u;
      const int64_t j = j0 + (jfast ? e % kSM : e / RC), c = c0 + (jfast ? e / kSM : e % RC);
      vL[u] = j < d && c < r ? L[j * l_sj + c * l_sc] : 0.f;
    }
  };
  load(0);
  for (int64_t j0 = 0; j0 < d; j0 += kSM) {
    __syncthreads();  // the previous tile is no longer read
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const int e = t + 256 * u, rr = e / kSM, cc = e % kSM;
      if (j0 < i0) sS[cc][rr] = vS[u];
      else sS[rr][cc] = vS[u];
    }
#pragma unroll
    for (int u = 0; u < LU; ++u) {
      const int e = t + 256 * u;
      sL[jfast ? e / kSM : e % RC][jfast ? e % kSM : e / RC] = vL[u];
    }
    if (j0 + kSM < d) load(j0 + kSM);
    __syncthreads();
    if (j0 == i0) {  // mirror the upper half of the diagonal tile
      for (int e = t; e < kSM * kSM; e += 256) {
        const int rr = e / kSM, cc = e % kSM;
        if (cc < rr) sS[rr][cc] = sS[cc][rr];
      }
      __syncthreads();
    }
#pragma unroll
    for (int ks = 0; ks < kSM; ks += 4) {
      const double fa = (double)sS[16 * w + li][ks + lk];
#pragma unroll
      for (int q = 0; q < NC; ++q)
        acc[q][(ks >> 2) & 1] = mfma_f64(fa, (double)sL[16 * q + li][ks + lk], acc[q][(ks >> 2) & 1]);
    }
  }
#pragma unroll
  for (int q = 0; q < NC; ++q)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t i = i0 + 16 * w + lk + 4 * u, c = c0 + 16 * q + li;
      if (i < d && c < r) out[(b * d + i) * r + c] = acc[q][0][u] + acc[q][1][u];
    }
}

template <typename ST>
hipError_t sym_mul(hipStream_t s, int64_t nb, int64_t d, int64_t r, const ST* S, int64_t s_bstride, const float* L,
                   int64_t l_bstride, int64_t l_sj, int64_t l_sc, double* out) {
  const unsigned gx = (unsigned)((d + kSM - 1) / kSM);
  if (r <= 16)
    k_sym_mul<ST, 1><<<dim3(gx, (unsigned)nb), 256, 0, s>>>(d, r, S, s_bstride, L, l_bstride, l_sj, l_sc, out);
  else
    k_sym_mul<ST, 2><<<dim3(gx, (unsigned)nb, (unsigned)((r + 31) / 32)), 256, 0, s>>>(d, r, S, s_bstride, L, l_bstride,
                                                                                       l_sj, l_sc, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ matrix-core tile products

// Per precision: panel width P (= output tile side), MFMA block side BLK and its K step.
template <typename T> struct Mf;
template <> struct Mf<float> {
  static constexpr int P = 128, BLK = 32, KS = 2, NR = 16;
  typedef f32x16_t acc_t;
  static LOCA_DEV acc_t mma(float a, float b, acc_t c) { return mfma_f32x2(a, b, c); }
  static LOCA_DEV int row(int lane, int r) { return mfma32_row(lane, r); }
  static LOCA_DEV int col(int lane) { return lane & 31; }
  static LOCA_DEV acc_t zero() { acc_t z; for (int r = 0; r < 16; ++r) z[r] = 0.f; return z; }
};
template <> struct Mf<double> {
  static constexpr int P = 64, BLK = 16, KS = 4, NR = 4;
  typedef f64x4_t acc_t;
  static LOCA_DEV acc_t mma(double a, double b, acc_t c) { return mfma_f64(a, b, c); }
  static LOCA_DEV int row(int lane, int r) { return (lane >> 4) + 4 * r; }
  static LOCA_DEV int col(int lane) { return lane & 15; }
  static LOCA_DEV acc_t zero() { return (acc_t){0.0, 0.0, 0.0, 0.0}; }
};

// acc[m][q] += sum_kk sP[kk][i] sQ[kk][j] over the wave's (P/2) x (P/2) quarter (wi, wj) of a
// P x P output tile; sP, sQ are K x (P + pad) row-major LDS panels.
template <typename T>
LOCA_DEV void tile_mma(const T* sP, const T* sQ, int ld, int K, int wi, int wj, int lane,
                       typename Mf<T>::acc_t (&acc)[2][2]) {
  constexpr int BLK = Mf<T>::BLK, KS = Mf<T>::KS, WT = Mf<T>::P / 2;
  const int kr = lane / BLK, cr = lane % BLK;
  for (int kk = 0; kk < K; kk += KS) {
    T a[2], b[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) a[m] = sP[(kk + kr) * ld + wi * WT + m * BLK + cr];
#pragma unroll
    for (int q = 0; q < 2; ++q) b[q] = sQ[(kk + kr) * ld + wj * WT + q * BLK + cr];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc[m][q] = Mf<T>::mma(a[m], b[q], acc[m][q]);
  }
}

// ------------------------------------------------------------------ fp32 panels on bf16 matrix cores

// A float a is carried as three bfloat16 parts, h = bf16(a), m = bf16(a - h),
// l = bf16(a - h - m) (each difference is exact in float), which hold a to about 2^-27
// relative.  The product of two split values keeps the six terms of order 2^-16 and
// larger (h*h, h*m, m*h, h*l, l*h, m*m) and drops m*l, l*m, l*l (order 2^-24 and
// below), so a product has float-class error while running on bf16 MFMA, which
// retires sixteen times the flops of the fp32 MFMA per cycle.
// The split is split3_pair (loca_bf16.h): hardware conversions, two values at a time.
// The kept terms, smallest first:
constexpr int kX6A[6] = {2, 0, 1, 1, 0, 0}, kX6B[6] = {0, 2, 1, 0, 1, 0};

LOCA_DEV float4 ld4_or_zero(const float* base, int64_t idx, bool ok) {
  const float4 v = *(const float4*)(base + (ok ? idx : 0));
  return ok ? v : make_float4(0.f, 0.f, 0.f, 0.f);
}
LOCA_DEV float4 ld4_or_zero_ro(const float* __restrict__ base, int64_t idx, bool ok) { return ld4_or_zero(base, idx, ok); }

// The first operand of a panel's products: stages of 16 rows x the panel's 128 columns of F,
// one 16-byte load (V4: d % 4 == 0) per four values, split once by the workgroup into three
// bf16 planes [16][kPanelLD] (the four rows a half-wave's transpose read takes start 64 bytes
// apart modulo 256: conflict-free).
constexpr int kPanelLD = 160, kPanelPlane = 16 * kPanelLD;
// The load takes the nearest element inside the matrix and panel_mask zeroes what lay outside,
// when the value is used: a load under a condition would be waited for where it is issued.
template <bool V4>
LOCA_DEV float4 panel_load(const float* F, int64_t d, int64_t row, int64_t col) {
  const float* r = F + (row < d ? row : d - 1) * d;
  if (V4) return *(const float4*)(r + (col < d ? col : d - 4));
  float4 v;
  v.x = r[col < d ? col : d - 1];
  v.y = r[col + 1 < d ? col + 1 : d - 1];
  v.z = r[col + 2 < d ? col + 2 : d - 1];
  v.w = r[col + 3 < d ? col + 3 : d - 1];
  return v;
}
LOCA_DEV float4 panel_mask(float4 v, int64_t d, int64_t row, int64_t col) {
  const bool ok = row < d;
  v.x = ok && col < d ? v.x : 0.f;
  v.y = ok && col + 1 < d ? v.y : 0.f;
  v.z = ok && col + 2 < d ? v.z : 0.f;
  v.w = ok && col + 3 < d ? v.w : 0.f;
  return v;
}
LOCA_DEV void panel_put(uint16_t* planes, int kk, int c4, const float4& v) {
  uint32_t h[2], m[2], l[2];
  split3_pair(v.x, v.y, h[0], m[0], l[0]);
  split3_pair(v.z, v.w, h[1], m[1], l[1]);
  const int o = kk * kPanelLD + c4;
  *(uint2*)(planes + o) = make_uint2(h[0], h[1]);
  *(uint2*)(planes + kPanelPlane + o) = make_uint2(m[0], m[1]);
  *(uint2*)(planes + 2 * kPanelPlane + o) = make_uint2(l[0], l[1]);
}

// As frag32_tr on the 16 rows of a stage, in the row order of a lane's own MFMA results: the
// operand of lane l is the rows 8 (e / 4) + 4 (l / 32) + e % 4, e = 0..7, of column c0 + l % 32.
LOCA_DEV bf16x8_t frag32_tr_own(const uint16_t* tile, int ld, int c0, int lane) {
  const int g = lane >> 4, w = lane & 15;
  const uint16_t* q = tile + (4 * (g >> 1) + (w >> 2)) * ld + c0 + 16 * (g & 1) + 4 * (w & 3);
  const s16x4_t lo = lds_read_tr16(q), hi = lds_read_tr16(q + 8 * ld);
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  const s16x8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8_t, v);
}

// The diagonal block's own strip update, eight waves: the ten 32 x 32 blocks on or above the
// diagonal of sum_kk F[kk][p + i] F[kk][p + j], rows kk in [k0, p), subtracted from sA.
template <bool V4, int LDA>
LOCA_DEV void diag_strip_update(const float* F, int64_t d, int64_t k0, int64_t p, uint16_t (&sP)[2][3 * kPanelPlane],
                                float* sA, int tid, int lane, int wid) {
  constexpr int D = 4;
  const int ns = (int)((p - k0) / 16);  // a multiple of 8
  const int kk = tid >> 5, c4 = 4 * (tid & 31);
  int bi[2], bj[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int u = wid + 8 * t < 10 ? wid + 8 * t : wid;
    bi[t] = u < 4 ? 0 : (u < 7 ? 1 : (u < 9 ? 2 : 3));
    bj[t] = u < 4 ? u : (u < 7 ? u - 3 : (u < 9 ? u - 5 : 3));
  }
  const int nt = wid < 2 ? 2 : 1;
  f32x16_t acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
  float4 rp[D];
#pragma unroll
  for (int u = 0; u < D; ++u) rp[u] = panel_load<V4>(F, d, k0 + 16 * u + kk, p + c4);
  panel_put(sP[0], kk, c4, panel_mask(rp[0], d, k0, p + c4));
  __syncthreads();
  for (int s0 = 0; s0 < ns; s0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int s = s0 + u, cur = u & 1;
      rp[u] = panel_load<V4>(F, d, k0 + 16 * (s + D) + kk, p + c4);  // past the last stage: not used
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        if (t >= nt) continue;
        bf16x8_t fa[3], fb[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          fa[x] = frag32_tr(sP[cur] + x * kPanelPlane, kPanelLD, 32 * bi[t], 0, lane);
          fb[x] = frag32_tr(sP[cur] + x * kPanelPlane, kPanelLD, 32 * bj[t], 0, lane);
        }
#pragma unroll
        for (int x = 0; x < 6; ++x) acc[t] = mfma32(fa[kX6A[x]], fb[kX6B[x]], acc[t]);
      }
      panel_put(sP[cur ^ 1], kk, c4, panel_mask(rp[(u + 1) % D], d, k0, p + c4));
      __syncthreads();
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t >= nt) continue;
    float* B = sA + 32 * bi[t] * LDA + 32 * bj[t] + (lane & 31);
    // the 16 x 16 block below the diagonal of a diagonal 32 x 32 one holds E's zeros
    const bool low = bi[t] == bj[t] && (lane & 31) < 16;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!(low && r >= 8)) B[mfma32_row(lane, r) * LDA] -= acc[t][r];
  }
}

// The rows [p, p + 128) of a panel right of its diagonal block, and of the right-hand sides:
//   A12 -= sum over kk in [k0, p) of F[kk][p + i] F[kk][j]   (the super-panel's earlier panels)
//   U12  = X^T A12,                                           X = U11^{-1} in the diagonal block.
// A wave owns 32 columns of all 128 rows (column block cb: the first nF in F, then R's), so the
// updated A12 is already, in the registers where the matrix cores left it, the second operand of
// the product with X: rows 16 c + 8 (e / 4) + 4 h + e % 4 of lane half h are one step's eight
// values, the first operand (X's rows, read in the same order) being staged as one more run of
// stages after the update's.  The second operand of the update is loaded by its owner straight
// into the matrix cores' layout (32 lanes on consecutive columns).  So a panel's rows cross HBM
// once in each direction where the update and the product, in a launch each, crossed it twice.
// NWV waves per workgroup share the staged operand: fewer when the launch leaves compute units
// idle (the rule and its figures stand at the launch).
template <int NWV, bool V4>
__global__ __launch_bounds__(64 * NWV) void k_panel_f32(int64_t d, int64_t k0, int64_t p, float* __restrict__ Fall,
                                                        float* __restrict__ Rall, int64_t m, int nF) {
  constexpr int NT = 64 * NWV, P = 128, QP = 512 / NT, D = 4;
  __shared__ __attribute__((aligned(16))) uint16_t sP[2][3 * kPanelPlane];
  const int64_t mi = blockIdx.y;
  float* F = Fall + mi * d * d;
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5;
  const int cb = (int)blockIdx.x * NWV + wid;
  const bool inF = cb < nF;
  float* B = inF ? F : Rall + mi * d * m;
  const int64_t ldb = inF ? d : m, c0 = inF ? p + P + 32 * (int64_t)cb : 32 * (int64_t)(cb - nF);
  const int64_t col = c0 + (lane & 31);
  const bool cok = col < ldb;  // false in the waves that the last workgroup has to spare
  const int pw = (int)((d - p) < P ? (d - p) : P);
  const int nk1 = (int)((p - k0) / 16);  // stages of the update (a multiple of 8), X's after them

  float4 rp[D][QP];
  auto load_p = [&](int slot, int s) {
#pragma unroll
    for (int q = 0; q < QP; ++q) {
      const int c = tid + NT * q;
      rp[slot][q] = panel_load<V4>(F, d, k0 + 16 * s + (c >> 5), p + 4 * (c & 31));
    }
  };
  auto put_p = [&](int buf, int slot, int s) {
#pragma unroll
    for (int q = 0; q < QP; ++q) {
      const int c = tid + NT * q, kk = c >> 5, c4 = 4 * (c & 31);
      panel_put(sP[buf], kk, c4, panel_mask(rp[slot][q], d, k0 + 16 * s + kk, p + c4));
    }
  };
  float rb[D][8];  // rows 8 h + e of a stage (columns past the edge read column 0: never stored)
  const uint32_t boff = (uint32_t)(4 * (8 * h * ldb + (cok ? col : 0)));
  auto load_b = [&](int slot, int s) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      rb[slot][e] = *(const float*)((const char*)(B + (k0 + 16 * (int64_t)s + e) * ldb) + boff);
  };
  auto split_b = [&](const float (&v)[8], bf16x8_t (&f)[3]) {
    uint32_t x[3][4];
#pragma unroll
    for (int e = 0; e < 4; ++e) split3_pair(v[2 * e], v[2 * e + 1], x[0][e], x[1][e], x[2][e]);
#pragma unroll
    for (int t = 0; t < 3; ++t) f[t] = __builtin_bit_cast(bf16x8_t, make_uint4(x[t][0], x[t][1], x[t][2], x[t][3]));
  };

#pragma unroll
  for (int u = 0; u < D; ++u) load_p(u, u);
  f32x16_t acc[4], old[4];  // the update's sum, then A12 less it; A12
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 32 * a + mfma32_row(lane, r);
      old[a][r] = B[(p + (row < pw ? row : 0)) * ldb + (cok ? col : 0)];  // rows past pw meet X's zero rows
      acc[a][r] = 0.f;
    }
  if (nk1 > 0)
#pragma unroll
    for (int u = 0; u < D; ++u) load_b(u, u);
  put_p(0, 0, 0);
  __syncthreads();
  for (int s0 = 0; s0 < nk1; s0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int s = s0 + u, cur = u & 1;
      load_p(u, s + D);
      bf16x8_t fb[3], fa[3][4];
      split_b(rb[u], fb);
      load_b(u, s + D < nk1 ? s + D : nk1 - 1);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) fa[t][a] = frag32_tr(sP[cur] + t * kPanelPlane, kPanelLD, 32 * a, 0, lane);
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] = mfma32(fa[kX6A[t]][a], fb[kX6B[t]], acc[a]);
      put_p(cur ^ 1, (u + 1) % D, s + 1);
      __syncthreads();
    }
  }
  f32x16_t out[4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc[a][r] = old[a][r] - acc[a][r];
      out[a][r] = 0.f;
    }
  // X's rows 16 c ..: zero left of the diagonal, so 32-row blocks of the output above row 16 c take nothing
#pragma unroll
  for (int c = 0; c < P / 16; ++c) {
    const int u = c % D, cur = c & 1;
    if (c + D < P / 16) load_p(u, nk1 + c + D);
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = acc[c >> 1][8 * (c & 1) + e];
    bf16x8_t fb[3], fa[3][4];
    split_b(v, fb);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
      for (int a = c >> 1; a < 4; ++a) fa[t][a] = frag32_tr_own(sP[cur] + t * kPanelPlane, kPanelLD, 32 * a, lane);
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int a = c >> 1; a < 4; ++a) out[a] = mfma32(fa[kX6A[t]][a], fb[kX6B[t]], out[a]);
    if (c + 1 < P / 16) {
      put_p(cur ^ 1, (u + 1) % D, nk1 + c + 1);
      __syncthreads();
    }
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int row = 32 * a + mfma32_row(lane, r);
      if (cok && row < pw) B[(p + row) * ldb + col] = out[a][r];
    }
}

// ------------------------------------------------------------------ diagonal block: factor and invert

// One workgroup per matrix factors the P x P diagonal block, A11 = U11^T U11, and inverts
// U11; X = U11^{-1} replaces the diagonal block of F (strict lower part zeroed), for the row
// panel and the back substitution apply it as a product.  The kernel is a serial chain on
// every panel's critical path, so it is built to make that chain short.
//
// The block is worked on as NB x NB blocks of 16 in LDS.  Eliminating the rows of [A | I]
// gives L^{-1} [A | I] = [U | E], E = U11^{-T}, so the inverse grows along with the factor: U
// takes the blocks right of the diagonal, E those left of it (E_rs starts as zero), and step q is
//   factor:    one wave factors A_qq and forms E_qq (chol_inv16),
//   row panel: block (q, s) <- E_qq block (q, s) for every s != q, one wave each; for s < q
//              that is the final E_qs, whose transpose goes straight to F,
//   update:    block (r, s) -= U_qr^T block (q, s) for r > q and s <= q or s >= r; wave 0 only
//              takes (q + 1, q + 1) and goes on to factor it while the others finish,
// the products on the 16x16x4 matrix cores (fp32, or fp64 for fp64 statistics).  Entries past
// the matrix (a ragged last block) are an identity extension.
//
// 128 x 128 in fp32, one matrix: 49.8 us blocked by 32 (a column of a block waited for an LDS
// round trip, and the inverse was assembled at the end); 64 x 64 in fp64: 68.6 us with one
// column of the whole block per step (two barriers and an fp64 square root and division each).
template <typename T> struct Dg;
template <> struct Dg<float> {
  typedef f32x4_t acc_t;
  static constexpr int LD_PAD = 20;  // row length = P + 20: operand reads of either kind fall on distinct banks
  static LOCA_DEV acc_t mma(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  static LOCA_DEV int row(int lane, int r) { return 4 * (lane >> 4) + r; }
  // the hardware estimate, whose error of up to an ulp leans one way, and a Newton step (without it
  // the solution leaned by -7e-8 to -9e-8, d = 896 to 5120; with it by -2e-8 to -4e-8)
  static LOCA_DEV float rsq(float v) {
    const float y = __builtin_amdgcn_rsqf(v), h = 0.5f * y, g = v * y;
    return fmaf(fmaf(-g, h, 0.5f), y, y);
  }
  template <int CTRL> static LOCA_DEV float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
  }
};
template <> struct Dg<double> {
  typedef f64x4_t acc_t;
  static constexpr int LD_PAD = 18;
  static LOCA_DEV acc_t mma(double a, double b, acc_t c) { return mfma_f64(a, b, c); }
  static LOCA_DEV int row(int lane, int r) { return (lane >> 4) + 4 * r; }
  // the hardware estimate and two Newton steps: y <- y + y (1 - v y^2) / 2
  static LOCA_DEV double rsq(double v) {
    double y = __builtin_amdgcn_rsq(v);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const double h = 0.5 * y, g = v * y;
      y = fma(fma(-g, h, 0.5), y, y);
    }
    return y;
  }
  template <int CTRL> static LOCA_DEV double dpp(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
  }
};
// lane I of each row of 16 lanes to all 16 (DPP row_newbcast)
template <int I, typename T>
LOCA_DEV T bcast16(T v) { return Dg<T>::template dpp<0x150 + I>(v); }

// Step J of the elimination of a 16 x 16 block: lane c (mod 16) holds column c of A in a[] and
// of E in e[].  The multipliers U[J][I] come from lane I by a DPP broadcast, so a step has no
// memory access; row J + 1 is updated first, since the next pivot waits for it.
template <int J, typename T, int... K>
LOCA_DEV void elim_rows(T (&a)[16], T (&e)[16], T uc, T nuc, T ec, std::integer_sequence<int, K...>) {
  auto row = [&](auto ic) {
    constexpr int I = J + 1 + decltype(ic)::value;
    const T m = bcast16<I>(nuc);
    a[I] = fma(m, uc, a[I]);
    e[I] = fma(m, ec, e[I]);
  };
  (row(std::integral_constant<int, K>{}), ...);
}
template <int J, typename T>
LOCA_DEV void elim_step(T (&a)[16], T (&e)[16], int& bad) {
  const T piv = bcast16<J>(a[J]);
  bad = (!(piv > (T)0) && bad == 16) ? J : bad;
  const T inv = Dg<T>::rsq(piv);
  const T uc = a[J] * inv, ec = e[J] * inv;
  e[J] = ec;
  elim_rows<J>(a, e, uc, -uc, ec, std::make_integer_sequence<int, 15 - J>{});
}
template <typename T, int... J>
LOCA_DEV void elim_all(T (&a)[16], T (&e)[16], int& bad, std::integer_sequence<int, J...>) {
  (elim_step<J>(a, e, bad), ...);
}

// One wave: A (16 x 16 at B, row stride ld; upper part used) = U^T U, E = U^{-T} over it (zero
// above its diagonal).  X = E^T to rows of the output (row stride ldx; rows and columns < valid).
// The first non-positive pivot among the first `valid` is reported (1-based, offset base).
template <typename T>
LOCA_DEV void chol_inv16(T* B, int ld, T* X, int64_t ldx, int lane, int valid, int64_t base, int32_t* info) {
  const int c = lane & 15;
  T a[16], e[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) a[r] = B[r * ld + c];
#pragma unroll
  for (int r = 0; r < 16; ++r) e[r] = r == c ? (T)1 : (T)0;
  int bad = 16;
  elim_all(a, e, bad, std::make_integer_sequence<int, 16>{});
  if (bad < 16 && bad < valid && lane == 0) atomicCAS(info, 0, (int32_t)(base + bad + 1));
  if (lane < 16) {
#pragma unroll
    for (int r = 0; r < 16; ++r) B[r * ld + c] = e[r];
    if (c < valid)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (r < valid) X[c * ldx + r] = e[r];
  }
}

// acc += Aop Bop for one 16 x 16 block with K = 16 from LDS: Aop[i][k] = Am[i ld + k], or
// Am[k ld + i] (TA); Bop[k][j] = Bm[k ld + j].
template <typename T, bool TA>
LOCA_DEV void mm16(typename Dg<T>::acc_t& acc, const T* Am, const T* Bm, int ld, int lane) {
  const int i = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int s = 0; s < 16; s += 4) {
    const int k = s + kq;
    acc = Dg<T>::mma(TA ? Am[k * ld + i] : Am[i * ld + k], Bm[k * ld + i], acc);
  }
}

// In fp32 the block first takes the update by its super-panel's earlier panels, A11 -= sum over
// the rows kk in [k0, p) of F[kk][p + i] F[kk][p + j] (diag_strip_update): in a launch of its own,
// with the rest of the panel's rows, that update was one more link of the chain.
template <typename T, int P, bool V4>
__global__ __launch_bounds__(4 * P) void k_diag_inv(int64_t d, int64_t k0, int64_t p, T* __restrict__ Fall,
                                                    int32_t* __restrict__ dev_info) {
  constexpr int NB = P / 16, LD = P + Dg<T>::LD_PAD, NT = 4 * P, NW = NT / 64;
  static_assert(NW == NB, "one wave per block of a row panel");
  __shared__ __attribute__((aligned(16))) T sA[P * LD];
  constexpr bool UPD = sizeof(T) == 4;
  __shared__ __attribute__((aligned(16))) uint16_t sP[UPD ? 2 : 1][UPD ? 3 * kPanelPlane : 8];
  const int64_t mi = blockIdx.x;
  T* F = Fall + mi * d * d + p * d + p;  // the diagonal block
  const int pw = (int)((d - p) < P ? (d - p) : P);
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15;
  {  // the upper part to LDS, all loads issued before the first use; zero below the diagonal
    constexpr int NE = P * P / NT;
    T v[NE];
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int e = tid + NT * u, r = e / P, c = e % P;
      v[u] = ld_or_zero(F, (int64_t)r * d + c, c >= r && c < pw);
    }
#pragma unroll
    for (int u = 0; u < NE; ++u) {
      const int e = tid + NT * u, r = e / P, c = e % P;
      sA[r * LD + c] = r == c && r >= pw ? (T)1 : v[u];
      if (c < r && r < pw) F[(int64_t)r * d + c] = (T)0;
    }
  }
  if constexpr (UPD)
    if (p > k0) diag_strip_update<V4, LD>(Fall + mi * d * d, d, k0, p, sP, sA, tid, lane, wid);
  __syncthreads();
  auto blk = [&](int r, int s) { return sA + 16 * r * LD + 16 * s; };
  auto update = [&](int q, int r, int s) {  // block (r, s) -= U_qr^T block (q, s)
    typename Dg<T>::acc_t acc = {};
    mm16<T, true>(acc, blk(q, r), blk(q, s), LD, lane);
    T* B = blk(r, s);
#pragma unroll
    for (int e = 0; e < 4; ++e) B[Dg<T>::row(lane, e) * LD + li] -= acc[e];
  };
  for (int q = 0; q < NB; ++q) {
    if (wid == 0) chol_inv16<T>(blk(q, q), LD, F + (int64_t)16 * q * d + 16 * q, d, lane, pw - 16 * q, p + 16 * q, dev_info + mi);
    __syncthreads();
    if (wid != q) {
      typename Dg<T>::acc_t acc = {};
      mm16<T, false>(acc, blk(q, q), blk(q, wid), LD, lane);
      T* B = blk(q, wid);
#pragma unroll
      for (int e = 0; e < 4; ++e) B[Dg<T>::row(lane, e) * LD + li] = acc[e];
      if (wid < q) {  // E_qs is final: X's block (s, q) is its transpose
        const int xr = 16 * wid + li;  // < pw: below a full block
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int xc = 16 * q + Dg<T>::row(lane, e);
          if (xc < pw) F[(int64_t)xr * d + xc] = acc[e];
        }
      }
    }
    if (q == NB - 1) break;
    __syncthreads();
    if (wid == 0) {
      update(q, q + 1, q + 1);
      wave_lds_sync();
    } else {
      for (int u = wid - 1; u < (NB - 1 - q) * NB; u += NW - 1) {
        const int r = q + 1 + u / NB, s = u % NB;
        if ((s > q && s < r) || (r == q + 1 && s == r)) continue;
        update(q, r, s);
      }
    }
  }
}

// ------------------------------------------------------------------ panel products (row panel, trailing update)

LOCA_DEV void upper_tile_c(int u, int T, int& I, int& J) {
  int i = 0;
  while (u >= T - i) { u -= T - i; ++i; }
  I = i;
  J = i + u;
}

// Out[i][j] (op)= sum_{kk < K} Pn[kk][i] Qn[kk][j] for one P x P output tile, with the
// K rows streamed through LDS in chunks of kKC rows, double-buffered via registers.
//   kRowPanel: Pn = U11^{-1} (diagonal block), Qn = the chunk's columns of the row
//              panel (F or R), Out = the same chunk, overwritten: U12 = U11^{-T} A12;
//   kTrailing: Pn, Qn = the row panel U12 (F) / its RHS rows (R), Out -= on the upper
//              tiles of the trailing matrix and on the RHS rows below the panel.
constexpr int kKC = 32;
enum PanelJob { kRowPanel = 0, kTrailing = 1 };

// kTrailing takes its K rows from [k0, k0 + kw) of F and R and updates the region of
// rows and columns >= off: every upper tile plus the RHS rows (strip = 0), or only the
// first row of tiles, rows [off, off + P) (strip = 1).  Job = blockIdx.x + job0, the
// upper tiles first, then the RHS tiles.
template <typename T, int JOB>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(2))) void k_panel_product(
    int64_t d, int64_t m, int64_t p, int64_t k0, int64_t kw, int64_t off, int strip, int job0, T* __restrict__ Fall,
    T* __restrict__ Rall) {
  constexpr int P = Mf<T>::P, LD = P + 4, PER = (kKC * P) / kT;
  __shared__ T sP[2][kKC * LD];
  __shared__ T sQ[2][kKC * LD];
  const int64_t mi = blockIdx.y;
  T* F = Fall + mi * d * d;
  T* R = Rall + mi * d * m;
  const int pw = JOB == kRowPanel ? (int)((d - p) < P ? (d - p) : P) : (int)kw;  // K rows
  if (JOB == kRowPanel) off = p + pw;
  const int64_t nrem = d - off;
  const int64_t nchF = (nrem + P - 1) / P;
  bool rhs, diag = false;
  int64_t orow, ocol, ocend;  // output tile origin (row in F/R, column) and column end
  const T* gP;                // row kk of Pn at gP + kk * ldp, column i at + i
  const T* gQ;
  int64_t ldq, prows_ok;
  if (JOB == kRowPanel) {
    const int64_t job = (int64_t)blockIdx.x + job0;
    rhs = job >= nchF;
    ocol = rhs ? (job - nchF) * P : off + job * P;
    ocend = rhs ? m : d;
    orow = p;
    gP = F + p * d + p;
    prows_ok = pw;
    gQ = rhs ? R + p * m + ocol : F + p * d + ocol;
    ldq = rhs ? m : d;
  } else {
    const int T2 = (int)((nrem + P - 1) / P);
    const int nU = strip ? T2 : T2 * (T2 + 1) / 2;
    const int TM = (int)((m + P - 1) / P);
    const int job = (int)blockIdx.x + job0;
    int I, J;
    rhs = job >= nU;
    if (!rhs) {
      if (strip) { I = 0; J = job; }
      else upper_tile_c(job, T2, I, J);
    } else { const int u = job - nU; I = u / TM; J = u % TM; }
    diag = !rhs && I == J;
    orow = off + (int64_t)I * P;
    ocol = rhs ? (int64_t)J * P : off + (int64_t)J * P;
    ocend = rhs ? m : d;
    gP = F + k0 * d + orow;
    prows_ok = d - orow;  // columns of Pn that exist
    gQ = rhs ? R + k0 * m + ocol : F + k0 * d + ocol;
    ldq = rhs ? m : d;
  }
  const int64_t pcols_ok = (JOB == kRowPanel) ? pw : prows_ok;
  const int64_t qcols_ok = ocend - ocol;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wid = tid >> 6, wi = wid >> 1, wj = wid & 1;
  const bool active = !(diag && wi > wj);  // strictly lower quarter of a diagonal tile

  T rp[PER], rq[PER];
  auto load_chunk = [&](int kc0) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + q * kT;
      const int kk = e / P, c = e % P;
      const bool okk = kc0 + kk < pw;
      rp[q] = ld_or_zero(gP, (int64_t)(kc0 + kk) * d + c, okk && c < pcols_ok);
      rq[q] = ld_or_zero(gQ, (int64_t)(kc0 + kk) * ldq + c, okk && c < qcols_ok);
    }
  };
  auto store_chunk = [&](int buf) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + q * kT;
      sP[buf][(e / P) * LD + e % P] = rp[q];
      sQ[buf][(e / P) * LD + e % P] = rq[q];
    }
  };

  typename Mf<T>::acc_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = Mf<T>::zero();
  const int nk = (pw + kKC - 1) / kKC;
  load_chunk(0);
  store_chunk(0);
  __syncthreads();
  for (int kc = 0; kc < nk; ++kc) {
    const int cur = kc & 1;
    if (kc + 1 < nk) load_chunk((kc + 1) * kKC);
    if (active) tile_mma<T>(sP[cur], sQ[cur], LD, kKC, wi, wj, lane, acc);
    if (kc + 1 < nk) store_chunk(cur ^ 1);
    __syncthreads();
  }
  if (!active) return;
  T* Out = rhs ? R : F;
  const int64_t ldo = rhs ? m : d;
  const int64_t rend = (JOB == kRowPanel) ? p + pw : d;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      T old[Mf<T>::NR];
      const int64_t col = ocol + wj * (P / 2) + b * Mf<T>::BLK + Mf<T>::col(lane);
      const int64_t rbase = orow + wi * (P / 2) + a * Mf<T>::BLK;
#pragma unroll
      for (int r = 0; r < Mf<T>::NR; ++r) {
        const int64_t row = rbase + Mf<T>::row(lane, r);
        const bool ok = row < rend && col < ocend && (JOB == kRowPanel || rhs || col >= row);
        if (JOB == kTrailing) old[r] = ld_or_zero(Out, row * ldo + col, ok);
      }
#pragma unroll
      for (int r = 0; r < Mf<T>::NR; ++r) {
        const int64_t row = rbase + Mf<T>::row(lane, r);
        const bool ok = row < rend && col < ocend && (JOB == kRowPanel || rhs || col >= row);
        if (ok) Out[row * ldo + col] = (JOB == kTrailing) ? old[r] - acc[a][b][r] : acc[a][b][r];
      }
    }
}

// ------------------------------------------------------------------ trailing update on bf16 matrix cores

// Trailing products on bf16 matrix cores, Out[i][j] -= sum_kk F[kk][i] Qn[kk][j], kk in [k0, k0 + kw):
//   kX6Trail: F on the upper 256 x 256 tiles of the trailing region [off, d), then (jobs past
//             the nF tiles) the right-hand sides' 256-row blocks, Qn and the output in R
//             (d x m per matrix, m % 4 == 0), all m columns;
//   kX6TrailRhs: only the right-hand-side jobs, in a layout for their few columns: a workgroup
//             takes 256 rows x 32 columns (eight waves of 32 x 32; columns 32 blockIdx.z ..),
//             so it does an eighth of the matrix-core work of a 256 x 256 tile.
// A stage is 16 rows of K: each operand is loaded into registers several stages ahead (a
// ring of D stages), split, and written to LDS as three bf16 planes [16][LD]; eight waves
// (2 x 4) read their MFMA operands with transpose reads (LD = 288: the four rows a
// half-wave reads start 64 bytes apart modulo 256, so the reads are conflict-free).
// Requires d % 4 == 0.
constexpr int kX6BK = 16, kX6LD = 288;
enum X6Mode { kX6Trail = 0, kX6TrailRhs = 1 };

template <int MODE>
__global__ __launch_bounds__(512) void k_panel_x6(int64_t d, int64_t k0, int64_t kw, int64_t off,
                                                  float* __restrict__ Fall, float* __restrict__ Rall, int64_t m,
                                                  int nF) {
  constexpr bool RH = MODE == kX6TrailRhs;
  constexpr int BR = 256;  // output rows per tile
  constexpr int BC = RH ? 32 : 256, WGN = RH ? 1 : 4, WGM = 8 / WGN;
  constexpr int WM = BR / WGM, WN = BC / WGN, NBM = WM / 32, NBN = WN / 32;
  constexpr int LD = kX6LD, PLANE = kX6BK * LD;
  constexpr int NQV = BC * kX6BK / 4;                                  // float4 values of a Qn stage
  constexpr int QP = BR * kX6BK / 4 / 512, QQ = (NQV + 511) / 512;     // float4 loads per thread
  __shared__ __attribute__((aligned(16))) uint16_t sm[2][6 * PLANE];  // [buffer][operand * 3 + part]
  const int64_t mi = blockIdx.y;
  float* F = Fall + mi * d * d;
  float* R = Rall + mi * d * m;
  const bool rhs = RH || (int)blockIdx.x >= nF;
  const int job = rhs && !RH ? (int)blockIdx.x - nF : (int)blockIdx.x;
  int64_t orow, ocol;
  bool diag = false;
  if (RH) {
    orow = off + (int64_t)job * BR;
    ocol = (int64_t)blockIdx.z * BC;
  } else if (rhs) {
    orow = off + (int64_t)job * BC;
    ocol = 0;
  } else {
    const int T2 = (int)((d - off + BC - 1) / BC);
    int I, J;
    upper_tile_c(job, T2, I, J);
    diag = I == J;
    orow = off + (int64_t)I * BC;
    ocol = off + (int64_t)J * BC;
  }
  const int64_t pcol = orow;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, wi = wid / WGN, wj = wid % WGN;
  const bool active = !(diag && (wj + 1) * WN <= wi * WM);
  const float* gP = F + k0 * d + pcol;
  float* Out = rhs ? R : F;                          // Qn and the output
  const int64_t ldq = rhs ? m : d, qend = rhs ? m : d;
  const float* gQ = Out + k0 * ldq + ocol;

  // a ring of D stages of global loads in flight: the loads of stage kc + D are issued
  // when stage kc is consumed, so D - 1 stages of matrix-core work cover their latency
  constexpr int D = MODE == kX6Trail ? 2 : 4;
  float4 rp[D][QP], rq[D][QQ];
  auto load = [&](int slot, int kc0) {
#pragma unroll
    for (int q = 0; q < QP; ++q) {
      const int c = tid + 512 * q, kk = c / (BR / 4), c4 = 4 * (c % (BR / 4));
      rp[slot][q] = ld4_or_zero(gP, (int64_t)(kc0 + kk) * d + c4, kc0 + kk < kw && pcol + c4 < d);
    }
#pragma unroll
    for (int q = 0; q < QQ; ++q) {
      const int c = tid + 512 * q, kk = c / (BC / 4), c4 = 4 * (c % (BC / 4));
      if (c < NQV)
        rq[slot][q] = ld4_or_zero(gQ, (int64_t)(kc0 + kk) * ldq + c4, kc0 + kk < kw && ocol + c4 < qend);
    }
  };
  auto put = [&](uint16_t* base, int kk, int c4, const float4& v) {
    uint32_t h[2], m[2], l[2];
    split3_pair(v.x, v.y, h[0], m[0], l[0]);
    split3_pair(v.z, v.w, h[1], m[1], l[1]);
    const int o = kk * LD + c4;
    *(uint2*)(base + o) = make_uint2(h[0], h[1]);
    *(uint2*)(base + PLANE + o) = make_uint2(m[0], m[1]);
    *(uint2*)(base + 2 * PLANE + o) = make_uint2(l[0], l[1]);
  };
  auto store = [&](int buf, int slot) {
#pragma unroll
    for (int q = 0; q < QP; ++q) {
      const int c = tid + 512 * q;
      put(&sm[buf][0], c / (BR / 4), 4 * (c % (BR / 4)), rp[slot][q]);
    }
#pragma unroll
    for (int q = 0; q < QQ; ++q) {
      const int c = tid + 512 * q;
      if (c < NQV) put(&sm[buf][3 * PLANE], c / (BC / 4), 4 * (c % (BC / 4)), rq[slot][q]);
    }
  };

  f32x16_t acc[NBM][NBN];
#pragma unroll
  for (int a = 0; a < NBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  const int nk = (int)((kw + kX6BK - 1) / kX6BK);
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (u < nk) load(u, u * kX6BK);
  store(0, 0);
  __syncthreads();
  for (int kc0 = 0; kc0 < nk; kc0 += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {  // stage kc = kc0 + u: in LDS buffer kc & 1; its register slot is u
      const int kc = kc0 + u;
      if (kc >= nk) break;
      const int cur = kc & 1;
      if (kc + D < nk) load(u, (kc + D) * kX6BK);
      bf16x8_t fa[3][NBM], fb[3][NBN];
#pragma unroll
      for (int t = 0; t < 3; ++t) {
#pragma unroll
        for (int a = 0; a < NBM; ++a) fa[t][a] = frag32_tr(&sm[cur][t * PLANE], LD, wi * WM + 32 * a, 0, lane);
#pragma unroll
        for (int b = 0; b < NBN; ++b)
          fb[t][b] = frag32_tr(&sm[cur][(3 + t) * PLANE], LD, wj * WN + 32 * b, 0, lane);
      }
      // each kept term runs over all blocks, so the MFMAs into one accumulator are NBM * NBN
      // instructions apart
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int a = 0; a < NBM; ++a)
#pragma unroll
          for (int b = 0; b < NBN; ++b) acc[a][b] = mfma32(fa[kX6A[t]][a], fb[kX6B[t]][b], acc[a][b]);
      if (kc + 1 < nk) store(cur ^ 1, (u + 1) % D);
      __syncthreads();
    }
  }
  if (!active) return;
#pragma unroll
  for (int a = 0; a < NBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      const int64_t col = ocol + wj * WN + 32 * b + mfma32_col(lane);
      const int64_t rb = orow + wi * WM + 32 * a;
      float old[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = rb + mfma32_row(lane, r);
        old[r] = ld_or_zero(Out, row * ldq + col, row < d && col < qend && (rhs || col >= row));
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = rb + mfma32_row(lane, r);
        if (row < d && col < qend && (rhs || col >= row)) Out[row * ldq + col] = old[r] - acc[a][b][r];
      }
    }
}

// ------------------------------------------------------------------ trailing update, fp32 rows split in registers

// The trailing update of a super-panel, F[i][j] -= sum_kk U[kk][i] U[kk][j] over its kw rows
// kk in [k0, k0 + kw), on the upper 256 x 256 tiles of the trailing region [off, d), with
// the fp32 rows of U read straight from F.  Stages of 16 rows x 256 columns (16 KB per
// panel) stream into a four-slot LDS ring by direct copies, three stages ahead; the 16-byte
// chunks of stage row r sit XOR-swizzled by 8 (r / 8), so that the two half-waves of an
// operand read (rows r and r + 8) fall on different banks.  The factor of the equilibrated
// matrix (unit diagonal) has |U[kk][i]| <= 1, so every operand, scaled by 2^8, is split in
// registers into two fp16 parts, u = h + l with h = fp16(2^8 u) and l = fp16(2^8 u - h)
// (22 bits of u; a part past the fp16 range cannot occur), and the three kept products
// l h, h l, h h (smallest first) run on the fp16 matrix cores, accumulated in fp32 and
// scaled back by 2^-16 (exact) when F is updated: half the matrix-core work of a three-part
// bf16 split, with product errors of the order of the fp32 accumulation's own rounding.
// A diagonal tile needs one panel (its second ring panel reads nothing).  Tiles, waves and
// the XCD-aware workgroup order are those of the Gram kernel.
// Requires d % 4 == 0, kw % 16 == 0 and 4 d^2 < 2^31 bytes per matrix.
constexpr int kS32BK = 16;  // K rows per stage
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_v __attribute__((ext_vector_type(2)));
LOCA_DEV f32x16_t mfma32h(f16x8_t a, f16x8_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}
// (2^8 a0, 2^8 a1) = h + l as packed fp16 pairs (a0 in the low halves); the difference is
// exact in float
LOCA_DEV void split2h_pair(float a0, float a1, uint32_t& hp, uint32_t& lp) {
  const float s0 = a0 * 256.f, s1 = a1 * 256.f;
  const f32x2_v v = {s0, s1};
  const f16x2_v h = __builtin_convertvector(v, f16x2_v);
  const float r0 = s0 - (float)h[0], r1 = s1 - (float)h[1];
  const f32x2_v r = {r0, r1};
  hp = __builtin_bit_cast(uint32_t, h);
  lp = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2_v));
}
// the 8 fp32 operand values of lane `lane` (rows 8 (lane / 32) + e of the stage, column
// c0 + lane % 32 of the panel) from a swizzled stage, split into two fp16 MFMA operands of
// 2^8 times their value
LOCA_DEV void frag_f32_split2h(const float* stage, int c0, int lane, f16x8_t& fh, f16x8_t& fl) {
  const int hw = lane >> 5, cc = c0 + (lane & 31);
  const float* p = stage + 8 * hw * 256 + 4 * ((cc >> 2) ^ (8 * hw)) + (cc & 3);
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = p[e * 256];
  uint32_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) split2h_pair(v[2 * e], v[2 * e + 1], h[e], l[e]);
  fh = __builtin_bit_cast(f16x8_t, make_uint4(h[0], h[1], h[2], h[3]));
  fl = __builtin_bit_cast(f16x8_t, make_uint4(l[0], l[1], l[2], l[3]));
}
__global__ __launch_bounds__(512) void k_syrk_f32_dl(int64_t d, int64_t k0, int64_t kw, int64_t off,
                                                     float* __restrict__ Fall, int ntile) {
  constexpr int BM = 256, NT = 512, WGN = 4, WM = 128, WN = 64, NBM = WM / 32, NBN = WN / 32;
  constexpr int TILE_F = kS32BK * BM;            // floats of one panel stage
  constexpr int NQ = TILE_F * 4 / 16 / NT;       // 16-byte copies per thread per panel
  constexpr int NCP = 2 * NQ;                    // copies per thread per stage
  static_assert(NCP == NBM, "one copy per fragment row of a stage");
  __shared__ __attribute__((aligned(1024))) float sb0[2 * TILE_F];
  __shared__ __attribute__((aligned(1024))) float sb1[2 * TILE_F];
  __shared__ __attribute__((aligned(1024))) float sb2[2 * TILE_F];
  __shared__ __attribute__((aligned(1024))) float sb3[2 * TILE_F];

  const int T = (int)((d - off + BM - 1) / BM);
  const int logical = xcd_logical((int)blockIdx.x, (int)gridDim.x);
  int I, J;
  upper_tile_c(logical % ntile, T, I, J);
  const int64_t mi = logical / ntile;
  float* F = Fall + mi * d * d;
  const bool diag = I == J;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int wi = wid / WGN, wj = wid % WGN;
  const bool active = !(diag && (wj + 1) * WN <= wi * WM);
  const int64_t cI = off + (int64_t)I * BM, cJ = off + (int64_t)J * BM;
  const int nk = (int)(kw / kS32BK);

  // copy q of this thread fills LDS chunk position (NQ wid + q) * 64 + lane of a panel stage:
  // stage row slot / 64, position slot % 64, holding global chunk position ^ 8 (row / 8)
  int lrow[NQ], lcol[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int slot = (NQ * wid + q) * 64 + lane;
    lrow[q] = slot >> 6;
    lcol[q] = 4 * ((slot & 63) ^ (8 * ((slot >> 9) & 1)));
  }
  const i32x4_t rs = buffer_rsrc(F, (uint32_t)(d * d * 4));
  // Copy j of stage kt: panel j / NQ, chunk j % NQ; stages past the last, and the second
  // panel of a diagonal tile, read nothing (out-of-range offsets return zeros).
  auto issue = [&](float* buf, int kt, int j) {
    const int pnl = j / NQ, q = j % NQ;
    const int64_t row = k0 + (int64_t)kt * kS32BK + lrow[q];
    const int64_t col = (pnl == 0 ? cI : cJ) + lcol[q];
    const bool ok = kt < nk && col < d && !(diag && pnl == 1);
    const uint32_t off_b = ok ? (uint32_t)(4 * (row * d + col)) : kBufOutside;
    const uint32_t dst = (uint32_t)(uintptr_t)(LOCA_LDS void*)buf + pnl * TILE_F * 4 + (NQ * wid + q) * 1024;
    lds_dma16_buf(off_b, rs, __builtin_amdgcn_readfirstlane(dst));
  };

  f32x16_t acc[NBM][NBN];
#pragma unroll
  for (int a = 0; a < NBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;

  const int bpanel = diag ? 0 : TILE_F;
  auto step = [&](float* cur, float* fill, int kt) {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * NCP));  // stage kt landed (this thread's copies)
    barrier_nofence();                               // ... everyone's; slot `fill` no longer read
    f16x8_t bh[NBN], bl[NBN];
#pragma unroll
    for (int b = 0; b < NBN; ++b) frag_f32_split2h(cur + bpanel, wj * WN + 32 * b, lane, bh[b], bl[b]);
#pragma unroll
    for (int a = 0; a < NBM; ++a) {
      __builtin_amdgcn_sched_barrier(0);
      issue(fill, kt + 3, a);
      __builtin_amdgcn_sched_barrier(0);
      f16x8_t ah, al;
      frag_f32_split2h(cur, wi * WM + 32 * a, lane, ah, al);
#pragma unroll
      for (int b = 0; b < NBN; ++b) {
        acc[a][b] = mfma32h(al, bh[b], acc[a][b]);
        acc[a][b] = mfma32h(ah, bl[b], acc[a][b]);
        acc[a][b] = mfma32h(ah, bh[b], acc[a][b]);
      }
    }
  };
#pragma unroll
  for (int j = 0; j < NCP; ++j) issue(sb0, 0, j);
#pragma unroll
  for (int j = 0; j < NCP; ++j) issue(sb1, 1, j);
#pragma unroll
  for (int j = 0; j < NCP; ++j) issue(sb2, 2, j);
  for (int kt = 0; kt < nk; kt += 4) {
    step(sb0, sb3, kt);
    if (kt + 1 < nk) step(sb1, sb0, kt + 1);
    if (kt + 2 < nk) step(sb2, sb1, kt + 2);
    if (kt + 3 < nk) step(sb3, sb2, kt + 3);
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // drain the look-ahead copies before the workgroup ends
  if (!active) return;
#pragma unroll
  for (int a = 0; a < NBM; ++a)
#pragma unroll
    for (int b = 0; b < NBN; ++b) {
      const int64_t col = cJ + wj * WN + 32 * b + mfma32_col(lane);
      const int64_t rb = cI + wi * WM + 32 * a;
      float old[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = rb + mfma32_row(lane, r);
        old[r] = ld_or_zero(F, row * d + col, row < d && col < d && col >= row);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = rb + mfma32_row(lane, r);
        if (row < d && col < d && col >= row) F[row * d + col] = old[r] - acc[a][b][r] * (1.0f / 65536.0f);
      }
    }
}

// ------------------------------------------------------------------ back substitution, one row block

// Right-looking back substitution for row block [p, p + pw) of U M' = Y, where the rows
// of R (= Y) have already received the contributions of every block below:
//   M'_p = U11^{-1} R_p                (computed by every workgroup, stored by x == 0)
//   R_r -= U_{r, p:p+pw} M'_p          for the rows r < p of this workgroup's chunk.
// Grid: x = P-row chunks above p (at least one), y = matrix.  The four waves split the
// P rows; each covers NQ MFMA blocks of the m right-hand-side columns (m <= NQ * BLK).
template <typename T, int NQ>
__global__ __launch_bounds__(kT) void k_back_step(int64_t d, int64_t m, int64_t p, const T* __restrict__ Fall,
                                                  T* __restrict__ Rall, T* __restrict__ Mpall) {
  constexpr int P = Mf<T>::P, BLK = Mf<T>::BLK, KS = Mf<T>::KS, NMB = P / 4 / BLK;
  constexpr int NC = NQ * BLK, LDK = P + 1, LDN = NC + 4;
  __shared__ T sA[P * LDK];  // U11^{-1}, then the rows above
  __shared__ T sB[P * LDN];  // R_p, then M'_p
  const int64_t mi = blockIdx.y;
  const T* F = Fall + mi * d * d;
  T* R = Rall + mi * d * m;
  T* Mp = Mpall + mi * d * m;
  const int pw = (int)((d - p) < P ? (d - p) : P);
  const int64_t r0 = (int64_t)blockIdx.x * P;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int kr = lane / BLK, cr = lane % BLK;
  g2s_block<T, P, P, kT>(sA, LDK, F + p * d + p, d, pw, pw);
  g2s_block<T, P, NC, kT>(sB, LDN, R + p * m, m, pw, m);
  __syncthreads();
  typename Mf<T>::acc_t acc[NMB][NQ];
  auto product = [&]() {
#pragma unroll
    for (int x = 0; x < NMB; ++x)
#pragma unroll
      for (int y = 0; y < NQ; ++y) acc[x][y] = Mf<T>::zero();
    for (int kk = 0; kk < pw; kk += KS) {
      T a[NMB], b[NQ];
#pragma unroll
      for (int x = 0; x < NMB; ++x) a[x] = sA[(wid * (P / 4) + x * BLK + cr) * LDK + kk + kr];
#pragma unroll
      for (int y = 0; y < NQ; ++y) b[y] = sB[(kk + kr) * LDN + y * BLK + cr];
#pragma unroll
      for (int x = 0; x < NMB; ++x)
#pragma unroll
        for (int y = 0; y < NQ; ++y) acc[x][y] = Mf<T>::mma(a[x], b[y], acc[x][y]);
    }
  };
  product();
  __syncthreads();  // everyone is done reading sA / sB
#pragma unroll
  for (int x = 0; x < NMB; ++x)
#pragma unroll
    for (int y = 0; y < NQ; ++y)
#pragma unroll
      for (int r = 0; r < Mf<T>::NR; ++r) {
        const int row = wid * (P / 4) + x * BLK + Mf<T>::row(lane, r);
        const int col = y * BLK + Mf<T>::col(lane);
        const T v = (row < pw && col < m) ? acc[x][y][r] : (T)0;
        sB[row * LDN + col] = v;
        if (blockIdx.x == 0 && row < pw && col < m) Mp[(p + row) * m + col] = v;
      }
  if (r0 >= p) return;  // no rows above in this chunk (only chunk 0 exists when p == 0)
  const int64_t rows = (p - r0) < P ? (p - r0) : P;
  g2s_block<T, P, P, kT>(sA, LDK, F + r0 * d + p, d, rows, pw);
  __syncthreads();
  product();
#pragma unroll
  for (int x = 0; x < NMB; ++x)
#pragma unroll
    for (int y = 0; y < NQ; ++y) {
      T old[Mf<T>::NR];
      const int col = y * BLK + Mf<T>::col(lane);
#pragma unroll
      for (int r = 0; r < Mf<T>::NR; ++r) {
        const int row = wid * (P / 4) + x * BLK + Mf<T>::row(lane, r);
        old[r] = ld_or_zero(R, (r0 + row) * m + col, row < rows && col < m);
      }
#pragma unroll
      for (int r = 0; r < Mf<T>::NR; ++r) {
        const int row = wid * (P / 4) + x * BLK + Mf<T>::row(lane, r);
        if (row < rows && col < m) R[(r0 + row) * m + col] = old[r] - acc[x][y][r];
      }
    }
}

// ------------------------------------------------------------------ back substitution, float

// One launch per row block p (descending) of U M' = Y, right-looking, with M'_p already
// in Mp: workgroups x >= 1 apply R_r -= U_{r,p} M'_p to kBackPer row blocks r above p each;
// workgroup 0 applies it to the block q just above p and then forms M'_q = U_qq^{-1} R_q
// (U_qq^{-1} sits in the diagonal block of F), so the next launch finds M'_q in Mp.  With
// `init`, workgroup 0 only forms M'_p of the last block.  The first operand of every
// product streams from F into registers: MFMA j of a K range of 32 takes k = 16 h + j
// in lane half h, for both operands, so a lane reads 16 consecutive floats of its row.
// The second operand (M'_p, or the updated R_q) sits transposed in LDS.
constexpr int kBackPer = 2;  // row blocks per updating workgroup (the launch waits on its slowest)
template <int NQ, bool V4>
__global__ __launch_bounds__(kT) void k_back_f32(int64_t d, int64_t m, int64_t p, int init, const float* __restrict__ Fall,
                                                 float* __restrict__ Rall, float* __restrict__ Mpall) {
  constexpr int P = 128, LDT = P + 4;
  __shared__ __attribute__((aligned(16))) float sT[NQ * 32 * LDT];  // [column][k]
  const int64_t mi = blockIdx.y;
  const float* F = Fall + mi * d * d;
  float* R = Rall + mi * d * m;
  float* Mp = Mpall + mi * d * m;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, li = lane & 31, h = lane >> 5;
  const int pw = (int)((d - p) < P ? (d - p) : P);

  // acc[q] = sum_{k < kmax} A[32 wid + li][k] T[k][32 q + li] for the wave's 32 rows
  // (rows >= rows_ok of A read as zero)
  auto product = [&](const float* A, int kmax, int rows_ok, f32x16_t (&acc)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    const bool rok = 32 * wid + li < rows_ok;
    const float* arow = A + (int64_t)(rok ? 32 * wid + li : 0) * d;
    // the lane's whole row slice (kmax <= P) is loaded before the first product
    float a[P / 2];
#pragma unroll
    for (int kc = 0; kc < P / 32; ++kc) {
      const int kb = 32 * kc + 16 * h;
      if (V4) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float4 t = ld4_or_zero_ro(arow, kb + 4 * v, rok && kb + 4 * v < kmax);
          a[16 * kc + 4 * v] = t.x; a[16 * kc + 4 * v + 1] = t.y; a[16 * kc + 4 * v + 2] = t.z;
          a[16 * kc + 4 * v + 3] = t.w;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) a[16 * kc + j] = ld_or_zero(arow, kb + j, rok && kb + j < kmax);
      }
    }
#pragma unroll
    for (int kc = 0; kc < P / 32; ++kc) {
      if (32 * kc >= kmax) break;
      const int kb = 32 * kc + 16 * h;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float* tb = sT + (32 * q + li) * LDT + kb;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float4 t = *(const float4*)(tb + 4 * v);
          acc[q] = mfma_f32x2(a[16 * kc + 4 * v], t.x, acc[q]);
          acc[q] = mfma_f32x2(a[16 * kc + 4 * v + 1], t.y, acc[q]);
          acc[q] = mfma_f32x2(a[16 * kc + 4 * v + 2], t.z, acc[q]);
          acc[q] = mfma_f32x2(a[16 * kc + 4 * v + 3], t.w, acc[q]);
        }
      }
    }
  };
  // sT[c][k] = src[k][c] for k < rows, c < m (zero elsewhere); all loads issued first
  auto load_t = [&](const float* src, int rows) {
    constexpr int PER = NQ * 32 * P / kT;
    float v[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + kT * u, k = e / (NQ * 32), c = e % (NQ * 32);
      v[u] = ld_or_zero(src, (int64_t)k * m + c, k < rows && c < m);
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int e = tid + kT * u, k = e / (NQ * 32), c = e % (NQ * 32);
      sT[c * LDT + k] = v[u];
    }
  };
  auto store_mp = [&](int64_t r0, int rows, const f32x16_t (&acc)[NQ]) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * wid + mfma32_row(lane, r), col = 32 * q + li;
        if (row < rows && col < m) Mp[(r0 + row) * m + col] = acc[q][r];
      }
  };

  f32x16_t acc[NQ];
  if (init) {  // M'_p of the last block from its forward-substituted rows
    load_t(R + p * m, pw);
    __syncthreads();
    product(F + p * d + p, pw, pw, acc);
    store_mp(p, pw, acc);
    return;
  }
  load_t(Mp + p * m, pw);
  __syncthreads();
  const int64_t nab = p / P;  // row blocks above p
  if (blockIdx.x == 0) {
    const int64_t r0 = p - P;
    float rv[NQ][16];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * wid + mfma32_row(lane, r), col = 32 * q + li;
        rv[q][r] = ld_or_zero(R, (r0 + row) * m + col, col < m);
      }
    product(F + r0 * d + p, pw, P, acc);
    __syncthreads();  // done with M'_p in LDS
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * wid + mfma32_row(lane, r), col = 32 * q + li;
        sT[col * LDT + row] = col < m ? rv[q][r] - acc[q][r] : 0.f;
      }
    __syncthreads();
    product(F + r0 * d + r0, P, P, acc);
    store_mp(r0, P, acc);
    return;
  }
  for (int c = 0; c < kBackPer; ++c) {
    const int64_t q0 = nab - 2 - kBackPer * ((int64_t)blockIdx.x - 1) - c;
    if (q0 < 0) break;
    const int64_t r0 = q0 * P;
    // the old values of the block's right-hand sides are loaded before the product
    float old[NQ][16];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int col = 32 * q + li;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * wid + mfma32_row(lane, r);
        old[q][r] = ld_or_zero(R, (r0 + row) * m + col, col < m);
      }
    }
    product(F + r0 * d + p, pw, P, acc);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int col = 32 * q + li;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 32 * wid + mfma32_row(lane, r);
        if (col < m) R[(r0 + row) * m + col] = old[q][r] - acc[q][r];
      }
    }
  }
}

// M = D M' (undo the equilibration), float output.
template <typename T>
__global__ void k_unscale(int64_t d, int64_t m, const T* __restrict__ Rall, const T* __restrict__ Dall,
                          float* __restrict__ Mout, int64_t m_bstride) {
  const int64_t mi = blockIdx.y;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= d * m) return;
  Mout[mi * m_bstride + e] = (float)(Dall[mi * d + e / m] * Rall[mi * d * m + e]);
}


// The panel rows in workgroups of eight waves (32 columns each), or four where eight would
// leave compute units idle: eight share the staging and splitting of the first operand, which a
// workgroup of two waves spends longer on than on its products.  Whole solves, two/four waves ->
// four/eight: one matrix of d = 2048 1396 -> 1346 us, 28 of 1536 1233 -> 1198 us, 84 of 3584
// 11.03 -> 10.90 ms (two waves everywhere: 11.16).
hipError_t launch_panel_f32(hipStream_t st, int64_t nm, int64_t d, int64_t k0, int64_t p, float* F, float* R, int64_t m) {
  const int64_t nrem = d - p - 128;
  const int nF = nrem > 0 ? (int)((nrem + 31) / 32) : 0, nc = nF + (int)((m + 31) / 32);
  const bool v4 = d % 4 == 0;
#define LOCA_PANEL(NWV)                                                                                          \
  {                                                                                                              \
    const dim3 g((unsigned)((nc + NWV - 1) / NWV), (unsigned)nm);                                                \
    if (v4) k_panel_f32<NWV, true><<<g, 64 * NWV, 0, st>>>(d, k0, p, F, R, m, nF);                               \
    else k_panel_f32<NWV, false><<<g, 64 * NWV, 0, st>>>(d, k0, p, F, R, m, nF);                                 \
  }
  if (nm * ((nc + 7) / 8) >= 256) LOCA_PANEL(8)
  else LOCA_PANEL(4)
#undef LOCA_PANEL
  return hipGetLastError();
}

template <typename T>
size_t solve_ws_t(int64_t nb, int64_t d, int64_t m, int64_t nl, int64_t r_prev) {
  const int64_t nm = nb * nl;
  size_t s = align256(sizeof(T) * nm * d * d);  // F
  s += align256(sizeof(T) * nm * d * m);         // R
  s += align256(sizeof(T) * nm * d);             // D
  s += align256(sizeof(T) * nm * d * m);         // M' (back substitution output)
  s += align256(sizeof(double) * nb * d * (r_prev > 0 ? r_prev : 1));  // S Lp
  s += 256;                                                            // lambdas
  return s;
}

// The launches of a solve group in submission order.  With `ops` null each launch is
// issued at once; otherwise it is kept as a closure (every value it needs copied in) for
// the caller, which interleaves the groups on the host: a group's launches then reach
// its stream while the other groups are still being submitted, instead of after them.
struct Emit {
  std::vector<std::function<hipError_t()>>* ops = nullptr;
  int stagger_at = -1;  // index of the op that records the stagger event, when kept
  hipError_t operator()(std::function<hipError_t()> f) {
    if (!ops) return f();
    ops->push_back(std::move(f));
    return hipSuccess;
  }
};

// The solve of the blocks [b0, b0 + nbg) (all their lambdas) on stream st; workspace
// regions are those of the whole call.  `after_diag`, when given, is recorded after the
// first diagonal-block launch.
template <typename T, typename ST>
hipError_t run_group(const SolveArgs& a, int64_t b0, int64_t nbg, hipStream_t st, T* Fw, T* Rw, T* Dw, T* Mpw,
                     double* SLpw, const double* dlam, hipEvent_t after_diag, Emit& emit) {
  const int64_t d = a.d, m = a.r_prev + a.k, nl = a.n_lambda, nm = nbg * nl, mi0 = b0 * nl;
  T* F = Fw + mi0 * d * d;
  T* R = Rw + mi0 * d * m;
  T* D = Dw + mi0 * d;
  T* Mp = Mpw + mi0 * d * m;
  // trailing updates through the direct-to-LDS kernel when a matrix fits 31-bit byte offsets
  const bool syrk_dl = sizeof(T) == 4 && d % 4 == 0 && 4 * d * d < ((int64_t)1 << 31);
  // an earlier call's factor (fp64 only): only the right-hand-side tiles of each launch run
  const bool reuse = a.reuse_factor && sizeof(T) == 8;
  if (a.reuse_factor && !reuse) return hipErrorNotSupported;
  double* SLp = SLpw + b0 * d * (a.r_prev > 0 ? a.r_prev : 1);
  int32_t* info = a.dev_info + mi0;
  const ST* S = (const ST*)a.S + b0 * a.s_bstride;
  const ST* K = (const ST*)a.K + b0 * a.k_bstride;
  const int64_t r_prev = a.r_prev, s_bstride = a.s_bstride, k_bstride = a.k_bstride;
  const float* lp = a.lp ? a.lp + b0 * a.lp_bstride : nullptr;
  const int64_t lp_bstride = a.lp_bstride;
  hipError_t e = emit([=]() {
    if (r_prev > 0) {
      hipError_t e = sym_mul<ST>(st, nbg, d, r_prev, S, s_bstride, lp, lp_bstride, r_prev, 1, SLp);
      if (e != hipSuccess) return e;
    }
    if (reuse) {  // D and F from the earlier call: the right-hand sides only
      dim3 gr((unsigned)((d * m + 255) / 256), (unsigned)nm);
      k_equil_rhs<T, ST><<<gr, 256, 0, st>>>(d, m, r_prev, K, k_bstride, SLp, (int)nl, D, R);
      return hipGetLastError();
    }
    dim3 g((unsigned)((d + 255) / 256), (unsigned)nm);
    k_equil_diag<T, ST><<<g, 256, 0, st>>>(d, S, s_bstride, dlam, (int)nl, D);
    dim3 g2((unsigned)((d + kEqRows - 1) / kEqRows), (unsigned)nbg);
    bool v4 = false;
    if constexpr (sizeof(T) == 4 && sizeof(ST) == 4)
      v4 = d % 4 == 0 && s_bstride % 4 == 0 && ((uintptr_t)S & 15) == 0;
    if (v4) {
      const dim3 g4((unsigned)((d + kEqRows - 1) / kEqRows), (unsigned)((d + kEqCols - 1) / kEqCols), (unsigned)nbg);
      k_equil_setup_v4<<<g4, kEqCols / 4, 0, st>>>(d, m, r_prev, (const float*)S, s_bstride, (const float*)K,
                                                   k_bstride, SLp, dlam, (int)nl, (const float*)D, (float*)F,
                                                   (float*)R);
    } else {
      k_equil_setup<T, ST><<<g2, 256, 0, st>>>(d, m, r_prev, S, s_bstride, K, k_bstride, SLp, dlam, (int)nl, D, F, R);
    }
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  // Blocked right-looking factorization with the forward substitution of the RHS
  // carried along.  The trailing matrix is updated once per super-panel of kSuper
  // panels (one pass over it per kSuper * P columns); inside a super-panel each panel
  // first receives the contributions of the super-panel's earlier panels (a strip
  // update of its own rows), then is factored (diagonal block) and solved (row panel).
  constexpr int P = Mf<T>::P, kSuper = 4;  // eight made the fp32 solves 5-20% slower (their strips' six products)
  const bool x6 = sizeof(T) == 4 && d % 4 == 0;
  const bool x6r = x6 && m % 4 == 0 && m <= 256;  // right-hand sides inside the same launches
  const int64_t TM = (m + P - 1) / P;
  for (int64_t P0 = 0; P0 < d; P0 += kSuper * P) {
    const int64_t P1 = (d - P0) < kSuper * P ? d : P0 + kSuper * P;
    for (int64_t pp = P0; pp < P1; pp += P) {
      const int64_t pw = (d - pp) < P ? (d - pp) : P;
      const int64_t nrem = d - pp - pw;
      const int64_t nchF = (nrem + P - 1) / P;
      if (pp > P0 && sizeof(T) == 8) {
        e = emit([=]() {
          const int64_t T2 = (d - pp + P - 1) / P;
          if (reuse)
            k_panel_product<T, kTrailing><<<dim3((unsigned)TM, (unsigned)nm), kT, 0, st>>>(
                d, m, 0, P0, pp - P0, pp, 1, (int)T2, F, R);
          else
            k_panel_product<T, kTrailing><<<dim3((unsigned)(T2 + TM), (unsigned)nm), kT, 0, st>>>(
                d, m, 0, P0, pp - P0, pp, 1, 0, F, R);
          return hipGetLastError();
        });
        if (e != hipSuccess) return e;
      }
      const bool rec = after_diag && pp == 0;
      if (rec && emit.ops) emit.stagger_at = (int)emit.ops->size();
      e = emit([=]() {
        if (!reuse) {
          if (d % 4 == 0) k_diag_inv<T, P, true><<<(unsigned)nm, 4 * P, 0, st>>>(d, P0, pp, F, info);
          else k_diag_inv<T, P, false><<<(unsigned)nm, 4 * P, 0, st>>>(d, P0, pp, F, info);
        }
        const hipError_t er = hipGetLastError();
        if (er != hipSuccess || !rec) return er;
        return hipEventRecord(after_diag, st);
      });
      if (e != hipSuccess) return e;
      e = emit([=]() {
        if constexpr (sizeof(T) == 4) {
          return launch_panel_f32(st, nm, d, P0, pp, (float*)F, (float*)R, m);
        } else if (reuse) {
          k_panel_product<T, kRowPanel><<<dim3((unsigned)TM, (unsigned)nm), kT, 0, st>>>(d, m, pp, 0, 0, 0, 0,
                                                                                          (int)nchF, F, R);
        } else {
          k_panel_product<T, kRowPanel><<<dim3((unsigned)(nchF + TM), (unsigned)nm), kT, 0, st>>>(
              d, m, pp, 0, 0, 0, 0, 0, F, R);
        }
        return hipGetLastError();
      });
      if (e != hipSuccess) return e;
    }
    if (P1 < d) {
      e = emit([=]() {
        const int64_t T2 = (d - P1 + P - 1) / P, nU = T2 * (T2 + 1) / 2;
        if (x6) {
          const int64_t T6 = (d - P1 + 255) / 256;
          const int nF = (int)(T6 * (T6 + 1) / 2);
          if (syrk_dl) {
            k_syrk_f32_dl<<<dim3((unsigned)(nF * nm)), 512, 0, st>>>(d, P0, P1 - P0, P1, (float*)F, nF);
            if (x6r)
              k_panel_x6<kX6TrailRhs><<<dim3((unsigned)T6, (unsigned)nm, (unsigned)((m + 31) / 32)), 512, 0, st>>>(
                  d, P0, P1 - P0, P1, (float*)F, (float*)R, m, 0);
          } else {
            k_panel_x6<kX6Trail><<<dim3((unsigned)(nF + (x6r ? T6 : 0)), (unsigned)nm), 512, 0, st>>>(
                d, P0, P1 - P0, P1, (float*)F, (float*)R, m, nF);
          }
          if (!x6r)
            k_panel_product<T, kTrailing><<<dim3((unsigned)(T2 * TM), (unsigned)nm), kT, 0, st>>>(
                d, m, 0, P0, P1 - P0, P1, 0, (int)nU, F, R);
        } else if (reuse) {
          k_panel_product<T, kTrailing><<<dim3((unsigned)(T2 * TM), (unsigned)nm), kT, 0, st>>>(
              d, m, 0, P0, P1 - P0, P1, 0, (int)nU, F, R);
        } else {
          k_panel_product<T, kTrailing><<<dim3((unsigned)(nU + T2 * TM), (unsigned)nm), kT, 0, st>>>(
              d, m, 0, P0, P1 - P0, P1, 0, 0, F, R);
        }
        return hipGetLastError();
      });
      if (e != hipSuccess) return e;
    }
  }
  if constexpr (sizeof(T) == 4) {
    const int64_t plast = ((d - 1) / P) * P;
    const int nq = (int)((m + 31) / 32);  // m <= 128 (checked by the API)
    auto back = [=](int64_t pp, int init, unsigned gx) {
      const dim3 grid(gx, (unsigned)nm);
      const bool v4 = d % 4 == 0 && m <= 128;
#define LOCA_BACK(NQ)                                                                                \
  if (v4) k_back_f32<NQ, true><<<grid, kT, 0, st>>>(d, m, pp, init, (const float*)F, (float*)R, (float*)Mp); \
  else k_back_f32<NQ, false><<<grid, kT, 0, st>>>(d, m, pp, init, (const float*)F, (float*)R, (float*)Mp);
      if (nq <= 1) { LOCA_BACK(1) }
      else if (nq <= 2) { LOCA_BACK(2) }
      else { LOCA_BACK(4) }
#undef LOCA_BACK
      return hipGetLastError();
    };
    if ((e = emit([=]() { return back(plast, 1, 1); })) != hipSuccess) return e;
    for (int64_t pp = plast; pp >= P; pp -= P) {
      const int64_t nab = pp / P;
      if ((e = emit([=]() { return back(pp, 0, (unsigned)(1 + (nab - 1 + kBackPer - 1) / kBackPer)); })) != hipSuccess)
        return e;
    }
  } else {
    for (int64_t pp = ((d - 1) / P) * P; pp >= 0; pp -= P) {
      e = emit([=]() {
        const dim3 grid((unsigned)(pp > 0 ? (pp + P - 1) / P : 1), (unsigned)nm);
        const int nq = (int)((m + Mf<T>::BLK - 1) / Mf<T>::BLK);  // m <= 128 (checked by the API)
        if (nq <= 1) k_back_step<T, 1><<<grid, kT, 0, st>>>(d, m, pp, F, R, Mp);
        else if (nq <= 2) k_back_step<T, 2><<<grid, kT, 0, st>>>(d, m, pp, F, R, Mp);
        else if (nq <= 4) k_back_step<T, 4><<<grid, kT, 0, st>>>(d, m, pp, F, R, Mp);
        else k_back_step<T, 8><<<grid, kT, 0, st>>>(d, m, pp, F, R, Mp);
        return hipGetLastError();
      });
      if (e != hipSuccess) return e;
    }
  }
  float* m_out = a.m_out + mi0 * a.m_bstride;
  const int64_t m_bstride = a.m_bstride;
  const bool dense = a.w_dense_out != nullptr;
  if (dense && r_prev != 0) return hipErrorNotSupported;
  const float* cb = dense ? a.credit_b + b0 * a.b_bstride : nullptr;
  const int64_t b_bstride = a.b_bstride, w_bstride = a.w_bstride;
  float* w_out = dense ? a.w_dense_out + mi0 * a.w_bstride : nullptr;
  return emit([=]() {
    k_unscale<T><<<dim3((unsigned)((d * m + 255) / 256), (unsigned)nm), 256, 0, st>>>(d, m, Mp, D, m_out, m_bstride);
    const hipError_t er = hipGetLastError();
    if (er != hipSuccess || !dense) return er;
    // W = M B~ (no earlier adapter: the right factor is B~ alone)
    return launch_lowrank_product(st, nm, d, d, m, m_out, m_bstride, m, cb, b_bstride, nl, d, w_out, w_bstride);
  });
}

// Extra streams and events per device, made on first use: the only state the library
// keeps.  The blocks of a large call are split into kGroups groups on the caller's stream
// and kGroups - 1 internal streams, group g started once group g - 1 has factored its
// first diagonal block: the latency-bound launches of one group (diagonal blocks,
// back substitution: few workgroups each) then run beside the matrix-core updates of the
// other instead of leaving most of the GPU idle.  A call whose factorizations are below
// kGroupFlops runs as one group: there the launches, not the matrix cores, set the time.
// Whole solves with one, two and three groups: 84 matrices of d = 3584 11.98 / 11.55 /
// 11.73 ms, 48 of 5120 18.91 / 17.84 / 17.98 ms; 28 of 1536 (3.4e10) 1253 / 1275 / 1332 us,
// 24 of 896 736 / 938 / 1125 us.
//
// The streams and events are shared by every call on a device, so creating them and the
// whole submission of a call that uses them (fork record, waits, launches, join records)
// happen under the device's mutex.  A wait on an event takes the event's state at the time
// the wait is enqueued, so once a call has left the critical section its internal work is
// ordered behind its own fork point and the next call may record the events again.
constexpr int kGroups = 2;
constexpr double kGroupFlops = 5e10;
constexpr int kMaxDevices = 64;
struct Aux {
  std::mutex mu;
  bool ready = false;
  hipStream_t s[kGroups] = {};
  hipEvent_t fork = nullptr;
  hipEvent_t stagger[kGroups] = {};
  hipEvent_t join[kGroups] = {};
};
Aux g_aux[kMaxDevices];

// With the device's mutex held: the internal streams and events exist.
hipError_t aux_ready(Aux& x) {
  if (x.ready) return hipSuccess;
  hipError_t e;
  for (int g = 1; g < kGroups; ++g) {
    if (!x.stagger[g] && (e = hipEventCreateWithFlags(&x.stagger[g], hipEventDisableTiming)) != hipSuccess) return e;
    if (!x.join[g] && (e = hipEventCreateWithFlags(&x.join[g], hipEventDisableTiming)) != hipSuccess) return e;
    if (!x.s[g] && (e = hipStreamCreateWithFlags(&x.s[g], hipStreamNonBlocking)) != hipSuccess) return e;
  }
  if (!x.fork && (e = hipEventCreateWithFlags(&x.fork, hipEventDisableTiming)) != hipSuccess) return e;
  x.ready = true;
  return hipSuccess;
}

template <typename T, typename ST>
hipError_t run_solve(const SolveArgs& a) {
  const int64_t d = a.d, m = a.r_prev + a.k, nl = a.n_lambda, nm = a.nb * nl;
  char* p = a.ws;
  T* F = (T*)p; p += align256(sizeof(T) * nm * d * d);
  T* R = (T*)p; p += align256(sizeof(T) * nm * d * m);
  T* D = (T*)p; p += align256(sizeof(T) * nm * d);
  T* Mp = (T*)p; p += align256(sizeof(T) * nm * d * m);
  double* SLp = (double*)p;
  Lams lams;
  for (int i = 0; i < 8; ++i) lams.v[i] = (i < nl) ? a.lambdas[i] : 0.0;
  double* dlam = (double*)(p + align256(sizeof(double) * a.nb * d * (a.r_prev > 0 ? a.r_prev : 1)));
  // the host lambdas travel by value into a one-wave kernel (no copy from pageable memory)
  k_set_lambdas<<<1, 64, 0, a.stream>>>(lams, dlam, (int)nl);
  k_fill_zero_i32<<<(unsigned)((nm + 255) / 256), 256, 0, a.stream>>>(a.dev_info, nm);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool large = (double)nm * (double)d * (double)d * (double)d / 3.0 >= kGroupFlops;
  const int G = large ? (int)(a.nb < kGroups ? a.nb : kGroups) : 1;
  if (G < 2) {
    Emit now;
    return run_group<T, ST>(a, 0, a.nb, a.stream, F, R, D, Mp, SLp, dlam, nullptr, now);
  }
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  Aux* x = &g_aux[dev];
  std::lock_guard<std::mutex> hold(x->mu);
  if ((e = aux_ready(*x)) != hipSuccess) return e;
  if ((e = hipEventRecord(x->fork, a.stream)) != hipSuccess) return e;
  // Every group's launches are recorded first, then submitted round-robin, one launch
  // per group in turn.  Group g joins once group g - 1 has submitted its first diagonal
  // block and the event after it; its stream waits for that event, so its GPU work
  // starts behind that block.
  std::vector<std::function<hipError_t()>> ops[kGroups];
  int stagger_at[kGroups];
  hipStream_t sts[kGroups];
  for (int g = 0; g < G; ++g) {
    const int64_t b0 = a.nb * g / G, b1 = a.nb * (g + 1) / G;
    sts[g] = g == 0 ? a.stream : x->s[g];
    hipEvent_t after = g + 1 < G ? x->stagger[g + 1] : nullptr;
    Emit keep;
    keep.ops = &ops[g];
    if ((e = run_group<T, ST>(a, b0, b1 - b0, sts[g], F, R, D, Mp, SLp, dlam, after, keep)) != hipSuccess) return e;
    stagger_at[g] = keep.stagger_at;
    if (after && keep.stagger_at < 0) return hipErrorUnknown;  // every group has a first diagonal block
  }
  size_t pos[kGroups] = {};
  bool joined[kGroups] = {};
  joined[0] = true;
  for (bool left = true; left;) {
    left = false;
    for (int g = 0; g < G; ++g) {
      if (!joined[g]) {
        if (!joined[g - 1] || pos[g - 1] <= (size_t)stagger_at[g - 1]) {
          left = true;
          continue;
        }
        if ((e = hipStreamWaitEvent(sts[g], x->fork, 0)) != hipSuccess) return e;
        if ((e = hipStreamWaitEvent(sts[g], x->stagger[g], 0)) != hipSuccess) return e;
        joined[g] = true;
      }
      if (pos[g] < ops[g].size()) {
        if ((e = ops[g][pos[g]++]()) != hipSuccess) return e;
        left = left || pos[g] < ops[g].size();
      }
    }
  }
  for (int g = 1; g < G; ++g) {
    if ((e = hipEventRecord(x->join[g], x->s[g])) != hipSuccess) return e;
    if ((e = hipStreamWaitEvent(a.stream, x->join[g], 0)) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

size_t ridge_solve_ws(int64_t nb, int64_t d, int64_t m, int64_t n_lambda, loca_dtype acc) {
  // m counts r_prev + k; the S Lp scratch is sized for m columns (>= r_prev)
  size_t s = acc == LOCA_F64 ? solve_ws_t<double>(nb, d, m, n_lambda, m) : solve_ws_t<float>(nb, d, m, n_lambda, m);
  return s;
}

hipError_t launch_chol_inv64(hipStream_t s, int64_t n, double* A, int32_t* info) {
  k_diag_inv<double, 64, true><<<1, 256, 0, s>>>(n, 0, 0, A, info);
  return hipGetLastError();
}

hipError_t launch_ridge_solve(const SolveArgs& a) {
  if (a.acc == LOCA_F64) return run_solve<double, double>(a);
  return run_solve<float, float>(a);
}

hipError_t launch_sym_mul_f64(hipStream_t s, int64_t nb, int64_t d, int64_t r, const double* S, int64_t s_bstride,
                              const float* L, int64_t l_bstride, int64_t l_sj, int64_t l_sc, double* out) {
  return sym_mul<double>(s, nb, d, r, S, s_bstride, L, l_bstride, l_sj, l_sc, out);
}

}  // namespace loca

// k_head.hip -- the head in the paper's order (Section S11): the top-layer error taken
// to the hidden width once for all blocks,
//   e_t = W_u^T E_t,   E_t = w_t (softmax(z_t) - onehot(y_t))   (the target's error term,
//                                                               Lemma S3.1's head error),
// so that each block then applies only V_k^T e_t (loca_credit_from_top_error).  It pays
// off when the blocks' folded factors A~ = W_u V_k together are wider than the hidden
// width (L k > d).
//
//   1. k_softmax_stats: per token the row maximum m_t and s_t = sum_c exp(z_tc - m_t)
//      (one workgroup per token, fixed-order combination of the partial pairs);
//   2. k_top_error_gemm: part_z = P W_u over the vocabulary range z, P_tc = w_t exp(z_tc -
//      m_t) / s_t formed in registers from the logits, split into bf16 hi + lo parts
//      (about 16 significant bits), each multiplied by the exact bf16 W_u on the matrix
//      cores (v_mfma_f32_32x32x16_bf16; W_u read transposed from LDS);
//   3. k_top_error_reduce: e = sum_z part_z in a fixed order (fp64), minus w_t W_u[y_t].
// With at most 64 columns the product takes one pass over the logits instead (an online
// softmax feeding the matrix cores, launch_softmax_product_online in k_fused.hip).
//
// The same product serves the folded order for a large vocabulary (loca_error_targets
// with bf16 A~): the right operand is then the blocks' A~ side by side (column j of
// group j / kc), so one launch forms Y_b = E A~_b for every block.
#include <algorithm>

#include "loca_launch.h"
#include "loca_bf16.h"

namespace loca {

namespace {

constexpr int kHT = 256;

// dev_info: INT32_MAX while no bad label is seen, then 1 + the smallest bad row, or
// LOCA_INFO_NONFINITE once a row's softmax sum is not finite; INT32_MAX becomes 0 at the end
__global__ void k_fill_i32_head(int32_t* p) {
  if (threadIdx.x == 0) *p = INT32_MAX;
}
__global__ void k_finish_info_head(int32_t* p) {
  if (threadIdx.x == 0 && *p == INT32_MAX) *p = 0;
}

// (m, s) of two disjoint parts of a row combined into one
LOCA_DEV void ms_combine(float& m, float& s, float m2, float s2) {
  if (s2 == 0.f) return;
  if (s == 0.f) { m = m2; s = s2; return; }
  const float mm = fmaxf(m, m2);
  s = s * __expf(m - mm) + s2 * __expf(m2 - mm);
  m = mm;
}

// 8 consecutive logits as floats (a 16-byte aligned bf16 chunk or two float4)
LOCA_DEV void load8(const uint16_t* p, float (&v)[8]) {
  const uint4 u = *(const uint4*)p;
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
LOCA_DEV void load8(const float* p, float (&v)[8]) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}

// One workgroup per token.  A 16-byte aligned row is read in chunks of 8 logits, two
// chunks in flight per thread: each chunk's maximum first rescales the running sum once,
// then its 8 terms are added.  Other rows (and the tail past a multiple of 8) go one
// logit at a time.
template <typename LT>
__global__ __launch_bounds__(kHT) void k_softmax_stats(int64_t n, int64_t V, const LT* __restrict__ z, int64_t ld,
                                                       const int32_t* __restrict__ labels, float* __restrict__ ms,
                                                       int32_t* __restrict__ dev_info) {
  __shared__ float sm[kHT], ss[kHT];
  const int64_t t = blockIdx.x;
  const LT* zt = z + t * ld;
  float m = -INFINITY, s = 0.f;  // s == 0: nothing seen yet
  auto add8 = [&](const float (&v)[8]) {
    float mx = v[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, v[i]);
    if (mx > m) {
      s *= __expf(m - mx);
      m = mx;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) s += __expf(v[i] - m);
  };
  int64_t c0 = 0;
  if ((((uintptr_t)zt) & 15) == 0) {
    const int64_t nch = V / 8;
    int64_t c = threadIdx.x;
    for (; c + kHT < nch; c += 2 * kHT) {
      float va[8], vb[8];
      load8(zt + 8 * c, va);
      load8(zt + 8 * (c + kHT), vb);
      add8(va);
      add8(vb);
    }
    for (; c < nch; c += kHT) {
      float va[8];
      load8(zt + 8 * c, va);
      add8(va);
    }
    c0 = nch * 8;
  }
  for (int64_t c = c0 + threadIdx.x; c < V; c += kHT) {
    const float v = load_as_f32(zt + c);
    if (v > m) {
      s = s * __expf(m - v) + 1.f;
      m = v;
    } else {
      s += __expf(v - m);
    }
  }
  sm[threadIdx.x] = m;
  ss[threadIdx.x] = s;
  __syncthreads();
  for (int h = kHT / 2; h > 0; h >>= 1) {  // pairs (i, i + h): a fixed tree
    if ((int)threadIdx.x < h) {
      float a = sm[threadIdx.x], b = ss[threadIdx.x];
      ms_combine(a, b, sm[threadIdx.x + h], ss[threadIdx.x + h]);
      sm[threadIdx.x] = a;
      ss[threadIdx.x] = b;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    ms[2 * t] = sm[0];
    ms[2 * t + 1] = ss[0];
    const int32_t yt = labels[t];
    if (yt < 0 || yt >= V) atomicMin(dev_info, (int32_t)(t + 1));
    // a NaN or +inf logit makes the sum NaN (a -inf logit is an excluded class and is fine)
    if (!__builtin_isfinite(ss[0])) atomicMin(dev_info, (int32_t)LOCA_INFO_NONFINITE);
  }
}

// Tiles of 128 tokens x 32 NB columns, one vocabulary range each; four waves of 32 tokens and all
// the columns.  The logits of a wave's tokens are the first operand as they lie: lane l's 16 bytes
// are token l % 32 and eight consecutive entries, so P = w exp(z - m) / s is formed in registers,
// once per column tile, and split into bf16 hi + lo (packed hardware conversions, loca_bf16.h).
// The right operand's rows go straight to LDS in blocks of 64 entries (two stages of 32 rows x 256
// columns, swizzled as in loca_common.h), double-buffered; a block's logits are loaded one block
// ahead.  The column tiles of one token tile are neighbours on an XCD, so the logits come from
// beyond its L2 once.  Column j of the right operand is column j % kc of group j / kc:
// W + (j / kc) w_bstride (V x kc bf16 each); d = total columns.  Requires ld % 8 == 0 (bf16) or % 4
// == 0 (f32), kc % 8 == 0, d % kc == 0, kchunk % 8 == 0.
//
// Bound by the matrix cores (the split doubles their work; busy for 54% of the cycles, at 1.73 GHz
// under this load) and the vector instructions beside them (exponentials and split, 46% of the
// cycles; the waves wait for 11%): n = 4096, V = 151936, 896 columns took 4.50 ms in 128-column tiles that formed P seven times and
// waited for each 32-entry stage's loads; the figures now stand at the launch.
__device__ const uint32_t g_zero16[4] __attribute__((aligned(16))) = {0, 0, 0, 0};
constexpr int kHT2 = 256, kHM = 128, kHK = 64;  // threads, token rows, vocabulary per block
template <typename LT> struct LogitChunk;       // eight logits
template <> struct LogitChunk<uint16_t> {
  uint4 v;
  // the chunk at p + c, of which [c, end) exists; past it the chunk at p + safe
  LOCA_DEV void load(const uint16_t* p, int64_t c, int64_t end, int64_t safe) { v = *(const uint4*)(p + (c < end ? c : safe)); }
  LOCA_DEV float get(int i) const {
    const uint32_t x = i < 2 ? v.x : (i < 4 ? v.y : (i < 6 ? v.z : v.w));
    return (i & 1) ? bf16_hi(x) : bf16_lo(x);
  }
};
template <> struct LogitChunk<float> {
  float4 a, b;
  LOCA_DEV void load(const float* p, int64_t c, int64_t end, int64_t safe) {
    a = *(const float4*)(p + (c < end ? c : safe));
    b = *(const float4*)(p + (c + 4 < end ? c + 4 : safe));
  }
  LOCA_DEV float get(int i) const {
    const float4 t = i < 4 ? a : b;
    return (i & 3) == 0 ? t.x : ((i & 3) == 1 ? t.y : ((i & 3) == 2 ? t.z : t.w));
  }
};

template <typename LT, int NB>
__global__ __launch_bounds__(kHT2, 2) void k_top_error_gemm(int64_t n, int64_t V, int64_t d, const LT* __restrict__ z,
                                                           int64_t ld, const float* __restrict__ w,
                                                           const float* __restrict__ ms,
                                                           const uint16_t* __restrict__ wu, int64_t kc,
                                                           int64_t w_bstride, int ntr, int nct, int64_t kchunk,
                                                           float* __restrict__ part) {
  constexpr int BLK = kHK * 256;  // bf16 of a block in LDS (rows of 256 columns, whatever NB)
  __shared__ __attribute__((aligned(1024))) uint16_t sb0[BLK];
  __shared__ __attribute__((aligned(1024))) uint16_t sb1[BLK];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6), lh = lane >> 5;
  const int logical = xcd_logical((int)blockIdx.x, (int)gridDim.x);
  const int ct = logical % nct, rt = (logical / nct) % ntr, sp = logical / (nct * ntr);
  const int64_t j0 = (int64_t)ct * 32 * NB, t0 = (int64_t)rt * kHM + 32 * wid;
  const int64_t cb = (int64_t)sp * kchunk, ce = std::min<int64_t>(V, cb + kchunk);
  const int nblk = (int)((ce - cb + kHK - 1) / kHK);

  const int64_t t = t0 + (lane & 31);
  const bool tok = t < n;
  const LT* zr = z + (tok ? t : 0) * ld;
  const float rmax = tok ? ms[2 * t] : 0.f;
  const float rscale = tok ? (w ? w[t] : 1.f) / ms[2 * t + 1] : 0.f;

  // copy q of this thread: row 8 q + tid / 32 of a block, 16-byte chunk ch of the columns (the same
  // for every q).  Rows past the range are zeros: they meet whatever the logits' row holds there,
  // kept finite by the cap of its exponent at 0 (no effect on the row's own entries).  Columns past
  // the last repeat it and are not stored.
  const int wrow = tid >> 5, ch = (tid & 31) ^ dl_swz(wrow);
  const int64_t jc = std::min<int64_t>(j0 + 8 * ch, d - 8), grp = jc / kc;
  const uint16_t* wp = wu + grp * w_bstride + (jc - grp * kc);
  auto issue = [&](uint16_t* buf, int64_t c0) {
    const uint32_t dst = (uint32_t)(uintptr_t)(LOCA_LDS void*)buf + (uint32_t)wid * 1024u;
    if (ch < 4 * NB)
#pragma unroll
      for (int q = 0; q < kHK / 8; ++q)
      {
        const int64_t r = c0 + 8 * q + wrow;
        lds_dma16(r < ce ? wp + r * kc : (const uint16_t*)g_zero16, __builtin_amdgcn_readfirstlane(dst + q * 4096u));
      }
  };
  auto load_z = [&](LogitChunk<LT> (&zb)[4], int64_t c0) {
#pragma unroll
    for (int s = 0; s < 4; ++s) zb[s].load(zr, c0 + 16 * s + 8 * lh, ce, cb);
  };

  f32x16_t acc[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;

  auto block = [&](uint16_t* cur, uint16_t* nxt, const LogitChunk<LT> (&zc)[4], LogitChunk<LT> (&zn)[4], int b) {
    const int64_t c0 = cb + (int64_t)b * kHK;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // this thread's copies and logits of the block landed
    barrier_nofence();                         // ... everyone's; the other buffer is no longer read
    if (b + 1 < nblk) {
      issue(nxt, c0 + kHK);
      load_z(zn, c0 + kHK);
    }
    // P of step s + 1 is formed beside the products of step s (and no further ahead: the
    // scheduling barrier keeps the registers of one step in flight)
    bf16x8_t fh, fl, gh, gl;
    auto form = [&](int s, bf16x8_t& oh, bf16x8_t& ol) {
      uint32_t ph[4], pl[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p0 = __expf(fminf(zc[s].get(2 * i) - rmax, 0.f)) * rscale;
        const float p1 = __expf(fminf(zc[s].get(2 * i + 1) - rmax, 0.f)) * rscale;
        ph[i] = cvt_pk_bf16(p0, p1);
        pl[i] = cvt_pk_bf16(p0 - bf16_lo(ph[i]), p1 - bf16_hi(ph[i]));
      }
      oh = __builtin_bit_cast(bf16x8_t, make_uint4(ph[0], ph[1], ph[2], ph[3]));
      ol = __builtin_bit_cast(bf16x8_t, make_uint4(pl[0], pl[1], pl[2], pl[3]));
    };
    form(0, fh, fl);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      __builtin_amdgcn_sched_barrier(0);
      bf16x8_t fb[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) fb[q] = frag32_tr_swz(cur + (s >> 1) * (BLK / 2), 32 * q, 16 * (s & 1), lane);
#pragma unroll
      for (int q = 0; q < NB; ++q) acc[q] = mfma32(fh, fb[q], acc[q]);
      if (s < 3) form(s + 1, gh, gl);
#pragma unroll
      for (int q = 0; q < NB; ++q) acc[q] = mfma32(fl, fb[q], acc[q]);
      fh = gh;
      fl = gl;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  LogitChunk<LT> za[4], zb[4];
  issue(sb0, cb);
  load_z(za, cb);
  for (int b = 0; b < nblk; b += 2) {
    block(sb0, sb1, za, zb, b);
    if (b + 1 < nblk) block(sb1, sb0, zb, za, b + 1);
  }
  float* out = part + (int64_t)sp * n * d;
#pragma unroll
  for (int q = 0; q < NB; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t tr = t0 + mfma32_row(lane, r), j = j0 + 32 * q + mfma32_col(lane);
      if (tr < n && j < d) out[tr * d + j] = acc[q][r];
    }
}

// out[(j / kc) o_bstride + t ld_o + j % kc] = sum_z part_z[t][j] (fp64, in order) - w_t W[y_t][j]
__global__ void k_top_error_reduce(int64_t n, int64_t d, int nsplit, const float* __restrict__ part,
                                   const float* __restrict__ w, const int32_t* __restrict__ labels, int64_t V,
                                   const uint16_t* __restrict__ wu, int64_t kc, int64_t w_bstride,
                                   float* __restrict__ out, int64_t ld_o, int64_t o_bstride) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * d) return;
  const int64_t t = e / d, j = e % d;
  const int64_t grp = j / kc, jc = j - grp * kc;
  double s = 0.0;
  for (int zc = 0; zc < nsplit; ++zc) s += (double)part[(int64_t)zc * n * d + e];
  const int32_t yt = labels[t];
  if (yt >= 0 && yt < V)
    s -= (double)(w ? w[t] : 1.f) * (double)bf16_to_f32(wu[grp * w_bstride + (int64_t)yt * kc + jc]);
  out[grp * o_bstride + t * ld_o + jc] = (float)s;
}

// Column tiles of at most 256, evenly cut in 32s (nb of them, as instantiated); the vocabulary in
// ns ranges of 32-entry multiples.  Never fewer ranges than 2048 tiles of 128 x 128 (of 128 x 64 up
// to 64 columns) would make, of at least 256 entries: the sums run in float32, and longer ones cost
// precision (n = 4096, V = 151936, 896 columns: rms error against float64 7.0e-8 in ranges of 594
// blocks, 6.2e-8 in ranges of 198, for 2% of the time).  From there up to twice as many, the count
// with the least rounds of 512 workgroups (two fit a compute unit; a last round of one each is the
// shorter) times blocks per range, an added range costing its partial sums' way through memory
// (about 1e-6 blocks per value, at 1.6 us a block and 5 TB/s).  Beyond twice the workspace would
// grow out of proportion.  `lean`: the fewest ranges, for calls whose workspace has to stay small.
struct HeadPlan {
  int ntr, nct, nb, ns;
  int64_t kchunk;
};
HeadPlan head_plan(int64_t n, int64_t V, int64_t cols, bool lean) {
  HeadPlan p;
  p.ntr = (int)((n + kHM - 1) / kHM);
  p.nct = (int)((cols + 255) / 256);
  p.nb = (int)((cols + 32 * p.nct - 1) / (32 * p.nct));
  p.nb = p.nb <= 2 ? 2 : (p.nb <= 4 ? 4 : p.nb);
  const int64_t tiles = (int64_t)p.ntr * p.nct, t128 = p.ntr * ((cols + 127) / 128);
  const int64_t want = std::max<int64_t>(1, std::min({(2048 + t128 - 1) / t128, (int64_t)32, (V + 255) / 256}));
  double best = 1e300;
  for (int64_t s = want; s <= (lean ? want : 2 * want); ++s) {
    const int64_t chunk = ((V + s - 1) / s + 31) / 32 * 32, ns = (V + chunk - 1) / chunk;
    const int64_t full = tiles * ns / 512, rest = tiles * ns % 512;
    const double rounds = (double)full + (rest == 0 ? 0.0 : rest <= 256 ? 0.6 : 1.0);
    const double t = rounds * (double)((chunk + kHK - 1) / kHK + 4) + (double)ns * (double)n * (double)cols * 1e-6;
    if (t < best) {
      best = t;
      p.kchunk = chunk;
      p.ns = (int)ns;
    }
  }
  return p;
}

template <typename LT>
void launch_product(const SoftmaxProductArgs& a, const HeadPlan& p, const float* ms, float* part) {
  const LT* z = (const LT*)a.logits;
  const int64_t cols = a.groups * a.kc;
  const unsigned grid = (unsigned)((int64_t)p.ntr * p.nct * p.ns);
  k_softmax_stats<LT><<<(unsigned)a.n, kHT, 0, a.stream>>>(a.n, a.V, z, a.ld_logits, a.labels, (float*)ms, a.dev_info);
#define LOCA_HEAD(NB)                                                                                          \
  k_top_error_gemm<LT, NB><<<grid, kHT2, 0, a.stream>>>(a.n, a.V, cols, z, a.ld_logits, a.w, ms, a.W, a.kc,     \
                                                       a.w_bstride, p.ntr, p.nct, p.kchunk, part)
  switch (p.nb) {
    case 2: LOCA_HEAD(2); break;
    case 4: LOCA_HEAD(4); break;
    case 5: LOCA_HEAD(5); break;
    case 6: LOCA_HEAD(6); break;
    case 7: LOCA_HEAD(7); break;
    default: LOCA_HEAD(8); break;
  }
#undef LOCA_HEAD
}

}  // namespace

// At most 64 columns (one tile of the single-pass kernel) the logits are read once, by the
// online-softmax product; wider products keep the statistics pass and a product pass per
// column tile.
// (Its buffer loads take 31-bit byte offsets within 128 rows of logits and 64 rows of the
// right operand.)
static bool product_online(const SoftmaxProductArgs& a) {
  const int64_t zb = a.logits_dtype == LOCA_BF16 ? 2 : 4;
  return a.groups * a.kc <= 64 && 128 * a.ld_logits * zb < ((int64_t)1 << 31) &&
         64 * ((a.V + 63) / 64) * 64 * 2 < ((int64_t)1 << 31);
}

static size_t two_pass_ws(int64_t n, int64_t V, int64_t cols, bool lean) {
  return align256(sizeof(float) * 2 * n) + align256(sizeof(float) * (size_t)head_plan(n, V, cols, lean).ns * n * cols);
}

size_t softmax_product_ws(int64_t n, int64_t V, int64_t cols, bool lean) {
  const size_t two = two_pass_ws(n, V, cols, lean);
  if (cols > 64) return two;
  const size_t one = softmax_product_online_ws(n, V, cols);
  return one > two ? one : two;  // the path is chosen at the launch (it also depends on the strides)
}

hipError_t launch_softmax_product(const SoftmaxProductArgs& a) {
  if (product_online(a)) return launch_softmax_product_online(a);
  float* ms = (float*)a.ws;
  float* part = (float*)(a.ws + align256(sizeof(float) * 2 * a.n));
  const int64_t cols = a.groups * a.kc;
  const HeadPlan pl = head_plan(a.n, a.V, cols, a.lean);
  hipStream_t st = a.stream;
  if (a.logits_dtype == LOCA_BF16) launch_product<uint16_t>(a, pl, ms, part);
  else launch_product<float>(a, pl, ms, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_top_error_reduce<<<(unsigned)((a.n * cols + 255) / 256), 256, 0, st>>>(
      a.n, cols, pl.ns, part, a.w, a.labels, a.V, a.W, a.kc, a.w_bstride, a.out, a.ld_o, a.o_bstride);
  return hipGetLastError();
}

size_t top_error_ws(int64_t n, int64_t V, int64_t d) { return softmax_product_ws(n, V, d, false); }

hipError_t launch_top_error(const TopErrorArgs& a) {
  hipStream_t st = a.stream;
  k_fill_i32_head<<<1, 64, 0, st>>>(a.dev_info);
  SoftmaxProductArgs p{st, a.n, a.V, a.logits, a.logits_dtype, a.ld_logits, a.labels, a.w, (const uint16_t*)a.wu,
                       1, a.d, 0, a.e_out, a.ld_e, 0, a.dev_info, a.ws, false};
  hipError_t e = launch_softmax_product(p);
  if (e != hipSuccess) return e;
  k_finish_info_head<<<1, 64, 0, st>>>(a.dev_info);
  return hipGetLastError();
}

}  // namespace loca

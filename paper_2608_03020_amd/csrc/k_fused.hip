// k_fused.hip -- the fused LM head ("Local Targets", Eq. 4; Lemma S3.1's head error; the
// head applied once per top error, Section S11).  From the final hidden states h (n x d) and
// the frozen head W_u (V x d), for a right operand Vm (V x c):
//   out_t = w_t ( sum_v softmax(z_t)_v Vm[v, :] - Vm[y_t, :] ),   z_t = W_u h_t,
// i.e. out = E Vm with E_t = w_t (softmax(z_t) - onehot(y_t)).  Vm = W_u gives the top error
// e_t = W_u^T E_t of the paper's order (then V_k^T e_t per block); Vm = [A~_1 | ... | A~_L]
// gives every block's credit coordinates Y_b = E A~_b at once.
//
// The logits are never stored.  A workgroup (8 waves) owns 256 tokens (128 for calls of at most
// 128), a tile of at most 64 columns of Vm and a contiguous range of the vocabulary, and walks
// that range in chunks of 256:
//   1. z^T (256 x tokens) = W_u[chunk] h_rows^T on the matrix cores (v_mfma_f32_32x32x16_bf16,
//      fp32 accumulation), both operands copied straight into LDS (buffer loads to LDS) in
//      64-wide slices of d through two slots that run across chunk boundaries;
//   2. an online softmax per token, in registers: the running maximum m and sums s (fp32)
//      are updated with the chunk, the accumulated output is rescaled by exp(m_old - m_new)
//      where m rose, and P = exp(z - m_new) is split into bf16 hi + lo parts (about 16
//      significant bits);
//   3. out += (P_hi + P_lo) Vm[chunk] on the matrix cores (Vm exact in bf16), P taken from
//      the registers of step 1 and Vm, laid out as the other operand beforehand, from cache.
// Each vocabulary range leaves (m, s) per token and its partial output; a second kernel
// combines the ranges in a fixed order in float64 and subtracts the label term.  Columns of
// Vm beyond one 64-wide tile recompute the logits (c / 64 passes over W_u).
#include <algorithm>

#include "loca_bf16.h"
#include "loca_launch.h"

namespace loca {

namespace {

constexpr int kFT = 512;        // threads: 8 waves, (vocabulary part wv) x (64-token part wt)
constexpr int kFV = 256;        // vocabulary per chunk
constexpr int kFC = 64;         // columns of Vm per tile
constexpr int kFK = 64;         // hidden width per stage: whole 128-byte lines of W_u and h
// Tile shapes by tokens TR: TR / 64 token parts, the rest of the eight waves splitting the
// vocabulary chunk; two ring slots of 64 KB (TR = 256) or 48 KB (TR = 128).
template <int TR> struct FusedTile {
  static constexpr int WT = TR / 64, WV = 8 / WT;      // waves along the tokens, along the vocabulary
  static constexpr int MV = kFV / WV / 32;             // 32-entry vocabulary blocks per wave
  static constexpr int STAGE = (kFV + TR) * kFK * 2;   // bytes per stage: W_u rows, then h rows (128 B each)
  static constexpr int COPIES = STAGE / 16 / kFT;      // 16-byte copies per thread per stage (8 or 6)
  // Buffer offsets are 31-bit, so a buffer of 256 rows takes rows of at most 2^22 values.  The
  // 128-token tile serves rows of up to 2^23: its chunk of W_u is addressed as two halves.
  static constexpr int WH = TR == 128 ? 2 : 1;         // buffers per chunk of W_u
  static constexpr int WR = kFV / WH;                  // rows of each
};
constexpr int64_t kMaxLd256 = (int64_t)1 << 22;        // longest row of h for 256 tokens a tile

// A stage holds 256 + TR rows of 128 bytes (64 bf16 of d): rows 0..255 the chunk's W_u rows,
// then the tile's h rows.  Chunk c (16 bytes) of row r sits at position c ^ ((r >> 1) & 7), so
// that the 16 lanes that read one chunk of 16 consecutive rows hit 16 distinct bank groups.
LOCA_DEV int fz_swz(int r) { return (r >> 1) & 7; }

// The logits are formed transposed, z^T = W_u[chunk] h_tile^T (vocabulary x tokens), so
// that lane l of a 32 x 32 result block holds token l % 32 and 16 vocabulary entries:
// the softmax statistics of a token stay within a lane pair (l, l ^ 32) and the waves
// that split the chunk's vocabulary, and the exponentials of a block are already
// the matrix-core operand of the product with Vm (the sum over the vocabulary taken in
// the order the result layout gives; k_vm_frag lays Vm out as the other operand).  The waves
// share a token's running maximum, exchanged once per chunk; each keeps the sum of its own
// exponentials, and the sums meet at the end.
//
// Bound by the matrix cores and the stream of W_u and h from L2 together: counters at the size below
// put the matrix cores at 52% of the cycles (1.76 GHz under this load), the L1 waiting for L2 at 34%
// and the waves in some wait at 43%.  A stage's copies are (256 + TR) rows for 256 TR products per
// unit of d, so 256 tokens a tile stream a third less per product than 128.  n = 4096, V = 151936, d = 2048, 64 columns: 5.35 ms with 128 tokens, slices of 32
// (half lines, each line fetched twice), run-time stage arithmetic and every exponential taken
// twice; 2.56 ms now (1.03 PFLOP/s).
template <int TR>
__global__ __launch_bounds__(kFT) void k_fused_head(int64_t n, int64_t V, int64_t d, int64_t c,
                                                    const uint16_t* __restrict__ h, int64_t ldh,
                                                    const uint16_t* __restrict__ wu,
                                                    const uint16_t* __restrict__ vmf, int ntr, int nct, int64_t vper,
                                                    int nsub, float* __restrict__ part_o,
                                                    float2* __restrict__ part_ms) {
  typedef FusedTile<TR> TL;
  constexpr int WT = TL::WT, WV = TL::WV, MV = TL::MV, VW = kFV / WV, NCP = TL::COPIES;
  constexpr int NQ = kFC / 32;  // 32-column output blocks per wave
  __shared__ __attribute__((aligned(1024))) uint8_t ring[2 * TL::STAGE];
  __shared__ float sEx[WV][TR];
  const int tid = threadIdx.x, lane = tid & 63, wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wv = wid / WT, wt = wid % WT, l32 = lane & 31, lh = lane >> 5;
  // tiles that share a vocabulary range are consecutive within an XCD (W_u read once there)
  const int logical = xcd_logical((int)blockIdx.x, (int)gridDim.x);
  const int rt = logical % ntr, ct = (logical / ntr) % nct, sp = logical / (ntr * nct);
  const int64_t r0 = (int64_t)rt * TR, c0 = (int64_t)ct * kFC;
  const int64_t vb = (int64_t)sp * vper, ve = (vb + vper < V) ? vb + vper : V;
  const int nks = (int)((d + kFK - 1) / kFK);
  const int nch = (int)((ve - vb + kFV - 1) / kFV);

  const int64_t nrow = (n - r0 < TR) ? n - r0 : TR;
  const i32x4_t rsH = buffer_rsrc(h + r0 * ldh, (uint32_t)(nrow * ldh * 2));
  const uint32_t ring_lds = (uint32_t)(uintptr_t)(LOCA_LDS void*)ring;
  // Copy j of a wave fills the 1 KB block (8 rows) wid + 8 j of a stage: W_u rows for j < 4, then
  // h rows.  Lane l takes row l / 8 of the block, position l % 8.  Byte offsets fit 31 bits (d <=
  // ldh <= 2^23 is checked by the caller, and rows past kMaxLd256 take the 128-token tile); rows
  // past V or n lie past the buffer and read zero.
  // Blocks eight apart hold rows 64 apart, which share the swizzle: one offset per operand.
  const int crow = 8 * wid + (lane >> 3);
  const uint32_t ck = 8u * (uint32_t)((lane & 7) ^ fz_swz(crow));  // the lane's first k in a slice
  const uint32_t offw = 2u * ((uint32_t)crow * (uint32_t)d + ck), offh = 2u * ((uint32_t)crow * (uint32_t)ldh + ck);
  const uint32_t stepw = 128u * (uint32_t)d, steph = 128u * (uint32_t)ldh;
  i32x4_t rsW[TL::WH];
  auto issue_stage = [&](int ks, int slot) {
    const uint32_t dst = ring_lds + (uint32_t)(slot * TL::STAGE + wid * 1024), k0 = (uint32_t)(ks * kFK);
    const bool in = k0 + ck < (uint32_t)d;
#pragma unroll
    for (int j = 0; j < NCP; ++j) {
      const uint32_t step = j < kFV / 64 ? (j % (TL::WR / 64)) * stepw : (j - kFV / 64) * steph;
      const uint32_t off = in ? (j < kFV / 64 ? offw : offh) + (step + 2u * k0) : kBufOutside;
      lds_dma16_buf(off, j < kFV / 64 ? rsW[j / (TL::WR / 64)] : rsH, dst + (uint32_t)(j * 8192));
    }
  };
  auto chunk_w = [&](int64_t v0) {
#pragma unroll
    for (int q = 0; q < TL::WH; ++q) {
      const int64_t v = v0 + q * TL::WR < V ? v0 + q * TL::WR : V, nvr = V - v < TL::WR ? V - v : TL::WR;
      rsW[q] = buffer_rsrc(wu + v * d, (uint32_t)(nvr * d * 2));
    }
  };

  f32x16_t o[2][NQ];
  float m_run[2], s_run[2];  // token l32 of block mt: the running maximum, and the sum of this lane's exponentials
  // operand addresses in a slot: row r's chunk 2 kk + lh at 128 r + 16 ((2 kk + lh) ^ swz(r)); rows
  // 32 apart share the swizzle
  const uint32_t ra = (uint32_t)(wv * VW + l32), rb = (uint32_t)(kFV + wt * 64 + l32);
  const uint32_t la = 128 * ra + 16 * (uint32_t)(lh ^ fz_swz((int)ra)), lb = 128 * rb + 16 * (uint32_t)(lh ^ fz_swz((int)rb));

  int slot = 0;
  for (int sub = 0; sub < nsub; ++sub) {  // the parts of the range, each with sums of its own
    const int j0 = sub == 0 ? 0 : (nch + 1) / 2, j1 = sub + 1 < nsub ? (nch + 1) / 2 : nch;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      m_run[mt] = -__builtin_inff();
      s_run[mt] = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[mt][q][r] = 0.f;
    }
    if (j0 < j1) {
      chunk_w(vb + (int64_t)j0 * kFV);
      issue_stage(0, slot);
    }
    for (int j = j0; j < j1; ++j) {
      const int64_t v0 = vb + (int64_t)j * kFV;
      // 1. z^T = W_u[chunk] h[tile]^T
      f32x16_t z[MV][2];
#pragma unroll
      for (int mv = 0; mv < MV; ++mv)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int r = 0; r < 16; ++r) z[mv][mt][r] = 0.f;
      for (int ks = 0; ks < nks; ++ks) {
        // the stage landed (this thread's copies), and this thread's reads of the other slot are done
        __builtin_amdgcn_s_waitcnt(kWaitMemLds);
        barrier_nofence();  // ... everyone's: the other slot may be overwritten
        if (ks + 1 < nks) {
          issue_stage(ks + 1, slot ^ 1);
        } else if (j + 1 < j1) {
          chunk_w(v0 + kFV);
          issue_stage(0, slot ^ 1);
        }
        const uint8_t* st = ring + slot * TL::STAGE;
#pragma unroll
        for (int kk = 0; kk < kFK / 16; ++kk) {
          bf16x8_t a[MV], b[2];
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) b[mt] = *(const bf16x8_t*)(st + (lb ^ (32u * kk)) + 4096 * mt);
#pragma unroll
          for (int mv = 0; mv < MV; ++mv) a[mv] = *(const bf16x8_t*)(st + (la ^ (32u * kk)) + 4096 * mv);
#pragma unroll
          for (int mv = 0; mv < MV; ++mv)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) z[mv][mt] = mfma32(a[mv], b[mt], z[mv][mt]);
        }
        slot ^= 1;
      }

      // 2. online softmax over the chunk.  Entry r of lane l in block (mv, mt): vocabulary
      // v0 + VW wv + 32 mv + 8 (r >> 2) + 4 lh + (r & 3), token 64 wt + 32 mt + l32.
      if (V - v0 < kFV) {  // the ragged last chunk: entries past V are excluded
        const int nv = (int)(V - v0);
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (VW * wv + 32 * mv + 8 * (r >> 2) + 4 * lh + (r & 3) >= nv) z[mv][0][r] = z[mv][1][r] = -__builtin_inff();
      }
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        float mx = z[0][mt][0];
#pragma unroll
        for (int mv = 0; mv < MV; ++mv)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, z[mv][mt][r]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (lh == 0) sEx[wv][wt * 64 + 32 * mt + l32] = mx;
      }
      wave_lds_sync();
      barrier_nofence();
      float al[2], ms[2];
#pragma unroll
      for (int mt = 0; mt < 2; ++mt) {
        const int tk = wt * 64 + 32 * mt + l32;
        float mn = m_run[mt];
#pragma unroll
        for (int u = 0; u < WV; ++u) mn = fmaxf(mn, sEx[u][tk]);
        ms[mt] = mn == -__builtin_inff() ? 0.f : mn;  // nothing but excluded entries so far
        al[mt] = __expf(m_run[mt] - ms[mt]);
        m_run[mt] = mn;
        s_run[mt] *= al[mt];
      }
      // rescale the output rows where a maximum rose: row r of an output block is token
      // 8 (r >> 2) + 4 lh + (r & 3)
      if (__ballot(al[0] != 1.f || al[1] != 1.f))
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float a_r = __shfl(al[mt], 8 * (r >> 2) + 4 * lh + (r & 3));
#pragma unroll
            for (int q = 0; q < NQ; ++q) o[mt][q][r] *= a_r;
          }
      // 3. out += (P_hi + P_lo) Vm[chunk]: k step (mv, ks2) takes the entries r = 8 ks2 .. 8 ks2 + 7
      float cs[2] = {0.f, 0.f};  // the chunk's own sums, short chains
      const uint4* vf = (const uint4*)vmf + (((v0 + VW * wv) / 16 * nct + ct) * NQ) * 64 + lane;
#pragma unroll
      for (int mv = 0; mv < MV; ++mv)
#pragma unroll
        for (int ks2 = 0; ks2 < 2; ++ks2) {
          bf16x8_t phi[2], plo[2], bv[NQ];
#pragma unroll
          for (int q = 0; q < NQ; ++q)
            bv[q] = __builtin_bit_cast(bf16x8_t, vf[((int64_t)(2 * mv + ks2) * nct * NQ + q) * 64]);
#pragma unroll
          for (int mt = 0; mt < 2; ++mt) {
            uint32_t hv[4], lv[4];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
              // hi and lo parts rounded to nearest even by the hardware conversion, in pairs
              const int r = 8 * ks2 + 2 * e2;
              const float p0 = __expf(z[mv][mt][r] - ms[mt]), p1 = __expf(z[mv][mt][r + 1] - ms[mt]);
              cs[mt] += p0 + p1;
              const uint32_t h2 = cvt_pk_bf16(p0, p1);
              hv[e2] = h2;
              lv[e2] = cvt_pk_bf16(p0 - bf16_lo(h2), p1 - bf16_hi(h2));
            }
            phi[mt] = __builtin_bit_cast(bf16x8_t, make_uint4(hv[0], hv[1], hv[2], hv[3]));
            plo[mt] = __builtin_bit_cast(bf16x8_t, make_uint4(lv[0], lv[1], lv[2], lv[3]));
          }
#pragma unroll
          for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
              o[mt][q] = mfma32(phi[mt], bv[q], o[mt][q]);
              o[mt][q] = mfma32(plo[mt], bv[q], o[mt][q]);
            }
        }
      s_run[0] += cs[0];
      s_run[1] += cs[1];
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();  // the ring is free: the vocabulary parts' sums and outputs meet there
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
      s_run[mt] += __shfl_xor(s_run[mt], 32);
      if (lh == 0) sEx[wv][wt * 64 + 32 * mt + l32] = s_run[mt];
    }
    // (the lane is opaque here, so that no address below is kept in a register over the products)
    int le = lane;
    asm volatile("" : "+v"(le));
    const int e32 = le & 31, eh = le >> 5;
    // partial outputs summed in a fixed order: (O_0 + O_2) + (O_1 + O_3), or O_0 + O_1
    float* red = (float*)ring;  // WV / 2 x TR tokens x (64 + 4) floats
    constexpr int RLD = kFC + 4;
    static_assert(WV / 2 * TR * RLD * 4 <= 2 * TL::STAGE, "the outputs fit the ring");
    auto put = [&](int slot2) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            red[(slot2 * TR + wt * 64 + 32 * mt + 8 * (r >> 2) + 4 * eh + (r & 3)) * RLD + 32 * q + e32] = o[mt][q][r];
    };
    auto add = [&](int slot2) {
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            o[mt][q][r] += red[(slot2 * TR + wt * 64 + 32 * mt + 8 * (r >> 2) + 4 * eh + (r & 3)) * RLD + 32 * q + e32];
    };
    if (WV == 4) {
      if (wv >= 2) put(wv - 2);
      __syncthreads();
      if (wv < 2) add(wv);
      __syncthreads();
    }
    if (wv == 1) put(0);
    __syncthreads();
    if (wv == 0) {
      add(0);
      const int64_t pi = (int64_t)sp * nsub + sub;
      float* po = part_o + pi * n * c;
#pragma unroll
      for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int tr = wt * 64 + 32 * mt + 8 * (r >> 2) + 4 * eh + (r & 3);
            const int64_t row = r0 + tr, col = c0 + 32 * q + e32;
            if (row < n && col < c) po[row * c + col] = o[mt][q][r];
          }
      if (ct == 0 && eh == 0)
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const int tk = wt * 64 + 32 * mt + e32;
          const int64_t row = r0 + tk;
          float sm = sEx[0][tk];
#pragma unroll
          for (int u = 1; u < WV; ++u) sm += sEx[u][tk];
          if (row < n) part_ms[pi * n + row] = make_float2(m_run[mt], sm);
        }
    }
    if (sub + 1 < nsub) __syncthreads();  // the ring and the sums are free for the next part
  }
}

// Vm as k_fused_head's second operand: 16 vocabulary entries x 32 columns a fragment of 64 lanes x
// 16 bytes, fragment (g, q) of vocabulary entries 16 g .. and columns 32 q .. (q < 2 nct) at 1 KB x
// (2 nct g + q); lane l holds column 32 q + l % 32 and the entries 8 (e / 4) + 4 (l / 32) + e % 4,
// e = 0..7 (the order in which the logits' result layout leaves them).  Zero past V and c.  One
// fragment per wave up to kFragBlocks workgroups (2^31 entries); larger operands loop, since one
// launch holds fewer than 2^32 threads.
constexpr int64_t kFragBlocks = (int64_t)1 << 20;
__global__ void k_vm_frag(int64_t V, int64_t c, const uint16_t* __restrict__ vm, int64_t ld_vm, int nq, int64_t nfrag,
                          uint4* __restrict__ vmf) {
  const int lane = threadIdx.x & 63;
  for (int64_t f = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); f < nfrag; f += (int64_t)gridDim.x * 4) {
    const int64_t g = f / nq, col = 32 * (f % nq) + (lane & 31);
    uint32_t x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t v = 16 * g + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
      x[e] = (v < V && col < c) ? vm[v * ld_vm + col] : (uint16_t)0;
    }
    vmf[f * 64 + lane] = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16));
  }
}

// dev_info protocol: INT32_MAX while nothing is wrong; atomicMin with 1 + a bad row or with
// LOCA_INFO_NONFINITE (which therefore takes precedence); INT32_MAX becomes 0 at the end
__global__ void k_fused_info_init(int32_t* p) {
  if (threadIdx.x == 0) *p = INT32_MAX;
}
__global__ void k_fused_info_finish(int32_t* p) {
  if (threadIdx.x == 0 && *p == INT32_MAX) *p = 0;
}

// Vm^T (c x ldvt, bf16, zero past V) from Vm given as column groups of kc: entry (v, j) at
// vm[(j / kc) gstride + v ld_vm + j % kc] (one group: kc = c); 32 x 32 tiles via LDS
__global__ void k_vm_transpose(int64_t V, int64_t c, const uint16_t* __restrict__ vm, int64_t ld_vm, int64_t kc,
                               int64_t gstride, uint16_t* __restrict__ vmt, int64_t ldvt) {
  __shared__ uint16_t t[32][33];
  const int64_t v0 = (int64_t)blockIdx.x * 32, j0 = (int64_t)blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: 32 x 8
  for (int r = ty; r < 32; r += 8) {
    const int64_t v = v0 + r, j = j0 + tx;
    t[r][tx] = (v < V && j < c) ? vm[(j / kc) * gstride + v * ld_vm + j % kc] : (uint16_t)0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    const int64_t j = j0 + r, v = v0 + tx;
    if (j < c && v < ldvt) vmt[j * ldvt + v] = t[tx][r];
  }
}

// out_t = w_t (sum_i O_i[t] e^{m_i - M} / S - Vm[y_t]), S = sum_i s_i e^{m_i - M}: the ranges (or
// their parts) in order, float64, each exponential taken by one thread (taken by all of them, 64
// parts cost the 4096-token head of a 2.6 ms call 0.1 ms).  One
// workgroup per token.  Column j of Vm and of the output is column
// j % kc of group j / kc (Vm entries as for k_vm_transpose; output at
// out[(j / kc) o_gstride + t ld_out + j % kc]).  A bad label drops the label term and is
// reported; a sum that is not finite or not positive is reported as non-finite data.  With
// ms_out the token's (M, S) are also written as floats (ms_out[2 t], ms_out[2 t + 1]).
__global__ __launch_bounds__(256) void k_fused_combine(int64_t n, int64_t c, int64_t V, int nsp,
                                                       const float* __restrict__ part_o,
                                                       const float2* __restrict__ part_ms,
                                                       const int32_t* __restrict__ labels, const float* __restrict__ w,
                                                       const uint16_t* __restrict__ vm, int64_t ld_vm, int64_t kc,
                                                       int64_t gstride, float* __restrict__ out, int64_t ld_out,
                                                       int64_t o_gstride, float* __restrict__ ms_out,
                                                       int32_t* __restrict__ info) {
  __shared__ double sc[2 * kMaxFusedSplits];
  __shared__ float2 sms[2 * kMaxFusedSplits];
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x;
  if (tid < nsp) sms[tid] = part_ms[(int64_t)tid * n + t];
  __syncthreads();
  // every part with a chunk has a finite s_i of at least 1; one without has m_i = -inf, s_i = 0
  double M = -__builtin_inf();
  for (int i = 0; i < nsp; ++i) M = fmax(M, (double)sms[i].x);
  if (tid < nsp) sc[tid] = exp((double)sms[tid].x - M);
  __syncthreads();
  double S = 0.0;
  for (int i = 0; i < nsp; ++i) S += (double)sms[i].y * sc[i];
  const int32_t y = labels[t];
  const bool bad = y < 0 || (int64_t)y >= V;
  const bool nonfin = !isfinite(M) || !isfinite(S) || !(S > 0.0);
  if (threadIdx.x == 0) {
    if (bad) atomicMin(info, (int32_t)(t + 1));
    if (nonfin) atomicMin(info, (int32_t)LOCA_INFO_NONFINITE);
    if (ms_out) {
      ms_out[2 * t] = (float)M;
      ms_out[2 * t + 1] = (float)S;
    }
  }
  const double wt = w ? (double)w[t] : 1.0;
  const double inv = nonfin ? 0.0 : 1.0 / S;
  for (int64_t j = threadIdx.x; j < c; j += blockDim.x) {
    double acc = 0.0;
    for (int i = 0; i < nsp; ++i) acc += (double)part_o[((int64_t)i * n + t) * c + j] * sc[i];
    const int64_t g = j / kc, jc = j - g * kc;
    const double lab = bad ? 0.0 : (double)__uint_as_float((uint32_t)vm[g * gstride + (int64_t)y * ld_vm + jc] << 16);
    out[g * o_gstride + t * ld_out + jc] = (float)(wt * (acc * inv - lab));
  }
}

// ------------------------------------------------------------------ single pass over stored logits
// The head error of Lemma S3.1 applied to a right operand from stored logits in one pass
// (what k_softmax_stats and k_top_error_gemm compute in two): a wave owns 32 tokens and the
// 64 columns of a tile of Vm, a workgroup 128 tokens, and walks a range of the vocabulary
// in steps of 16 entries, one k step of v_mfma_f32_32x32x16_bf16.  The logits enter as the
// A operand (lane l: token l % 32, the 8 entries 8 (l / 32) .. 8 (l / 32) + 7 of the step),
// under an online softmax whose running maximum is raised only when a chunk of 64 entries
// exceeds it (the accumulated rows are then rescaled); P = exp(z - m) is split into bf16
// hi + lo against the bf16 Vm^T slice.  Both are copied straight into LDS by buffer loads:
// the logits through a three-slot ring, two chunks ahead, and the Vm^T slice (read from L2,
// where the tiles of one vocabulary range on an XCD share it) double-buffered one chunk
// ahead; one barrier per chunk.  ZT: bf16 (uint16_t, ld % 8 == 0) or float (ld % 4 == 0) logits with
// 16-byte aligned rows; entries past V are masked, reads stay inside the row's stride.
constexpr int kOnlineChunk = 64;
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kOnlineStages = 3;  // logits ring slots: two chunks in flight while one is read
// LDS staging of a chunk's logits: 128 token rows of 64 entries (bf16: 128 bytes, 8 chunks of
// 16 bytes; float: 256 bytes, 16 chunks), chunk c of row r at position c ^ swz(r), so that the
// 16 lanes of a half wave reading one chunk of 16 consecutive rows hit distinct bank groups.
template <typename ZT> LOCA_DEV int zo_swz(int r) { return sizeof(ZT) == 2 ? ((r >> 1) & 7) : (r & 15); }
// the Vm^T slice of a chunk: 64 rows (columns of Vm) of 64 entries (128 bytes), swizzled alike
LOCA_DEV int bo_swz(int r) { return (r >> 1) & 7; }
template <typename ZT>
__global__ __launch_bounds__(256) void k_head_online(int64_t n, int64_t V, const ZT* __restrict__ z, int64_t ldz,
                                                     const uint16_t* __restrict__ vmt, int64_t ldvt, int64_t c,
                                                     int ntr, int nct, int64_t vper, float* __restrict__ part_o,
                                                     float2* __restrict__ part_ms) {
  constexpr int RB = kOnlineChunk * (int)sizeof(ZT);   // bytes per staged logits row
  constexpr int CPR = RB / 16;                         // 16-byte chunks per row
  constexpr int STAGE = 128 * RB;                      // bytes per stage
  constexpr int NA = STAGE / 16 / 256;                 // copies per thread per stage (4 or 8)
  constexpr int RPB = 1024 / RB;                       // rows per 1 KB copy block
  constexpr int KS = kOnlineChunk / 16;
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kOnlineStages * STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t sB[2][64 * 128];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, l32 = lane & 31, lh = lane >> 5;
  const int wq = __builtin_amdgcn_readfirstlane(wid);
  const int logical = xcd_logical((int)blockIdx.x, (int)gridDim.x);
  const int rt = logical % ntr, ct = (logical / ntr) % nct, sp = logical / (ntr * nct);
  const int64_t r0 = (int64_t)rt * 128;
  const int64_t tok0 = r0 + 32 * wid;
  const int64_t t = tok0 + l32;
  const int64_t c0 = (int64_t)ct * 64;
  const int64_t vb = (int64_t)sp * vper, ve = (vb + vper < V) ? vb + vper : V;
  const int nchunk = (int)((ve - vb + kOnlineChunk - 1) / kOnlineChunk);
  // byte offsets fit 31 bits: 128 rows x ldz and 64 rows x ldvt (V <= 2^23 is checked)
  const int64_t nrow = (n - r0 < 128) ? n - r0 : 128;
  const i32x4_t rsZ = buffer_rsrc(z + r0 * ldz, (uint32_t)(nrow * ldz * sizeof(ZT)));
  const int64_t ncol = (c - c0 < 64) ? c - c0 : 64;
  const i32x4_t rsB = buffer_rsrc(vmt + c0 * ldvt, (uint32_t)(ncol * ldvt * 2));
  const uint32_t ring_lds = (uint32_t)(uintptr_t)(LOCA_LDS void*)ring;
  const uint32_t sb_lds = (uint32_t)(uintptr_t)(LOCA_LDS void*)sB;
  auto issue_a = [&](int g) {  // chunk g's logits into ring slot g % 3 (entries past the row's data masked later)
    const int64_t v0 = vb + (int64_t)g * kOnlineChunk;
    const uint32_t slot = ring_lds + (uint32_t)((g % kOnlineStages) * STAGE);
#pragma unroll
    for (int j = 0; j < NA; ++j) {
      const int blk = wq * NA + j;
      const int row = RPB * blk + lane / CPR, pos = lane % CPR;
      const int ch = pos ^ zo_swz<ZT>(row);
      const uint32_t off = (uint32_t)((row * ldz + v0) * (int64_t)sizeof(ZT)) + 16u * (uint32_t)ch;
      lds_dma16_buf(off, rsZ, slot + (uint32_t)blk * 1024u);
    }
  };
  auto issue_b = [&](int g) {  // chunk g's Vm^T slice into sB[g & 1] (rows of 64 entries, zero past V and c)
    const int64_t v0 = vb + (int64_t)g * kOnlineChunk;
    const uint32_t base = sb_lds + (uint32_t)((g & 1) * 64 * 128);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int blk = wq * 2 + j;  // 1 KB = 8 rows of 128 bytes
      const int row = 8 * blk + (lane >> 3), pos = lane & 7;
      const uint32_t off = 2u * (uint32_t)(row * ldvt + v0 + 8 * (pos ^ bo_swz(row)));
      lds_dma16_buf(off, rsB, base + (uint32_t)blk * 1024u);
    }
  };
  auto wait_vm = [&](int a) {
    if (a == NA) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NA));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  };
  f32x16_t o[2];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[q][r] = 0.f;
  float m_run = -__builtin_inff(), s_lane = 0.f;
  // prologue: chunks 0 .. kOnlineStages - 2 and the first Vm^T slice
  for (int g = 0; g < kOnlineStages - 1 && g < nchunk; ++g) issue_a(g);
  issue_b(0);
  const int arow = 32 * wid + l32;
  for (int g = 0; g < nchunk; ++g) {
    // chunk g's logits (issued kOnlineStages - 1 iterations ago) and its Vm^T slice (issued at
    // the top of iteration g - 1, before chunk g + 1's logits): only that copy may be pending
    wait_vm(g >= 1 && g + kOnlineStages - 2 < nchunk ? NA : 0);
    __syncthreads();  // every thread's copies landed; the slots refilled below are free
    if (g + 1 < nchunk) issue_b(g + 1);
    if (g + kOnlineStages - 1 < nchunk) issue_a(g + kOnlineStages - 1);
    const int64_t v0 = vb + (int64_t)g * kOnlineChunk;
    const uint8_t* st = ring + (g % kOnlineStages) * STAGE;
    const uint8_t* sb = sB[g & 1];
    // the chunk's logits of this lane's token: entry e of step ks is vocabulary v0 + 16 ks + 8 lh + e
    float zv[KS][8];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if constexpr (sizeof(ZT) == 2) {
        const int ch = 2 * ks + lh;
        const uint4 u = *(const uint4*)(st + arow * RB + 16 * (ch ^ zo_swz<ZT>(arow)));
        const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          zv[ks][2 * e] = __uint_as_float(w4[e] << 16);
          zv[ks][2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
        }
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int ch = 4 * ks + 2 * lh + h;
          const uint4 u = *(const uint4*)(st + arow * RB + 16 * (ch ^ zo_swz<ZT>(arow)));
          zv[ks][4 * h] = __uint_as_float(u.x);
          zv[ks][4 * h + 1] = __uint_as_float(u.y);
          zv[ks][4 * h + 2] = __uint_as_float(u.z);
          zv[ks][4 * h + 3] = __uint_as_float(u.w);
        }
      }
    }
    if (v0 + kOnlineChunk > ve) {  // the range's ragged last chunk: entries past ve out (p = 0)
      const int rem = (int)(ve - v0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (16 * ks + 8 * lh + e >= rem) zv[ks][e] = -__builtin_inff();
    }
    float cm = -__builtin_inff();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) cm = fmaxf(cm, zv[ks][e]);
    cm = fmaxf(cm, __shfl_xor(cm, 32));
    if (__any(cm > m_run)) {  // raise the running maximum of the tokens that need it
      const float mn = fmaxf(m_run, cm);
      const float al = __expf(m_run - mn);
      s_lane *= al;
      m_run = mn;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a_r = __shfl(al, 8 * (r >> 2) + 4 * lh + (r & 3));
#pragma unroll
        for (int q = 0; q < 2; ++q) o[q][r] *= a_r;
      }
    }
    const float m2 = m_run * kLog2e;  // exp(z - m) = 2^(z log2(e) - m log2(e))
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t hv[4], lv[4];
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        // p = exp(z - m), 0 for the masked entries (m_run is finite); hi and lo parts rounded
        // to nearest even by the hardware conversion, two values per instruction
        const float p0 = __builtin_amdgcn_exp2f(fmaf(zv[ks][2 * e2], kLog2e, -m2)),
                    p1 = __builtin_amdgcn_exp2f(fmaf(zv[ks][2 * e2 + 1], kLog2e, -m2));
        s_lane += p0;
        s_lane += p1;
        const uint32_t h2 = cvt_pk_bf16(p0, p1);
        hv[e2] = h2;
        lv[e2] = cvt_pk_bf16(p0 - bf16_lo(h2), p1 - bf16_hi(h2));
      }
      const bf16x8_t phi = __builtin_bit_cast(bf16x8_t, make_uint4(hv[0], hv[1], hv[2], hv[3]));
      const bf16x8_t plo = __builtin_bit_cast(bf16x8_t, make_uint4(lv[0], lv[1], lv[2], lv[3]));
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        // B lane l: Vm[v0 + 16 ks + 8 lh + e][c0 + 32 q + l % 32] = Vm^T row 32 q + l % 32
        const int row = 32 * q + l32, ch = 2 * ks + lh;
        const bf16x8_t bq = *(const bf16x8_t*)(sb + row * 128 + 16 * (ch ^ bo_swz(row)));
        o[q] = mfma32(phi, bq, o[q]);
        o[q] = mfma32(plo, bq, o[q]);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  const float s_tok = s_lane + __shfl_xor(s_lane, 32);
  float* po = part_o + (int64_t)sp * n * c;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t row = tok0 + 8 * (r >> 2) + 4 * lh + (r & 3), col = c0 + 32 * q + l32;
      if (row < n && col < c) po[row * c + col] = o[q][r];
    }
  if (ct == 0 && lh == 0 && t < n) part_ms[(int64_t)sp * n + t] = make_float2(m_run, s_tok);
}

struct FusedPlan {
  int ct, tr, ntr, nct, nsp, nsub;  // nsp ranges, each summed in nsub parts
  int64_t vper, ldvt;
};

FusedPlan fused_plan(int64_t n, int64_t V, int64_t c) {
  FusedPlan p;
  p.ct = kFC;  // a wider column tile holds more accumulators than the register file keeps
  // 256 tokens a tile unless half of them would be empty
  p.tr = n > 128 ? 256 : 128;
  p.ntr = (int)((n + p.tr - 1) / p.tr);
  p.nct = (int)((c + p.ct - 1) / p.ct);
  const int64_t tiles = (int64_t)p.ntr * p.nct, nchunk = (V + kFV - 1) / kFV;
  // One workgroup fits a compute unit: the number of vocabulary ranges with the least rounds of
  // 256 workgroups times chunks per range (and half a chunk's time for a prologue and a write of
  // partial outputs).  Never fewer ranges than 1024 workgroups of 128 tokens would make, and at most
  // twice as many: beyond, the partial outputs would grow out of proportion to the output (n = 51085,
  // V = 156192, d = 256, 142 columns: a workspace of 560 MB and 19.7 ms in 17 ranges, 119 MB and
  // 20.2 ms now).
  //
  // The sums run in float32, so their length costs precision: in the 128-token tile four waves share
  // a chunk's vocabulary, in the 256-token tile two, whose sums are twice as long.  Such a range is
  // summed in two parts where it is longer than half the longest (n = 4096, V = 151936, 64 columns,
  // ranges of 19 chunks, rms error against float64 in one part, in two and in the 128-token tile: d =
  // 2048 5.17e-8, 5.03e-8 and 5.13e-8; an operand of ones, whose output is 0, 6.6e-8, 3.4e-8 and
  // 3.7e-8; 2.52 ms in one part and in two).
  const int64_t wgs = ((n + 127) / 128) * p.nct;
  const int64_t want = std::max<int64_t>(1, std::min({(int64_t)kMaxFusedSplits, (1024 + wgs - 1) / wgs, nchunk}));
  const int64_t longest = (nchunk + want - 1) / want;
  int64_t best = longest;
  double cost = 1e300;
  for (int64_t s = want; s <= std::min({(int64_t)kMaxFusedSplits, 2 * want, nchunk}); ++s) {
    const int64_t per = (nchunk + s - 1) / s, ns = (nchunk + per - 1) / per;
    const int parts = p.tr == 256 && 2 * per > longest + 1 ? 2 : 1;
    const double t = (double)((tiles * ns + 255) / 256) * ((double)per + 0.5 * parts);
    if (t < cost) {
      cost = t;
      best = per;
      p.nsub = parts;
    }
  }
  p.vper = best * kFV;
  p.nsp = (int)((V + p.vper - 1) / p.vper);  // every range holds at least one chunk
  p.ldvt = nchunk * kFV;
  return p;
}

}  // namespace

namespace {
struct OnlinePlan {
  int ntr, nct, nsp;
  int64_t vper, ldvt;
};
OnlinePlan online_plan(int64_t n, int64_t V, int64_t cols) {
  OnlinePlan p;
  p.ntr = (int)((n + 127) / 128);
  p.nct = (int)((cols + 63) / 64);
  const int64_t tiles = (int64_t)p.ntr * p.nct, nchunk = (V + kOnlineChunk - 1) / kOnlineChunk;
  int64_t want = (512 + tiles - 1) / tiles;  // about two workgroups per compute unit
  if (want > kMaxFusedSplits) want = kMaxFusedSplits;
  if (want > nchunk) want = nchunk;
  if (want < 1) want = 1;
  p.vper = ((nchunk + want - 1) / want) * kOnlineChunk;
  p.nsp = (int)((V + p.vper - 1) / p.vper);
  p.ldvt = nchunk * kOnlineChunk;
  return p;
}
}  // namespace

size_t softmax_product_online_ws(int64_t n, int64_t V, int64_t cols) {
  const OnlinePlan p = online_plan(n, V, cols);
  size_t s = align256(sizeof(float) * 2 * n);  // (m, s) per token, first (the e_out writer reads it there)
  s += align256(sizeof(float) * p.nsp * n * cols);
  s += align256(sizeof(float2) * p.nsp * n);
  s += align256(sizeof(uint16_t) * cols * p.ldvt);
  return s;
}

hipError_t launch_softmax_product_online(const SoftmaxProductArgs& a) {
  const int64_t cols = a.groups * a.kc;
  const OnlinePlan p = online_plan(a.n, a.V, cols);
  char* w = a.ws;
  float* ms = (float*)w; w += align256(sizeof(float) * 2 * a.n);
  float* part_o = (float*)w; w += align256(sizeof(float) * p.nsp * a.n * cols);
  float2* part_ms = (float2*)w; w += align256(sizeof(float2) * p.nsp * a.n);
  uint16_t* vmt = (uint16_t*)w;
  hipStream_t st = a.stream;
  k_vm_transpose<<<dim3((unsigned)((p.ldvt + 31) / 32), (unsigned)((cols + 31) / 32)), 256, 0, st>>>(
      a.V, cols, a.W, a.kc, a.kc, a.w_bstride, vmt, p.ldvt);
  const unsigned grid = (unsigned)((int64_t)p.ntr * p.nct * p.nsp);
  if (a.logits_dtype == LOCA_BF16)
    k_head_online<uint16_t><<<grid, 256, 0, st>>>(a.n, a.V, (const uint16_t*)a.logits, a.ld_logits, vmt, p.ldvt,
                                                   cols, p.ntr, p.nct, p.vper, part_o, part_ms);
  else
    k_head_online<float><<<grid, 256, 0, st>>>(a.n, a.V, (const float*)a.logits, a.ld_logits, vmt, p.ldvt, cols,
                                                p.ntr, p.nct, p.vper, part_o, part_ms);
  k_fused_combine<<<(unsigned)a.n, 256, 0, st>>>(a.n, cols, a.V, p.nsp, part_o, part_ms, a.labels, a.w, a.W, a.kc,
                                                 a.kc, a.w_bstride, a.out, a.ld_o, a.o_bstride, ms, a.dev_info);
  return hipGetLastError();
}

size_t fused_head_ws(int64_t n, int64_t V, int64_t c) {
  const FusedPlan p = fused_plan(n, V, c);
  const int64_t np = (int64_t)p.nsp * p.nsub;
  size_t s = align256(sizeof(float) * np * n * c);
  s += align256(sizeof(float2) * np * n);
  s += align256(sizeof(uint16_t) * p.nct * kFC * p.ldvt);
  return s;
}

hipError_t launch_fused_head(const FusedArgs& a) {
  FusedPlan p = fused_plan(a.n, a.V, a.c);
  if (p.tr == 256 && a.ldh > kMaxLd256) {  // the same ranges in tiles of 128 tokens
    p.tr = 128;
    p.ntr = (int)((a.n + 127) / 128);
  }
  char* w = a.ws;
  const int64_t np = (int64_t)p.nsp * p.nsub;
  float* part_o = (float*)w; w += align256(sizeof(float) * np * a.n * a.c);
  float2* part_ms = (float2*)w; w += align256(sizeof(float2) * np * a.n);
  uint16_t* vmf = (uint16_t*)w;
  hipStream_t st = a.stream;
  k_fused_info_init<<<1, 64, 0, st>>>(a.dev_info);
  const int nq = p.nct * (kFC / 32);
  const int64_t nfrag = p.ldvt / 16 * nq;
  k_vm_frag<<<(unsigned)std::min<int64_t>((nfrag + 3) / 4, kFragBlocks), 256, 0, st>>>(a.V, a.c, a.vm, a.ld_vm, nq, nfrag, (uint4*)vmf);
  const unsigned grid = (unsigned)((int64_t)p.ntr * p.nct * p.nsp);
  if (p.tr == 256)
    k_fused_head<256><<<grid, kFT, 0, st>>>(a.n, a.V, a.d, a.c, a.h, a.ldh, a.wu, vmf, p.ntr, p.nct, p.vper, p.nsub,
                                            part_o, part_ms);
  else
    k_fused_head<128><<<grid, kFT, 0, st>>>(a.n, a.V, a.d, a.c, a.h, a.ldh, a.wu, vmf, p.ntr, p.nct, p.vper, p.nsub,
                                            part_o, part_ms);
  k_fused_combine<<<(unsigned)a.n, 256, 0, st>>>(a.n, a.c, a.V, (int)np, part_o, part_ms, a.labels, a.w, a.vm, a.ld_vm,
                                                 a.c, 0, a.out, a.ld_out, 0, nullptr, a.dev_info);
  k_fused_info_finish<<<1, 64, 0, st>>>(a.dev_info);
  return hipGetLastError();
}

}  // namespace loca

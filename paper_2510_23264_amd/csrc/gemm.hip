// Grouped GEMMs on the CDNA4 matrix cores.
//
// gemm_fp8: val = (A_codes * W_codes^T) * row_scale * col_scale, then the
//   epilogue of GemmProb (bias, GELU, residual add, second output).  Both
//   operands are FP8 E4M3 codes with K contiguous, K padded with zero codes to
//   a multiple of 128.  The kernels:
//
//   gemm_x_k (exact sums, the default): codes are decoded to fp16 in registers
//   (V_CVT_SCALEF32_PK_F16_FP8, exact) and multiplied by V_MFMA_F32_16X16X32_F16:
//   exact products, fp32 sums.  Slabs of 128 K-bytes go from global memory
//   straight into LDS (GLOBAL_LOAD_LDS_DWORDX4), two stages, one barrier per
//   slab.  128 x 128 tile, four wavefronts of 64 x 64 (two decodes per MFMA; a
//   smaller wave tile is bound by instruction issue, not by the matrix cores), or
//   smaller ones where those would leave compute units idle (pick_exact_tile).
//   gemm_s_k: the smallest tiles, one per workgroup; gemm_p_k: the large problems; gemm_w_k: the
//   large plain ones (gemm8_wide_ok).
//
//   gemm_fp8_k (PAHQ_MMA_FP8): V_MFMA_SCALE_F32_16X16X128_F8F6F4 with unit block
//   scales; its adder keeps a fixed-point window below the largest product of
//   an instruction (about 2^-13 of sum |a w| in the worst case).  128 x 64 tile,
//   slabs staged through registers into LDS rows padded to 144 bytes.
//
//   In these (not in gemm_p_k and gemm_w_k), W is the first MFMA operand, so a lane owns one output row of a
//   16 x 16 tile and four consecutive columns (16-byte stores); row scales,
//   column scales and the instance / row split are fetched before the K loop so
//   that the epilogue does not wait on them.  The workgroup -> tile map gives
//   each XCD (workgroup id mod 8) a contiguous range of tiles, column tiles
//   innermost, so the A rows of a tile are fetched into one L2 only.
//
// gemm_f32: plain fp32 C = A * W (+ bias) with V_MFMA_F32_16X16X4_F32 (true
//   fp32 multiply-accumulate) for the heads in fp32 and the all-fp32 mode.
#include <algorithm>
#include <atomic>
#include "kernels.h"
#include "device_util.h"
#include "mma_util.h"
#include "tile_rules.h"

namespace pahq {

#define LDS_ROW 144   // gemm_fp8_k: 128 data bytes + 16 pad

// One result element (the slow path: ragged column tail or unaligned rows).
__device__ __forceinline__ void epilogue_store(const GemmProb& P, int n, float acc, float sa, float sw, int inst,
                                               int r) {
  float val = acc * (sa * sw);
  float v = val;
  if (P.bias) v += GCF(P.bias)[n];
  if (P.act == 1) v = gelu_tanh(v);
  long long off = (long long)r * P.ldc + n;
  if (P.add) v += GCF(P.add)[inst * P.add_is + off];
  GF(P.C)[inst * P.c_is + off] = v;
  if (P.aux) {
    float x = val;
    if (P.aux_sub) x -= GCF(P.aux_sub)[off];
    GF(P.aux)[inst * P.aux_is + off] = x;
  }
}

// What the epilogue needs besides the accumulators: fetched before the K loop.
template <int TM, int TN>
struct EpiPre {
  float sa[TM];      // row scale of row (mbase + 16 i + li)
  int inst[TM];      // its instance and row within the instance
  int row[TM];
  float sw[TN];      // column scale of columns nbase + 16 j + 4 lg .. + 3 (they share one weight slice)
  float4 bias[TN];   // bias of those columns (zero without a bias)
};
__device__ __forceinline__ int wscale_index(const GemmProb& P, int n) {
  if (P.wscale_block >= P.N) return 0;
  return P.ws_shift >= 0 ? (n >> P.ws_shift) : n / P.wscale_block;
}
template <int TM, int TN>
__device__ __forceinline__ void epi_prefetch(EpiPre<TM, TN>& E, const GemmProb& P, int m0, int i0, int r0, int mbase,
                                             int nbase, int li, int lg) {
#pragma unroll
  for (int i = 0; i < TM; i++) {
    int m = min(mbase + i * 16 + li, P.M - 1);
    split_row(i0, r0, m - m0, P.rpi, P.rp0, E.inst[i], E.row[i]);
    E.sa[i] = GCF(P.ascale)[E.inst[i] * P.as_is + (long long)E.row[i] * P.as_stride];
  }
#pragma unroll
  for (int j = 0; j < TN; j++) {
    int nb = nbase + j * 16 + lg * 4;
    E.sw[j] = GCF(P.wscale)[wscale_index(P, min(nb, P.N - 1))];
    // one 16-byte load, no divergence: a group past the last one re-reads the last one (its results are
    // never stored), and the last group may read up to three floats behind bias[N - 1] (the bias
    // arrays of this library are followed by padding; the values land in the padding of the C row)
    E.bias[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (P.bias) E.bias[j] = gload4(P.bias + min(nb, (P.N - 1) & ~3));
  }
}
// acc[i][j] holds, for lane (li, lg), row mbase + 16 i + li and columns nbase + 16 j + 4 lg .. + 3.
// Every store is 16 bytes: rows, instance strides and pointers are 16-byte aligned and a last,
// partial group of columns is written whole into the padding the row has behind column N
// (gemm8_prob_ok on the host guarantees all of this).
template <int TM, int TN>
__device__ __forceinline__ void epi_store(const EpiPre<TM, TN>& E, const GemmProb& P, const v4f (&acc)[TM][TN],
                                          int mbase, int nbase, int li, int lg) {
#pragma unroll
  for (int i = 0; i < TM; i++) {
    if (mbase + i * 16 + li >= P.M) continue;
    const int inst = E.inst[i], row = E.row[i];
    const float sa = E.sa[i];
#pragma unroll
    for (int j = 0; j < TN; j++) {
      int nb = nbase + j * 16 + lg * 4;
      if (nb >= P.N) continue;
      float s2 = sa * E.sw[j];
      float4 val = make_float4(acc[i][j][0] * s2, acc[i][j][1] * s2, acc[i][j][2] * s2, acc[i][j][3] * s2);
      float4 v = val;
      if (P.bias) { v.x += E.bias[j].x; v.y += E.bias[j].y; v.z += E.bias[j].z; v.w += E.bias[j].w; }
      if (P.act == 1) { v.x = gelu_tanh(v.x); v.y = gelu_tanh(v.y); v.z = gelu_tanh(v.z); v.w = gelu_tanh(v.w); }
      long long off = (long long)row * P.ldc + nb;
      if (P.add) { float4 a = gload4(P.add + inst * P.add_is + off); v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w; }
      gstore4(P.C + inst * P.c_is + off, v);
      if (P.aux) {
        if (P.aux_sub) { float4 u = gload4(P.aux_sub + off); val.x -= u.x; val.y -= u.y; val.z -= u.z; val.w -= u.w; }
        gstore4(P.aux + inst * P.aux_is + off, val);
      }
    }
  }
}

// The log-softmax / KL epilogue (the unembedding of a scored pass): nothing of a row has to reach
// memory but, per 64-column part of it, the running maximum, the sum of exponentials against it and
// the part's share of sum_v p_ref[v] (ref[v] - x[v]), p_ref[v] = exp(ref[v] - logz_ref).  A lane holds 16 values of a row (four groups
// of four columns); the four lanes that share the row combine through two shuffles.  Columns past N
// count as -3e38 (their exponentials vanish) and have p_ref = 0.  The order of every sum is fixed by the lane layout alone, so equal
// logits give equal parts whatever the problem's number of rows.
template <int TM, int TN>
__device__ __forceinline__ void epi_kl(const EpiPre<TM, TN>& E, const GemmProb& P, const v4f (&acc)[TM][TN],
                                       int mbase, int nbase, int li, int lg, int part) {
  const float NEG = -3.0e38f;
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int m = mbase + i * 16 + li;
    const bool row_on = m < P.M;
    const int inst = E.inst[i], row = E.row[i];
    float c[TN][4];
    float mx = NEG;
    const float lzr = P.kl_ref ? (float)P.kl_ref_logz[row] : 0.f;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int nb = nbase + j * 16 + lg * 4;
      const float s2 = E.sa[i] * E.sw[j];
      float4 v = make_float4(acc[i][j][0] * s2, acc[i][j][1] * s2, acc[i][j][2] * s2, acc[i][j][3] * s2);
      if (P.bias) { v.x += E.bias[j].x; v.y += E.bias[j].y; v.z += E.bias[j].z; v.w += E.bias[j].w; }
      if (P.C && row_on && nb < P.N) gstore4(P.C + inst * P.c_is + (long long)row * P.ldc + nb, v);
      c[j][0] = nb + 0 < P.N ? v.x : NEG; c[j][1] = nb + 1 < P.N ? v.y : NEG;
      c[j][2] = nb + 2 < P.N ? v.z : NEG; c[j][3] = nb + 3 < P.N ? v.w : NEG;
      mx = fmaxf(fmaxf(mx, fmaxf(c[j][0], c[j][1])), fmaxf(c[j][2], c[j][3]));
    }
    float se = 0.f, a = 0.f;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int nb = nbase + j * 16 + lg * 4;
#pragma unroll
      for (int r = 0; r < 4; r++) se += (c[j][r] > -1.0e38f) ? __expf(c[j][r] - mx) : 0.f;
      if (P.kl_ref && row_on && nb < P.N) {
        // reference probabilities from the reference logits (one fast exponential each, relative error 1e-6,
        // instead of a second load); a column past N has p = 0 exactly through the select
        const float4 rr = gload4(P.kl_ref + (long long)row * P.ldc + nb);
        const float p0 = __expf(rr.x - lzr), p1 = nb + 1 < P.N ? __expf(rr.y - lzr) : 0.f,
                    p2 = nb + 2 < P.N ? __expf(rr.z - lzr) : 0.f, p3 = nb + 3 < P.N ? __expf(rr.w - lzr) : 0.f;
        a += p0 * (rr.x - c[j][0]) + p1 * (rr.y - c[j][1]) + p2 * (rr.z - c[j][2]) + p3 * (rr.w - c[j][3]);
      }
    }
    float ma = fmaxf(mx, __shfl_xor(mx, 16, 64));
    ma = fmaxf(ma, __shfl_xor(ma, 32, 64));
    se *= __expf(mx - ma);                 // 0 * exp(0) for a lane whose columns are all past N
    se += __shfl_xor(se, 16, 64); se += __shfl_xor(se, 32, 64);
    a += __shfl_xor(a, 16, 64); a += __shfl_xor(a, 32, 64);
    if (lg == 0 && row_on) gstore4(P.kl_part + ((long long)m * P.kl_npart + part) * 4, make_float4(ma, se, a, 0.f));
  }
}

// ------------------------------------------------------------------ exact sums (fp16 matrix cores)
// LDS rows are 128 bytes without padding; the 16-byte chunk c of row r sits at chunk position
// c ^ (r & 7), so the 16-byte operand reads of 8 consecutive rows cover all 32 banks.  A load
// instruction fills 8 rows: lane l writes LDS bytes [16 l, 16 l + 16) behind a wave-uniform base,
// i.e. row l >> 3, position l & 7, and therefore fetches chunk (l & 7) ^ (l >> 3) of its row.
// Rows past M or N are clamped to the last valid row: they feed only results that are never stored.
// One 16-byte operand read feeds two MFMA steps: step 2 q + s takes bytes [64 q + 16 g + 8 s, + 8)
// of every row, the same k positions for both operands.
//
// Workgroups are persistent: the gridDim.x / 8 workgroups of an XCD walk that XCD's tile range
// round-robin, so that the first slab of the next tile, its scales and its bias can be requested
// while the last slab of this tile is multiplied, and the next K loop starts while the stores of
// this tile are still in flight.

// B16: the rows hold bfloat16 patterns instead of e4m3 codes.  Nothing changes on the way into LDS (rows of 128
// bytes, K counted in bytes); a 16-byte operand read is then eight elements, one step of V_MFMA_F32_16X16X32_BF16,
// with no conversion (products of two bfloat16 numbers are exact in binary32, as those of two e4m3 codes are).
template <int WAVES_M, int WAVES_N, int TM, int TN, bool B16 = false>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 2) void gemm_x_k(const GemmProb* probs) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int BM = WAVES_M * TM * 16, BN = WAVES_N * TN * 16, ROWS = BM + BN;
  constexpr int NI = ROWS / 8 / NW;            // load instructions per wave and slab (8 rows each)
  constexpr int STAGE = ROWS * 128;
  static_assert(ROWS % (8 * NW) == 0, "rows must split evenly over the waves");
  static_assert(TM * TN < 64, "vmcnt has six bits");
  __shared__ __attribute__((aligned(1024))) uint8_t st0[STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[STAGE];

  const GemmProb P = probs[blockIdx.y];
  const int mt = (P.M + BM - 1) / BM, nt = (P.N + BN - 1) / BN, total = mt * nt;
  const int chunk = (total + 7) >> 3, xcd = blockIdx.x & 7, per = gridDim.x >> 3;
  const int jend = min(chunk, total - xcd * chunk);
  int j = blockIdx.x >> 3;
  if (j >= jend) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int li = lane & 15, lg = lane >> 4;

  const uint8_t* src[NI];
  const int cg = ((lane & 7) ^ (lane >> 3)) * 16;
  auto set_src = [&](int m0, int n0) {
    int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
#pragma unroll
    for (int t = 0; t < NI; t++) {
      int r = 8 * (wave * NI + t) + (lane >> 3);
      if (r < BM) {
        int m = min(m0 + r, P.M - 1), inst, row;
        split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
        src[t] = (const uint8_t*)P.A + (long long)inst * P.a_is + (long long)row * P.lda + cg;
      } else {
        int n = min(n0 + r - BM, P.N - 1);
        src[t] = (const uint8_t*)P.W + (long long)n * P.ldw + cg;
      }
    }
  };
  auto issue = [&](const uint8_t* st, int k0) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds_addr_of(st) + wave * NI * 1024);
#pragma unroll
    for (int t = 0; t < NI; t++) slab_load16(src[t] + k0, base + t * 1024);
  };

  const int offA = (wm * TM * 16 + li) * 128, offB = (BM + wn * TN * 16 + li) * 128;
  const int sw0 = (lg ^ (li & 7)) * 16, sw1 = ((4 + lg) ^ (li & 7)) * 16;
  v4f acc[TM][TN];
  auto compute = [&](const uint8_t* st) {
    const uint8_t* sA = st + offA;
    const uint8_t* sB = st + offB;
    if constexpr (B16) {
#pragma unroll
      for (int q = 0; q < 2; q++) {
        const int sw = q ? sw1 : sw0;
        union U { uint4 u; v8bf h; };
        U ha[TM];
#pragma unroll
        for (int i = 0; i < TM; i++) ha[i].u = *(const uint4*)(sA + i * 2048 + sw);
#pragma unroll
        for (int jj = 0; jj < TN; jj++) {
          U hb; hb.u = *(const uint4*)(sB + jj * 2048 + sw);
#pragma unroll
          for (int i = 0; i < TM; i++) acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hb.h, ha[i].h, acc[i][jj], 0, 0, 0);
        }
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int sw = q ? sw1 : sw0;
      v8h ha[TM][2];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        uint4 w = *(const uint4*)(sA + i * 2048 + sw);
        ha[i][0] = decode8(w.x, w.y);
        ha[i][1] = decode8(w.z, w.w);
      }
#pragma unroll
      for (int jj = 0; jj < TN; jj++) {
        uint4 w = *(const uint4*)(sB + jj * 2048 + sw);
        v8h hb0 = decode8(w.x, w.y), hb1 = decode8(w.z, w.w);
#pragma unroll
        for (int i = 0; i < TM; i++) {
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb0, ha[i][0], acc[i][jj], 0, 0, 0);
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb1, ha[i][1], acc[i][jj], 0, 0, 0);
        }
      }
    }
  };

  int lin = xcd * chunk + j;
  // Order of an XCD's tiles: neighbours share the larger operand.  With more weight rows than activation rows (the
  // unembedding: 50 257 columns against a few thousand rows) consecutive tiles walk down the rows of one column tile, so
  // that the weights cross HBM once and the small activation block is what the L2 re-serves; otherwise row tile first.
  const bool col_first = P.N > P.M;
  auto origin = [&](int t, int& mo, int& no) {
    if (col_first) { mo = (t % mt) * BM; no = (t / mt) * BN; } else { mo = (t / nt) * BM; no = (t % nt) * BN; }
  };
  int m0, n0;
  origin(lin, m0, n0);
  set_src(m0, n0);
  issue(st0, 0);
  // With an even number of slabs the last slab of a tile sits in st1 while st0 is idle: the first
  // slab of the next tile is requested there, a whole slab of MFMAs before it is needed, and the
  // K loop of the next tile starts with nothing but a barrier while the stores of this tile are
  // still in flight.  Row scales, column scales and bias of a tile are requested when its K loop
  // starts and are waited for together with its second slab.
  const bool even = (P.K & 255) == 0;
  bool slab0_here = false;           // this wave's part of slab 0 of the current tile has been waited for

  for (;;) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int jj = 0; jj < TN; jj++) acc[i][jj] = (v4f){0.f, 0.f, 0.f, 0.f};

    const int mbase = m0 + wm * TM * 16, nbase = n0 + wn * TN * 16;
    const int jn = j + per;
    const bool more = jn < jend;
    int m0n = 0, n0n = 0;
    if (more) origin(xcd * chunk + jn, m0n, n0n);
    const bool early = even && more;

    // slab 0 has landed for every wave; st1 is free
    if (slab0_here) wg_barrier();
    else wait_all_then_barrier();
    if (128 < P.K) issue(st1, 128);
    EpiPre<TM, TN> E;
    { int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0); epi_prefetch<TM, TN>(E, P, m0, i0, r0, mbase, nbase, li, lg); }
    compute(st0);
    for (int k0 = 128; k0 < P.K; k0 += 256) {        // slabs k0 (in st1) and k0 + 128 (in st0)
      wait_all_then_barrier();                       // the slab has landed for everyone, the other stage is free
      const bool last = k0 + 128 >= P.K;
      if (!last) issue(st0, k0 + 128);
      else if (early) { set_src(m0n, n0n); issue(st0, 0); }
      compute(st1);
      if (last) break;
      wait_all_then_barrier();
      if (k0 + 256 < P.K) issue(st1, k0 + 256);
      compute(st0);
    }

    if (!early) {
      wg_barrier();                                  // every wave is done with both stages
      if (more) { set_src(m0n, n0n); issue(st0, 0); }
    }
    // scales, bias and this wave's part of the next slab 0: requested at least a slab ago when
    // `early`; after this wait nothing the wave has to wait for precedes the stores
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if (P.kl_part) epi_kl<TM, TN>(E, P, acc, mbase, nbase, li, lg, (n0 / BN) * WAVES_N + wn);
    else epi_store<TM, TN>(E, P, acc, mbase, nbase, li, lg);
    if (!more) break;
    slab0_here = true;       // the barrier at the top publishes slab 0
    j = jn; m0 = m0n; n0 = n0n;
  }
}

// ------------------------------------------------------------------ exact sums, problems of few tiles
// A problem with fewer 128 x 128 tiles than the chip has room for leaves compute units idle and the others waiting for
// their loads slab by slab.  Here tiles are smaller (their number fills the chip), a workgroup has one tile, and NS
// stages of LDS keep NS - 1 slabs on their way.  Operand order, steps and epilogue are those of gemm_x_k: same bits.
template <int WAVES_M, int WAVES_N, int TM, int TN, int NS, bool B16>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64, 2) void gemm_s_k(const GemmProb* probs) {
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int BM = WAVES_M * TM * 16, BN = WAVES_N * TN * 16, ROWS = BM + BN;
  constexpr int NI = ROWS / 8 / NW;            // load instructions per wave and slab (8 rows each)
  constexpr int STAGE = ROWS * 128;
  static_assert(ROWS % (8 * NW) == 0 && BM % 8 == 0, "rows must split evenly over the waves");
  __shared__ __attribute__((aligned(1024))) uint8_t st[NS * STAGE];

  const GemmProb P = probs[blockIdx.y];
  const int mt = (P.M + BM - 1) / BM, nt = (P.N + BN - 1) / BN;
  const int lin = xcd_tile(blockIdx.x, mt * nt);
  if (blockIdx.x >= (unsigned)((mt * nt + 7) / 8 * 8) || lin >= mt * nt) return;
  const bool col_first = P.N > P.M;            // as in gemm_x_k
  const int m0 = (col_first ? lin % mt : lin / nt) * BM, n0 = (col_first ? lin / mt : lin % nt) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int li = lane & 15, lg = lane >> 4;
  const int mbase = m0 + wm * TM * 16, nbase = n0 + wn * TN * 16;
  int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
  EpiPre<TM, TN> E;                            // in front of the slabs, so that the counted waits cover it
  epi_prefetch<TM, TN>(E, P, m0, i0, r0, mbase, nbase, li, lg);

  const uint8_t* src[NI];
  const int cg = ((lane & 7) ^ (lane >> 3)) * 16;
#pragma unroll
  for (int t = 0; t < NI; t++) {
    const int r = 8 * (wave * NI + t) + (lane >> 3);
    if (r < BM) {
      int m = min(m0 + r, P.M - 1), inst, row;
      split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
      src[t] = (const uint8_t*)P.A + (long long)inst * P.a_is + (long long)row * P.lda + cg;
    } else {
      src[t] = (const uint8_t*)P.W + (long long)min(n0 + r - BM, P.N - 1) * P.ldw + cg;
    }
  }
  const uint32_t lds0 = lds_addr_of(st);
  auto issue = [&](int stage) {
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + wave * NI * 1024);
#pragma unroll
    for (int t = 0; t < NI; t++) { slab_load16(src[t], base + t * 1024); src[t] += 128; }
  };
  const int offA = (wm * TM * 16 + li) * 128, offB = (BM + wn * TN * 16 + li) * 128;
  v4f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const uint8_t* s) {
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int sw = ((4 * q + lg) ^ (li & 7)) * 16;
      uint4 wa[TM], wb[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) wa[i] = *(const uint4*)(s + offA + i * 2048 + sw);
#pragma unroll
      for (int j = 0; j < TN; j++) wb[j] = *(const uint4*)(s + offB + j * 2048 + sw);
      if constexpr (B16) {
        union U { uint4 u; v8bf h; };
#pragma unroll
        for (int j = 0; j < TN; j++) {
          U hb; hb.u = wb[j];
#pragma unroll
          for (int i = 0; i < TM; i++) { U ha; ha.u = wa[i]; acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hb.h, ha.h, acc[i][j], 0, 0, 0); }
        }
      } else {
        v8h ha[TM][2];
#pragma unroll
        for (int i = 0; i < TM; i++) { ha[i][0] = decode8(wa[i].x, wa[i].y); ha[i][1] = decode8(wa[i].z, wa[i].w); }
#pragma unroll
        for (int j = 0; j < TN; j++) {
          const v8h hb0 = decode8(wb[j].x, wb[j].y), hb1 = decode8(wb[j].z, wb[j].w);
#pragma unroll
          for (int i = 0; i < TM; i++) {
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb0, ha[i][0], acc[i][j], 0, 0, 0);
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb1, ha[i][1], acc[i][j], 0, 0, 0);
          }
        }
      }
    }
  };
  const int nslab = P.K >> 7;
#pragma unroll
  for (int k = 0; k < NS - 1; k++) if (k < nslab) issue(k);
  int sc = 0, sr = NS - 1;                     // stage of the slab to multiply, of the next request
  for (int k = 0; k < nslab; k++) {
    wait_slab_barrier<NS, NI>(nslab - 1 - k);  // the slab has landed for everyone, the previous one's stage is free
    if (k + NS - 1 < nslab) issue(sr);
    compute(st + sc * STAGE);
    sr = sc;
    sc = (sc == NS - 1) ? 0 : sc + 1;
  }
  if (P.kl_part) epi_kl<TM, TN>(E, P, acc, mbase, nbase, li, lg, (n0 / BN) * WAVES_N + wn);
  else epi_store<TM, TN>(E, P, acc, mbase, nbase, li, lg);
}

// ------------------------------------------------------------------ exact sums, three-stage pipeline
// The large problems.  What bounds gemm_x_k is the distance between requesting a slab and needing
// it: one slab of MFMAs, less than the latency of the loads under load.  Here one workgroup of
// eight wavefronts (4 x 2, 64 x 64 each) owns a 256 x 128 tile per compute unit, LDS holds three
// stages of 48 KB, and a slab is requested two slabs before it is multiplied.  The slabs of all
// tiles a workgroup walks form one stream: the request side runs two slabs ahead of the compute
// side across tile boundaries, so a tile's stores drain while the next tile is multiplied.
// Everything that is loaded goes through LDS, also the scales and the bias of a tile (one
// GLOBAL_LOAD_LDS_DWORD per wave when the tile's first slab is multiplied; read back by the
// epilogue), so that the only vector-memory operations the compiler knows of are stores and the
// residual loads of the epilogue, and the waits can be counted: a wave waits for slab c with
// "at most (6 if slab c+1 is requested) + (stores issued since) operations outstanding".
template <int UNUSED>
__global__ __launch_bounds__(512, 1) void gemm_p_k(const GemmProb* probs) {
  constexpr int BM = 256, BN = 128, TM = 4, TN = 4, NW = 8;
  constexpr int ROWS = BM + BN, NI = ROWS / 8 / NW, STAGE = ROWS * 128, NS = 3;
  static_assert(NI == 6, "six slab loads per wave: the wait counts below assume it");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  float* const e_rs = (float*)(smem + NS * STAGE);      // row scales of the tile [BM]
  float* const e_cs = e_rs + BM;                        // column scales [BN]
  float* const e_bi = e_cs + BN;                        // bias [BN]

  const GemmProb P = probs[blockIdx.y];
  const int mt = (P.M + BM - 1) / BM, nt = (P.N + BN - 1) / BN, total = mt * nt;
  const int chunk = (total + 7) >> 3, xcd = blockIdx.x & 7, per = gridDim.x >> 3;
  const int jend = min(chunk, total - xcd * chunk);
  int j = blockIdx.x >> 3;
  if (j >= jend) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lg = lane >> 4;
  const int nslab = P.K >> 7;
  const uint32_t lds0 = lds_addr_of(smem);

  // ---- request side
  const uint8_t* src[NI];
  const int cg = ((lane & 7) ^ (lane >> 3)) * 16;
  auto set_src = [&](int m0, int n0) {
    int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
#pragma unroll
    for (int t = 0; t < NI; t++) {
      int r = 8 * (wave * NI + t) + (lane >> 3);
      if (r < BM) {
        int m = min(m0 + r, P.M - 1), inst, row;
        split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
        src[t] = (const uint8_t*)P.A + (long long)inst * P.a_is + (long long)row * P.lda + cg;
      } else {
        // LDS row 16 jj + li of a wave's 64-column block holds column 4 li + jj of the block, so that a lane's four
        // accumulators of one tile row are four neighbouring columns (see the epilogue)
        const int q = r - BM;
        int n = min(n0 + (q & 64) + (q & 15) * 4 + ((q >> 4) & 3), P.N - 1);
        src[t] = (const uint8_t*)P.W + (long long)n * P.ldw + cg;
      }
    }
  };
  auto tile_origin = [&](int jj, int& m0, int& n0) {
    int lin = xcd * chunk + jj;
    m0 = (lin / nt) * BM; n0 = (lin % nt) * BN;
  };
  int ji = j, ki = 0, si = 0;          // tile, slab and stage of the next request
  bool requesting = true;
  auto request = [&]() -> bool {
    if (!requesting) return false;
    const uint32_t base = __builtin_amdgcn_readfirstlane(lds0 + si * STAGE + wave * NI * 1024);
#pragma unroll
    for (int t = 0; t < NI; t++) slab_load16(src[t] + ki * 128, base + t * 1024);
    si = (si == NS - 1) ? 0 : si + 1;
    if (++ki == nslab) {
      ki = 0; ji += per;
      if (ji < jend) { int a, b; tile_origin(ji, a, b); set_src(a, b); }
      else requesting = false;
    }
    return true;
  };
  // scales and bias of a tile: one dword per lane and wave
  auto request_scales = [&](int m0, int n0) {
    const float* g;
    float* dst;
    if (wave < 4) {
      int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
      int m = min(m0 + wave * 64 + lane, P.M - 1), inst, row;
      split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
      g = P.ascale + inst * P.as_is + (long long)row * P.as_stride;
      dst = e_rs + wave * 64;
    } else {
      int n = min(n0 + (wave & 1) * 64 + lane, P.N - 1);
      if (wave >= 6 && P.bias) { g = P.bias + n; dst = e_bi + (wave & 1) * 64; }
      else { g = P.wscale + wscale_index(P, n); dst = ((wave >= 6) ? e_bi : e_cs) + (wave & 1) * 64; }
    }
    lds_load4(g, __builtin_amdgcn_readfirstlane(lds_addr_of(dst)));
  };

  // ---- compute side
  const int offA = (wm * 64 + li) * 128, offB = (BM + wn * 64 + li) * 128;
  const int sw0 = (lg ^ (li & 7)) * 16, sw1 = ((4 + lg) ^ (li & 7)) * 16;
  v4f acc[TM][TN];
  auto compute = [&](const uint8_t* st) {
    const uint8_t* sA = st + offA;
    const uint8_t* sB = st + offB;
    // all operand reads of the slab are issued before the first convert, so that the reads of the
    // second half are in flight while the first half is multiplied
    uint4 ra[2][TM], rb[2][TN];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int sw = q ? sw1 : sw0;
#pragma unroll
      for (int i = 0; i < TM; i++) ra[q][i] = *(const uint4*)(sA + i * 2048 + sw);
#pragma unroll
      for (int jj = 0; jj < TN; jj++) rb[q][jj] = *(const uint4*)(sB + jj * 2048 + sw);
    }
    __builtin_amdgcn_sched_barrier(0);       // keep the scheduler from sinking the reads to their uses
#pragma unroll
    for (int q = 0; q < 2; q++) {
      v8h ha[TM][2];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        ha[i][0] = decode8(ra[q][i].x, ra[q][i].y);
        ha[i][1] = decode8(ra[q][i].z, ra[q][i].w);
      }
#pragma unroll
      for (int jj = 0; jj < TN; jj++) {
        v8h hb0 = decode8(rb[q][jj].x, rb[q][jj].y), hb1 = decode8(rb[q][jj].z, rb[q][jj].w);
#pragma unroll
        for (int i = 0; i < TM; i++) {
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i][0], hb0, acc[i][jj], 0, 0, 0);
          acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i][1], hb1, acc[i][jj], 0, 0, 0);
        }
      }
    }
  };

  int m0, n0;
  tile_origin(j, m0, n0);
  set_src(m0, n0);
  request();
  bool next_requested = request();      // is the slab after the one about to be multiplied on its way?
  int stores = 0;                       // stores this wave issued since that slab was requested (0, 16 or 32)
  int sc = 0;                           // stage of the slab about to be multiplied

  for (;;) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int jj = 0; jj < TN; jj++) acc[i][jj] = (v4f){0.f, 0.f, 0.f, 0.f};

    for (int k = 0; k < nslab; k++) {
      // this wave's part of the slab has landed: everything but what was issued after it is complete
      if (next_requested) {
        if (stores == 0) wait_vm<6>(); else if (stores == 16) wait_vm<22>(); else wait_vm<38>();
      } else {
        if (stores == 0) wait_vm<0>(); else if (stores == 16) wait_vm<16>(); else wait_vm<32>();
      }
      stores = 0;
      wg_barrier();                     // everyone's part has; the stage of the previous slab is free
      if (k == 0) request_scales(m0, n0);
      next_requested = request();       // two slabs ahead, into the stage just freed
      compute(smem + sc * STAGE);
      sc = (sc == NS - 1) ? 0 : sc + 1;
    }
    if (nslab == 1) { wait_vm<0>(); wg_barrier(); }     // the scales were requested in this very slab

    // ---- epilogue: scales and bias from LDS, 16-byte stores
    // Accumulator acc[i][jj][r] of lane (li, lg) is tile row 16 i + 4 lg + r and, with the column order the
    // request side gave the W rows, column 4 li + jj of the wave's block: a lane stores the four jj values of one
    // row as 16 bytes, and the 16 lanes of a group cover 256 contiguous bytes of that row.  Neighbouring lanes
    // writing neighbouring addresses is what the store path wants: the same bytes stored as 16 rows x 64 bytes
    // per instruction take a fifth longer end to end.
    const int nbase = n0 + wn * 64 + li * 4;
    const bool interior = (m0 + BM <= P.M) && (n0 + BN <= P.N);
    const bool col_on = interior || nbase < P.N;
    int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
    const float cs = e_cs[wn * 64 + li * 4];
    const float4 bias = *(const float4*)(e_bi + wn * 64 + li * 4);
    int inst[TM][4];
    int roff[TM][4];           // within one instance's block: far below 2^31 elements
    bool live[TM][4];
    float4 sa[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) {
      sa[i] = *(const float4*)(e_rs + wm * 64 + i * 16 + lg * 4);
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int m = m0 + wm * 64 + i * 16 + lg * 4 + r;
        live[i][r] = col_on && (interior || m < P.M);
        int row;
        split_row(i0, r0, min(m, P.M - 1) - m0, P.rpi, P.rp0, inst[i][r], row);
        roff[i][r] = row * (int)P.ldc + nbase;
      }
    }
    // the residual tile first, all of it, so that its loads are in flight together
    float4 addv[TM][4];
    if (P.add) {
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int r = 0; r < 4; r++)
          addv[i][r] = live[i][r] ? gload4_nt(P.add + inst[i][r] * P.add_is + roff[i][r]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < TM; i++) {
      const float sar[4] = {sa[i].x, sa[i].y, sa[i].z, sa[i].w};
#pragma unroll
      for (int r = 0; r < 4; r++) {
        if (!live[i][r]) continue;
        const float s2 = sar[r] * cs;
        float4 val = make_float4(acc[i][0][r] * s2, acc[i][1][r] * s2, acc[i][2][r] * s2, acc[i][3][r] * s2);
        float4 v = val;
        if (P.bias) { v.x += bias.x; v.y += bias.y; v.z += bias.z; v.w += bias.w; }
        // (no activation here: problems that ask for one are refused for this kernel's sizes by gemm8_prob_ok; the code
        // of 64 inlined GELUs cost every tile's epilogue 1.5-2 % of a K = 768 product although no problem used it)
        if (P.add) { v.x += addv[i][r].x; v.y += addv[i][r].y; v.z += addv[i][r].z; v.w += addv[i][r].w; }
        gstore4_nt(P.C + inst[i][r] * P.c_is + roff[i][r], v);
        if (P.aux) {
          if (P.aux_sub) { float4 u = gload4(P.aux_sub + roff[i][r]); val.x -= u.x; val.y -= u.y; val.z -= u.z; val.w -= u.w; }
          gstore4_nt(P.aux + inst[i][r] * P.aux_is + roff[i][r], val);
        }
      }
    }
    if (interior) stores = P.aux ? 32 : 16;     // every wave issued exactly that many
    else {                                      // ragged tile: the count is not uniform, so drain
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0F70);
      stores = 0;
    }
    j += per;
    if (j >= jend) break;
    tile_origin(j, m0, n0);
  }
}

// ------------------------------------------------------------------ exact sums, the large plain problems
// gemm_w_k: one instance, no second output (gemm8_wide_ok).  256 x 256 tile, eight wavefronts (4 x 2) of 64 x 128, one persistent
// workgroup per compute unit, slabs of 128 bytes of K in two stages of 64 KB.  gemm_p_k, which these problems took before,
// spent its time on four things that this shape and schedule remove:
//   - all waves read their operands behind the slab's barrier and multiplied afterwards, so that the matrix cores idled
//     while LDS worked and the other way round.  Here the next half slab's reads, its conversions and the requests for the slab after
//     it stand between the matrix instructions of the present one (step below);
//   - two conversions per matrix instruction (a wave of 64 x 64); one and a half here, and half the LDS reads per product;
//   - 24 bytes per clock and unit from L2; 16 here.  (Slabs of 64 bytes in more stages ask L2 for half lines: 15 % slower.)
//   - an epilogue that placed every row by itself, 5 k clocks a tile: rows are equidistant here, one offset per lane.
// Tiles at the right and lower edge are moved inwards until they end there and overlap their neighbours: no guard anywhere, and
// the overlap is written twice with the same bits (so C may not be `add`).
// Elements are the sums of the other kernels in the same order: same bits.  us, before and now (one MI355X): 102400 x 2304 x 768
// 498 -> 353, 102400 x 3072 x 768 582 -> 431, 102400 x 768 x 3072 521 -> 423, 24576 x 4096 x 1024 224 -> 169, 4096 x 12288 x 4096
// 354 -> 292 (1.4 PFLOP/s).  What bounds it now: at K = 768 the stores (1.26 GB of them; a slab requested behind the stores of
// a tile is not seen to have landed before they have), at long K the chip's power: the shader clock falls to 1.75 GHz.
// The wave's 256 registers do not quite suffice: 18 (bfloat16: 13) spill, 72 and 56 bytes of scratch a lane, and a few come back
// inside the K loop.  The counted waits bear that: operations the compiler adds make them stricter.  Recomputing such values
// instead was slower.
// Measured and not kept: two workgroups of 256 x 128 per unit with slabs of 64 bytes (530 us where this takes 431), one wave of
// 64 x 128 per SIMD whose finished tile leaves during the next one (747), V_MFMA_F32_32X32X16_F16 (the same bits, 15 % slower: the
// clock falls further).
template <bool B16>
__global__ __launch_bounds__(512, 2) void gemm_w_k(const GemmProb* probs) {
  constexpr int BM = 256, BN = 256, NI = 8, STAGE = (BM + BN) * 128;
  static_assert(STAGE == 65536, "the stages differ in one address bit");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  float* const e_base = (float*)(smem + 2 * STAGE);      // per tile parity: row scales, column scales, bias [256 each]
  const GemmProb P = probs[blockIdx.y];
  const int mt = (P.M + BM - 1) / BM, nt = (P.N + BN - 1) / BN, total = mt * nt;
  const int chunk = (total + 7) >> 3, xcd = blockIdx.x & 7, per = gridDim.x >> 3;
  const int jend = min(chunk, total - xcd * chunk);
  int j = blockIdx.x >> 3;
  if (j >= jend) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lg = lane >> 4;
  const int nslab = P.K >> 7;
  auto tile_origin = [&](int jj, int& m0, int& n0) {
    const int lin = xcd * chunk + jj, tm = lin / nt;
    m0 = min(tm * BM, P.M - BM); n0 = min((lin - tm * nt) * BN, P.N - BN);
  };

  // ---- request side: waves 0-3 load 64 rows of A each, waves 4-7 of W.  LDS row 16 q + i of a 64-row block of W holds row 4 i + q
  // of the block, so that a lane's accumulators of four 16-column tiles are neighbouring columns (see the epilogue).
  const bool is_a = wave < 4;
  const int ldo = is_a ? P.lda : P.ldw;
  const uint32_t lane_off = (uint32_t)((lane >> 3) * (is_a ? 1 : 4) * ldo + ((lane & 7) ^ (lane >> 3)) * 16);
  const uint8_t* src;
  auto set_src = [&](int m0, int n0) {
    src = is_a ? (const uint8_t*)P.A + (long long)(m0 + wave * 64) * P.lda : (const uint8_t*)P.W + (long long)(n0 + (wave - 4) * 64) * P.ldw;
  };
  int ji = j, ki = 0;                    // tile and slab of the next request
  uint32_t to = __builtin_amdgcn_readfirstlane(lds_addr_of(smem) + wave * NI * 1024);      // and where it goes
  auto request_one = [&](int t) {
    slab_load16s(src + (long long)(is_a ? 8 * t : 32 * (t & 1) + (t >> 1)) * ldo, lane_off, to + t * 1024);
  };
  auto request_end = [&]() {
    src += 128;
    to ^= STAGE;
    if (++ki == nslab) {
      ki = 0; ji += per;
      if (ji < jend) { int a, b; tile_origin(ji, a, b); set_src(a, b); }
      else { src -= 128; ki = nslab - 1; ji -= per; }      // behind the last tile its last slab again (nobody reads it): no branch in the loop
    }
  };
  auto request_scales = [&](int m0, int n0, float* e) {
    const uint32_t o = (uint32_t)((wave & 3) * 64 + lane) * 4;
    if (is_a) {
      lds_load4s(P.ascale + m0, o, __builtin_amdgcn_readfirstlane(lds_addr_of(e + wave * 64)));
      lds_load4(P.wscale + wscale_index(P, n0 + wave * 64 + lane), __builtin_amdgcn_readfirstlane(lds_addr_of(e + 256 + wave * 64)));
    } else if (P.bias) {
      lds_load4s(P.bias + n0, o, __builtin_amdgcn_readfirstlane(lds_addr_of(e + 512 + (wave & 3) * 64)));
    }
  };

  // ---- compute side.  LDS offsets of the operands' first tiles in the first half (64 bytes of K) of the stage at hand; the
  // other half is at ^ 64, the other stage at ^ STAGE.
  uint32_t at_a = (wm * 64 + li) * 128 + (lg ^ (li & 7)) * 16, at_b = (BM + wn * 128 + li) * 128 + (lg ^ (li & 7)) * 16;
  v4f acc[4][8];
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  union U { uint4 u; v8bf h; };
  U ra[2][4], rb[8];                     // a half slab's operands as they lie in LDS ([1] with B16 only)
  v8h ha[4], hb[2];                      // decoded: all of A and two of W, of one step
  auto dec = [&](const U& w, int s) -> v8h { return s ? decode8(w.u.z, w.u.w) : decode8(w.u.x, w.u.y); };
  auto read_a = [&](int h, int i, uint32_t a) { ra[h][i].u = *(const uint4*)(smem + a + i * 2048); };
  auto read_b = [&](int jj, uint32_t b) { rb[jj].u = *(const uint4*)(smem + b + jj * 2048); };
  // One step, 32 k, of the half slab in ra, rb: the decoded operands for it are there, those of the next step are made on the
  // way.  rd: the other half (at a, b) is read into the registers that this step sets free; rq: a slab is requested.
  auto step = [&](int s, bool first, bool rd, bool rq, uint32_t a, uint32_t b) {
#pragma unroll
    for (int jj = 0; jj < 8; jj++) {
      if (jj < 7) hb[(jj + 1) & 1] = dec(rb[jj + 1], s);
      if (rd) { if (jj < 4) read_a(0, jj, a); read_b(jj, b); }
#pragma unroll
      for (int i = 0; i < 4; i++) {
        acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i], hb[jj & 1], first ? zero : acc[i][jj], 0, 0, 0);
        if (jj == 7) { ha[i] = dec(ra[0][i], s ^ 1); __builtin_amdgcn_sched_barrier(0); }
      }
      if (jj == 7) hb[0] = dec(rb[0], s ^ 1);
      if (rq) request_one(jj);
      if (jj < 7) {                      // a conversion behind every matrix instruction
#pragma unroll
        for (int q = 0; q < 4; q++) { __builtin_amdgcn_sched_group_barrier(0x8, 1, 0); __builtin_amdgcn_sched_group_barrier(0x2, 1, 0); }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // bfloat16: a half slab is one step, its operands need no conversion
  auto step16 = [&](int h, bool first, bool rq, uint32_t a, uint32_t b) {
#pragma unroll
    for (int jj = 0; jj < 8; jj++) {
      if (jj < 4) read_a(h ^ 1, jj, a);
#pragma unroll
      for (int i = 0; i < 4; i++)
        acc[i][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[h][i].h, rb[jj].h, first ? zero : acc[i][jj], 0, 0, 0);
      read_b(jj, b);
      if (rq) request_one(jj);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto read_first = [&]() {              // the operands of a tile's first step, from the slab at hand
#pragma unroll
    for (int i = 0; i < 4; i++) read_a(0, i, at_a);
#pragma unroll
    for (int jj = 0; jj < 8; jj++) read_b(jj, at_b);
    if constexpr (!B16) {
#pragma unroll
      for (int i = 0; i < 4; i++) ha[i] = dec(ra[0][i], 0);
      hb[0] = dec(rb[0], 0);
    }
  };

  int m0, n0;
  tile_origin(j, m0, n0);
  set_src(m0, n0);
#pragma unroll
  for (int q = 0; q < 2; q++) {
#pragma unroll
    for (int t = 0; t < NI; t++) request_one(t);
    request_end();
  }
  wait_vm<NI>();
  wg_barrier();
  read_first();
  int par = 0;
  bool stored = false;                   // has this wave stored a tile since the next slab was requested?
  const bool has_bias = P.bias != nullptr, has_add = P.add != nullptr;

  for (;;) {
    float* const e = e_base + par * 768; // (the other parity's may still be read by a wave that is behind)
    request_scales(m0, n0, e);
    for (int k = 0; k < nslab; k++) {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (B16) {
        if (k == 0) step16(0, true, false, at_a ^ 64, at_b ^ 64);
        else step16(0, false, false, at_a ^ 64, at_b ^ 64);
      } else {
        if (k == 0) step(0, true, false, false, 0, 0);
        else step(0, false, false, false, 0, 0);
        step(1, false, true, false, at_a ^ 64, at_b ^ 64);
        step(0, false, false, false, 0, 0);
      }
      // The next slab has landed for this wave: only a tile's 32 stores (and scales) were issued after it.  All of this slab's
      // operands are in registers, so behind the barrier its stage is free.
      if (stored) wait_vm_barrier<32>(); else wait_vm_barrier<0>();
      stored = false;
      at_a ^= STAGE; at_b ^= STAGE;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (B16) step16(1, false, true, at_a, at_b);
      else step(1, false, true, true, at_a, at_b);
      request_end();
    }

    // ---- epilogue.  Accumulator acc[i][4 b + q][r] of lane (li, lg) is tile row 64 wm + 16 i + 4 lg + r and column
    // 128 wn + 64 b + 4 li + q: a lane stores 16 bytes of a row, the 16 lanes of a group 256 contiguous ones.
    const long long row = (long long)P.ldc * 4, origin = (long long)(m0 + wm * 64) * P.ldc + n0 + wn * 128;
    uint8_t* const out = (uint8_t*)(P.C + origin);
    const uint8_t* const res = (const uint8_t*)(P.add + origin);
    const uint32_t vo = (uint32_t)(lg * 4 * P.ldc + li * 4) * 4;
    float4 bias[2], sa[4];
    float cs[2];
#pragma unroll
    for (int b = 0; b < 2; b++) {
      cs[b] = e[256 + wn * 128 + b * 64 + li * 4];
      bias[b] = has_bias ? *(const float4*)(e + 512 + wn * 128 + b * 64 + li * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < 4; i++) sa[i] = *(const float4*)(e + wm * 64 + i * 16 + lg * 4);
    auto store4 = [&](int g, const float4 (&addv)[4], bool add) {          // group g = 4 b + i: four rows
      const int b = g >> 2, i = g & 3;
      const float sar[4] = {sa[i].x, sa[i].y, sa[i].z, sa[i].w};
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const float s2 = sar[r] * cs[b];
        float4 v = make_float4(acc[i][4 * b][r] * s2, acc[i][4 * b + 1][r] * s2, acc[i][4 * b + 2][r] * s2, acc[i][4 * b + 3][r] * s2);
        if (has_bias) { v.x += bias[b].x; v.y += bias[b].y; v.z += bias[b].z; v.w += bias[b].w; }
        if (add) { v.x += addv[r].x; v.y += addv[r].y; v.z += addv[r].z; v.w += addv[r].w; }
        gstore4_nt((float*)(out + (16 * i + r) * row + b * 256 + vo), v);
      }
    };
    if (!has_add) {
      const float4 none[4] = {};
#pragma unroll
      for (int g = 0; g < 8; g++) { store4(g, none, false); __builtin_amdgcn_sched_barrier(0); }
    } else {
      // The residual tile comes four groups ahead of the one that is stored: loads and stores complete in order, and one
      // group at a time each would wait for the stores in front of it (102400 x 768 x 3072 542 -> 423 us).
      constexpr int D = 4;
      float4 addv[D][4];
      auto load4 = [&](int g) {
#pragma unroll
        for (int r = 0; r < 4; r++) addv[g % D][r] = gload4_nt((const float*)(res + (16 * (g & 3) + r) * row + (g >> 2) * 256 + vo));
      };
#pragma unroll
      for (int g = 0; g < D; g++) load4(g);
#pragma unroll
      for (int g = 0; g < 8; g++) {
        store4(g, addv[g % D], true);
        if (g + D < 8) load4(g + D);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    read_first();                        // once more: what the last slab read ahead has left its registers to the epilogue
    stored = true;
    j += per;
    if (j >= jend) break;
    tile_origin(j, m0, n0);
    par ^= 1;
  }
  wait_vm<0>();                          // no load may still be on its way into LDS that is another workgroup's by then
}

// ------------------------------------------------------------------ FP8 matrix-core instruction
// Lane layout of the instruction (lane = 16*g + i): the operand of lane (i, g) is row i, bytes
// [32g, 32g+32) of the slab.  WAVES_M x WAVES_N wavefronts; each owns a (BM / WAVES_M) x
// (BN / WAVES_N) sub-tile.
template <int BM, int BN, int WAVES_M, int WAVES_N>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_fp8_k(const GemmProb* probs) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int TM = WM / 16, TN = WN / 16;
  constexpr int A_CH = BM * 8 / NT;     // 16-byte chunks per thread
  constexpr int B_CH = BN * 8 / NT;
  __shared__ __attribute__((aligned(16))) uint8_t sA[BM * LDS_ROW];
  __shared__ __attribute__((aligned(16))) uint8_t sB[BN * LDS_ROW];

  const GemmProb P = probs[blockIdx.y];
  const int mt = (P.M + BM - 1) / BM, nt = (P.N + BN - 1) / BN;
  const int lin = xcd_tile(blockIdx.x, mt * nt);
  if (lin >= mt * nt) return;
  const int m0 = (lin / nt) * BM, n0 = (lin % nt) * BN;
  const uint8_t* W = (const uint8_t*)P.W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int li = lane & 15, lg = lane >> 4;

  // global row pointers of this thread's chunks (rows of A may straddle instances)
  const uint8_t* pa[A_CH];
  const uint8_t* pb[B_CH];
#pragma unroll
  for (int c = 0; c < A_CH; c++) {
    int ch = tid + c * NT, r = ch >> 3, kc = ch & 7;
    int m = m0 + r;
    int inst, row; row_origin(m, P.rpi, P.rp0, inst, row);
    pa[c] = (m < P.M) ? (const uint8_t*)P.A + (long long)inst * P.a_is + (long long)row * P.lda + kc * 16 : nullptr;
  }
#pragma unroll
  for (int c = 0; c < B_CH; c++) {
    int ch = tid + c * NT, r = ch >> 3, kc = ch & 7;
    int n = n0 + r;
    pb[c] = (n < P.N) ? W + (long long)n * P.ldw + kc * 16 : nullptr;
  }
  uint4 ra[A_CH], rb[B_CH];
  auto load_slab = [&](int k0) {
#pragma unroll
    for (int c = 0; c < A_CH; c++) ra[c] = pa[c] ? *(const uint4*)(pa[c] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < B_CH; c++) rb[c] = pb[c] ? *(const uint4*)(pb[c] + k0) : make_uint4(0, 0, 0, 0);
  };
  auto store_slab = [&]() {
#pragma unroll
    for (int c = 0; c < A_CH; c++) {
      int ch = tid + c * NT, r = ch >> 3, kc = ch & 7;
      *(uint4*)(sA + r * LDS_ROW + kc * 16) = ra[c];
    }
#pragma unroll
    for (int c = 0; c < B_CH; c++) {
      int ch = tid + c * NT, r = ch >> 3, kc = ch & 7;
      *(uint4*)(sB + r * LDS_ROW + kc * 16) = rb[c];
    }
  };

  v4f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  load_slab(0);
  const int mbase = m0 + wm * WM, nbase = n0 + wn * WN;
  EpiPre<TM, TN> E;
  { int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0); epi_prefetch<TM, TN>(E, P, m0, i0, r0, mbase, nbase, li, lg); }
  for (int k0 = 0; k0 < P.K; k0 += 128) {
    __syncthreads();                 // previous slab fully consumed
    store_slab();
    __syncthreads();
    if (k0 + 128 < P.K) load_slab(k0 + 128);
    v8i fa[TM];
#pragma unroll
    for (int i = 0; i < TM; i++) {
      const uint8_t* p = sA + (wm * WM + i * 16 + li) * LDS_ROW + lg * 32;
      uint4 lo = *(const uint4*)p, hi = *(const uint4*)(p + 16);
      fa[i] = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
    }
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const uint8_t* p = sB + (wn * WN + j * 16 + li) * LDS_ROW + lg * 32;
      uint4 lo = *(const uint4*)p, hi = *(const uint4*)(p + 16);
      v8i fb = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
#pragma unroll
      for (int i = 0; i < TM; i++)
        acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb, fa[i], acc[i][j], 0, 0, 0, 0x7F7F7F7F, 0,
                                                                     0x7F7F7F7F);
    }
  }
  epi_store<TM, TN>(E, P, acc, mbase, nbase, li, lg);
}

// grid of the persistent kernel: at most `per` workgroups (limited by LDS) per compute unit
template <int WAVES_M, int WAVES_N, int TM, int TN, bool B16>
static hipError_t launch_x(const GemmProb* probs, int n_probs, int M, int N, int per, hipStream_t s) {
  constexpr int BM = WAVES_M * TM * 16, BN = WAVES_N * TN * 16;
  const long long tiles = (long long)((M + BM - 1) / BM) * ((N + BN - 1) / BN);
  const int gx = (int)std::min<long long>((tiles + 7) / 8 * 8, 256LL * per);
  hipLaunchKernelGGL((gemm_x_k<WAVES_M, WAVES_N, TM, TN, B16>), dim3(gx, n_probs), dim3(256), 0, s, probs);
  return hipGetLastError();
}
template <int TM, bool B16>
static hipError_t launch_s(const GemmProb* probs, int n_probs, int M, int N, hipStream_t s) {
  const long long tiles = (long long)((M + 32 * TM - 1) / (32 * TM)) * ((N + 63) / 64);
  if (tiles > 0x7ffffff0LL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_s_k<2, 2, TM, 2, 3, B16>), dim3((unsigned)((tiles + 7) / 8 * 8), n_probs), dim3(256), 0, s, probs);
  return hipGetLastError();
}
template <bool B16>
static hipError_t launch_tile(ExactTile t, const GemmProb* probs, int n_probs, int M, int N, hipStream_t s) {
  switch (t) {
    case TILE_64x128: return launch_x<2, 2, 2, 4, B16>(probs, n_probs, M, N, 3, s);
    case TILE_128x64: return launch_x<4, 1, 2, 4, B16>(probs, n_probs, M, N, 3, s);
    case TILE_64x64: return launch_s<2, B16>(probs, n_probs, M, N, s);
    case TILE_32x64: return launch_s<1, B16>(probs, n_probs, M, N, s);
    default: return launch_x<2, 2, 4, 4, B16>(probs, n_probs, M, N, 2, s);
  }
}

// Problems with the log-softmax / KL epilogue: the 128-column tilings that the number of parts per row
// (kl_parts_per_row) is derived from.
hipError_t launch_gemm_fp8_kl(const GemmProb* probs, int n_probs, int max_M, int max_N, int K, int b16, hipStream_t s) {
  if (n_probs == 0 || max_M == 0 || max_N == 0) return hipSuccess;
  const ExactTile t = pick_exact_tile(n_probs, max_M, max_N, K, b16 != 0, true, false, false);
  return b16 ? launch_tile<true>(t, probs, n_probs, max_M, max_N, s) : launch_tile<false>(t, probs, n_probs, max_M, max_N, s);
}

// The kernels of one workgroup per compute unit use more LDS than a launch gets by default.  The attribute belongs to the
// kernel's code object on one device: set once per device (atomically, so that models on several streams or host threads may
// launch concurrently).
static hipError_t launch_one_per_cu(const void* kernel, std::atomic<bool>* set, int lds_bytes, int tiles, int n_probs,
                                    const GemmProb* probs, hipStream_t s) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (!set[dev].load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
    if (e != hipSuccess) return e;
    set[dev].store(true, std::memory_order_release);
  }
  void* args[] = {(void*)&probs};
  return hipLaunchKernel(kernel, dim3(std::min((tiles + 7) / 8 * 8, 256), n_probs), dim3(512), args, lds_bytes, s);
}
template <bool B16>
static hipError_t launch_w(const GemmProb* probs, int n_probs, int M, int N, hipStream_t s) {
  static std::atomic<bool> set[64];
  return launch_one_per_cu((const void*)gemm_w_k<B16>, set, 2 * 512 * 128 + 2 * 768 * 4, ((M + 255) / 256) * ((N + 255) / 256), n_probs, probs, s);
}

hipError_t launch_gemm_fp8(const GemmProb* probs, int n_probs, int max_M, int max_N, int K, int exact, int b16, bool wide, bool residual, hipStream_t s) {
  if (n_probs == 0 || max_M == 0 || max_N == 0) return hipSuccess;
  if (b16 && !exact) return hipErrorInvalidValue;        // bfloat16 operands: exact sums only
  if (exact) {
    const ExactTile t = pick_exact_tile(n_probs, max_M, max_N, K, b16 != 0, false, wide, residual);
    if (t == TILE_256x256) return b16 ? launch_w<true>(probs, n_probs, max_M, max_N, s) : launch_w<false>(probs, n_probs, max_M, max_N, s);
    if (t == TILE_256x128) {
      // three 48 KB stages + 2 KB of scales
      static std::atomic<bool> set[64];
      return launch_one_per_cu((const void*)gemm_p_k<0>, set, 3 * 384 * 128 + 2048, ((max_M + 255) / 256) * ((max_N + 127) / 128), n_probs, probs, s);
    }
    return b16 ? launch_tile<true>(t, probs, n_probs, max_M, max_N, s) : launch_tile<false>(t, probs, n_probs, max_M, max_N, s);
  } else {
    int tiles = ((max_M + 127) / 128) * ((max_N + 63) / 64);
    dim3 grid((tiles + 7) / 8 * 8, n_probs);
    hipLaunchKernelGGL((gemm_fp8_k<128, 64, 4, 1>), grid, dim3(256), 0, s, probs);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ fp32
// 64 x 64 tile, K slabs of 32, four waves as 2 x 2, each 32 x 32 (2 x 2 MFMA tiles).
// MFMA 16x16x4 f32: A operand of lane (i, g) = A[i][g], B operand = B[g][i],
// result lane (i, g) holds C[4g + r][i].  Global loads are 16 bytes per lane where rows allow them.  For what the
// kernel below does not take: K not a multiple of 32 (heads of 16, an MLP of such a width).
__global__ __launch_bounds__(256) void gemm_f32_k(const GemmProb* probs) {
  __shared__ float sA[64][33];
  __shared__ float sB[32][65];
  const GemmProb P = probs[blockIdx.z];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  if (m0 >= P.M || n0 >= P.N) return;
  const float* W = (const float*)P.W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  // A tile 64 x 32 floats = 512 float4: thread -> rows (tid >> 3) and (tid >> 3) + 32, float4 column tid & 7
  const float* pa[2];
#pragma unroll
  for (int c = 0; c < 2; c++) {
    int m = m0 + (tid >> 3) + 32 * c;
    int inst, row; row_origin(m, P.rpi, P.rp0, inst, row);
    pa[c] = (m < P.M) ? (const float*)P.A + (long long)inst * P.a_is + (long long)row * P.lda + (tid & 7) * 4 : nullptr;
  }
  // B tile 32 x 64 floats = 512 float4: thread -> k rows (tid >> 4) and (tid >> 4) + 16, float4 column tid & 15
  const int bn = n0 + (tid & 15) * 4;
  v4f acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int j = 0; j < 2; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  for (int k0 = 0; k0 < P.K; k0 += 32) {
    float4 va[2], vb[2];
#pragma unroll
    for (int c = 0; c < 2; c++) {
      int k = k0 + (tid & 7) * 4;
      va[c] = (pa[c] && k + 3 < P.K) ? *(const float4*)(pa[c] + k0) : make_float4(0, 0, 0, 0);
      if (pa[c] && k < P.K && k + 3 >= P.K) {             // ragged K tail
        float t[4] = {0, 0, 0, 0};
        for (int q = 0; q < 4 && k + q < P.K; q++) t[q] = pa[c][k0 + q];
        va[c] = make_float4(t[0], t[1], t[2], t[3]);
      }
      int kb = k0 + (tid >> 4) + 16 * c;
      if (kb < P.K && bn + 3 < P.N && ((P.ldw & 3) == 0)) vb[c] = *(const float4*)(W + (long long)kb * P.ldw + bn);
      else {
        float t[4] = {0, 0, 0, 0};
        if (kb < P.K) for (int q = 0; q < 4 && bn + q < P.N; q++) t[q] = W[(long long)kb * P.ldw + bn + q];
        vb[c] = make_float4(t[0], t[1], t[2], t[3]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; c++) {
      int r = (tid >> 3) + 32 * c, k = (tid & 7) * 4;
      sA[r][k] = va[c].x; sA[r][k + 1] = va[c].y; sA[r][k + 2] = va[c].z; sA[r][k + 3] = va[c].w;
      int kb = (tid >> 4) + 16 * c, n = (tid & 15) * 4;
      sB[kb][n] = vb[c].x; sB[kb][n + 1] = vb[c].y; sB[kb][n + 2] = vb[c].z; sB[kb][n + 3] = vb[c].w;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 32; kk += 4) {
      float fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; i++) fa[i] = sA[wm * 32 + i * 16 + li][kk + lg];
#pragma unroll
      for (int j = 0; j < 2; j++) fb[j] = sB[kk + lg][wn * 32 + j * 16 + li];
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int i = 0; i < 2; i++)
#pragma unroll
    for (int r = 0; r < 4; r++) {
      int m = m0 + wm * 32 + i * 16 + lg * 4 + r;
      if (m >= P.M) continue;
      int inst, row; row_origin(m, P.rpi, P.rp0, inst, row);
#pragma unroll
      for (int j = 0; j < 2; j++) {
        int n = n0 + wn * 32 + j * 16 + li;
        if (n >= P.N) continue;
        epilogue_store(P, n, acc[i][j][r], 1.0f, 1.0f, inst, row);
      }
    }
}

// The fp32 product for K a multiple of 32 and 16-byte aligned rows of A.  Per element the same sum as gemm_f32_k: one
// V_MFMA_F32_16X16X4_F32 per four k, ascending.  W is the first operand here, so that a lane owns one row and four
// neighbouring columns (16-byte stores).  Slabs of 32 k go from global memory straight into LDS, two stages; a lane reads
// its single k of a step (a wider read would hand it four k of one row and change the order of the sum).  STEP slabs make a
// step: they are requested together and one wait and barrier stand in front of them.
// LDS rows have no padding: chunk c (16 bytes) of row r of A sits at chunk c ^ (r & 7), chunk c of row k of W
// at c ^ swz(k), so that the 64 words a read of W takes lie in 64 banks and those of A in at least 32.
// Bound by the fp32 matrix cores' issue once the chip is full (121 to 130 TFLOP/s, where a loop of nothing but these
// instructions reaches 138), by a wave's chain of waits, reads and products before that: the tile and the step are chosen by how
// the launch fills the chip (pick_f32_tile).  Three or four stages instead of two, or the next operands read in front
// of the present products, gain nothing there and cost up to a tenth where the chip is full.
// STEP 0: the rows of W are not 16-byte aligned (an unembedding with an odd vocabulary) and W comes word by word, a slab a step.
template <int WAVES_M, int WAVES_N, int TM, int TN, int STEP>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void gemm_f32_x_k(const GemmProb* probs, int n_probs, int mt, int nt, int col_first) {
  constexpr bool WV4 = STEP > 0;
  constexpr int SUB = WV4 ? STEP : 1;
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int BM = WAVES_M * TM * 16, BN = WAVES_N * TN * 16;
  constexpr int IA = BM / 8 / NW;                       // load instructions per wave and slab: A (8 rows each)
  constexpr int IB = (WV4 ? BN / 8 : BN / 2) / NW;      // and W (256 or 64 words each)
  constexpr int ABYTES = BM * 128, STAGE = ABYTES + BN * 128;
  static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && BN >= 32, "rows must split evenly over the waves");
  __shared__ __attribute__((aligned(1024))) uint8_t st[2 * SUB * STAGE];
  // all problems' tiles of a row tile are neighbours on one XCD (heads read the same rows); with more columns than
  // rows the row tiles of one column tile are
  const int lin = xcd_tile(blockIdx.x, mt * nt * n_probs);
  if (lin >= mt * nt * n_probs) return;
  const int pi = col_first ? lin / (mt * nt) : (lin / nt) % n_probs;
  const int m0 = (col_first ? lin % mt : lin / (nt * n_probs)) * BM, n0 = (col_first ? (lin / mt) % nt : lin % nt) * BN;
  const GemmProb P = probs[pi];
  if (m0 >= P.M || n0 >= P.N) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int li = lane & 15, lg = lane >> 4;
  auto swz = [](int k) { return BN == 32 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); };

  const uint8_t* srcA[IA];
  const uint8_t* srcB[IB];
  int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
#pragma unroll
  for (int t = 0; t < IA; t++) {
    const int m = min(m0 + 8 * (wave * IA + t) + (lane >> 3), P.M - 1);
    int inst, row; split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
    srcA[t] = (const uint8_t*)((const float*)P.A + (long long)inst * P.a_is + (long long)row * P.lda) + ((lane & 7) ^ (lane >> 3)) * 16;
  }
#pragma unroll
  for (int t = 0; t < IB; t++) {
    const int f = WV4 ? ((wave * IB + t) * 64 + lane) * 4 : (wave * IB + t) * 64 + lane;      // word of the W slab in LDS
    const int k = f / BN, c = (f % BN) >> 2;
    const int n = n0 + ((c ^ swz(k)) << 2) + (f & 3);
    srcB[t] = (const uint8_t*)((const float*)P.W + (long long)k * P.ldw + min(n, P.N - (WV4 ? 4 : 1)));
  }
  const long long stepB = 32LL * P.ldw * 4;
  const uint32_t lds0 = lds_addr_of(st);
  auto issue_slab = [&](int stage) {
    const uint32_t ba = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + wave * IA * 1024);
    const uint32_t bb = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + ABYTES + wave * IB * (WV4 ? 1024 : 256));
#pragma unroll
    for (int t = 0; t < IA; t++) { slab_load16(srcA[t], ba + t * 1024); srcA[t] += 128; }
#pragma unroll
    for (int t = 0; t < IB; t++) {
      if (WV4) slab_load16(srcB[t], bb + t * 1024); else lds_load4(srcB[t], bb + t * 256);
      srcB[t] += stepB;
    }
  };
  v4f acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  int offB[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) offB[j] = ABYTES + (lg * BN + ((((wn * TN + j) * 4 + (li >> 2)) ^ swz(lg)) << 2) + (li & 3)) * 4;
  const int offA = (wm * TM * 16 + li) * 128 + lg * 4;
  auto compute = [&](const uint8_t* s) {
#pragma unroll
    for (int q = 0; q < 8; q++) {
      float fa[TM], fb[TN];
      const int sw = (q ^ (li & 7)) * 16;
#pragma unroll
      for (int i = 0; i < TM; i++) fa[i] = *(const float*)(s + offA + i * 2048 + sw);
#pragma unroll
      for (int j = 0; j < TN; j++) fb[j] = *(const float*)(s + offB[j] + q * (16 * BN));
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  };
  const int nslab = P.K >> 5, nstep = (nslab + SUB - 1) / SUB;
  auto issue = [&](int step) {
#pragma unroll
    for (int u = 0; u < SUB; u++) if (SUB == 1 || step * SUB + u < nslab) issue_slab((step & 1) * SUB + u);
  };
  issue(0);
  for (int k = 0; k < nstep; k++) {
    wait_vm_barrier<0>();                               // the step's slabs have landed for everyone, the previous one's stage is free
    if (k + 1 < nstep) issue(k + 1);
    const uint8_t* s = st + (k & 1) * (SUB * STAGE);
    if (SUB == 1 || (k + 1) * SUB <= nslab) {
#pragma unroll
      for (int u = 0; u < SUB; u++) compute(s + u * STAGE);
    } else {
      for (int u = 0; k * SUB + u < nslab; u++) compute(s + u * STAGE);
    }
  }
  // 16-byte accesses where rows, strides and pointers allow them
  const bool al = ((P.ldc | P.c_is | (P.add ? P.add_is : 0) | (P.aux ? P.aux_is : 0)) & 3) == 0 &&
                  (((uintptr_t)P.C | (uintptr_t)P.add | (uintptr_t)P.aux | (uintptr_t)P.aux_sub) & 15) == 0;
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int m = m0 + wm * TM * 16 + i * 16 + li;
    if (m >= P.M) continue;
    int inst, row; split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int n = n0 + wn * TN * 16 + j * 16 + lg * 4;
      if (al && n + 3 < P.N) {
        const float4 val = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        float4 v = val;
        if (P.bias) { v.x += GCF(P.bias)[n]; v.y += GCF(P.bias)[n + 1]; v.z += GCF(P.bias)[n + 2]; v.w += GCF(P.bias)[n + 3]; }
        if (P.act == 1) { v.x = gelu_tanh(v.x); v.y = gelu_tanh(v.y); v.z = gelu_tanh(v.z); v.w = gelu_tanh(v.w); }
        const long long off = (long long)row * P.ldc + n;
        if (P.add) { const float4 a = gload4(P.add + inst * P.add_is + off); v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w; }
        gstore4(P.C + inst * P.c_is + off, v);
        if (P.aux) {
          float4 x = val;
          if (P.aux_sub) { const float4 u = gload4(P.aux_sub + off); x.x -= u.x; x.y -= u.y; x.z -= u.z; x.w -= u.w; }
          gstore4(P.aux + inst * P.aux_is + off, x);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++) if (n + r < P.N) epilogue_store(P, n + r, acc[i][j][r], 1.0f, 1.0f, inst, row);
      }
    }
  }
}

// Output projections of the fp32 heads of a layer, summed:
//   C[m] = (run_in[m] + bias) + (((add[m] + z_0 W_0) + z_1 W_1) + ...)        (run_in null: the bracket alone)
// probs[h] is head h's projection (A = the head's columns of the rows of all heads, which lie side by side: probs[0].A and
// 4 K bytes per head); rows, C and `add` are probs[0]'s, W and the second output (aux = z_h W_h - aux_sub) each head's own.
// One launch per head moved the running sum through memory H times: with eight heads of 64 and 16384 rows of 512 the heads'
// 25 us each were 20 us of traffic, and at 1024 rows 14 us each were latency.  Here the sum stays in registers.
// Every head's product starts from zero and is then added, ascending: the bits of the launches one by one.
// Slabs, operand layout and tiles as in gemm_f32_x_k; the slabs of all heads are one stream.  A head has few slabs (two of
// 64 columns), so nothing may stand between the heads: the pointers of the next one come by scalar loads ahead of time,
// aux_sub through LDS while the head's last slab is multiplied, and the stores of aux are counted: vector memory operations retire
// in order, so the wait for a slab allows as many as were issued behind it.  (With aux_sub, a head's stores are retired by the next
// head's wait for its subtrahend.)
// Two stages: a third one, requested two slabs ahead, gains nothing where the chip is not full and costs workgroups where it is
// (45 KB instead of 33 with 32 x 64 tiles, three instead of four per unit: 6 heads of 32, 10700 x 192 with aux 23.2 / 16.4 us).  Of
// 400 random launches of 2 to 16 heads none takes longer by more than 3 % than with the waits between heads, in the mean 0.88.
template <int TM, int TN>
__global__ __launch_bounds__(256) void gemm_f32_heads_k(const GemmProb* probs, int n_heads, int mt, int nt, const float* run_in,
                                                         long long run_is, const float* bias) {
  constexpr int BM = 32 * TM, BN = 32 * TN, IA = BM / 32, IB = BN / 32;
  constexpr int ABYTES = BM * 128, STAGE = ABYTES + BN * 128;
  static_assert(BN == 64 || BN == 32, "swz below");
  __shared__ __attribute__((aligned(1024))) uint8_t st[2 * STAGE + 4 * TM * TN * 1024];
  const int lin = xcd_tile(blockIdx.x, mt * nt);
  if (lin >= mt * nt) return;
  const int m0 = (lin / nt) * BM, n0 = (lin % nt) * BN;
  const GemmProb P = probs[0];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lg = lane >> 4;
  auto swz = [](int k) { return BN == 32 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); };
  int i0, r0; row_origin(m0, P.rpi, P.rp0, i0, r0);
  const uint8_t* srcA[IA];
  long long offW[IB];
#pragma unroll
  for (int t = 0; t < IA; t++) {
    const int m = min(m0 + 8 * (wave * IA + t) + (lane >> 3), P.M - 1);
    int inst, row; split_row(i0, r0, m - m0, P.rpi, P.rp0, inst, row);
    srcA[t] = (const uint8_t*)((const float*)P.A + (long long)inst * P.a_is + (long long)row * P.lda) + ((lane & 7) ^ (lane >> 3)) * 16;
  }
#pragma unroll
  for (int t = 0; t < IB; t++) {
    const int f = ((wave * IB + t) * 64 + lane) * 4, k = f / BN, c = (f % BN) >> 2;
    offW[t] = (long long)k * P.ldw + min(n0 + ((c ^ swz(k)) << 2), P.N - 4);
  }
  const int spk = P.K >> 5, nslab = spk * n_heads;      // slabs of a head, of all
  const uint32_t lds0 = lds_addr_of(st);
  // the heads' pointers by scalar loads (a vector load of them would wait for the requested slabs and the stores too)
  const auto* const cp = (const __attribute__((address_space(4))) GemmProb*)(uintptr_t)probs;
  int rh = 0, rk = 0;                                   // head and slab of the next request
  const float* rw = (const float*)P.W;
  const float* rw_next = (const float*)cp[min(1, n_heads - 1)].W;
  auto issue = [&](int stage) {
    const uint32_t ba = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + wave * IA * 1024);
    const uint32_t bb = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGE + ABYTES + wave * IB * 1024);
#pragma unroll
    for (int t = 0; t < IA; t++) { slab_load16(srcA[t], ba + t * 1024); srcA[t] += 128; }
#pragma unroll
    for (int t = 0; t < IB; t++) slab_load16((const uint8_t*)(rw + offW[t]), bb + t * 1024);
    rw += 32LL * P.ldw;
    if (++rk == spk) { rk = 0; rh++; rw = rw_next; rw_next = (const float*)cp[min(rh + 1, n_heads - 1)].W; }
  };
  int offB[TN];
#pragma unroll
  for (int j = 0; j < TN; j++) offB[j] = ABYTES + (lg * BN + ((((wn * TN + j) * 4 + (li >> 2)) ^ swz(lg)) << 2) + (li & 3)) * 4;
  const int offA = (wm * TM * 16 + li) * 128 + lg * 4;
  v4f acc[TM][TN], tot[TM][TN];
  // what a lane adds to: its row and the columns n .. n + 3 of every 16 x 16 block
  int inst[TM], row[TM];
  bool on[TM];
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int m = m0 + wm * TM * 16 + i * 16 + li;
    on[i] = m < P.M;
    split_row(i0, r0, min(m, P.M - 1) - m0, P.rpi, P.rp0, inst[i], row[i]);
  }
  const int nb = n0 + wn * TN * 16 + lg * 4;
  int nc[TN];                                           // those columns, or the last ones
#pragma unroll
  for (int j = 0; j < TN; j++) nc[j] = min(nb + j * 16, P.N - 4);
  // -0 + x is x
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) {
      tot[i][j] = (v4f){-0.f, -0.f, -0.f, -0.f};
      if (P.add) { const float4 a = gload4(P.add + inst[i] * P.add_is + (long long)row[i] * P.ldc + nc[j]); tot[i][j] = (v4f){a.x, a.y, a.z, a.w}; }
    }
  const uint32_t lds_u = __builtin_amdgcn_readfirstlane(lds0 + 2 * STAGE + wave * TM * TN * 1024);
  const uint8_t* const own_u = st + 2 * STAGE + wave * TM * TN * 1024 + lane * 16;
  issue(0);
  int slab = 0;
  bool stored = false;                                  // has a second output left behind the previous slab?
  for (int h = 0; h < n_heads; h++) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    float* const aux = cp[h].aux;
    const float* const sub = cp[h].aux_sub;
    const long long aux_is = cp[h].aux_is;
    for (int k = 0; k < spk; k++, slab++) {
      // the slab has landed for everyone, the other stage is free; younger than the slab's loads are the stores behind the
      // previous slab alone
      if (stored) wait_vm_barrier<TM * TN>(); else wait_vm_barrier<0>();
      stored = false;
      if (k == spk - 1 && aux && sub) {                 // each lane's own values, through LDS: in front of the next request
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) slab_load16((const uint8_t*)(sub + (long long)row[i] * P.ldc + nc[j]), lds_u + (i * TN + j) * 1024);
      }
      if (slab + 1 < nslab) issue((slab + 1) & 1);
      const uint8_t* s = st + (slab & 1) * STAGE;
#pragma unroll
      for (int q = 0; q < 8; q++) {
        float fa[TM], fb[TN];
        const int sw = (q ^ (li & 7)) * 16;
#pragma unroll
        for (int i = 0; i < TM; i++) fa[i] = *(const float*)(s + offA + i * 2048 + sw);
#pragma unroll
        for (int j = 0; j < TN; j++) fb[j] = *(const float*)(s + offB[j] + q * (16 * BN));
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j], fa[i], acc[i][j], 0, 0, 0);
      }
    }
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) tot[i][j] += acc[i][j];
    if (aux) {
      stored = true;
      if (sub) {                                        // this head's subtrahend (and with it the stores of the head before)
        if (slab < nslab) wait_vm<IA + IB>(); else wait_vm<0>();
      }
      // every lane stores, so that a wave has TM * TN stores whatever its rows and columns are: past the end a lane's
      // operands, and so its value, are those of the last row or column
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++) {
          float4 x = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
          if (sub) { const float4 u = *(const float4*)(own_u + (i * TN + j) * 1024); x.x -= u.x; x.y -= u.y; x.z -= u.z; x.w -= u.w; }
          gstore4(aux + inst[i] * aux_is + (long long)row[i] * P.ldc + nc[j], x);
        }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) {
      const int n = nb + j * 16;
      if (!on[i] || n >= P.N) continue;
      const long long off = (long long)row[i] * P.ldc + n;
      float4 v = make_float4(tot[i][j][0], tot[i][j][1], tot[i][j][2], tot[i][j][3]);
      if (run_in) {
        float4 r = gload4(run_in + inst[i] * run_is + off);
        if (bias) { const float4 b = gload4(bias + n); r.x += b.x; r.y += b.y; r.z += b.z; r.w += b.w; }
        v.x = r.x + v.x; v.y = r.y + v.y; v.z = r.z + v.z; v.w = r.w + v.w;
      }
      gstore4(P.C + inst[i] * P.c_is + off, v);
    }
}
hipError_t launch_gemm_f32_heads(const GemmProb* probs, int n_heads, int M, int N, const float* run_in, long long run_is,
                                 const float* bias, hipStream_t s) {
  if (n_heads == 0 || M == 0 || N == 0) return hipSuccess;
  auto tiles = [&](int bm, int bn) { return (long long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
  auto grid = [](long long t) { return dim3((unsigned)((t + 7) / 8 * 8)); };
  if (tiles(32, 32) > 0x7ffffff0LL) return hipErrorInvalidValue;
  // from two tiles of 64 x 64 per compute unit on those, below that smaller ones, so that every unit has waves to switch between
  if (tiles(64, 64) >= 512) hipLaunchKernelGGL((gemm_f32_heads_k<2, 2>), grid(tiles(64, 64)), dim3(256), 0, s, probs, n_heads, (M + 63) / 64, (N + 63) / 64, run_in, run_is, bias);
  else if (tiles(64, 64) >= 96) hipLaunchKernelGGL((gemm_f32_heads_k<1, 2>), grid(tiles(32, 64)), dim3(256), 0, s, probs, n_heads, (M + 31) / 32, (N + 63) / 64, run_in, run_is, bias);
  else hipLaunchKernelGGL((gemm_f32_heads_k<1, 1>), grid(tiles(32, 32)), dim3(256), 0, s, probs, n_heads, (M + 31) / 32, (N + 31) / 32, run_in, run_is, bias);
  return hipGetLastError();
}

template <int WAVES_M, int WAVES_N, int TM, int TN, int STEP>
static hipError_t launch_f32_x(const GemmProb* probs, int n_probs, int M, int N, hipStream_t s) {
  const int BM = WAVES_M * TM * 16, BN = WAVES_N * TN * 16, mt = (M + BM - 1) / BM, nt = (N + BN - 1) / BN;
  const long long tiles = (long long)mt * nt * n_probs;
  if (tiles > 0x7ffffff0LL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_f32_x_k<WAVES_M, WAVES_N, TM, TN, STEP>), dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(256), 0, s, probs,
                     n_probs, mt, nt, n_probs == 1 && N > M ? 1 : 0);
  return hipGetLastError();
}
// form: the smallest gemm32_form of the problems.  K: that of all of them.
hipError_t launch_gemm_f32(const GemmProb* probs, int n_probs, int max_M, int max_N, int K, int form, hipStream_t s) {
  if (n_probs == 0 || max_M == 0 || max_N == 0) return hipSuccess;
  if (form == 2) {
    switch (pick_f32_tile(n_probs, max_M, max_N, K)) {
      case F32_128x128: return launch_f32_x<2, 2, 4, 4, 1>(probs, n_probs, max_M, max_N, s);
      case F32_64x64: return launch_f32_x<2, 2, 2, 2, 1>(probs, n_probs, max_M, max_N, s);
      case F32_32x64_STEP4: return launch_f32_x<2, 2, 1, 2, 4>(probs, n_probs, max_M, max_N, s);
      case F32_32x64: return launch_f32_x<2, 2, 1, 2, 1>(probs, n_probs, max_M, max_N, s);
      case F32_32x32_STEP4: return launch_f32_x<2, 2, 1, 1, 4>(probs, n_probs, max_M, max_N, s);
      case F32_32x32: return launch_f32_x<2, 2, 1, 1, 1>(probs, n_probs, max_M, max_N, s);
    }
  }
  const long long t = tile_count(n_probs, max_M, max_N, 64, 64);
  if (form == 1) return t >= 256 ? launch_f32_x<2, 2, 2, 2, 0>(probs, n_probs, max_M, max_N, s)
                                 : launch_f32_x<2, 2, 1, 1, 0>(probs, n_probs, max_M, max_N, s);
  dim3 grid((max_N + 63) / 64, (max_M + 63) / 64, n_probs);
  hipLaunchKernelGGL(gemm_f32_k, grid, dim3(256), 0, s, probs);
  return hipGetLastError();
}

}  // namespace pahq

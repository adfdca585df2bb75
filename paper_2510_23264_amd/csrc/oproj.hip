// Output projection of all heads of a layer fused with the stream update:
//   next[m][:] = run[m][:] + b_O + extra[m][:] + sum_h (z_h[m] W_O^h) * s_z[m][h] * s_w[h]
// Each head is a part of K (in oproj_fused_k a slab of 128 bytes padded with zeros, in
// oproj_x_k and oproj_w_k its codes alone, the heads side by side) with its own row and
// weight scale, so the MFMA result of a head is scaled and added to the running total in
// registers; the per-head sender outputs never go to HBM unless a receiver needs one
// (HeadAux: the head's output, optionally minus the corrupted run's, is written next to the
// total).  `extra` carries the fp32 head's contribution, computed by the fp32 GEMM.
// oproj_fused_k, for other head sizes: tile 128 x 64, four wavefronts of 32 x 64; operands staged
// through LDS as in the fp8 GEMM (144-byte rows), next head prefetched into registers.
#include "kernels.h"
#include "device_util.h"
#include "mma_util.h"
#include <atomic>
#include <cmath>
#include <type_traits>

namespace pahq {

#define LDS_ROW 144

template <bool EXACT>
__global__ __launch_bounds__(256) void oproj_fused_k(const OprojDesc* descs, int di, const HeadAux* auxs) {
  constexpr int BM = 128, BN = 64, TM = 2, TN = 4;
  __shared__ __attribute__((aligned(16))) uint8_t sA[BM * LDS_ROW];
  __shared__ __attribute__((aligned(16))) uint8_t sB[BN * LDS_ROW];
  const OprojDesc D = descs[di];
  const int mt = (D.M + BM - 1) / BM, nt = (D.N + BN - 1) / BN;
  const int chunk = (mt * nt + 7) >> 3;
  const int lin = (blockIdx.x & 7) * chunk + (blockIdx.x >> 3);
  if (lin >= mt * nt) return;
  const int m0 = (lin / nt) * BM, n0 = (lin % nt) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;

  // this thread's chunks: A rows (tid>>3) + 32c, B rows (tid>>3) + 32c; 16-byte column kc
  const int kc = tid & 7;
  const uint8_t* pa[4];
  const uint8_t* pb[2];
#pragma unroll
  for (int c = 0; c < 4; c++) {
    int m = m0 + (tid >> 3) + 32 * c;
    int inst, row; row_origin(m, D.rpi, D.rp0, inst, row);
    pa[c] = (m < D.M) ? D.zc + (long long)inst * D.zc_is + (long long)row * D.H * D.Kz + kc * 16 : nullptr;
  }
#pragma unroll
  for (int c = 0; c < 2; c++) {
    int n = n0 + (tid >> 3) + 32 * c;
    pb[c] = (n < D.N) ? D.W + (long long)n * D.Kz + kc * 16 : nullptr;
  }
  uint4 ra[4], rb[2];
  // codes beyond d_head are zero padding: neither loaded nor (with the fp16 matrix cores) multiplied
  const bool real_chunk = kc * 16 < D.dh;
  const int nkk = (D.dh + 31) >> 5;
  auto load_head = [&](int h) {
#pragma unroll
    for (int c = 0; c < 4; c++)
      ra[c] = (pa[c] && real_chunk) ? *(const uint4*)(pa[c] + (long long)h * D.Kz) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int c = 0; c < 2; c++)
      rb[c] = (pb[c] && real_chunk) ? *(const uint4*)(pb[c] + (long long)h * D.N * D.Kz) : make_uint4(0, 0, 0, 0);
  };
  auto skipped = [&](int h) { return ((D.skip_mask >> h) & 1ull) != 0; };
  auto next_head = [&](int h) { h++; while (h < D.H && skipped(h)) h++; return h; };

  // W is the first MFMA operand, so lane (i, g) owns row i of a 16-row tile and columns 4g .. 4g+3
  int row_m[TM];
  const float* zs_p[TM];
#pragma unroll
  for (int i = 0; i < TM; i++) {
    int m = m0 + wave * 32 + i * 16 + li;
    row_m[i] = m;
    int mm = m < D.M ? m : D.M - 1;
    int inst, row; row_origin(mm, D.rpi, D.rp0, inst, row);
    zs_p[i] = D.zs + (long long)inst * D.zs_is + (long long)row * D.H;
  }

  v4f tot[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) tot[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  int h = next_head(-1);
  if (h < D.H) load_head(h);
  for (; h < D.H; h = next_head(h)) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; c++) *(uint4*)(sA + ((tid >> 3) + 32 * c) * LDS_ROW + kc * 16) = ra[c];
#pragma unroll
    for (int c = 0; c < 2; c++) *(uint4*)(sB + ((tid >> 3) + 32 * c) * LDS_ROW + kc * 16) = rb[c];
    __syncthreads();
    int hn = next_head(h);
    if (hn < D.H) load_head(hn);

    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
    if (EXACT) {
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
        if (kk >= nkk) break;
        v8h ha[TM];
#pragma unroll
        for (int i = 0; i < TM; i++) {
          uint2 w = *(const uint2*)(sA + (wave * 32 + i * 16 + li) * LDS_ROW + kk * 32 + lg * 8);
          ha[i] = decode8(w.x, w.y);
        }
#pragma unroll
        for (int j = 0; j < TN; j++) {
          uint2 w = *(const uint2*)(sB + (j * 16 + li) * LDS_ROW + kk * 32 + lg * 8);
          v8h hb = decode8(w.x, w.y);
#pragma unroll
          for (int i = 0; i < TM; i++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb, ha[i], acc[i][j], 0, 0, 0);
        }
      }
    } else {
      v8i fa[TM];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        const uint8_t* p = sA + (wave * 32 + i * 16 + li) * LDS_ROW + lg * 32;
        uint4 lo = *(const uint4*)p, hi = *(const uint4*)(p + 16);
        fa[i] = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
      }
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const uint8_t* p = sB + (j * 16 + li) * LDS_ROW + lg * 32;
        uint4 lo = *(const uint4*)p, hi = *(const uint4*)(p + 16);
        v8i fb = (v8i){(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
#pragma unroll
        for (int i = 0; i < TM; i++)
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb, fa[i], acc[i][j], 0, 0, 0, 0x7F7F7F7F, 0,
                                                                       0x7F7F7F7F);
      }
    }
    // scale this head's result, add it to the total, and hand it out if some receiver needs it
    const float sw = D.ws[h];
    HeadAux ax; ax.dst = nullptr; ax.dst_is = 0; ax.sub = nullptr;
    if (D.aux_begin >= 0) ax = auxs[D.aux_begin + h];
#pragma unroll
    for (int i = 0; i < TM; i++) {
      float sc = zs_p[i][h] * sw;
      int m = row_m[i];
#pragma unroll
      for (int j = 0; j < TN; j++) {
        float4 val = make_float4(acc[i][j][0] * sc, acc[i][j][1] * sc, acc[i][j][2] * sc, acc[i][j][3] * sc);
        tot[i][j][0] += val.x; tot[i][j][1] += val.y; tot[i][j][2] += val.z; tot[i][j][3] += val.w;
        if (ax.dst) {
          int nb = n0 + j * 16 + lg * 4;
          if (m < D.M && nb < D.N) {
            int inst, row; row_origin(m, D.rpi, D.rp0, inst, row);
            long long off = (long long)row * D.N + nb;
            if (ax.sub) { float4 u = *(const float4*)(ax.sub + off); val.x -= u.x; val.y -= u.y; val.z -= u.z; val.w -= u.w; }
            *(float4*)(ax.dst + (long long)inst * ax.dst_is + off) = val;
          }
        }
      }
    }
  }

#pragma unroll
  for (int i = 0; i < TM; i++) {
    int m = row_m[i];
    if (m >= D.M) continue;
    int inst, row; row_origin(m, D.rpi, D.rp0, inst, row);
    long long roff = (long long)row * D.N;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      int nb = n0 + j * 16 + lg * 4;
      if (nb >= D.N) continue;
      float4 v = *(const float4*)(D.run_in + inst * D.run_in_is + roff + nb);
      if (D.bias) { float4 b = *(const float4*)(D.bias + nb); v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w; }
      v.x += tot[i][j][0]; v.y += tot[i][j][1]; v.z += tot[i][j][2]; v.w += tot[i][j][3];
      // the fp32 head goes in last: (stream + bias + other heads) + fp32 head, the same association
      // the candidate path uses when it adds that head to a precomputed sum of the others
      if (D.extra) { float4 e = *(const float4*)(D.extra + inst * D.extra_is + roff + nb); v.x += e.x; v.y += e.y; v.z += e.z; v.w += e.w; }
      *(float4*)(D.run_out + inst * D.run_out_is + roff + nb) = v;
    }
  }
}

// ------------------------------------------------------------------ exact sums, d_head 64 or 128
// The same projection with the slab pipeline of the exact GEMM: slabs of 128 code bytes (one head
// of 128, or two heads of 64, which lie side by side in the rows of both operands) go straight into
// swizzled LDS.  128 x 64 tile, eight wavefronts of 32 x 32 (two workgroups
// per compute unit, four waves per SIMD: a tile is a chain of short dependent steps - six slabs of 16
// matrix instructions per wave, then the stream tile - and it is the number of waves in flight that
// hides their latencies; four waves of 32 x 64 took a tenth longer).  A head's
// partial result is complete after one (d_head 64) or two (d_head 128) 64-byte halves of a slab;
// it is scaled by z-scale[row][head] * w-scale[head] and added to the running total in registers.
// A head that is computed in fp32 elsewhere (skip mask) is multiplied like the others and left out of the sum.
// Three stages of 25 KB, a slab requested two slabs before it is multiplied: with one slab of
// look-ahead a workgroup waits for memory at every slab (a slab is far less work than the latency
// of its loads under load).  For the waits to be countable every
// load inside the loop goes into LDS by the same path, also the row scales of a slab's heads (one
// dword per lane and wave with each slab) and the weight scales (once, before slab 0): a wave
// waits for slab s with "at most the four operations of slab s + 1 outstanding".  A layer that
// hands out per-head results issues stores and loads of its own inside the loop; it drains
// instead of counting.
// DH: bytes of a head's row of codes (64 or 128).  B16: they are bfloat16 patterns (d_head = DH / 2), multiplied
// without conversion by V_MFMA_F32_16X16X32_BF16, one step per 16-byte operand read; everything else is the same.
// BM: rows of a tile, 128 or 32 (four wavefronts of 16 x 32; for problems of few tiles, see launch_oproj_fused).
constexpr int OPX_STAGES = 3;
constexpr int opx_oper(int BM) { return (BM + 64) * 128; }                                     // operand bytes of a stage
constexpr int opx_stage(int BM) { return opx_oper(BM) + 1024; }                                // + row scales [heads of the slab][BM]
constexpr int opx_lds(int BM) { return OPX_STAGES * opx_stage(BM) + 256; }                     // + weight scales [64]
template <int DH, bool B16, int BM>
__global__ __launch_bounds__(BM == 128 ? 512 : 256, 4) void oproj_x_k(const OprojDesc* descs, int di, const HeadAux* auxs) {
  constexpr int BN = 64, TM = BM == 128 ? 2 : 1, TN = 2, NI = 3, NS = OPX_STAGES, STAGE = opx_stage(BM);
  static_assert(BM == 128 || BM == 32, "waves: BM / (16 TM) x 2, three loads each");
  constexpr int HPS = 128 / DH;            // heads per slab
  static_assert(NI + 1 == 4, "four loads per slab and wave: the wait counts below assume it");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const float* const e_ws = (const float*)(smem + NS * STAGE);
  const OprojDesc D = descs[di];
  const int mt = (D.M + BM - 1) / BM, nt = (D.N + BN - 1) / BN;
  const int lin = xcd_tile(blockIdx.x, mt * nt);
  if (lin >= mt * nt) return;
  const int m0 = (lin / nt) * BM, n0 = (lin % nt) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lg = lane >> 4;
  const int nslab = D.H / HPS;
  const uint32_t lds0 = lds_addr_of(smem);

  // lane l of a load instruction fills LDS row l >> 3, chunk position l & 7, i.e. logical chunk
  // c = (l & 7) ^ (l >> 3) of the slab
  const int c = (lane & 7) ^ (lane >> 3);
  const uint8_t* src[NI];
#pragma unroll
  for (int t = 0; t < NI; t++) {
    int r = 8 * (wave * NI + t) + (lane >> 3);
    if (r < BM) {
      int m = min(m0 + r, D.M - 1), inst, row;
      row_origin(m, D.rpi, D.rp0, inst, row);
      src[t] = D.zc + (long long)inst * D.zc_is + (long long)row * D.H * DH + c * 16;
    } else {
      int n = min(n0 + r - BM, D.N - 1);
      src[t] = D.W + (long long)n * D.H * DH + c * 16;
    }
  }
  // row scales of a slab: entry [q][r] (head q of the slab, tile row r) is lane's if 64 wave + lane = BM q + r;
  // waves past the last entry repeat what earlier ones fetch (so that all waves count alike), and with one head per slab
  // the entries behind the first BM repeat the rows into the unused part
  const float* zsrc;
  {
    const int e = (wave & 3) * 64 + lane;
    const int q = (HPS == 2) ? (e / BM) & 1 : 0;
    int inst, row; row_origin(min(m0 + e % BM, D.M - 1), D.rpi, D.rp0, inst, row);
    zsrc = D.zs + (long long)inst * D.zs_is + (long long)row * D.H + q;
  }
  int si = 0;                              // stage of the next request
  auto issue = [&]() {                     // fetches the next slab and advances
    const uint32_t st = lds0 + si * STAGE;
    const uint32_t base = __builtin_amdgcn_readfirstlane(st + wave * NI * 1024);
#pragma unroll
    for (int t = 0; t < NI; t++) { slab_load16(src[t], base + t * 1024); src[t] += 128; }
    lds_load4(zsrc, __builtin_amdgcn_readfirstlane(st + opx_oper(BM) + (wave & 3) * 256));
    zsrc += HPS;
    si = (si == NS - 1) ? 0 : si + 1;
  };
  const int mbase = m0 + wm * TM * 16, nbase = n0 + wn * 32;
  // weight scales of all heads, the same 64 dwords from every wave (so that all waves count alike)
  lds_load4(D.ws + min(lane, D.H - 1), __builtin_amdgcn_readfirstlane(lds0 + NS * STAGE));
  issue();
  if (1 < nslab) issue();

  const int offA = (wm * TM * 16 + li) * 128, offB = (BM + wn * 32 + li) * 128;
  const int sw0 = (lg ^ (li & 7)) * 16, sw1 = ((4 + lg) ^ (li & 7)) * 16;
  v4f tot[TM][TN], acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) tot[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  // adds head h's finished partial result to the total and hands it out if some receiver needs it
  auto fold = [&](auto aux_tag, int h, const float (&zsc)[TM]) {
    constexpr bool AUX = decltype(aux_tag)::value;
    // a head computed in fp32 elsewhere adds nothing here: its codes and scales are whatever an earlier pass left
    // (the total starts at +0 and so never is -0: leaving the head out gives the bits of adding zeros)
    if ((D.skip_mask >> h) & 1ull) return;
    const float sw = e_ws[h];
    HeadAux ax; ax.dst = nullptr; ax.dst_is = 0; ax.sub = nullptr;
    if constexpr (AUX) ax = auxs[D.aux_begin + h];
#pragma unroll
    for (int i = 0; i < TM; i++) {
      const float sc = zsc[i] * sw;
#pragma unroll
      for (int j = 0; j < TN; j++) {
        float4 val = make_float4(acc[i][j][0] * sc, acc[i][j][1] * sc, acc[i][j][2] * sc, acc[i][j][3] * sc);
        tot[i][j][0] += val.x; tot[i][j][1] += val.y; tot[i][j][2] += val.z; tot[i][j][3] += val.w;
        if constexpr (AUX) if (ax.dst) {
          int m = mbase + i * 16 + li, nb = nbase + j * 16 + lg * 4;
          if (m < D.M && nb < D.N) {
            int inst, row; row_origin(m, D.rpi, D.rp0, inst, row);
            long long off = (long long)row * D.N + nb;
            if (ax.sub) { float4 u = gload4(ax.sub + off); val.x -= u.x; val.y -= u.y; val.z -= u.z; val.w -= u.w; }
            gstore4(ax.dst + (long long)inst * ax.dst_is + off, val);
          }
        }
      }
    }
  };
  auto compute = [&](auto aux_tag, const uint8_t* st, int s) {
    const uint8_t* sA = st + offA;
    const uint8_t* sB = st + offB;
    const float* zrow = (const float*)(st + opx_oper(BM)) + wm * TM * 16 + li;
    float zsc[HPS][TM];                      // requested now, used after the MFMAs of the half
#pragma unroll
    for (int q = 0; q < HPS; q++)
#pragma unroll
      for (int i = 0; i < TM; i++) zsc[q][i] = zrow[q * BM + i * 16];
    // all operand reads of the slab first (the scheduler would otherwise sink them to their uses)
    uint4 ra[2][TM], rb[2][TN];
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int sw = q ? sw1 : sw0;
#pragma unroll
      for (int i = 0; i < TM; i++) ra[q][i] = *(const uint4*)(sA + i * 2048 + sw);
#pragma unroll
      for (int j = 0; j < TN; j++) rb[q][j] = *(const uint4*)(sB + j * 2048 + sw);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 2; q++) {
      if (HPS == 2 || q == 0) {
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
      }
      if constexpr (B16) {
        union U { uint4 u; v8bf h; };
#pragma unroll
        for (int j = 0; j < TN; j++) {
          U hb; hb.u = rb[q][j];
#pragma unroll
          for (int i = 0; i < TM; i++) {
            U ha; ha.u = ra[q][i];
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hb.h, ha.h, acc[i][j], 0, 0, 0);
          }
        }
      } else {
      v8h ha[TM][2];
#pragma unroll
      for (int i = 0; i < TM; i++) {
        ha[i][0] = decode8(ra[q][i].x, ra[q][i].y);
        ha[i][1] = decode8(ra[q][i].z, ra[q][i].w);
      }
#pragma unroll
      for (int j = 0; j < TN; j++) {
        v8h hb0 = decode8(rb[q][j].x, rb[q][j].y), hb1 = decode8(rb[q][j].z, rb[q][j].w);
#pragma unroll
        for (int i = 0; i < TM; i++) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb0, ha[i][0], acc[i][j], 0, 0, 0);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(hb1, ha[i][1], acc[i][j], 0, 0, 0);
        }
      }
      }
      if (HPS == 2) fold(aux_tag, 2 * s + q, zsc[q]);
      else if (q == 1) fold(aux_tag, s, zsc[0]);
    }
  };

  int sc = 0;                                // stage of the slab about to be multiplied
  if (D.aux_begin < 0) {
    // no vector-memory operation inside the loop but the slab requests (the code that hands out per-head results is
    // not even compiled into this loop: the wait for its descriptor would sit where the two paths merge)
    for (int s = 0; s < nslab; s++) {
      // this wave's part of slab s has landed: all but the four operations of slab s + 1 are complete
      if (s + 1 < nslab) wait_vm<4>(); else wait_vm<0>();
      wg_barrier();                          // everyone's part has; the stage of slab s - 1 is free
      if (s + 2 < nslab) issue();
      compute(std::false_type{}, smem + sc * STAGE, s);
      sc = (sc == NS - 1) ? 0 : sc + 1;
    }
  } else {
    for (int s = 0; s < nslab; s++) {
      wait_all_then_barrier();
      if (s + 2 < nslab) issue();
      compute(std::true_type{}, smem + sc * STAGE, s);
      sc = (sc == NS - 1) ? 0 : sc + 1;
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);        // nothing is outstanding; said with the builtin so that the compiler knows

#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int m = mbase + i * 16 + li;
    if (m >= D.M) continue;
    int inst_i, row_i; row_origin(m, D.rpi, D.rp0, inst_i, row_i);
    const long long roff = (long long)row_i * D.N;
#pragma unroll
    for (int j = 0; j < TN; j++) {
      int nb = nbase + j * 16 + lg * 4;
      if (nb >= D.N) continue;
      float4 v = gload4(D.run_in + inst_i * D.run_in_is + roff + nb);
      if (D.bias) { float4 b = gload4(D.bias + nb); v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w; }
      v.x += tot[i][j][0]; v.y += tot[i][j][1]; v.z += tot[i][j][2]; v.w += tot[i][j][3];
      // the fp32 head goes in last, as in oproj_fused_k
      if (D.extra) { const float4 e = gload4(D.extra + inst_i * D.extra_is + roff + nb); v.x += e.x; v.y += e.y; v.z += e.z; v.w += e.w; }
      gstore4(D.run_out + inst_i * D.run_out_is + roff + nb, v);
    }
  }
}

// The same projection for many rows without per-head results: 128 x 128 tile, four wavefronts of 64 x 64, two stages of 32 KB,
// two workgroups per compute unit, so that one multiplies while the other reads and writes its stream tile.  It moves 0.7 GB of
// stream for 0.08 of codes (100 000 rows of 768, 12 heads) and is bound by that: 318 -> 239 us, 3.3 TB/s.  Against the kernel
// above an operand is read half as often from L2, a wave's conversions serve twice the products, and a lane's four columns are
// neighbours, so that 16 lanes read and write 256 bytes of a row of the stream instead of four lanes 64.  24 600 rows of 1024, 16
// heads: 133 -> 100 us; 4096 rows of 4096, 32 heads of 128: 190 -> 155.  Loading part or all of the stream tile in front of the
// last products gains nothing (252 us; 269 with half of it).  Same sums in the same order.
// A tile row's offset in its instance (row * N) is kept in 32 bits: a handle's tile (rows of an instance * N floats) would have to be
// 8 GB for more, and its workspace beyond 290 GB with the fewest and smallest heads there can be.
template <int DH, bool B16>
__global__ __launch_bounds__(256, 2) void oproj_w_k(const OprojDesc* descs, int di) {
  constexpr int BM = 128, BN = 128, TM = 4, TN = 4, NI = 8, HPS = 128 / DH;
  constexpr int OPER = (BM + BN) * 128, STAGE = OPER + HPS * BM * 4;         // operands, row scales [heads of the slab][BM]
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * STAGE + 256 + BM * 8];
  float* const e_ws = (float*)(smem + 2 * STAGE);                            // weight scales [64]
  int2* const e_row = (int2*)(smem + 2 * STAGE + 256);                       // a tile row's instance and element offset in it
  const OprojDesc D = descs[di];
  const int mt = (D.M + BM - 1) / BM, nt = (D.N + BN - 1) / BN;
  const int lin = xcd_tile(blockIdx.x, mt * nt);
  if (lin >= mt * nt) return;
  const int m0 = (lin / nt) * BM, n0 = (lin % nt) * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int li = lane & 15, lg = lane >> 4;
  const int nslab = D.H / HPS;
  const uint32_t lds0 = lds_addr_of(smem);
  int i0, r0; row_origin(m0, D.rpi, D.rp0, i0, r0);

  // load t of a wave: eight rows of A (t < 4) or of W.  LDS row 16 q + i of a 64-row block of W holds row 4 i + q of the block, so
  // that a lane's accumulators of four 16-column tiles are neighbouring columns.
  const uint8_t* src[NI];
  const int c = ((lane & 7) ^ (lane >> 3)) * 16;
#pragma unroll
  for (int t = 0; t < NI; t++) {
    const int r = 8 * (wave * 4 + (t & 3)) + (lane >> 3);
    if (t < 4) {
      int inst, row; split_row(i0, r0, min(m0 + r, D.M - 1) - m0, D.rpi, D.rp0, inst, row);
      src[t] = D.zc + (long long)inst * D.zc_is + (long long)row * D.H * DH + c;
    } else {
      src[t] = D.W + (long long)min(n0 + (r & 64) + (r & 15) * 4 + ((r >> 4) & 3), D.N - 1) * D.H * DH + c;
    }
  }
  // row scales of a slab's heads: entry 64 wave + lane = BM q + r is head q's of tile row r (with one head per slab the upper two
  // waves repeat the rows of the lower two)
  const float* zsrc;
  {
    const int e = wave * 64 + lane;
    int inst, row; split_row(i0, r0, min(m0 + e % BM, D.M - 1) - m0, D.rpi, D.rp0, inst, row);
    zsrc = D.zs + (long long)inst * D.zs_is + (long long)row * D.H + (HPS == 2 ? e / BM : 0);
    if (e < BM) e_row[e] = make_int2(inst, row * D.N);
  }
  auto issue = [&](int stage) {
    const uint32_t st = lds0 + stage * STAGE;
    const uint32_t a = __builtin_amdgcn_readfirstlane(st + wave * 4096);
#pragma unroll
    for (int t = 0; t < NI; t++) { slab_load16(src[t], a + (t < 4 ? 0 : BM * 128) + (t & 3) * 1024); src[t] += 128; }
    lds_load4(zsrc, __builtin_amdgcn_readfirstlane(st + OPER + (HPS == 2 ? wave : wave & 1) * 256));
    zsrc += HPS;
  };
  lds_load4(D.ws + min(lane, D.H - 1), __builtin_amdgcn_readfirstlane(lds0 + 2 * STAGE));
  issue(0);

  const int offA = (wm * 64 + li) * 128, offB = (BM + wn * 64 + li) * 128;
  const int sw0 = (lg ^ (li & 7)) * 16, sw1 = ((4 + lg) ^ (li & 7)) * 16;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  v4f tot[TM][TN], acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++) tot[i][j] = zero;
  union U { uint4 u; v8bf h; };
  for (int s = 0; s < nslab; s++) {
    wait_vm_barrier<0>();                    // the slab has landed for everyone, the other stage is free
    if (s + 1 < nslab) issue((s + 1) & 1);
    const uint8_t* st = smem + (s & 1) * STAGE;
#pragma unroll
    for (int q = 0; q < 2; q++) {
      const int sw = q ? sw1 : sw0;
      U ra[TM], rb[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) ra[i].u = *(const uint4*)(st + offA + i * 2048 + sw);
#pragma unroll
      for (int j = 0; j < TN; j++) rb[j].u = *(const uint4*)(st + offB + j * 2048 + sw);
      const bool first = HPS == 2 || q == 0;
      if constexpr (B16) {
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
          for (int i = 0; i < TM; i++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[i].h, rb[j].h, first ? zero : acc[i][j], 0, 0, 0);
      } else {
        v8h ha[TM][2];
#pragma unroll
        for (int i = 0; i < TM; i++) { ha[i][0] = decode8(ra[i].u.x, ra[i].u.y); ha[i][1] = decode8(ra[i].u.z, ra[i].u.w); }
#pragma unroll
        for (int j = 0; j < TN; j++) {
          const v8h hb0 = decode8(rb[j].u.x, rb[j].u.y), hb1 = decode8(rb[j].u.z, rb[j].u.w);
#pragma unroll
          for (int i = 0; i < TM; i++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i][0], hb0, first ? zero : acc[i][j], 0, 0, 0);
#pragma unroll
          for (int i = 0; i < TM; i++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ha[i][1], hb1, acc[i][j], 0, 0, 0);
        }
      }
      if (HPS == 1 && q == 0) continue;
      const int h = HPS == 2 ? 2 * s + q : s;
      if ((D.skip_mask >> h) & 1ull) continue;             // as in oproj_x_k
      const float w = e_ws[h];
      const float* z = (const float*)(st + OPER) + (HPS == 2 ? q * BM : 0) + wm * 64 + lg * 4;
#pragma unroll
      for (int i = 0; i < TM; i++) {
        const float4 zi = *(const float4*)(z + i * 16);
        const float f[4] = {zi.x * w, zi.y * w, zi.z * w, zi.w * w};
#pragma unroll
        for (int j = 0; j < TN; j++)
#pragma unroll
          for (int r = 0; r < 4; r++) { const float v = acc[i][j][r] * f[r]; tot[i][j][r] += v; }
      }
    }
  }
  // next = (stream + bias + sum of the heads) + fp32 head.  tot[i][q][r] of lane (li, lg) is row 64 wm + 16 i + 4 lg + r, column 64 wn + 4 li + q.
  const int n = n0 + wn * 64 + li * 4;
  if (n >= D.N) return;
  const float4 bias = D.bias ? gload4(D.bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < TM; i++) {
    const int rt = wm * 64 + i * 16 + lg * 4;
    float4 x[4], e[4];
    int2 at[4];
#pragma unroll
    for (int r = 0; r < 4; r++) {
      at[r] = e_row[rt + r];
      x[r] = gload4(D.run_in + at[r].x * D.run_in_is + at[r].y + n);
      if (D.extra) e[r] = gload4(D.extra + at[r].x * D.extra_is + at[r].y + n);
    }
#pragma unroll
    for (int r = 0; r < 4; r++) {
      if (m0 + rt + r >= D.M) continue;
      float4 v = x[r];
      if (D.bias) { v.x += bias.x; v.y += bias.y; v.z += bias.z; v.w += bias.w; }
      v.x += tot[i][0][r]; v.y += tot[i][1][r]; v.z += tot[i][2][r]; v.w += tot[i][3][r];
      if (D.extra) { v.x += e[r].x; v.y += e[r].y; v.z += e[r].z; v.w += e[r].w; }
      gstore4(D.run_out + at[r].x * D.run_out_is + at[r].y + n, v);
    }
  }
}
template <int DH, bool B16>
static hipError_t launch_oproj_w(int M, int N, hipStream_t s, const OprojDesc* descs, int desc_index) {
  const int tiles = ((M + 127) / 128) * ((N + 127) / 128);
  hipLaunchKernelGGL((oproj_w_k<DH, B16>), dim3((tiles + 7) / 8 * 8), dim3(256), 0, s, descs, desc_index);
  return hipGetLastError();
}

// The kernel's 75 KB of dynamic LDS need the attribute, which belongs to the kernel's code object on one device:
// set once per device and instantiation (atomically: models on several streams or host threads may launch at once).
template <int DH, bool B16, int BM>
static hipError_t launch_oproj_bm(int M, int N, hipStream_t s, const OprojDesc* descs, int desc_index, const HeadAux* auxs) {
  if (BM == 128) {
    static std::atomic<bool> attr_set[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
      hipError_t e = hipFuncSetAttribute((const void*)oproj_x_k<DH, B16, BM>, hipFuncAttributeMaxDynamicSharedMemorySize, opx_lds(BM));
      if (e != hipSuccess) return e;
      attr_set[dev].store(true, std::memory_order_release);
    }
  }
  const int tiles = ((M + BM - 1) / BM) * ((N + 63) / 64);
  hipLaunchKernelGGL((oproj_x_k<DH, B16, BM>), dim3((tiles + 7) / 8 * 8), dim3(BM == 128 ? 512 : 256), opx_lds(BM), s, descs, desc_index, auxs);
  return hipGetLastError();
}
// A tile is a chain of dependent steps whatever its height; with fewer 128-row tiles than compute units the chip waits for
// that chain with units idle, and tiles of 32 rows make the chain's steps shorter (1024 rows of 512, 64 tiles against 256:
// four-layer circuit 2.28 -> 2.16 ms, its sweep 21.8 -> 21.2 ms, both with four such layers a pass).  They also read the
// weights four times as often, so near a full chip it depends on the slabs (128 bytes of codes) a chain has.  Time with 32
// rows over that with 128, means over 1300 random sizes: up to 7 slabs 0.78 at 96 .. 127 tiles, 0.94 at 192 .. 255; from 8 on
// 0.73 at 96 .. 127, 0.89 at 160 .. 191, 1.04 at 192 .. 255 (1.10 at the worst).  With bfloat16 rows, up to 3 slabs 0.84 and
// 0.97; from 4 on 0.81, 0.93 and 1.07 (1.47), and from 12 on 1.00 at 128 .. 191 already (1.14).
// 128 x 128 tiles (oproj_w_k, no per-head results): a round of 512 of them takes 1.5 times one of 128 x 64, a last round between
// its share and a whole one.  Of 400 random sizes (150 tiles and more) 177 take them, at 0.68 to 1.04 of the other's time, mean 0.83.
template <int DH, bool B16>
static hipError_t launch_oproj_x(int M, int N, int H, hipStream_t s, const OprojDesc* descs, int desc_index, const HeadAux* auxs) {
  auto rounds = [&](int bn) { const double t = (double)((M + 127) / 128) * ((N + bn - 1) / bn) / 512; return 0.5 * (std::ceil(t) + t); };
  if (!auxs && 0.4 + 1.5 * rounds(128) <= rounds(64)) return launch_oproj_w<DH, B16>(M, N, s, descs, desc_index);
  const int slabs = H * DH / 128, few = slabs < (B16 ? 4 : 8) ? 256 : (!B16 || slabs < 12 ? 192 : 128);
  if (((M + 127) / 128) * ((N + 63) / 64) < few) return launch_oproj_bm<DH, B16, 32>(M, N, s, descs, desc_index, auxs);
  return launch_oproj_bm<DH, B16, 128>(M, N, s, descs, desc_index, auxs);
}

hipError_t launch_oproj_fused(const OprojDesc* descs, int desc_index, const HeadAux* auxs, int M, int N, int H, int dh,
                              int exact, int b16, hipStream_t s) {
  if (M == 0) return hipSuccess;
  int tiles = ((M + 127) / 128) * ((N + 63) / 64);
  dim3 grid((tiles + 7) / 8 * 8);
  if (b16) {
    // bfloat16 attention outputs: heads of 32 or 64 values (64 or 128 bytes)
    if (!oproj_side_by_side(H, 2 * dh, N, exact != 0)) return hipErrorInvalidValue;
    if (dh == 32) return launch_oproj_x<64, true>(M, N, H, s, descs, desc_index, auxs);
    return launch_oproj_x<128, true>(M, N, H, s, descs, desc_index, auxs);
  }
  if (oproj_side_by_side(H, dh, N, exact != 0)) {
    if (dh == 64) return launch_oproj_x<64, false>(M, N, H, s, descs, desc_index, auxs);
    return launch_oproj_x<128, false>(M, N, H, s, descs, desc_index, auxs);
  } else if (exact) hipLaunchKernelGGL(oproj_fused_k<true>, grid, dim3(256), 0, s, descs, desc_index, auxs);
  else hipLaunchKernelGGL(oproj_fused_k<false>, grid, dim3(256), 0, s, descs, desc_index, auxs);
  return hipGetLastError();
}

}  // namespace pahq

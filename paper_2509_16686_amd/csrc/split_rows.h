// MFMA split kernel of EG-MLA decode for latents wider than 128 (bf16
// storage, 16 heads per work-group; built for d_c 320, d_r 64).  Included by
// decode.hip after split_slice.h, whose unit scheme it follows: a wave owns
// 16-token units of all dims, loads their rows and gate rows in whole lines,
// gates them (exact fp32 products, one rounding to fp16), stages them in its
// own LDS tile, and takes both MFMA operands from there, so the waves share
// nothing until they merge.
//
// What bounds it: the memory system (768 + 640 bytes of rows and gate rows per
// token).  A unit is 88 registers of loads, so one unit is in flight per wave
// (90 KB per compute unit with one work-group of 4 waves); it goes out as soon
// as the previous one is staged.  The kernel it replaced split a
// row's dimensions over the waves, in the layout of the MFMA operand (64-byte
// pieces of rows), with a barrier and an exchange of partial scores per 32
// tokens: the call
// took 196 us at 256 sequences of 2048 tokens, 117 here (split kernel 182 and
// 100: 7.3 TB/s of rows and gate rows).  The balanced schedule of the d_c 128
// kernel gained 2 % at mixed lengths and cost 4 % at equal ones: not taken.
#pragma once

namespace egmla {

template <int DC, int DR, int NW>
struct RowsCfg {
  static constexpr int DQ = DC + DR;
  static constexpr int NC = DC / 32, NR = DR / 32;   // 32-dim score chunks
  static constexpr int NB = DC / 16;                 // 16-dim value blocks
  static constexpr int NLI = 16 * DC / 8 / 64;       // latent (and gate) load instructions per unit
  static constexpr int NRI = 16 * DR / 8 / 64;       // RoPE load instructions per unit
  static constexpr int TS = DQ + 8;                  // tile row: latent (fp16) | RoPE key (bf16) | 16 bytes (4 banks mod 64)
  static constexpr int CAP = kMaxSplitTokens;        // tokens listed
  static constexpr int LDS_LIST = CAP * 8;
  static constexpr int LDS_TILE = NW * 16 * TS * 2;
  static constexpr int LDS_Q = 16 * TS * 2;          // query rows [q_lat fp16 | q^R bf16] (in registers they spill)
  static constexpr int LDS_MAIN = LDS_LIST + LDS_TILE + LDS_Q;
  static constexpr int LDS_BYTES = LDS_MAIN + 2 * NW * 16 * 4;
  static_assert(DC % 32 == 0 && DR % 32 == 0 && (16 * DC / 8) % 64 == 0 && (16 * DR / 8) % 64 == 0 && NB % 2 == 0,
                "whole load instructions; value blocks in two halves");
  static_assert(NW * (NB / 2) * 64 * 16 <= LDS_MAIN, "half of the waves' accumulators");
};

template <int DC, int DR, int NW>
__global__ __launch_bounds__(NW * 64, 2) void split_rows_kernel(SplitArgs a) {
  using C = RowsCfg<DC, DR, NW>;
  constexpr int NC = C::NC, NR = C::NR, NB = C::NB, NLI = C::NLI, NRI = C::NRI, DQ = C::DQ, TS = C::TS, NT = NW * 64;
  __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS_BYTES];
  int2* list = reinterpret_cast<int2*>(lds);
  uint16_t* tile_all = reinterpret_cast<uint16_t*>(lds + C::LDS_LIST);  // [NW][16][TS]
  uint16_t* q_s = reinterpret_cast<uint16_t*>(lds + C::LDS_LIST + C::LDS_TILE);  // [16][TS]
  f32x4_t* obuf = reinterpret_cast<f32x4_t*>(lds);                      // [NW][NB / 2][64], after the units
  float* mbuf = reinterpret_cast<float*>(lds + C::LDS_MAIN);            // [NW][16]
  float* lbuf = mbuf + NW * 16;

  const int item = xcd_logical_block(blockIdx.x, gridDim.x);
  const int hg = item % a.groups, s = (item / a.groups) % a.s_max, b = item / (a.groups * a.s_max);
  const int t0 = s * a.split;
  const int64_t row = static_cast<int64_t>(b) * a.s_max + s;  // partial row
  const int n = min(a.split, clamp_len(a.seq_lens[b], a.cap) - t0);
  if (n <= 0) return;  // no tokens: the merge reads no partial of it (uniform over the work-group)
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- token list ----
  {
    constexpr int PER = C::CAP / NT;
    const int nper = (n + NT - 1) / NT;  // uniform
    int pp[PER], psl[PER], pid[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) pp[e] = min(tid + e * NT, n - 1);
    split_slots(a, b, t0, pp, psl, nper);
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (e < nper) pid[e] = a.ids[psl[e]];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = tid + e * NT;
      if (e < nper && j < n) list[j] = make_int2(psl[e], clamp_id(pid[e], a.V));
    }
  }
  // query rows: absorbed query in fp16, RoPE query (a stored bf16 value: exact)
  for (int i = tid; i < 16 * (DQ / 8); i += NT) {
    const int h = i / (DQ / 8), c = 8 * (i % (DQ / 8));
    const float* src = a.qfull + (static_cast<int64_t>(b) * a.H + hg * 16 + h) * DQ + c;
    const f32x4_t x = *reinterpret_cast<const f32x4_t*>(src), y = *reinterpret_cast<const f32x4_t*>(src + 4);
    u32x4_t v;
    if (c < DC) v = u32x4_t{pack_f16x2(x[0], x[1]), pack_f16x2(x[2], x[3]), pack_f16x2(y[0], y[1]), pack_f16x2(y[2], y[3])};
    else v = u32x4_t{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
    *reinterpret_cast<u32x4_t*>(q_s + h * TS + c) = v;
  }
  __syncthreads();

  const uint16_t* __restrict__ cache = static_cast<const uint16_t*>(a.cache);
  const uint16_t* __restrict__ gate = static_cast<const uint16_t*>(a.gate);
  struct Regs {
    u32x4_t lat[NLI], gat[NLI], rop[NRI];
  };
  Regs rg;
  // piece c * 64 + lane of a unit: token and first dim (latent, RoPE)
  constexpr int PL = DC / 8, PR = DR / 8;
  auto issue = [&](int i) {
    const int j0 = (w + i * NW) * 16;
#pragma unroll
    for (int c = 0; c < NLI; ++c) {
      const int p = c * 64 + lane, t = p / PL, d = 8 * (p % PL);
      const int2 e = list[min(j0 + t, n - 1)];
      rg.lat[c] = __builtin_nontemporal_load(
          reinterpret_cast<const u32x4_t*>(cache + static_cast<int64_t>(e.x) * DQ + d));
      rg.gat[c] = *reinterpret_cast<const u32x4_t*>(gate + static_cast<int64_t>(e.y) * DC + d);
    }
#pragma unroll
    for (int c = 0; c < NRI; ++c) {
      const int p = c * 64 + lane, t = p / PR, d = 8 * (p % PR);
      rg.rop[c] = __builtin_nontemporal_load(
          reinterpret_cast<const u32x4_t*>(cache + static_cast<int64_t>(list[min(j0 + t, n - 1)].x) * DQ + DC + d));
    }
  };

  const int nunits = (n + 15) / 16;
  const int nu = nunits > w ? (nunits - w + NW - 1) / NW : 0;
  f32x4_t o[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  if (nu > 0) {
    issue(0);
    uint16_t* tile = tile_all + w * 16 * TS;
    const uint16_t* arow = tile + r16 * TS + 8 * g;
    const uint16_t* qrow = q_s + r16 * TS + 8 * g;
    uint16_t* tread = tile + (4 * g + (r16 >> 2)) * TS + 4 * (r16 & 3);
    for (int i = 0; i < nu; ++i) {
      const int nt = n - (w + i * NW) * 16;  // valid tokens of the unit (>= 1)
#pragma unroll
      for (int c = 0; c < NLI; ++c) {
        const int p = c * 64 + lane;
        *reinterpret_cast<u32x4_t*>(tile + (p / PL) * TS + 8 * (p % PL)) = gate_chunk_f16(rg.lat[c], rg.gat[c]);
      }
#pragma unroll
      for (int c = 0; c < NRI; ++c) {
        const int p = c * 64 + lane;
        *reinterpret_cast<u32x4_t*>(tile + (p / PR) * TS + DC + 8 * (p % PR)) = rg.rop[c];
      }
      issue(i + 1);  // past the last unit: the last token again, never used
      wave_lds_sync();
      // S^T[token 4g + q][head r16]
      f32x4_t acc = {0.f, 0.f, 0.f, 0.f}, acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < NC; ++c)
        acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const f16x8_t*>(arow + 32 * c),
                                                     *reinterpret_cast<const f16x8_t*>(qrow + 32 * c), acc, 0, 0, 0);
#pragma unroll
      for (int c = 0; c < NR; ++c)
        acc2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(arow + DC + 32 * c),
                                                       *reinterpret_cast<const bf16x8_t*>(qrow + DC + 32 * c), acc2, 0,
                                                       0, 0);
      acc += acc2;
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = 4 * g + q < nt ? acc[q] * a.scale_log2 : -INFINITY;
      const float mt = max_over_row_groups(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      const float m_new = fmaxf(m_run, mt);
      const bool grow = m_new > m_run + kLazyRescale;
      if (__builtin_amdgcn_ballot_w64(grow)) {
        const float alpha = grow ? __builtin_amdgcn_exp2f(m_run - m_new) : 1.0f;
        m_run = grow ? m_new : m_run;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < NB; ++db) o[db] *= alpha;
      }
      // (-inf only while every score so far overflowed to it: those tokens weigh nothing)
      const float m_ref = m_run == -INFINITY ? 0.f : m_run;
      float p[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        p[q] = __builtin_amdgcn_exp2f(x[q] - m_ref);
        l_run += p[q];
      }
      const f16x4_t pb = __builtin_bit_cast(f16x4_t, u32x2_t{pack_f16x2(p[0], p[1]), pack_f16x2(p[2], p[3])});
#pragma unroll
      for (int db = 0; db < NB; ++db) {
        const s16x4_t at =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(tread + db * 16));
        o[db] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4_t, at), pb, o[db], 0, 0, 0);
      }
      wave_lds_sync();
    }
  }

  // ---- merge of the waves, the value blocks in two halves ----
  l_run = sum_over_row_groups(l_run);
  if (g == 0) mbuf[w * 16 + r16] = m_run;
  __syncthreads();  // also: every wave is done with the list and its tile (obuf aliases them)
  float M = -INFINITY;
#pragma unroll
  for (int v = 0; v < NW; ++v) M = fmaxf(M, mbuf[v * 16 + r16]);
  const float sc = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - M);
  if (g == 0) lbuf[w * 16 + r16] = l_run * sc;
  const int64_t prow = row * a.H + hg * 16 + r16;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    if (half) __syncthreads();  // the first half's sums are read
#pragma unroll
    for (int db = 0; db < NB / 2; ++db) obuf[(w * (NB / 2) + db) * 64 + lane] = o[half * (NB / 2) + db] * sc;
    __syncthreads();
    for (int db = w; db < NB / 2; db += NW) {
      f32x4_t sum = obuf[db * 64 + lane];
#pragma unroll
      for (int v = 1; v < NW; ++v) sum += obuf[(v * (NB / 2) + db) * 64 + lane];
      __builtin_nontemporal_store(
          sum, reinterpret_cast<f32x4_t*>(a.part_o + prow * DC + (half * (NB / 2) + db) * 16 + 4 * g));
    }
  }
  if (w == 0 && g == 0) {
    float Ls = 0.f;
#pragma unroll
    for (int v = 0; v < NW; ++v) Ls += lbuf[v * 16 + r16];
    *reinterpret_cast<float2*>(a.part_ml + prow * 2) = make_float2(M, Ls);
  }
}

}  // namespace egmla

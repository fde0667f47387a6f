// fp32 matrix-core split kernel of EG-MLA decode: fp32 or bf16 storage, any
// head count, latent dim <= DCM, RoPE dim <= 64.  Included by decode.hip after
// SplitArgs.  The layers it serves (fp32 storage; 12 heads of 64 with d_c 16
// to 256) have no 16-bit fast path, and every product here stays fp32: the
// gated latent is the fp32 product c * g (exact for bf16 storage), queries,
// probabilities and sums are fp32, and both contractions run on
// v_mfma_f32_16x16x4_f32.
//
// One work-group of NW waves per (sequence, context split, block of 16 heads;
// heads past H are computed on a copy of the last and not stored).  As in the
// d_c 128 kernel, the split's slots and ids go to an LDS list first, the list
// forms 16-token units, and unit u belongs to wave u % NW, so the waves share
// nothing until they merge.  Per unit a wave
//   * loads the latent, gate and RoPE pieces (16 bytes per lane and
//     instruction, consecutive lanes on consecutive pieces of a row, D units
//     ahead, every load unconditional: pieces past the unit repeat its last),
//   * gates and writes the rows as fp32 into its own LDS tile,
//   * scores S^T[token][head]: one 16-byte LDS read of the tile and one of the
//     query feed four products (lane group g holds dims 16 c + 4 g .. + 3 of
//     chunk c: the four k-slots of product j are dims 4 g' + j, g' = 0 .. 3),
//   * runs the online softmax in the accumulator layout, and
//   * adds O^T[dim][head] += C~^T P^T: the lane's probability of token 4 g + i
//     is the B operand of product i as it stands, the A operand a 4-byte read
//     of the tile's token 4 g + i.
// The tile row is a multiple of 16 dwords plus 4: the 16-byte reads of 16 rows
// and the 4-byte reads of rows 4 g + i fall on distinct banks.
//
// What bounds it: for the small layers it serves, latency (list, rows, merge)
// and the fp32 matrix rate (as much as the vector rate, but with one LDS read
// per four products).  It replaced a vector kernel that kept one score per
// thread and read both operands of every fma from LDS.  12 heads, d_c 64, 64
// sequences of 100 to 3003 tokens: 22 us against 301 (call 28.2 against 317).
//
// ONE: the whole decode in one launch for layers whose weights are small and
// contexts of at most kOneMaxTokens: the work-group also absorbs its heads'
// queries first (fp32 sums over slices of the head dim, added in slice order)
// and up-projects the merged rows at the end, so nothing passes through the
// workspace and no other kernel runs.  4 heads, d_c 32, fp32, one sequence of
// 128 tokens: one launch of 9.3 us (call 9.5 us) against 4.6 + 28.3 + 4.7 (35.8).
#pragma once

namespace egmla {

constexpr int kOnePre = 4;  // ONE: W_UV pieces a thread loads before the units

template <bool BF16, int DCM, int NW, bool ONE>
struct F32Cfg {
  static constexpr int DRM = 64;
  static constexpr int EPP = BF16 ? 8 : 4;                          // elements per 16-byte piece
  static constexpr int NLL = (16 * DCM / EPP + 63) / 64;            // latent (and gate) loads per unit
  static constexpr int NLR = (16 * DRM / EPP + 63) / 64;            // RoPE loads per unit
  static constexpr int NB = DCM / 16;                               // 16-dim value blocks
  static constexpr int REGS = (2 * NLL + NLR) * 4;                  // registers of a unit in flight
  static constexpr int D = REGS >= 48 ? 1 : 2;                      // units in flight
  static constexpr int TS = DCM + DRM + 4;                          // tile / query row (dwords)
  static constexpr int CAP = ONE ? kOneMaxTokens : kMaxSplitTokens;  // tokens listed in LDS
  static constexpr int LDS_LIST = CAP * 8;
  static constexpr int LDS_Q = 16 * TS * 4;
  static constexpr int LDS_TILE = NW * 16 * TS * 4;
  static constexpr int LDS_MAIN = LDS_LIST + LDS_Q + LDS_TILE;
  static constexpr int LDS_BYTES = LDS_MAIN + 2 * NW * 16 * 4;
  static_assert(DCM % 16 == 0 && NW * NB * 64 * 16 <= LDS_MAIN && LDS_BYTES <= 160 * 1024, "LDS budget");
  static_assert(!ONE || (16 * DCM * 4 + NW * NB * 64 * 16 <= LDS_MAIN), "merged rows beside the waves' sums");
  static_assert(CAP % (NW * 64) == 0, "list chunk");
};

// What the single-launch form needs beyond SplitArgs (storage-typed tensors).
struct OneArgs {
  const void* q;     // [B, H, DH + DR]
  const void* w_uk;  // [H, DH, DC]
  const void* w_uv;  // [H, DV, DC]
  void* out;         // [B, H, DV]
  int DV;
  int slices;        // head-dim slices of the absorption: tasks (head, piece, slice) fill the work-group
  int tpo;           // threads per output of the up-projection (power of two, at most 8)
};

// 16 bytes of the storage type as fp32.
template <bool BF16>
__device__ __forceinline__ void widen_piece(u32x4_t w, float (&o)[BF16 ? 8 : 4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (BF16) {
      o[2 * e] = bf16_lo(w[e]);
      o[2 * e + 1] = bf16_hi(w[e]);
    } else {
      o[e] = __uint_as_float(w[e]);
    }
  }
}

template <bool BF16, int DCM, int NW, bool ONE>
__global__ __launch_bounds__(NW * 64, DCM <= 128 ? 2 : 1) void split_f32_kernel(SplitArgs a, OneArgs one) {
  using C = F32Cfg<BF16, DCM, NW, ONE>;
  constexpr int EPP = C::EPP, NLL = C::NLL, NLR = C::NLR, NB = C::NB, TS = C::TS, D = C::D, NT = NW * 64;
  constexpr int DQM = DCM + C::DRM;
  __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS_BYTES];
  int2* list = reinterpret_cast<int2*>(lds);
  float* q_s = reinterpret_cast<float*>(lds + C::LDS_LIST);                  // [16][TS]
  float* tile_all = reinterpret_cast<float*>(lds + C::LDS_LIST + C::LDS_Q);  // [NW][16][TS]
  f32x4_t* obuf = reinterpret_cast<f32x4_t*>(lds);                           // [NW][NB][64], after the units
  float* mbuf = reinterpret_cast<float*>(lds + C::LDS_MAIN);                 // [NW][16]
  float* lbuf = mbuf + NW * 16;                                              // [NW][16]

  const int item = xcd_logical_block(blockIdx.x, gridDim.x);
  const int hg = item % a.groups;
  const int s = ONE ? 0 : (item / a.groups) % a.s_max;
  const int b = ONE ? item / a.groups : item / (a.groups * a.s_max);
  const int t0 = s * a.split;
  const int L = clamp_len(a.seq_lens[b], a.cap);
  const int h0 = hg * 16, nh = min(16, a.H - h0);
  const int tid = threadIdx.x, lane = tid & 63, r16 = lane & 15, g = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (t0 >= L) {  // uniform over the work-group
    if constexpr (ONE) {
      for (int i = tid; i < nh * one.DV; i += NT) st<BF16>(one.out, (static_cast<int64_t>(b) * a.H + h0) * one.DV + i, 0.f);
    }
    return;
  }
  const int n = min(t0 + a.split, L) - t0;
  const int DC = a.DC, DR = a.DR, DQ = DC + DR;
  constexpr int EB = BF16 ? 2 : 4;
  // absorption tasks (ONE)
  const int DH = a.DH, pc = DC / EPP, np = nh * pc, ks = ONE ? min(one.slices, DH) : 1, kper = (DH + ks - 1) / ks;

  // ---- token list: slot and id of every position (all loads first) ----
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
    if constexpr (!ONE) {
      // the absorbed query (rows past the block's heads repeat the last one)
      const int per_row = DQ / 4;
      for (int i = tid; i < 16 * per_row; i += NT) {
        const int h = i / per_row, c = 4 * (i - h * per_row);
        *reinterpret_cast<float4*>(q_s + h * TS + c) =
            *reinterpret_cast<const float4*>(a.qfull + (static_cast<int64_t>(b) * a.H + h0 + min(h, nh - 1)) * DQ + c);
      }
    }
    if constexpr (ONE) {
      // ---- absorption: q_lat[h][c] = sum_k q^C[h][k] W_UK[h][k][c] ----
      // a task is (head, piece of EPP columns, slice of the head dim); the
      // slices' sums meet in the tile region
      for (int i = tid; i < np * ks; i += NT) {
        const int sl = i / np, hp = i - sl * np, h = hp / pc, c = EPP * (hp - h * pc);
        const int k0 = sl * kper, k1 = min(DH, k0 + kper);
        const int64_t qrow = (static_cast<int64_t>(b) * a.H + h0 + h) * (DH + DR);
        const int64_t wrow = static_cast<int64_t>(h0 + h) * DH * DC + c;
        float acc[EPP];
#pragma unroll
        for (int e = 0; e < EPP; ++e) acc[e] = 0.f;
#pragma unroll 4
        for (int k = k0; k < k1; ++k) {
          const float qk = ld<BF16>(one.q, qrow + k);
          float wv[EPP];
          widen_piece<BF16>(*reinterpret_cast<const u32x4_t*>(static_cast<const unsigned char*>(one.w_uk) +
                                                              (wrow + static_cast<int64_t>(k) * DC) * EB),
                            wv);
#pragma unroll
          for (int e = 0; e < EPP; ++e) acc[e] = fmaf(qk, wv[e], acc[e]);
        }
#pragma unroll
        for (int e = 0; e < EPP; ++e) tile_all[(sl * nh + h) * DC + c + e] = acc[e];
      }
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = tid + e * NT;
      if (e < nper && j < n) list[j] = make_int2(psl[e], clamp_id(pid[e], a.V));
    }
  }
  // zero the columns past d_c + d_r of the query and of the tiles: the products run over DQM dims
  const int npad = (DQM - DQ) / 4;  // 16-byte pieces
  if constexpr (!ONE) {
    for (int i = tid; i < 16 * (NW + 1) * npad; i += NT)
      *reinterpret_cast<float4*>(q_s + (i / npad) * TS + DQ + 4 * (i % npad)) = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  __syncthreads();

  // this lane's pieces of a unit: token (bits 16..) and first element of latent and RoPE instruction c
  const int pl = DC / EPP, pr = DR / EPP;
  int el[NLL], er[NLR];
#pragma unroll
  for (int c = 0; c < NLL; ++c) {
    const int p = min(c * 64 + lane, 16 * pl - 1);
    el[c] = ((p / pl) << 16) | (EPP * (p % pl));
  }
#pragma unroll
  for (int c = 0; c < NLR; ++c) {
    const int p = pr > 0 ? min(c * 64 + lane, 16 * pr - 1) : 0;
    er[c] = pr > 0 ? ((p / pr) << 16) | (EPP * (p % pr)) : 0;
  }
  const unsigned char* __restrict__ cache = static_cast<const unsigned char*>(a.cache);
  const unsigned char* __restrict__ gate = static_cast<const unsigned char*>(a.gate);
  struct Regs {
    u32x4_t lat[NLL], gat[NLL], rop[NLR];
  };
  auto issue = [&](Regs& rg, int i) {
    const int j0 = (w + i * NW) * 16;
#pragma unroll
    for (int c = 0; c < NLL; ++c) {
      const int2 e = list[min(j0 + (el[c] >> 16), n - 1)];
      const int col = el[c] & 0xffff;
      rg.lat[c] = __builtin_nontemporal_load(
          reinterpret_cast<const u32x4_t*>(cache + (static_cast<int64_t>(e.x) * DQ + col) * EB));
      rg.gat[c] = *reinterpret_cast<const u32x4_t*>(gate + (static_cast<int64_t>(e.y) * DC + col) * EB);
    }
    if (pr > 0) {
#pragma unroll
      for (int c = 0; c < NLR; ++c) {
        const int2 e = list[min(j0 + (er[c] >> 16), n - 1)];
        rg.rop[c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(
            cache + (static_cast<int64_t>(e.x) * DQ + DC + (er[c] & 0xffff)) * EB));
      }
    }
  };

  const int nunits = (n + 15) / 16;
  const int nu = nunits > w ? (nunits - w + NW - 1) / NW : 0;  // this wave's units
  f32x4_t o[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  Regs ring[D];
  if (nu > 0) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      issue(ring[u], u);  // a unit past the list repeats the last token, never used
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // ONE: the slices' sums, added in slice order, and q^R; the first W_UV pieces of this thread's output
  u32x4_t wpre[ONE ? kOnePre : 1];
  if constexpr (ONE) {
    if (tid / one.tpo < nh * one.DV) {
      const unsigned char* wrow = static_cast<const unsigned char*>(one.w_uv) +
                                  (static_cast<int64_t>(h0) * one.DV + tid / one.tpo) * DC * EB;
#pragma unroll
      for (int k = 0; k < kOnePre; ++k)
        wpre[k] = *reinterpret_cast<const u32x4_t*>(wrow + 16 * min(tid % one.tpo + k * one.tpo, pc - 1));
    }
    for (int i = tid; i < 16 * DQM; i += NT) {
      const int h = i / DQM, c = i - h * DQM, hh = min(h, nh - 1);
      float v = 0.f;
      if (c < DC) {
        for (int sl = 0; sl < ks; ++sl) v += tile_all[(sl * nh + hh) * DC + c];
      } else if (c < DQ) {
        v = ld<BF16>(one.q, (static_cast<int64_t>(b) * a.H + h0 + hh) * (DH + DR) + DH + c - DC);
      }
      q_s[h * TS + c] = v;
    }
    __syncthreads();  // the slices' sums are read before the tiles are written
    for (int i = tid; i < 16 * NW * npad; i += NT)
      *reinterpret_cast<float4*>(tile_all + (i / npad) * TS + DQ + 4 * (i % npad)) = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
  }
  if (nu > 0) {
    float* tile = tile_all + w * 16 * TS;
    const float* arow = tile + r16 * TS + 4 * g;
    const float* qrow = q_s + r16 * TS + 4 * g;
    const float* vrow = tile + 4 * g * TS + r16;
    auto process = [&](Regs& rg, int i, bool refill) {
      const int nt = n - (w + i * NW) * 16;  // valid tokens of the unit (>= 1)
#pragma unroll
      for (int c = 0; c < NLL; ++c) {
        float x[EPP], y[EPP];
        widen_piece<BF16>(rg.lat[c], x);
        widen_piece<BF16>(rg.gat[c], y);
        float* dst = tile + (el[c] >> 16) * TS + (el[c] & 0xffff);
#pragma unroll
        for (int e = 0; e < EPP; e += 4)
          *reinterpret_cast<float4*>(dst + e) =
              make_float4(x[e] * y[e], x[e + 1] * y[e + 1], x[e + 2] * y[e + 2], x[e + 3] * y[e + 3]);
      }
      if (pr > 0) {
#pragma unroll
        for (int c = 0; c < NLR; ++c) {
          float x[EPP];
          widen_piece<BF16>(rg.rop[c], x);
          float* dst = tile + (er[c] >> 16) * TS + DC + (er[c] & 0xffff);
#pragma unroll
          for (int e = 0; e < EPP; e += 4)
            *reinterpret_cast<float4*>(dst + e) = make_float4(x[e], x[e + 1], x[e + 2], x[e + 3]);
        }
      }
      if (refill) issue(rg, i + D);
      wave_lds_sync();
      // S^T[token 4g + q][head r16], two accumulator chains
      f32x4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < DQM; c += 16) {
        const float4 av = *reinterpret_cast<const float4*>(arow + c);
        const float4 bv = *reinterpret_cast<const float4*>(qrow + c);
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, s1, 0, 0, 0);
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, s1, 0, 0, 0);
      }
      s0 += s1;
      float x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = 4 * g + q < nt ? s0[q] * a.scale_log2 : -INFINITY;
      const float mt = max_over_row_groups(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      const float m_new = fmaxf(m_run, mt);
      const bool grow = m_new > m_run + kLazyRescale;
      if (__builtin_amdgcn_ballot_w64(grow)) {
        const float alpha = grow ? exp2f(m_run - m_new) : 1.0f;  // exp2(-inf) = 0
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
        p[q] = exp2f(x[q] - m_ref);
        l_run += p[q];
      }
#pragma unroll
      for (int db = 0; db < NB; ++db) {
        // (blocks past d_c sum RoPE or zero columns and are not stored)
        float av[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) av[q] = vrow[q * TS + 16 * db];
#pragma unroll
        for (int q = 0; q < 4; ++q) o[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], p[q], o[db], 0, 0, 0);
      }
      wave_lds_sync();  // the tile is read before the next unit overwrites it
    };
    // full groups of D units, then the rest straight-line (one loop exit with
    // the same loads in flight on every path keeps the wait counts exact)
    const int nfull = nu / D;
    for (int i0 = 0; i0 < nfull * D; i0 += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        __builtin_amdgcn_sched_barrier(0);
        process(ring[u], i0 + u, true);
      }
    }
#pragma unroll
    for (int u = 0; u < D - 1; ++u) {
      __builtin_amdgcn_sched_barrier(0);
      if (nfull * D + u < nu) process(ring[u], nfull * D + u, false);
    }
  }

  // ---- merge of the waves ----
  l_run = sum_over_row_groups(l_run);
  if (g == 0) mbuf[w * 16 + r16] = m_run;
  __syncthreads();  // also: every wave is done with the list, the query and its tile (obuf aliases them)
  float M = -INFINITY;
#pragma unroll
  for (int v = 0; v < NW; ++v) M = fmaxf(M, mbuf[v * 16 + r16]);
  const float sc = m_run == -INFINITY ? 0.f : exp2f(m_run - M);
#pragma unroll
  for (int db = 0; db < NB; ++db) obuf[(w * NB + db) * 64 + lane] = o[db] * sc;
  if (g == 0) lbuf[w * 16 + r16] = l_run * sc;
  __syncthreads();
  float Ls = 0.f;
#pragma unroll
  for (int v = 0; v < NW; ++v) Ls += lbuf[v * 16 + r16];
  if constexpr (!ONE) {
    const int64_t prow = (static_cast<int64_t>(b) * a.s_max + s) * a.H + h0 + r16;
    if (r16 < nh) {
      for (int db = w; 16 * db < DC; db += NW) {
        f32x4_t sum = obuf[db * 64 + lane];
#pragma unroll
        for (int v = 1; v < NW; ++v) sum += obuf[(v * NB + db) * 64 + lane];
        // lane holds O^T[dim 16 db + 4 g + q][head r16]; d_c is a multiple of 4
        if (16 * db + 4 * g < DC) *reinterpret_cast<f32x4_t*>(a.part_o + prow * DC + 16 * db + 4 * g) = sum;
      }
      if (w == 0 && g == 0) *reinterpret_cast<float2*>(a.part_ml + prow * 2) = make_float2(M, Ls);
    }
  } else {
    // merged rows o / l into LDS ([16][DCM], past the waves' sums), then W_UV
    float* o_s = reinterpret_cast<float*>(lds + NW * NB * 64 * 16);
    const float inv = 1.f / Ls;
    for (int db = w; 16 * db < DC; db += NW) {
      f32x4_t sum = obuf[db * 64 + lane];
#pragma unroll
      for (int v = 1; v < NW; ++v) sum += obuf[(v * NB + db) * 64 + lane];
      *reinterpret_cast<f32x4_t*>(o_s + r16 * DCM + 16 * db + 4 * g) = sum * inv;
    }
    __syncthreads();
    // tpo threads per output, each every tpo-th piece of its row
    const int sub = tid % one.tpo;
    for (int i = tid / one.tpo, first = 1; i < nh * one.DV; i += NT / one.tpo, first = 0) {
      const float* orow = o_s + (i / one.DV) * DCM;
      const unsigned char* wrow = static_cast<const unsigned char*>(one.w_uv) +
                                  (static_cast<int64_t>(h0) * one.DV + i) * DC * EB;
      float acc = 0.f;
      auto add = [&](u32x4_t v, int p) {
        float wv[EPP];
        widen_piece<BF16>(v, wv);
#pragma unroll
        for (int e = 0; e < EPP; ++e) acc = fmaf(wv[e], orow[p * EPP + e], acc);
      };
      if (first) {
#pragma unroll
        for (int k = 0; k < kOnePre; ++k)
          if (sub + k * one.tpo < pc) add(wpre[k], sub + k * one.tpo);
      }
#pragma unroll 4
      for (int p = sub + (first ? kOnePre * one.tpo : 0); p < pc; p += one.tpo)
        add(*reinterpret_cast<const u32x4_t*>(wrow + 16 * p), p);
      for (int m = 1; m < one.tpo; m <<= 1) acc += __shfl_xor(acc, m, 64);
      if (sub == 0) st<BF16>(one.out, (static_cast<int64_t>(b) * a.H + h0) * one.DV + i, acc);
    }
  }
}

}  // namespace egmla

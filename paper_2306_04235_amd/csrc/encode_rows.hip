// encode_rows.hip -- the encoder for more than 64 rows in two launches per
// layer: attention (a block per head and sentence), then everything row-local
// (a block per 16 or 32 rows): output projection and residual, LayerNorm,
// feed-forward and residual, the next LayerNorm, and the next layer's Q/K/V.
//
// The row-local part streams the layer's weights through each CU as the
// row-wise decoder does (decode_rows.hip, rows.hpp), with 16 (or 2 x 16) rows
// against every fragment, so that nothing but the residual rows, Q/K/V codes
// and the context passes through memory.  As launches per operator, the
// mobile model's layer over 3840 rows took 55 us: four GEMMs of 5.5-8.2 us
// and two LayerNorms of 4.3 us, each mostly launch and memory latency, and an
// attention of 16 us.
#include "blocks.hpp"
#include "internal.h"
#include "rows.hpp"
#include "rows_plan.hpp"

namespace mnmt {
namespace {

// The stream of one blob: 0 o, 1 w1, 2 w2, 3 the next layer's qkv.
template <int KQ_, int FQ_>
struct EncShape {
  static constexpr int KQ = KQ_, FQ = FQ_, D = 64 * KQ, F = 64 * FQ;
  static constexpr int WAVES = rows_waves(D);
  static constexpr int C = KQ <= 2 ? 1 : KQ == 6 ? 3 : 2;
  static constexpr int kRing = KQ == 1 ? 2 : 4;
  static constexpr int NCH = KQ / C, NCH2 = FQ / C;
  static constexpr int TD = 4 * KQ / WAVES, TQ = 3 * TD, TF = 4 * FQ / WAVES;
  static constexpr int kO = 0, kW1 = kO + TD * NCH, kW2 = kW1 + TF * NCH, kQkv = kW2 + TD * NCH2, kEnd = kQkv + TQ * NCH;
  __host__ __device__ static constexpr BatchAt at(int b) {
    return b < kW1    ? batch_in(0, b - kO, NCH)
           : b < kW2  ? batch_in(1, b - kW1, NCH)
           : b < kQkv ? batch_in(2, b - kW2, NCH2)
                      : batch_in(3, b - kQkv, NCH);
  }
  __host__ __device__ static constexpr EncOff off(bool w4) { return enc_off(D, F, w4); }
  static_assert(KQ % C == 0 && FQ % C == 0 && 4 * KQ % WAVES == 0 && 4 * FQ % WAVES == 0, "");
};

struct EncHdr {
  float ff_inv, next_inv, sa_gamma, ff_gamma;
};

// One block: rows blockIdx.x * RB .. + RB - 1 (at most 16 MT).  g.first: the
// input rows (embedded here, or in x), their LayerNorm and Q/K/V; else from
// the attention context and the residual rows x to the next layer's Q/K/V, or
// g.last: to the encoder's int8 output.
template <int KQ, int FQ, bool W4, int MT>
__global__ __launch_bounds__((64 * EncShape<KQ, FQ>::WAVES)) void k_enc_rows(EncRowsArgs g) {
  using S = EncShape<KQ, FQ>;
  constexpr int D = S::D, WAVES = S::WAVES, THREADS = 64 * WAVES;
  constexpr int XS = D + 4, AS = D + 16, QS = 3 * D + 16, HS = S::F + 16;
  constexpr EncOff O = enc_off(D, S::F, W4);
  extern __shared__ __attribute__((aligned(16))) int8_t lds[];
  const int RB = g.RB;
  float* xs = reinterpret_cast<float*>(lds);
  float* lns = reinterpret_cast<float*>(lds + RB * XS * 4);
  int8_t* as = lds + RB * XS * 4 + 16 * D;
  int8_t* act = as + RB * AS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row0 = blockIdx.x * RB, rows = min(RB, g.R - row0);
  // nothing to do for rows past their sentence's end (they are never read)
  bool live = false;
  for (int b = row0 / g.S; b * g.S < row0 + rows; ++b)  // (lengths clamped to 1..S, as the attention reads them)
    live = live || max(row0, b * g.S) < b * g.S + min(max(g.len[b], 1), g.S);
  if (!live) return;

  const Blob bl = blob_rsrc<S, W4>(g.blob);
  Ring<S, W4> ring;
  const auto* hp = (const __attribute__((address_space(4))) float*)(uintptr_t)g.blob;  // (scalar loads)
  const EncHdr H{hp[0], hp[1], hp[2], hp[3]};
  constexpr int LN4 = 4 * D / 4;
  static_assert(LN4 <= THREADS && O.ln[1] == O.ln[0] + 8 * D, "");
  auto load_ln = [&] {
    if (tid < LN4) *(float4*)(lns + 4 * tid) = *(const float4*)(g.blob + O.ln[0] + 16 * tid);
  };
  const int koff = 16 * (lane >> 4);
  const int l16 = lane & 15;
  const int8_t *arow = as + min(l16, rows - 1) * AS + koff, *hrow = act + min(l16, rows - 1) * HS + koff;
  // tile 1's rows: 16 further, or (past the block's last row) tile 0's again
  const int step = MT > 1 && l16 + 16 < rows ? 16 : 0;

  auto norm = [&](int ln, int do_ln, float inv_s, bool replace) {
    for (int i = wave; i < rows; i += WAVES) {
      float gj[KQ], bj[KQ];
#pragma unroll
      for (int j = 0; j < KQ; ++j) {
        gj[j] = lns[2 * D * ln + lane + 64 * j];
        bj[j] = lns[2 * D * ln + D + lane + 64 * j];
      }
      norm_row<KQ>(xs + i * XS, do_ln, gj, bj, g.eps, inv_s, replace, as + i * AS, lane);
    }
    lds_barrier();
  };
  auto resid = [&](float gamma) {
    return [=](int m, int tile, const v4i acc, const float4 sc, const float4 bi) {
      if (l16 + 16 * m < rows) {
        float4* xp = reinterpret_cast<float4*>(xs + (l16 + 16 * m) * XS + 16 * tile + 4 * (lane >> 4));
        float4 x = *xp;
        x.x = fmaf(gamma, x.x, fmaf((float)acc[0], sc.x, bi.x));
        x.y = fmaf(gamma, x.y, fmaf((float)acc[1], sc.y, bi.y));
        x.z = fmaf(gamma, x.z, fmaf((float)acc[2], sc.z, bi.z));
        x.w = fmaf(gamma, x.w, fmaf((float)acc[3], sc.w, bi.w));
        *xp = x;
      }
    };
  };
  auto qkv = [&] {  // the next layer's Q/K/V from as, and the residual rows, to memory
    linear<S, W4, S::kQkv, S::kEnd, MT, S::kEnd>(
        ring, arow, step * AS, bl, bl, false, wave, lane,
        [&](int m, int tile, const v4i acc, const float4 sc, const float4 bi) {
          if (l16 + 16 * m < rows)
            *(int*)(act + (l16 + 16 * m) * QS + 16 * tile + 4 * (lane >> 4)) = pack_codes<false>(acc, sc, bi);
        });
    lds_barrier();
    for (int i = tid; i < rows * (D / 4); i += THREADS) {
      const int r = i / (D / 4), c = i % (D / 4);
      *(float4*)(g.x + (size_t)(row0 + r) * D + 4 * c) = *(const float4*)(xs + r * XS + 4 * c);
    }
    for (int i = tid; i < rows * (3 * D / 16); i += THREADS) {
      const int r = i / (3 * D / 16), c = i % (3 * D / 16);
      *(v4i*)(g.out + (size_t)(row0 + r) * 3 * D + 16 * c) = *(const v4i*)(act + r * QS + 16 * c);
    }
  };

  if (g.first) {
#pragma unroll
    for (int b = S::kQkv; b < S::kQkv + S::kRing; ++b) issue(ring, b, bl, bl, wave, lane);
    load_ln();
    for (int i = wave; i < rows; i += WAVES) {
      const size_t r = row0 + i;
      float v[KQ];
      if (g.tok) {
        int tk = g.tok[r];
        tk = tk < 0 ? 0 : (tk >= g.V ? g.V - 1 : tk);
        const float c = g.c_emb[tk];
        const size_t pos = r % (size_t)g.S;
#pragma unroll
        for (int j = 0; j < KQ; ++j)
          v[j] = fmaf((float)g.E[(size_t)tk * D + lane + 64 * j], c, g.pe[pos * D + lane + 64 * j]);
      } else {
#pragma unroll
        for (int j = 0; j < KQ; ++j) v[j] = g.x[r * D + lane + 64 * j];
      }
#pragma unroll
      for (int j = 0; j < KQ; ++j) xs[i * XS + lane + 64 * j] = v[j];
    }
    lds_barrier();
    norm(1, !g.post, H.next_inv, false);
    qkv();
    return;
  }
#pragma unroll
  for (int b = 0; b < S::kRing; ++b) issue(ring, b, bl, bl, wave, lane);
  load_ln();
  for (int i = tid; i < rows * (D / 16); i += THREADS) {
    const int r = i / (D / 16), c = i % (D / 16);
    *(v4i*)(as + r * AS + 16 * c) = *(const v4i*)(g.ctx + (size_t)(row0 + r) * D + 16 * c);
  }
  for (int i = tid; i < rows * (D / 4); i += THREADS) {
    const int r = i / (D / 4), c = i % (D / 4);
    *(float4*)(xs + r * XS + 4 * c) = *(const float4*)(g.x + (size_t)(row0 + r) * D + 4 * c);
  }
  lds_barrier();
  const bool more = !g.last;
  linear<S, W4, S::kO, S::kW1, MT, S::kQkv>(ring, arow, step * AS, bl, bl, more, wave, lane, resid(H.sa_gamma));
  lds_barrier();
  norm(0, 1, H.ff_inv, g.post);
  linear<S, W4, S::kW1, S::kW2, MT, S::kQkv>(
      ring, arow, step * AS, bl, bl, more, wave, lane,
      [&](int m, int tile, const v4i acc, const float4 sc, const float4 bi) {
        if (l16 + 16 * m < rows)
          *(int*)(act + (l16 + 16 * m) * HS + 16 * tile + 4 * (lane >> 4)) = pack_codes<true>(acc, sc, bi);
      });
  lds_barrier();
  linear<S, W4, S::kW2, S::kQkv, MT, S::kQkv>(ring, hrow, step * HS, bl, bl, more, wave, lane, resid(H.ff_gamma));
  lds_barrier();
  norm(1, 1, H.next_inv, g.post);
  if (!g.last) {
    qkv();
    return;
  }
  for (int i = tid; i < rows * (D / 16); i += THREADS) {
    const int r = i / (D / 16), c = i % (D / 16);
    *(v4i*)(g.out + (size_t)(row0 + r) * D + 16 * c) = *(const v4i*)(as + r * AS + 16 * c);
  }
}

// Encoder self-attention, block = (head, sentence), heads of at most 64: the
// sentence's keys of the head in LDS, its values transposed there (a word =
// four keys of one column), wave w working on query rows 8 w .. 8 w + 7, then
// 8 w + 64 and so on.  The scores of 8 rows come from v_mfma_i32_16x16x64_i8
// (exact); the softmax runs in the canonical layout (key = lane + 64 i), four
// rows at a time so that their butterflies overlap; the context takes one fma
// per key and row in ascending order, each value converted once for 8 rows.
// Bound by VALU issue: 64 keys of 64 columns cost 64 fma per row, about 4 us
// of a CU for a sentence of 60.  The one-row-at-a-time form (k_attn_shared:
// dot products per row, a conversion per key and row) took 16 us per layer
// for 64 sentences of 10-60 tokens and 34 us for 128 of 20-64, 8 heads.
struct EncAttnArgs {
  const int8_t* qkv;   // [B * S, 3d]
  const int32_t* len;
  int8_t* ctx;         // [B * S, d]
  int S, d, dh;
  float c_qk, c_pv;
};

template <int NP>
__global__ __launch_bounds__(512) void k_attn_enc(EncAttnArgs a) {
  constexpr int NI = NP / 64, KS = 80, VS = NP / 4 + 1;
  __shared__ __attribute__((aligned(16))) int8_t kl[NP * KS];
  __shared__ int vt[64 * VS];
  __shared__ __attribute__((aligned(16))) int sc[8][8][NP];
  const int hd = blockIdx.x, b = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int d = a.d, dh = a.dh, nc = dh / 16;
  int n = a.len[b];
  n = n < 1 ? 1 : (n > a.S ? a.S : n);
  const size_t ld = 3 * (size_t)d;
  const int8_t* q = a.qkv + (size_t)b * a.S * ld + hd * dh;
  const int8_t *k = q + d, *v = q + 2 * d;
  const int l16 = lane & 15, ch = lane >> 4;
  auto qfrag = [&](int u) { return *(const v4i*)(q + (size_t)min(8 * u + (lane & 7), n - 1) * ld + 16 * min(ch, nc - 1)); };
  v4i qf = qfrag(wave);
  for (int i = tid; i < n * 4; i += 512) {
    const int t = i >> 2, c = i & 3;
    v4i x = {0, 0, 0, 0};
    if (c < nc) x = *(const v4i*)(k + (size_t)t * ld + 16 * c);
    *(v4i*)(kl + t * KS + 16 * c) = x;  // (chunks past the head: zero, so that they add nothing)
  }
  for (int i = tid; i < (n + 3) / 4 * nc; i += 512) {
    const int g = i / nc, c = i - g * nc;
    v4i x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = *(const v4i*)(v + (size_t)min(4 * g + u, n - 1) * ld + 16 * c);
    int w[16];
    transpose_chunks(x, w);
#pragma unroll
    for (int j = 0; j < 16; ++j) vt[(16 * c + j) * VS + g] = w[j];
  }
  lds_barrier();
  for (int u = wave; 8 * u < n; u += 8) {
    int(&s)[8][NP] = sc[wave];
    for (int kt = 0; 16 * kt < n; ++kt) {
      const v4i kf = *(const v4i*)(kl + (16 * kt + l16) * KS + 16 * ch);
      const v4i acc = mfma16(qf, kf, v4i{0, 0, 0, 0});
      // element i of lane l: query row 4 (l / 16) + i (rows 8..15 repeat 0..7), key l % 16
      if (lane < 32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[4 * ch + i][16 * kt + l16] = acc[i];
      }
    }
    qf = qfrag(min(u + 8, (n - 1) / 8));
    wave_sync();  // the scores visible to every lane of the wave
#pragma unroll
    for (int r0 = 0; r0 < 8; r0 += 4) {
      float sv[4][NI], mx[4], part[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        mx[r] = -FLT_MAX;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          const int t = lane + 64 * i;
          sv[r][i] = (float)s[r0 + r][t] * a.c_qk;
          if (t < n) mx[r] = fmaxf(mx[r], sv[r][i]);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) mx[r] = wave_max(mx[r]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        part[r] = 0.0f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (64 * i < n) {
            sv[r][i] = lane + 64 * i < n ? canon_exp(sv[r][i] - mx[r]) : 0.0f;
            part[r] = part[r] + sv[r][i];
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) part[r] = 1.0f / wave_sum(part[r]);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < NI; ++i)
          if (64 * i < n) s[r0 + r][lane + 64 * i] = __float_as_int(sv[r][i] * part[r]);
    }
    wave_sync();  // the weights
    float acc[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) acc[r] = 0.0f;
#pragma unroll 1
    for (int t0 = 0; t0 < n; t0 += 16) {  // (keys past n: weight zero)
      float vf[16];
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int w = vt[lane * VS + t0 / 4 + g];
        vf[4 * g] = (float)(int8_t)w;
        vf[4 * g + 1] = (float)(int8_t)(w >> 8);
        vf[4 * g + 2] = (float)(int8_t)(w >> 16);
        vf[4 * g + 3] = (float)(w >> 24);
      }
#pragma unroll
      for (int r = 0; r < 8; ++r) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const float4 p = *(const float4*)&s[r][t0 + 4 * g];
          acc[r] = fmaf(p.x, vf[4 * g], acc[r]);
          acc[r] = fmaf(p.y, vf[4 * g + 1], acc[r]);
          acc[r] = fmaf(p.z, vf[4 * g + 2], acc[r]);
          acc[r] = fmaf(p.w, vf[4 * g + 3], acc[r]);
        }
      }
    }
    if (lane < dh) {
#pragma unroll
      for (int r = 0; r < 8; ++r)
        if (8 * u + r < n) a.ctx[((size_t)b * a.S + 8 * u + r) * d + hd * dh + lane] = code_of(acc[r] * a.c_pv);
    }
    wave_sync();  // every lane done with the rows before the next ones
  }
}

int enc_lds(int d, int F, int RB) {
  return RB * (d + 4) * 4 + 16 * d + RB * (d + 16) + RB * ((3 * d > F ? 3 * d : F) + 16);
}

template <int KQ, int FQ, int MT>
hipError_t launch_shape(const EncRowsArgs& g, int blocks, int lds, hipStream_t s) {
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kRowsMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * EncShape<KQ, FQ>::WAVES), lds, s, g);
    return hipGetLastError();
  };
  return g.w4 ? go(k_enc_rows<KQ, FQ, true, MT>) : go(k_enc_rows<KQ, FQ, false, MT>);
}

template <int KQ>
hipError_t launch_kq(const EncRowsArgs& g, int blocks, int lds, hipStream_t s) {
  if (g.RB > 16)
    return g.F == 2 * g.d ? launch_shape<KQ, 2 * KQ, 2>(g, blocks, lds, s) : launch_shape<KQ, 4 * KQ, 2>(g, blocks, lds, s);
  return g.F == 2 * g.d ? launch_shape<KQ, 2 * KQ, 1>(g, blocks, lds, s) : launch_shape<KQ, 4 * KQ, 1>(g, blocks, lds, s);
}

}  // namespace

// Rows per block: as few as keep the grid within one block per CU (weights
// cost a block the same for 1 to 32 rows), up to two tiles of 16; past that,
// the fewest rounds of 256 blocks, evenly filled.
hipError_t launch_enc_rows(const EncRowsArgs& args, hipStream_t s) {
  if (args.R < 1 || !dec_rows_shape(args.d, args.dh, args.F)) return hipErrorInvalidValue;
  EncRowsArgs g = args;
  const int rounds = (g.R + 256 * 32 - 1) / (256 * 32);
  g.RB = (g.R + 256 * rounds - 1) / (256 * rounds);
  const int blocks = (g.R + g.RB - 1) / g.RB, lds = enc_lds(g.d, g.F, g.RB);
  if (lds > kRowsMaxLds) return hipErrorInvalidValue;
  switch (g.d) {
    case 64: return launch_kq<1>(g, blocks, lds, s);
    case 128: return launch_kq<2>(g, blocks, lds, s);
    case 256: return launch_kq<4>(g, blocks, lds, s);
    case 384: return launch_kq<6>(g, blocks, lds, s);
    default: return launch_kq<8>(g, blocks, lds, s);
  }
}

hipError_t launch_attn_enc_rows(const int8_t* qkv, const int32_t* len, int B, int S, int d, int h, float c_qk,
                                float c_pv, int8_t* ctx, hipStream_t s) {
  const EncAttnArgs a{qkv, len, ctx, S, d, d / h, c_qk, c_pv};
  if (B < 1 || S < 1 || S > kMaxAttnLen || a.dh > 64 || a.dh % 16) return hipErrorInvalidValue;
  if (S <= 64)
    hipLaunchKernelGGL(k_attn_enc<64>, dim3(h, B), dim3(512), 0, s, a);
  else if (S <= 128)
    hipLaunchKernelGGL(k_attn_enc<128>, dim3(h, B), dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL(k_attn_enc<256>, dim3(h, B), dim3(512), 0, s, a);
  return hipGetLastError();
}

size_t enc_rows_blob_bytes(int d, int F, bool w4) { return enc_off(d, F, w4).bytes; }

// Blob of the pass after layer L's attention up to the next layer's Q/K/V
// (next; null after the last layer), or (L null) of the first Q/K/V alone.
// ln_next, next_inv: the LayerNorm and 1 / input scale of what follows.
hipError_t launch_enc_rows_pack(const LayerDev* L, const LinearDev* next, const LnDev& ln_ff, const LnDev& ln_next,
                                float next_inv, int d, int F, bool w4, int8_t* blob, hipStream_t s) {
  const EncOff O = enc_off(d, F, w4);
  RowsPack p{};
  p.blob = blob;
  const float hdr[4] = {L ? L->w1.inv_in : 0.0f, next_inv, L ? L->sa_gamma : 0.0f, L ? L->ff_gamma : 0.0f};
  for (int i = 0; i < 4; ++i) p.hdr[i] = hdr[i];
  const LnDev* ln[2] = {L ? &ln_ff : nullptr, &ln_next};
  for (int i = 0; i < 2; ++i)
    if (ln[i]) {
      rows_pack_add(p, ln[i]->g, O.ln[i], d);
      rows_pack_add(p, ln[i]->b, O.ln[i] + 4 * d, d);
    }
  const LinearDev* lin[4] = {L ? &L->o : nullptr, L ? &L->w1 : nullptr, L ? &L->w2 : nullptr, next};
  return launch_rows_pack(p, lin, 4, O.c, O.n, O.w, w4, s);
}

}  // namespace mnmt

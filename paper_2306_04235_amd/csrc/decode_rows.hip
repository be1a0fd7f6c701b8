// decode_rows.hip -- every decoder layer of one step in one launch, for
// batches of rows (beam search of any width, greedy search of 3 rows and
// more).
//
// The rows of a step do not depend on each other between the logits of one
// step and the next (each has its own cache row and history, and attends over
// its own sentence's source), so a block can take a few rows through all
// layers by itself: LayerNorms, projections, attention and feed-forward, with
// the rows' residual stream and int8 activations in LDS and no exchange with
// any other block.  The launch-per-operator form paid 6 (d 256) to 10 (d 512)
// dependent launches per layer of 4-9 us each, most of it dispatch and memory
// latency.
//
// What bounds it: a block streams every weight of the layer through its CU,
// whose vector memory path moves 64 bytes per clock: 115-130 GB/s measured
// with 64-256 such blocks resident (the 8 L2s and the last-level cache supply
// them all, since the blocks of an XCD read the same weights at about the
// same time).  That rate needs each wave's load to be one contiguous
// kilobyte: from row-major weights, where a matrix-core fragment gathers 64
// bytes of 16 rows, the same loop reached 37 GB/s.  So the session keeps a
// copy of the decoder's weights in fragment order (per tile of 16 output
// columns and slice of 64 inputs, lane l's 16 bytes, or 8 of packed 4-bit
// codes, next to lane l + 1's), in one blob per layer with the layer's
// constants (RowsOff), so that every address is the layer's base plus a
// compile-time offset: pointers fetched from a table cost half a microsecond
// of scalar-load latency per phase.
//
// The weights of a layer are one stream of batches per wave, through all six
// linear layers and on into the next decoder layer: each wave keeps a ring of
// kRing batches in flight, and the batch that is used makes room for the
// batch kRing further on, whatever phase it belongs to.  So the memory pipe
// stays busy through the LayerNorms, attention and barriers in between (a
// version that loaded one batch ahead within a phase took 43 us for the mobile
// decoder's two layers at 256 rows and 327 us for the base model's six at 512;
// this one 35 and 278 us, against about 66 and 370 us for the launches per
// operator).  Clock stamps put a base layer at 46 us: the linear layers 35
// (3.7 MB at about 105 GB/s), self-attention 4.8, cross-attention 2.5, the
// three LayerNorms 3.
//
// Rows per block: as few as let the grid reach one block per CU (up to 16,
// the rows of a matrix-core tile): weights cost the same for 1 or 16 rows,
// attention and LayerNorm cost per row.
//
// The arithmetic is that of the other decoder kernels, in the same canonical
// order (canon.hpp): exact int32 sums, one fma per requantization, LayerNorm
// sums in lane order, one fma per key for the attention context.
#include "blocks.hpp"
#include "internal.h"
#include "rows.hpp"
#include "rows_plan.hpp"

namespace mnmt {
namespace {

struct RowsParams {
  RowsArgs g;
  RowsLds l;
};

// The scalars of a layer, first in its blob.
struct RowsHdr {
  float sa_inv, ca_inv, ff_inv;  // 1 / input scale of qkv, cq, w1
  float sa_cqk, sa_cpv, ca_cqk, ca_cpv;
  float sa_gamma, ca_gamma, ff_gamma;
};

// Shapes of the decoder the kernel is compiled for: d = 64 KQ, F = 64 FQ.
// WAVES divides the tiles of every linear layer (4 KQ, 12 KQ, 4 FQ); a batch
// is C slices of a tile, kRing batches are in flight per wave (C * kRing
// kilobytes of int8 weights), and the batches of a layer are a multiple of
// kRing, so that a batch's ring slot is the same in every layer.
template <int KQ_, int FQ_>
struct Shape {
  static constexpr int KQ = KQ_, FQ = FQ_, D = 64 * KQ, F = 64 * FQ;
  static constexpr int WAVES = rows_waves(D);
  static constexpr int C = KQ <= 2 ? 1 : KQ == 6 ? 3 : 2;
  static constexpr int kRing = KQ == 1 ? 2 : 4;
  static constexpr int NCH = KQ / C, NCH2 = FQ / C;             // batches per tile: K = d, K = F
  static constexpr int TD = 4 * KQ / WAVES, TQ = 3 * TD, TF = 4 * FQ / WAVES;  // tiles per wave
  static constexpr int kQkv = 0, kO = kQkv + TQ * NCH, kCq = kO + TD * NCH, kCo = kCq + TD * NCH,
                       kW1 = kCo + TD * NCH, kW2 = kW1 + TF * NCH, kEnd = kW2 + TD * NCH2;  // first batches
  __host__ __device__ static constexpr BatchAt at(int b) {
    return b < kO    ? batch_in(0, b - kQkv, NCH)
           : b < kCq ? batch_in(1, b - kO, NCH)
           : b < kCo ? batch_in(2, b - kCq, NCH)
           : b < kW1 ? batch_in(3, b - kCo, NCH)
           : b < kW2 ? batch_in(4, b - kW1, NCH)
                     : batch_in(5, b - kW2, NCH2);
  }
  __host__ __device__ static constexpr RowsOff off(bool w4) { return rows_off(D, F, w4); }
  static_assert(KQ % C == 0 && FQ % C == 0 && 4 * KQ % WAVES == 0 && 4 * FQ % WAVES == 0 && kEnd % kRing == 0, "");
};

// Chunk c = lane % 4 (16 bytes) of the keys or values of positions t0 + 4 pp
// + u, pp = lane / 4, of one head: SELF: position pos of the sentence's cache
// row hist[pos] (base: its first row), at column `at` (byte offsets below
// 2^31, which the launcher checks); else row pos of one sentence's source keys
// or values.  Positions past the last of `cached` repeat it.  hist holds a
// valid row for every position up to the next multiple of 64.
template <bool SELF>
__device__ __forceinline__ void load_chunks(v4i (&r)[4], const int8_t* base, const uint8_t* hist, int T, unsigned ld,
                                            unsigned at, int cached, int t0, int pp) {
  const int last = max(cached - 1, 0);
  unsigned h = 0;
  if constexpr (SELF) h = *(const unsigned*)(hist + t0 + 4 * pp);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const unsigned pos = min(t0 + 4 * pp + u, last);
    r[u] = *(const v4i*)(base + ((SELF ? (h >> (8 * u) & 255u) * T + pos : pos) * ld + at));
  }
}

__device__ __forceinline__ int dot16(const v4i a, const v4i b) {
  int acc = __builtin_amdgcn_sdot4(a.x, b.x, 0, false);
  acc = __builtin_amdgcn_sdot4(a.y, b.y, acc, false);
  acc = __builtin_amdgcn_sdot4(a.z, b.z, acc, false);
  return __builtin_amdgcn_sdot4(a.w, b.w, acc, false);
}

// Attention of one query row for one head (at most 64 wide) by one wave over
// `cached` keys (load_chunks; kr holds the first 64 positions') and, SELF,
// the row's own, not yet in the cache: its key at q + d and its value at
// q + 2d in LDS.  The four lanes of a position sum their partial dot products
// (exact), and the lane keeps u = c, so that lane l holds the score of key t0
// + l, the canonical softmax's layout, without a pass through LDS.  A lane's
// value chunks of four consecutive positions are transposed in registers and
// stored as words of four keys per column, so that the context chain (one fma
// per key, ascending) reads four values at a time.
template <bool SELF>
__device__ __forceinline__ void attend_row(v4i (&kr)[4], const int8_t* kb, const int8_t* vb, const uint8_t* hist, int T,
                                           unsigned ld, unsigned at, int cached, int dh, const int8_t* q, int d,
                                           float c_qk, float c_pv, float* p, int* vt, int8_t* out, int lane) {
  const int c = lane & 3, pp = lane >> 2, nc = dh / 16, cc = min(c, nc - 1), n = cached + (SELF ? 1 : 0);
  const v4i qc = *(const v4i*)(q + 16 * cc);
  int own = 0;
  if constexpr (SELF) {
    own = dot16(*(const v4i*)(q + d + 16 * cc), qc);
    own = quad_sum(c < nc ? own : 0);
  }
  // scores of 64 keys at a time into p (each lane its own keys' slots)
  float mx = -FLT_MAX;
#pragma unroll 1
  for (int t0 = 0; t0 < n; t0 += 64) {
    if (t0 > 0) load_chunks<SELF>(kr, kb, hist, T, ld, at + 16u * cc, cached, t0, pp);
    int s[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int x = dot16(kr[u], qc);
      s[u] = quad_sum(c < nc ? x : 0);
    }
    int mine = c == 0 ? s[0] : c == 1 ? s[1] : c == 2 ? s[2] : s[3];
    if (SELF && t0 + lane == cached) mine = own;
    const float sv = (float)mine * c_qk;
    if (t0 + lane < n) mx = fmaxf(mx, sv);
    p[t0 + lane] = sv;
  }
  // the first values, in flight during the softmax
  v4i v[4];
  load_chunks<SELF>(v, vb, hist, T, ld, at + 16u * cc, cached, 0, pp);
  asm volatile("" ::: "memory");
  // softmax (the canonical order; weights past n are zero and add nothing)
  mx = wave_max(mx);
  float part = 0.0f;
#pragma unroll 1
  for (int t0 = 0; t0 < n; t0 += 64) {
    const float e = t0 + lane < n ? canon_exp(p[t0 + lane] - mx) : 0.0f;
    part = part + e;
    p[t0 + lane] = e;
  }
  const float inv = 1.0f / wave_sum(part);
  float w = 0.0f;
#pragma unroll 1
  for (int t0 = 0; t0 < n; t0 += 64) {
    w = p[t0 + lane] * inv;
    p[t0 + lane] = t0 + lane < cached ? w : 0.0f;
  }
  // the own key is the last of the last group
  const float w_own = SELF ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), cached & 63)) : 0.0f;
  // context
  float acc = 0.0f;
  const int* mine = vt + lane * kVtStride;
#pragma unroll 1
  for (int t0 = 0; t0 < cached; t0 += 64) {
    if (t0 > 0) load_chunks<SELF>(v, vb, hist, T, ld, at + 16u * cc, cached, t0, pp);
    int w[16];
    transpose_chunks(v, w);
#pragma unroll
    for (int k = 0; k < 16; ++k) vt[(16 * c + k) * kVtStride + pp] = w[k];
    wave_sync();  // the weights and the transposed values visible to the wave
    const int m = min(64, cached - t0);
    const float* pw = p + t0;
#pragma unroll 1
    for (int t = 0; t < m; t += 8) {  // (keys past the last: weight zero)
      const float4 pa = *(const float4*)(pw + t), pb = *(const float4*)(pw + t + 4);
      const int va = mine[t / 4], vb2 = mine[t / 4 + 1];
      acc = fmaf(pa.x, (float)(int8_t)va, acc);
      acc = fmaf(pa.y, (float)(int8_t)(va >> 8), acc);
      acc = fmaf(pa.z, (float)(int8_t)(va >> 16), acc);
      acc = fmaf(pa.w, (float)(va >> 24), acc);
      acc = fmaf(pb.x, (float)(int8_t)vb2, acc);
      acc = fmaf(pb.y, (float)(int8_t)(vb2 >> 8), acc);
      acc = fmaf(pb.z, (float)(int8_t)(vb2 >> 16), acc);
      acc = fmaf(pb.w, (float)(vb2 >> 24), acc);
    }
    wave_sync();  // every lane done with vt (and p) before they are written again
  }
  if (lane < dh) {
    if (SELF) acc = fmaf(w_own, (float)q[2 * d + lane], acc);
    out[lane] = code_of(acc * c_pv);
  }
}

template <int KQ, int FQ, bool W4>
__global__ __launch_bounds__((64 * Shape<KQ, FQ>::WAVES)) void k_dec_rows(RowsParams P) {
  using S = Shape<KQ, FQ>;
  constexpr int D = S::D, WAVES = S::WAVES, THREADS = 64 * WAVES;
  constexpr int XS = D + 4, AS = D + 16;
  constexpr RowsOff O = rows_off(D, S::F, W4);
  extern __shared__ __attribute__((aligned(16))) int8_t lds[];
  const RowsArgs& g = P.g;
  float* xs = reinterpret_cast<float*>(lds);
  float* lns = reinterpret_cast<float*>(lds + P.l.ln);
  int8_t* as = lds + P.l.a;
  int8_t* act = lds + P.l.act;
  uint8_t* hs = reinterpret_cast<uint8_t*>(lds + P.l.hist);
  constexpr int QS = 3 * D + 16, HS = S::F + 16;  // row strides of act: q|k|v, hidden rows
  int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = blockIdx.x * g.RB, rows = min(g.RB, g.R - row0);
  const int dh = g.dh, h = g.h, T = g.T, nc = dh / 16, units = rows * h;
  const int hs_s = (T + 63) / 64 * 64;
  // the wave's first (row, head) unit of the attention phases, and the steps
  // to its next ones (units wave, wave + WAVES, ...); the sentence's first row
  const int i0 = wave / h, hd0 = wave - i0 * h, di = WAVES / h, dhd = WAVES - di * h;
  float* pw = reinterpret_cast<float*>(lds + P.l.p + min(wave, min(WAVES, g.RB * h) - 1) * (P.l.np * 4 + kVtBytes));
  int* vt = reinterpret_cast<int*>(pw + P.l.np);

  auto layer_base = [&](int l) {
    return g.blobs + (size_t)__builtin_amdgcn_readfirstlane(g.index ? g.index[l] : l) * O.bytes;
  };
  const int8_t* base = layer_base(0);
  Ring<S, W4> ring;
#pragma unroll
  for (int b = 0; b < S::kRing; ++b) issue(ring, b, blob_rsrc<S, W4>(base), blob_rsrc<S, W4>(base), wave, lane);
  const int t = g.t >= 0 ? g.t : min(max(*g.step, 0), T - 1);

  // A layer's LayerNorm constants (gain and bias of its three LayerNorms, 6 d
  // floats next to each other in the blob) pass through registers into LDS,
  // one 16-byte word per thread: read from memory where they are used, they
  // would wait behind the weights in flight (loads return in order).
  constexpr int LN4 = 6 * D / 4;
  static_assert(LN4 <= THREADS && O.ln[1] == O.ln[0] + 8 * D && O.ln[2] == O.ln[1] + 8 * D, "");
  auto load_ln = [&](const int8_t* layer) { return *(const float4*)(layer + O.ln[0] + 16 * min(tid, LN4 - 1)); };
  auto store_ln = [&](const float4 v) {
    if (tid < LN4) *(float4*)(lns + 4 * tid) = v;
  };
  store_ln(load_ln(base));
  // the step's input rows: embeddings (tok) or rows another kernel wrote
  for (int i = wave; i < rows; i += WAVES) {
    const size_t r = row0 + i;
    float v[KQ];
    if (g.tok) {
      int tk = g.tok[r];
      tk = tk < 0 ? 0 : (tk >= g.V ? g.V - 1 : tk);
      const float c = g.c_emb[tk];
#pragma unroll
      for (int j = 0; j < KQ; ++j)
        v[j] = fmaf((float)g.E[(size_t)tk * D + lane + 64 * j], c, g.pe[(size_t)t * D + lane + 64 * j]);
    } else {
#pragma unroll
      for (int j = 0; j < KQ; ++j) v[j] = g.x[r * D + lane + 64 * j];
    }
#pragma unroll
    for (int j = 0; j < KQ; ++j) xs[i * XS + lane + 64 * j] = v[j];
  }
  // the rows of the sentence that hold each earlier position's key and value
  // (without a history, and past the last position: the row's own)
  for (int i = wave; i < rows; i += WAVES) {
    const int r = row0 + i, first = r / g.W * g.W;
    for (int j = lane; j < hs_s; j += 64)
      hs[i * hs_s + j] = (uint8_t)((g.hist && j < T ? g.hist[((size_t)(t & 1) * g.R + r) * T + j] : r) - first);
  }
  // the first unit's sentence
  auto keys_of = [&](int b) {
    const int n = g.len[b];
    return n < 1 ? 1 : (n > g.S ? g.S : n);
  };
  const int b0 = (row0 + min(i0, rows - 1)) / g.W, n0 = keys_of(b0);
  auto cache_at = [&](int i) { return (unsigned)((row0 + i) / g.W * g.W) * T * D; };
  lds_barrier();

  for (int l = 0; l < g.n_layers; ++l) {
    // the lane and wave indexes opaque to the compiler in each layer: it would otherwise
    // compute every phase's LDS and memory offsets before the loop and spill
    asm volatile("" : "+v"(lane), "+v"(tid), "+s"(wave));
    const int l16 = min(lane & 15, rows - 1), koff = 16 * (lane >> 4);
    const bool real = (lane & 15) < rows;  // the lane's row of a tile is one of the block's
    const int8_t* next = layer_base(min(l + 1, g.n_layers - 1));
    const bool more = l + 1 < g.n_layers;
    const auto* hp = (const __attribute__((address_space(4))) float*)(uintptr_t)base;  // (scalar loads)
    const RowsHdr H{hp[0], hp[1], hp[2], hp[3], hp[4], hp[5], hp[6], hp[7], hp[8], hp[9]};
    int8_t* kc = g.kcache + l * g.cache_stride;
    int8_t* vc = g.vcache + l * g.cache_stride;
    const int8_t* ckv = g.cross + l * g.cross_stride;
    const int8_t* arow = as + l16 * AS + koff;
    const int8_t* hrow = act + l16 * HS + koff;

    // LayerNorm + quantization of the block's rows, one wave per row
    auto norm = [&](int ln, int do_ln, float inv_s, bool replace) {
      if (wave < rows) {
        float gj[KQ], bj[KQ];
#pragma unroll
        for (int j = 0; j < KQ; ++j) {
          gj[j] = lns[2 * D * ln + lane + 64 * j];
          bj[j] = lns[2 * D * ln + D + lane + 64 * j];
        }
        norm_row<KQ>(xs + wave * XS, do_ln, gj, bj, g.eps, inv_s, replace, as + wave * AS, lane);
      }
      lds_barrier();
    };
    auto resid = [&](float gamma) {
      return [=](int, int tile, const v4i acc, const float4 sc, const float4 bi) {
        if (real) {
          float4* xp = reinterpret_cast<float4*>(xs + (lane & 15) * XS + 16 * tile + 4 * (lane >> 4));
          float4 x = *xp;
          x.x = fmaf(gamma, x.x, fmaf((float)acc[0], sc.x, bi.x));
          x.y = fmaf(gamma, x.y, fmaf((float)acc[1], sc.y, bi.y));
          x.z = fmaf(gamma, x.z, fmaf((float)acc[2], sc.z, bi.z));
          x.w = fmaf(gamma, x.w, fmaf((float)acc[3], sc.w, bi.w));
          *xp = x;
        }
      };
    };
    auto codes = [&](int, int tile, const v4i acc, const float4 sc, const float4 bi) {
      if (real) *(int*)(act + (lane & 15) * QS + 16 * tile + 4 * (lane >> 4)) = pack_codes<false>(acc, sc, bi);
    };
    auto relu_codes = [&](int, int tile, const v4i acc, const float4 sc, const float4 bi) {
      if (real) *(int*)(act + (lane & 15) * HS + 16 * tile + 4 * (lane >> 4)) = pack_codes<true>(acc, sc, bi);
    };
    const Blob lb = blob_rsrc<S, W4>(base), nb = blob_rsrc<S, W4>(next);
    const int cc = min(lane & 3, nc - 1), pp = lane >> 2;
    v4i kv[4];

    // self-attention: the cached keys of the wave's first unit go out before the LayerNorm and the projection
    if (wave < units) load_chunks<true>(kv, kc + (size_t)b0 * g.W * T * D, hs + i0 * hs_s, T, D, hd0 * dh + 16 * cc, t, 0, pp);
    norm(0, !(g.post && l == 0), H.sa_inv, g.post);
    linear<S, W4, S::kQkv, S::kO, 1, S::kEnd>(ring, arow, 0, lb, nb, more, wave, lane, codes);
    lds_barrier();
    for (int u = wave, i = i0, hd = hd0; u < units; u += WAVES) {
      const int8_t* qr = act + i * QS + hd * dh;
      const unsigned at = u == wave ? (unsigned)b0 * g.W * T * D : cache_at(i);
      if (u != wave) load_chunks<true>(kv, kc + at, hs + i * hs_s, T, D, hd * dh + 16 * cc, t, 0, pp);
      attend_row<true>(kv, kc + at, vc + at, hs + i * hs_s, T, D, hd * dh, t, dh, qr, D, H.sa_cqk, H.sa_cpv, pw, vt,
                       as + i * AS + hd * dh, lane);
      i += di;
      if ((hd += dhd) >= h) {
        hd -= h;
        ++i;
      }
    }
    // the new keys and values into the cache (no block reads position t of this step)
    for (int i = tid; i < rows * (D / 16); i += THREADS) {
      const int r = i / (D / 16), ch = i % (D / 16);
      const size_t o = ((size_t)(row0 + r) * T + t) * D + 16 * ch;
      *(v4i*)(kc + o) = *(const v4i*)(act + r * QS + D + 16 * ch);
      *(v4i*)(vc + o) = *(const v4i*)(act + r * QS + 2 * D + 16 * ch);
    }
    lds_barrier();
    linear<S, W4, S::kO, S::kCq, 1, S::kEnd>(ring, arow, 0, lb, nb, more, wave, lane, resid(H.sa_gamma));
    // cross-attention
    const int8_t* ck = ckv + (size_t)b0 * g.S * 2 * D + hd0 * dh;
    if (wave < units) load_chunks<false>(kv, ck, nullptr, 0, 2 * D, 16 * cc, n0, 0, pp);
    lds_barrier();
    norm(1, 1, H.ca_inv, g.post);
    linear<S, W4, S::kCq, S::kCo, 1, S::kEnd>(ring, arow, 0, lb, nb, more, wave, lane, codes);
    lds_barrier();
    int n = n0;
    for (int u = wave, i = i0, hd = hd0; u < units; u += WAVES) {
      if (u != wave) {
        const int b = (row0 + i) / g.W;
        n = keys_of(b);
        ck = ckv + (size_t)b * g.S * 2 * D + hd * dh;
        load_chunks<false>(kv, ck, nullptr, 0, 2 * D, 16 * cc, n, 0, pp);
      }
      attend_row<false>(kv, ck, ck + D, nullptr, 0, 2 * D, 0, n, dh, act + i * QS + hd * dh, D, H.ca_cqk, H.ca_cpv,
                        pw, vt, as + i * AS + hd * dh, lane);
      i += di;
      if ((hd += dhd) >= h) {
        hd -= h;
        ++i;
      }
    }
    lds_barrier();
    linear<S, W4, S::kCo, S::kW1, 1, S::kEnd>(ring, arow, 0, lb, nb, more, wave, lane, resid(H.ca_gamma));
    lds_barrier();
    // feed-forward
    norm(2, 1, H.ff_inv, g.post);
    const float4 ln_next = load_ln(next);
    linear<S, W4, S::kW1, S::kW2, 1, S::kEnd>(ring, arow, 0, lb, nb, more, wave, lane, relu_codes);
    store_ln(ln_next);
    lds_barrier();
    linear<S, W4, S::kW2, S::kEnd, 1, S::kEnd>(ring, hrow, 0, lb, nb, more, wave, lane, resid(H.ff_gamma));
    lds_barrier();
    base = next;
  }
  // the final LayerNorm (post-LN: the last feed-forward's): the output
  // projection's int8 input, and the residual rows
  if (wave < rows) {
    float gj[KQ], bj[KQ];
#pragma unroll
    for (int j = 0; j < KQ; ++j) {
      gj[j] = g.fin_ln.g[lane + 64 * j];
      bj[j] = g.fin_ln.b[lane + 64 * j];
    }
    float* xr = xs + wave * XS;
    const size_t o = (size_t)(row0 + wave) * D;
#pragma unroll
    for (int j = 0; j < KQ; ++j) g.x[o + lane + 64 * j] = xr[lane + 64 * j];
    norm_row<KQ>(xr, 1, gj, bj, g.eps, g.inv_fin, false, as + wave * AS, lane);
    wave_sync();
    for (int i = lane; i < D / 4; i += 64) *(int*)(g.out + o + 4 * i) = *(const int*)(as + wave * AS + 4 * i);
  }
}

template <int KQ, int FQ>
hipError_t launch_shape(const RowsParams& P, int blocks, hipStream_t s) {
  auto go = [&](auto kern) -> hipError_t {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kRowsMaxLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64 * Shape<KQ, FQ>::WAVES), P.l.total, s, P);
    return hipGetLastError();
  };
  return P.g.w4 ? go(k_dec_rows<KQ, FQ, true>) : go(k_dec_rows<KQ, FQ, false>);
}

template <int KQ>
hipError_t launch_kq(const RowsParams& P, int blocks, hipStream_t s) {
  return P.g.F == 2 * P.g.d ? launch_shape<KQ, 2 * KQ>(P, blocks, s) : launch_shape<KQ, 4 * KQ>(P, blocks, s);
}

// A blob from its parts, in one launch: block a < arrays copies a float array
// (block 0 also the scalars), the others 256 fragment chunks each: a lane's 16
// bytes (W4: 8) of tile t, slice j of a linear layer (launch_pack_fragments'
// order).
template <bool W4>
__global__ __launch_bounds__(256) void k_rows_pack(RowsPack p) {
  const int a = blockIdx.x, tid = threadIdx.x;
  if (a < p.arrays) {
    float* dst = reinterpret_cast<float*>(p.blob + p.off[a]);
    for (int i = tid; i < p.n[a]; i += 256) dst[i] = p.src[a][i];
    if (a == 0 && tid < 16) reinterpret_cast<float*>(p.blob)[tid] = p.hdr[tid];
    return;
  }
  unsigned c = (unsigned)(a - p.arrays) * 256 + tid;
  for (int i = 0; i < p.lins; ++i) {
    const RowsPack::Lin& L = p.lin[i];
    const unsigned ks = L.K / 64, chunks = L.N / 16 * ks * 64;
    if (c >= chunks) {
      c -= chunks;
      continue;
    }
    const unsigned lane = c % 64, j = c / 64 % ks, t = c / (64 * ks);
    const size_t at = (size_t)(16 * t + (lane & 15)) * L.K + 64 * j + 16 * (lane >> 4);  // code
    if constexpr (W4)
      *(uint2*)(p.blob + L.out + 8 * (size_t)c) = *(const uint2*)(L.W + at / 2);
    else
      *(int4*)(p.blob + L.out + 16 * (size_t)c) = *(const int4*)(L.W + at);
    return;
  }
}

}  // namespace

// Shapes the kernel is compiled for: the usual feed-forward ratios, heads of
// at most 64.
bool dec_rows_shape(int d, int dh, int F) {
  return (d == 64 || d == 128 || d == 256 || d == 384 || d == 512) && (F == 2 * d || F == 4 * d) && dh <= 64 &&
         dh % 16 == 0;
}

size_t dec_rows_blob_bytes(int d, int F, bool w4) { return rows_off(d, F, w4).bytes; }

hipError_t launch_rows_pack(RowsPack& p, const LinearDev* const* lin, int n, const unsigned* c, const unsigned* cols,
                            const unsigned* w, bool w4, hipStream_t s) {
  size_t chunks = 0;
  for (int i = 0; i < n; ++i)
    if (lin[i]) {
      rows_pack_add(p, lin[i]->scale, c[i], lin[i]->N);
      rows_pack_add(p, lin[i]->bias, c[i] + 4 * cols[i], lin[i]->N);
      p.lin[p.lins++] = RowsPack::Lin{w4 ? reinterpret_cast<const int8_t*>(lin[i]->w4) : lin[i]->w, lin[i]->N, lin[i]->K, w[i]};
      chunks += (size_t)lin[i]->N * lin[i]->K / 16;
    }
  const dim3 grid(p.arrays + (unsigned)((chunks + 255) / 256));
  if (w4)
    k_rows_pack<true><<<grid, dim3(256), 0, s>>>(p);
  else
    k_rows_pack<false><<<grid, dim3(256), 0, s>>>(p);
  return hipGetLastError();
}

// Reorder decoder layer L into its blob.  ln_self: the LayerNorm in front of
// the layer's Q/K/V projection (post-LN: the previous layer's last).
hipError_t launch_dec_rows_pack(const LayerDev& L, const LnDev& ln_self, bool post, bool w4, int8_t* blob,
                                hipStream_t s) {
  const int d = L.o.N, F = L.w1.N;
  const RowsOff O = rows_off(d, F, w4);
  const LinearDev* lin[6] = {&L.qkv, &L.o, &L.cq, &L.co, &L.w1, &L.w2};
  // post-LN: the rows in front of a sublayer are normalized by the sublayer before it
  const LnDev* ln[3] = {&ln_self, post ? &L.sa_ln : &L.ca_ln, post ? &L.ca_ln : &L.ff_ln};
  RowsPack p{};
  p.blob = blob;
  const float hdr[10] = {L.qkv.inv_in, L.cq.inv_in, L.w1.inv_in, L.sa_cqk,   L.sa_cpv,
                         L.ca_cqk,     L.ca_cpv,    L.sa_gamma,  L.ca_gamma, L.ff_gamma};
  for (int i = 0; i < 10; ++i) p.hdr[i] = hdr[i];
  for (int i = 0; i < 3; ++i) {
    rows_pack_add(p, ln[i]->g, O.ln[i], d);
    rows_pack_add(p, ln[i]->b, O.ln[i] + 4 * d, d);
  }
  return launch_rows_pack(p, lin, 6, O.c, O.n, O.w, w4, s);
}

hipError_t launch_dec_rows(const RowsArgs& args, hipStream_t s) {
  if ((size_t)args.R * args.T * args.d >> 31) return hipErrorInvalidValue;  // load_chunks' offsets
  if (args.R < 1 || args.t >= args.T || (args.t < 0 && !args.step) || !dec_rows_shape(args.d, args.dh, args.F))
    return hipErrorInvalidValue;
  RowsParams P{args, {}};
  const RowsPlan plan = rows_plan(RowsSizes{args.R, args.d, args.h, args.F, args.T, args.S, args.t});
  P.g.RB = plan.rows;
  P.l = plan.lds;
  if (P.l.total > kRowsMaxLds) return hipErrorInvalidValue;
  const int blocks = plan.blocks;
  switch (args.d) {
    case 64: return launch_kq<1>(P, blocks, s);
    case 128: return launch_kq<2>(P, blocks, s);
    case 256: return launch_kq<4>(P, blocks, s);
    case 384: return launch_kq<6>(P, blocks, s);
    default: return launch_kq<8>(P, blocks, s);
  }
}

}  // namespace mnmt

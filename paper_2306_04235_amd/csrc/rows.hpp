// rows.hpp -- device pieces of the row-wise kernels (decode_rows.hip,
// encode_rows.hip): a block takes a few rows through several linear layers,
// streaming the layers' weights in fragment order through its CU.
//
// A stream S describes the linear layers of one pass over a blob: d, F, the
// block's waves, C slices of 64 inputs per batch, kRing batches in flight per
// wave, kEnd batches in the pass, S::at(b) the place of batch b, and
// S::off(w4) the blob's byte offsets (scales and biases c[], columns n[],
// weights w[] of each linear layer, total bytes).
#pragma once

#include "blocks.hpp"

namespace mnmt {

// Where a batch of the stream lies: linear layer (0..5), the wave's tile, the
// tile's batch, slices per tile.
struct BatchAt {
  int lin, tile, ch, nch;
};
__host__ __device__ constexpr BatchAt batch_in(int lin, int b, int nch) { return BatchAt{lin, b / nch, b % nch, nch}; }

// The wave's weights in flight: batch b in slot b % kRing, with the tile's
// scale and bias of the lane's four columns beside its last batch.
template <class S, bool W4>
struct Ring {
  WFrag<W4> f[S::kRing][S::C];
  float4 sc[S::kRing], bi[S::kRing];
};

// A layer's blob as a buffer descriptor: a load's address is then the lane's
// offset plus scalars, with no vector address arithmetic per load, and loads
// past the blob return zero.
typedef __amdgpu_buffer_rsrc_t Blob;
template <class S, bool W4>
__device__ __forceinline__ Blob blob_rsrc(const int8_t* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(base), 0, S::off(W4).bytes, 0x00020000);
}

// Issue the loads of batch b (constant after unrolling; past the layer's last
// batch: the next layer's) into its slot.
template <class S, bool W4>
__device__ __forceinline__ void issue(Ring<S, W4>& r, int b, Blob layer, Blob next, int wave, int lane) {
  constexpr auto O = S::off(W4);
  const Blob base = b < S::kEnd ? layer : next;
  const int slot = b % S::kRing;
  const BatchAt at = S::at(b < S::kEnd ? b : b - S::kEnd);
  const int tile = wave + S::WAVES * at.tile;
  const unsigned w = O.w[at.lin] + ((unsigned)(tile * at.nch + at.ch) * S::C) * (W4 ? 512u : 1024u);
#pragma unroll
  for (int u = 0; u < S::C; ++u) {
    if constexpr (W4) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(base, 8 * lane, w + 512 * u, 0);
      r.f[slot][u].p = make_uint2(v[0], v[1]);
    } else {
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(base, 16 * lane, w + 1024 * u, 0);
      r.f[slot][u].v = v4i{(int)v[0], (int)v[1], (int)v[2], (int)v[3]};
    }
  }
  if (at.ch == at.nch - 1) {
    const unsigned c = O.c[at.lin] + 64 * tile, l = 16 * (lane >> 4);
    const auto x = __builtin_amdgcn_raw_buffer_load_b128(base, l, c, 0);
    const auto y = __builtin_amdgcn_raw_buffer_load_b128(base, l, c + 4 * O.n[at.lin], 0);
    r.sc[slot] = make_float4(__uint_as_float(x[0]), __uint_as_float(x[1]), __uint_as_float(x[2]), __uint_as_float(x[3]));
    r.bi[slot] = make_float4(__uint_as_float(y[0]), __uint_as_float(y[1]), __uint_as_float(y[2]), __uint_as_float(y[3]));
  }
}

// One linear layer: batches B0 .. B1 - 1 of the stream over the int8 rows in
// LDS (the lane's row of tile 0 and its chunk at arow; MT tiles of 16 rows,
// tile_bytes apart, against each weight fragment).  The weights are the A
// operand, so element i of lane l is column 4 (l / 16) + i of row l % 16: a
// lane finishes four consecutive columns of one row.  Batches from kMore on
// are only fetched if `more`.  epi(m, tile, acc, scale, bias).
template <class S, bool W4, int B0, int B1, int MT, int kMore, class Epi>
__device__ __forceinline__ void linear(Ring<S, W4>& r, const int8_t* arow, int tile_bytes, Blob layer, Blob next,
                                       bool more, int wave, int lane, Epi&& epi) {
  v4i acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = v4i{0, 0, 0, 0};
#pragma unroll
  for (int b = B0; b < B1; ++b) {
    const int slot = b % S::kRing;
    const BatchAt at = S::at(b);
#pragma unroll
    for (int u = 0; u < S::C; ++u)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        acc[m] = mfma16(r.f[slot][u].get(), *(const v4i*)(arow + m * tile_bytes + 64 * (at.ch * S::C + u)), acc[m]);
    const float4 sc = r.sc[slot], bi = r.bi[slot];
    if (b + S::kRing < kMore || more) issue(r, b + S::kRing, layer, next, wave, lane);
    asm volatile("" ::: "memory");  // (the loads stay here: the compiler would sink them to their use)
    if (at.ch == at.nch - 1) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        epi(m, wave + S::WAVES * at.tile, acc[m], sc, bi);
        acc[m] = v4i{0, 0, 0, 0};
      }
    }
  }
}

// Four requantized codes of one row (columns col .. col + 3) as one word.
template <bool RELU>
__device__ __forceinline__ int pack_codes(const v4i acc, const float4 sc, const float4 bi) {
  const float y[4] = {fmaf((float)acc[0], sc.x, bi.x), fmaf((float)acc[1], sc.y, bi.y),
                      fmaf((float)acc[2], sc.z, bi.z), fmaf((float)acc[3], sc.w, bi.w)};
  unsigned w = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w |= (unsigned)(uint8_t)code_of(RELU ? fmaxf(y[i], 0.0f) : y[i]) << (8 * i);
  return (int)w;
}

// LayerNorm (if do_ln) and quantization of the row x [d] in LDS by one wave,
// into the int8 row q; the normalized row replaces x if `replace`.
template <int KQ>
__device__ __forceinline__ void norm_row(float* x, int do_ln, const float (&gj)[KQ], const float (&bj)[KQ], float eps,
                                         float inv_s, bool replace, int8_t* q, int lane) {
  constexpr int D = 64 * KQ;
  float v[KQ];
#pragma unroll
  for (int j = 0; j < KQ; ++j) v[j] = x[lane + 64 * j];
  if (do_ln) ln_row<KQ>(v, gj, bj, D, eps);
#pragma unroll
  for (int j = 0; j < KQ; ++j) {
    q[lane + 64 * j] = code_of(v[j] * inv_s);
    if (replace) x[lane + 64 * j] = v[j];
  }
}

// The 4x4 byte transposes of a lane's 16-byte value chunks of four consecutive
// positions: word k of the result holds column k of the four positions.
__device__ __forceinline__ void transpose_chunks(const v4i (&v)[4], int (&w)[16]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const unsigned a0 = __builtin_amdgcn_perm((unsigned)v[1][k], (unsigned)v[0][k], 0x05010400u);
    const unsigned a1 = __builtin_amdgcn_perm((unsigned)v[1][k], (unsigned)v[0][k], 0x07030602u);
    const unsigned b0 = __builtin_amdgcn_perm((unsigned)v[3][k], (unsigned)v[2][k], 0x05010400u);
    const unsigned b1 = __builtin_amdgcn_perm((unsigned)v[3][k], (unsigned)v[2][k], 0x07030602u);
    w[4 * k] = (int)__builtin_amdgcn_perm(b0, a0, 0x05040100u);
    w[4 * k + 1] = (int)__builtin_amdgcn_perm(b0, a0, 0x07060302u);
    w[4 * k + 2] = (int)__builtin_amdgcn_perm(b1, a1, 0x05040100u);
    w[4 * k + 3] = (int)__builtin_amdgcn_perm(b1, a1, 0x07060302u);
  }
}

// the sum over the 4 lanes of a quad
__device__ __forceinline__ int quad_sum(int v) {
  v += __builtin_amdgcn_mov_dpp(v, 0xB1, 0xf, 0xf, false);  // lanes 1 0 3 2
  v += __builtin_amdgcn_mov_dpp(v, 0x4E, 0xf, 0xf, false);  // lanes 2 3 0 1
  return v;
}

}  // namespace mnmt

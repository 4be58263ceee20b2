// bf16 attention of short sequences (32 NRB keys, all of them in LDS): what the exact and the insert kernel share.
//
// A wave takes units of 32 query rows of one head, the next unit's rows on their way during the products of this one; the
// workgroup takes as many K/V heads ("tiles") as give its four waves a unit each (few tiles: a part of one tile's units each),
// copies their K and V once, and meets at one barrier.  All scores of a unit are in registers before the first weight is formed
// (S^T = K Q^T, a lane: 16 keys of one query row a block), so the softmax takes one pass and no rescaling, and the weights can
// be normalised before they are rounded.
// K and V are copied, permuted and read as in exact.hip.
#pragma once
#include "common.hpp"

namespace ac {

struct ShortArgs {
  const bf16_t *Q, *K, *V;   // [items][Lc][Hq | Hkv][S][D]
  bf16_t* O;
  const int32_t *row_sel, *key_len;   // by item, or nullptr
  int32_t Hq, Hkv, Lc;
  int32_t n_tiles;        // (item, layer, K/V head)
  int32_t tiles_per_wg;   // up to kShortTiles
  int32_t parts;          // workgroups that share a tile's units (tiles_per_wg is 1 then)
  int32_t xcd_bits;       // 3 if those get ids equal mod 8 (one XCD, one L2), else 0
  float scale_log2e;
};
constexpr int kShortTiles = 4;

inline size_t short_lds(const ShortArgs& a, int S, int D) {
  return ((size_t)2 * a.tiles_per_wg * S * D + 4 * 16 * kSmallOutStride) * sizeof(bf16_t);
}
// Tiles of a workgroup and parts of a tile (as many as the chip holds at once: a second round of workgroups takes longer than
// units one after the other: 192 tiles of 4 heads on one of 128 x 128, causal 21.3 us in four parts, 17.9 in two); the grid.
// In large launches of 32 rows a workgroup takes four units again, those of a tile on one XCD: they read and write closer together (K and V,
// which the others find in the L2, are few bytes there).  us per call, one workgroup a tile / so, exact: 8,192 tiles of eight heads on one K and V of 32 x 128
// 238 / 207 (228 in the resident kernel), 32,768 954 / 841; 2,048 of sixteen 100 / 99; 32 x 64, 8,192 of twelve 158 / 149, of eight 105 / 104, 4,096 47.5 / 48.4.
// With 64 rows and more it costs what it gains or more: 8,192 tiles of four heads of 64 x 128 246 / 254, inserted packed 280 / 305.
inline unsigned short_plan(ShortArgs& a, int S, int D) {
  const int units = a.Hq / a.Hkv * (S >> 5), slots = 256 * (D == 64 ? (S <= 64 ? 4 : 3) : S == 32 ? 3 : 2);
  a.tiles_per_wg = units < 4 ? 4 / units : 1;
  const int most = (units + 3) / 4, fit = slots / a.n_tiles;
  a.parts = fit < 1 ? 1 : fit < most ? fit : most;
  if (a.tiles_per_wg > 1) a.parts = 1;
  a.xcd_bits = 0;
  const size_t apart = (size_t)a.n_tiles * most;   // (a grid has 2^32 threads at most)
  if (S == 32 && units > 4 && units % 4 == 0 && apart >= (D == 64 ? 16384 : 8192) && apart < (size_t)1 << 23) {
    a.parts = most;
    a.xcd_bits = 3;
    return (unsigned)((size_t)((a.n_tiles + 7) / 8 * 8) * a.parts);
  }
  return (unsigned)((size_t)((a.n_tiles + a.tiles_per_wg - 1) / a.tiles_per_wg) * a.parts);
}

__device__ __forceinline__ int short_tile0(const ShortArgs& a) {   // first tile of the workgroup
  if (a.parts == 1) return (int)blockIdx.x * a.tiles_per_wg;   // (a division less in small launches)
  const unsigned group = (blockIdx.x >> a.xcd_bits) / a.parts;
  return (int)(group << a.xcd_bits | (blockIdx.x & ((1u << a.xcd_bits) - 1))) * a.tiles_per_wg;
}

struct ShortUnit { int t, head, rb, tile, b, len; };   // tile of the workgroup, head of all, 32-row block, tile of all, item, its keys

// NORM: weights are divided by their sum before they are rounded, else the result is.  weights(unit, block, w) sees the packed
// weights of a 32-key block, finish(unit, n) follows those of the n blocks that hold a visible key.
template <int D, bool CAUSAL, int NRB, bool NORM, typename Weights, typename Finish>
__device__ __forceinline__ void short_attention(const ShortArgs& a, bf16_t* smem, Weights weights, Finish finish) {
  constexpr int S = 32 * NRB, PPR = D / 8, NCOPY = S * PPR / kWave / 4;   // copy instructions per wave, tensor and tile
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int T = a.tiles_per_wg, g = a.Hq / a.Hkv, per = g * NRB;
  bf16_t* kb = smem;                          // [T][S][D]
  bf16_t* vb = smem + (size_t)T * S * D;      // [T][S][D]
  bf16_t* ost = smem + (size_t)2 * T * S * D + wave * (16 * kSmallOutStride);
  const int tile0 = short_tile0(a), part = a.parts == 1 ? 0 : (int)((blockIdx.x >> a.xcd_bits) % a.parts);
  // as a scalar that a vector instruction wrote (see exact.hip)
  const float scale = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.scale_log2e) + (lane & 0)));

  int len[kShortTiles];   // keys of the tiles, 0: nothing to do
  bool any = false;
#pragma unroll
  for (int t = 0; t < kShortTiles; ++t) {
    len[t] = 0;
    if (t < T && tile0 + t < a.n_tiles) {
      const int b = (tile0 + t) / (a.Hkv * a.Lc);
      if (!(a.row_sel && a.row_sel[b] >= 0)) {
        len[t] = a.key_len ? min(max(a.key_len[b], 1), S) : S;
        any = true;
      }
    }
  }
  if (!any) return;
  // (rows rotate with the head, so that the heavy ones under a causal mask fall to all waves in turn)
  auto unit = [&](int u) {
    ShortUnit w;
    w.t = u / per;
    w.head = u % per / NRB;
    w.rb = (u + w.head) % NRB;
    w.tile = tile0 + w.t;
    w.b = w.tile / (a.Hkv * a.Lc);
    w.head += w.tile % a.Hkv * g;
    w.len = w.t == 0 ? len[0] : w.t == 1 ? len[1] : w.t == 2 ? len[2] : len[3];
    return w;
  };
  auto row_at = [&](const ShortUnit& w) {   // first row of the unit in Q and O
    return ((size_t)(w.tile / a.Hkv) * a.Hq + w.head) * (size_t)(S * D) + 32 * w.rb * D;
  };
  struct Rows { u32x4 q[D / 16]; };
  auto load_q = [&](int u) {
    Rows r;
    const ShortUnit w = unit(u);
    if (w.len == 0) return r;
    const bf16_t* qrow = a.Q + row_at(w) + il * D + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) r.q[ks] = *reinterpret_cast<const u32x4*>(qrow + 16 * ks);
    return r;
  };
  const int share = a.parts > 1 ? (per + 4 * a.parts - 1) / (4 * a.parts) * 4 : T * per;   // units of the workgroup
  const int u_end = a.parts > 1 ? min(share * (part + 1), per) : T * per;
  int u = share * part + wave;
  Rows now;
  if (u < u_end) now = load_q(u);

  const int slot0 = kWave * wave + lane, crow = slot0 / PPR, cpos = slot0 % PPR;
  const unsigned koff0 = (unsigned)(crow * D + 8 * (cpos ^ k_piece_swizzle<D>(crow)));
  const unsigned voff0 = (unsigned)(crow * D + 8 * (cpos ^ v_piece_swizzle<D>(crow)));
#pragma unroll
  for (int t = 0; t < kShortTiles; ++t)
    if (len[t] > 0) {
      const bf16_t* K = a.K + (size_t)(tile0 + t) * (S * D);
      const bf16_t* V = a.V + (size_t)(tile0 + t) * (S * D);
#pragma unroll
      for (int i = 0; i < NCOPY; ++i) {
        __builtin_amdgcn_global_load_lds(K + (koff0 + 2048u * i), kb + t * (S * D) + kWave * 8 * (wave + 4 * i), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(V + (voff0 + 2048u * i), vb + t * (S * D) + kWave * 8 * (wave + 4 * i), 16, 0, 0);
      }
    }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  int koff[D / 16], voff[2][D / 32];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) koff[ks] = il * D + 8 * ((2 * ks + kh) ^ k_piece_swizzle<D>(il));
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      const int t = lane & 15, j = 4 * kh + 8 * half + (t >> 2), d0 = 32 * db + 16 * (il >> 4) + 4 * (t & 3);
      voff[half][db] = j * D + 8 * ((d0 >> 3) ^ v_piece_swizzle<D>(j)) + (d0 & 7);
    }

  for (; u < u_end; u += 4) {
    Rows next;
    if (u + 4 < u_end) next = load_q(u + 4);
    const ShortUnit w = unit(u);
    if (w.len > 0) {
      const bf16_t* k = kb + w.t * (S * D);
      const bf16_t* v = vb + w.t * (S * D);
      const int n = min(CAUSAL ? w.rb + 1 : NRB, (w.len + 31) >> 5);   // blocks that hold a visible key
      f32x16 s[NRB];
      float mx = -INFINITY;
#pragma unroll
      for (int jb = 0; jb < NRB; ++jb)
        if (jb < n) {
#pragma unroll
          for (int x = 0; x < 16; ++x) s[jb][x] = 0.f;
#pragma unroll
          for (int ks = 0; ks < D / 16; ++ks)
            s[jb] = mfma_bf16(*reinterpret_cast<const bf16x8*>(k + koff[ks] + 32 * jb * D), __builtin_bit_cast(bf16x8, now.q[ks]), s[jb]);
          if ((CAUSAL && jb == w.rb) || 32 * jb + 32 > w.len) {   // wave-uniform
            const int limit = (CAUSAL ? min(32 * w.rb + il, w.len - 1) : w.len - 1) - 32 * jb;
#pragma unroll
            for (int x = 0; x < 16; ++x)
              if (mfma_row(x, kh) > limit) s[jb][x] = -INFINITY;
          }
#pragma unroll
          for (int x = 0; x < 16; x += 2) mx = fmaxf(fmaxf(mx, s[jb][x]), s[jb][x + 1]);
        }
      const float m = max_with_other_half(mx) * scale;
      float sum = 0.f, inv = 1.f;
      if (NORM) {
#pragma unroll
        for (int jb = 0; jb < NRB; ++jb)
          if (jb < n)
#pragma unroll
            for (int x = 0; x < 16; ++x) {
              s[jb][x] = __builtin_amdgcn_exp2f(fmaf(s[jb][x], scale, -m));
              sum += s[jb][x];
            }
        inv = 1.0f / (sum + __shfl_xor(sum, 32));
      }
      f32x16 acc[D / 32];
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc[db][x] = 0.f;
#pragma unroll
      for (int jb = 0; jb < NRB; ++jb)
        if (jb < n) {
          u32x4 p[2];
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            const float e0 = s[jb][2 * x], e1 = s[jb][2 * x + 1];
            if (NORM) {
              p[x >> 2][x & 3] = pack_bf16(e0 * inv, e1 * inv);
            } else {   // the sum is that of the rounded weights, which V is multiplied with
              p[x >> 2][x & 3] = pack_bf16(__builtin_amdgcn_exp2f(fmaf(e0, scale, -m)), __builtin_amdgcn_exp2f(fmaf(e1, scale, -m)));
              const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
              const uint32_t pair = p[x >> 2][x & 3];
              sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), ones, sum, false);
            }
          }
          weights(w, jb, p);
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int db = 0; db < D / 32; ++db) {
              const int base = (32 * jb + 16 * s2) * D;
              const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (s16x4 __attribute__((address_space(3)))*)(v + voff[0][db] + base));
              const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (s16x4 __attribute__((address_space(3)))*)(v + voff[1][db] + base));
              const s16x8 op = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
              acc[db] = mfma_bf16(__builtin_bit_cast(bf16x8, op), __builtin_bit_cast(bf16x8, p[s2]), acc[db]);
            }
        }
      finish(w, n);
      store_tile_bf16_small<D>(acc, NORM ? 1.0f : 1.0f / (sum + __shfl_xor(sum, 32)), ost, a.O + row_at(w), lane);
    }
    now = next;
  }
}

}  // namespace ac

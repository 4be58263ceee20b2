// Database building on the device (Fig. 3, steps 2 and 3): the recompute branch of Algorithm 2
// for inputs that are to be remembered.  For every selected item the kernel computes
// O = softmax(scale * Q K^T) V like attention_exact, and ALSO writes the normalised map
// A = softmax(scale * Q K^T) of every (layer, head), rounded once to bf16, into the item's slot
// of the map store, in the store's layout, and copies the item's feature vector into the same
// slot of the feature store.  A later search that hits the slot makes
// attncache_apply reproduce this O from the stored map.
//
// The map has to be normalised before it is written, so the row statistics must be known before
// the first weight leaves: two passes over the keys.  Pass 1 forms the scores and keeps only the
// row maximum m and the row sum l of 2^(score - m); pass 2 forms the scores again, turns them
// into a = 2^(score - m) / l, rounds to bf16, stores them and multiplies the ROUNDED weights
// with V (so O is exactly what the stored map yields, up to summation order).  Same transposed
// products and register hand-over as the exact kernel: S^T = K Q^T (a lane holds 16 keys of one
// query row), O^T = V^T A^T with A taken from the first product's result registers.
// For S <= 128 K and V are staged in LDS once per group of query heads that share them and both
// passes of every head read them there; longer sequences stream 64-key chunks through two LDS
// stages, once per pass.
//
// Packed layout (see pack_maps_kernel): the result registers of one 32 x 32 score block map onto
// packed 16 x 32 blocks directly -- register group q (4 registers) of lane (row i, half kh) is
// elements 4 kh .. 4 kh + 3 of piece (16 q + i % 16), i.e. one 8-byte store per group, and the 32
// lanes of a 16-row half fill a contiguous 256-byte run.
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "short_tile.hpp"
#include "split_tile.hpp"
#include <type_traits>

namespace ac {

struct InsertArgs {
  const void *Q, *K, *V;
  void *O, *maps;
  const int32_t *slot, *row_sel, *key_len;
  const u32x4* feat;      // [B][feat_pieces] or nullptr
  u32x4* emb;             // the feature store, rows of feat_pieces
  int32_t feat_pieces;    // 16-byte pieces of a feature vector
  int32_t B, M, L, layer_begin, Lc, Hq, Hkv, S;
  int32_t n_tiles;   // KV groups: (item, layer, KV head)
  float scale_log2e;
};

// One workgroup = up to 128 query rows of one (item, layer, group of query heads that share K and V),
// walking the keys in chunks of 64 -- twice, see above.  K and V reach the matrix cores
// the way they do in the exact kernel: every chunk is copied global -> LDS directly (no data
// registers, no ALU work) into one of two stages, rows unpadded with the 16-byte pieces
// permuted (k_piece_swizzle, v_piece_swizzle), V^T fetched with the transposing LDS read.
//   RESIDENT (S <= 128): both chunks sit in the two stages for the whole tile and the workgroup
//   walks all g query heads of the group -- K and V come from HBM once per group, and after the
//   one barrier behind the copy the four waves never meet again.
//   Streaming (S > 128): the row blocks of all g heads of the group are units of 32 rows of one
//   head, numbered row block first, head second, and a workgroup takes four consecutive ones, one
//   per wave (g = 4: the same rows of all four heads).  Its waves see (nearly) the same keys, K and V
//   are copied once for all of them.  The fours are counted from the first rows, as in the exact
//   kernel (57 items x 12 heads, 160 x 128, causal: 42 us counted from the end, 38 so).
//   The copy of chunk c + 1 is in flight while chunk c is multiplied, one barrier per chunk;
//   the statistics pass needs no V and copies none.
// Chunks and blocks beyond the sentence's length are not multiplied: their weights are zeros.
// 16 items x 4 layers x 32 heads on 8 K and V, 288 x 128, causal, padded: 203 us per call with 128
// rows of one head per workgroup and all keys multiplied, 132 to 139 us so (several boxes),
// without an extra launch for the feature vectors (520 MB, 93 us at the copy rate).
constexpr int kIChunk = 64;   // keys per staged chunk
constexpr float kNoScore = -3.402823466e38f;

template <int D, bool CAUSAL, bool PACKED, bool RESIDENT>
__global__ __launch_bounds__(kThreads, (D == 64 ? 3 : 2)) void insert_bf16_kernel(const InsertArgs a) {
  constexpr int PPR = D / 8;                          // 16-byte pieces per row
  constexpr int NCOPY = kIChunk * PPR / kWave / 4;    // copy instructions per wave, tensor, chunk
  __shared__ __attribute__((aligned(16))) bf16_t kb0[kIChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t vb0[kIChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t kb1[kIChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t vb1[kIChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t ost_small[4 * 16 * kSmallOutStride];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int S = a.S, g = a.Hq / a.Hkv;

  // all workgroups of a KV group get ids equal mod 8 (one XCD, one L2), heaviest first.
  // RESIDENT (S <= 128): both chunks of K and V sit in the two stages for the whole tile and the
  // workgroup walks all g query heads that share them; between the one barrier after the copy
  // and the end of the tile the four waves never meet again.
  const int bid = blockIdx.x;
  const int n_units = RESIDENT ? 4 : g * (S >> 5), per_tile = (n_units + 3) >> 2;
  const int slot_id = bid >> 3;
  const int grp = slot_id / per_tile * 8 + (bid & 7);   // (item, layer, KV head)
  const int low = 4 * (per_tile - 1 - slot_id % per_tile), top = min(low + 3, n_units - 1);
  const int unit = RESIDENT ? wave : low + 3 - wave;
  if (grp >= a.n_tiles) return;
  const int kvh = grp % a.Hkv;
  const int l = (grp / a.Hkv) % a.Lc;
  const int b = grp / (a.Hkv * a.Lc);
  if (a.row_sel && a.row_sel[b] >= 0) return;
  const int len = a.key_len ? min(max(a.key_len[b], 1), S) : S;
  const int entry = a.slot ? a.slot[b] : -1;
  const bool keep = entry >= 0 && entry < a.M;   // anything else: compute O only
  // the item's first workgroup also copies its feature vector into the same slot
  if (a.feat && keep && l == 0 && kvh == 0 && slot_id % per_tile == 0)
    for (int p = tid; p < a.feat_pieces; p += kThreads)
      a.emb[(size_t)entry * a.feat_pieces + p] = a.feat[(size_t)b * a.feat_pieces + p];

  const size_t kv = (((size_t)b * a.Lc + l) * a.Hkv + kvh) * (size_t)S * D;
  const bf16_t* Ksrc = reinterpret_cast<const bf16_t*>(a.K) + kv;
  const bf16_t* Vsrc = reinterpret_cast<const bf16_t*>(a.V) + kv;
  // chunks the workgroup walks (the same for all four waves): up to its last diagonal, and only
  // those that hold a visible key
  const int last = RESIDENT || !CAUSAL ? S : 32 * (top / g + 1);
  const int n_chunk = (min(last, len) + kIChunk - 1) / kIChunk;
  const int r0 = RESIDENT ? 32 * unit : 32 * (min(unit, top) / g);
  const bool active = RESIDENT ? r0 < S : unit <= top;
  const int n32 = S >> 5;
  const size_t tile_elems = PACKED ? (size_t)packed_blocks(S, CAUSAL) * 512 : (size_t)S * S;
  bf16_t* At = nullptr;   // the current head's map in the store

  // ---- copies: instruction k = wave + 4 i fills LDS slots [64 k, 64 k + 64), slot = row * PPR +
  // position; from one instruction to the next the row grows by 256 / PPR, which leaves both
  // permutations unchanged.  Rows past the end of a ragged last chunk repeat its last row
  // (finite, and never multiplied: the block count below stops before them).
  const int slot0 = kWave * wave + lane;
  const int crow = slot0 / PPR, cpos = slot0 % PPR;
  const int kpiece = cpos ^ k_piece_swizzle<D>(crow);
  const int vpiece = cpos ^ v_piece_swizzle<D>(crow);
  auto copy_in = [&](bf16_t* to, const bf16_t* from, int piece, int c) {
    const int nj = min(kIChunk, S - c * kIChunk);
    const bf16_t* src = from + (size_t)c * kIChunk * D;
#pragma unroll
    for (int i = 0; i < NCOPY; ++i) {
      const int rr = min(crow + (256 / PPR) * i, nj - 1);
      __builtin_amdgcn_global_load_lds(src + (size_t)rr * D + 8 * piece, to + kWave * 8 * (wave + 4 * i), 16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto copy_k = [&](bf16_t* kb, int c) { copy_in(kb, Ksrc, kpiece, c); };
  auto copy_v = [&](bf16_t* vb, int c) { copy_in(vb, Vsrc, vpiece, c); };
  // this wave's copies have landed (they are counted like loads), then everybody's; the
  // barrier also retires the stage that the next copy overwrites
  auto publish = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };

  // ---- operand addresses (elements, relative to a stage), as in the exact kernel
  int koff[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) koff[ks] = il * D + 8 * ((2 * ks + kh) ^ k_piece_swizzle<D>(il));
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  int voff[2][D / 32];
  {
    const int t = lane & 15;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        const int j = 4 * kh + 8 * half + (t >> 2);
        const int d0 = 32 * db + 16 * (il >> 4) + 4 * (t & 3);
        voff[half][db] = j * D + 8 * ((d0 >> 3) ^ v_piece_swizzle<D>(j)) + (d0 & 7);
      }
  }
  // V^T operand of contraction step s2 of key block jb: slot e of lane half kh is key
  // 16 s2 + 8 (e / 4) + 4 kh + e % 4 of the block, where the first product left the scores
  auto vop = [&](const bf16_t* vb, int db, int jb, int s2) {
    const int base = (32 * jb + 16 * s2) * D;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(vb + voff[0][db] + base));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(vb + voff[1][db] + base));
    s16x8 w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, w);
  };

  u32x4 q[D / 16];
  // 32-key blocks of a row of this wave's maps, and those of chunk c that hold a visible key
  const int row_blocks = CAUSAL ? (r0 >> 5) + 1 : n32;
  auto blocks = [&](int c) {
    if (!active) return 0;
    return max(min(min(2, row_blocks - 2 * c), (len - c * kIChunk + 31) >> 5), 0);
  };
  // scores^T of key block jb of the staged chunk c (keys beyond the diagonal or in the padding
  // hidden; the first block of a row always has a visible key, so the running maximum is
  // finite from then on)
  auto scores = [&](const bf16_t* kb, int c, int jb) {
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      s = mfma_bf16(*reinterpret_cast<const bf16x8*>(kb + koff[ks] + 32 * jb * D),
                    __builtin_bit_cast(bf16x8, q[ks]), s);
    const int j00 = c * kIChunk + 32 * jb;
    if ((CAUSAL && j00 == r0) || j00 + 32 > len) {   // wave-uniform: most blocks skip the tests
      int limit = len - 1 - j00;
      if (CAUSAL) limit = min(limit, r0 + il - j00);
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (mfma_row(v, kh) > limit) s[v] = -INFINITY;
    }
    return s;
  };

  // Every lane has the running maximum and the sum of ITS keys of a row (half of them); the halves meet between the passes.
  // (The lowest finite value stands for "none yet": a lane may see no key in the first blocks.)
  float m_run = kNoScore, l_run = 0.f, inv_l = 0.f;
  f32x16 acc[D / 32];
  // where register group q4 (scores 4 q4 .. 4 q4 + 3 of this lane) of 32-key block kb goes
  const int r16 = (r0 >> 4) + (il >> 4);
  auto map_piece = [&](int kb, int q4) -> u32x2* {
    if (PACKED) {
      const int blk = (CAUSAL ? packed_prefix(r16) : r16 * n32) + kb;
      return reinterpret_cast<u32x2*>(At + (size_t)blk * 512 + (16 * q4 + (il & 15)) * 8 + 4 * kh);
    }
    return reinterpret_cast<u32x2*>(At + (size_t)(r0 + il) * S + 32 * kb + 8 * q4 + 4 * kh);
  };

  // First pass: row maximum m (log2 domain, scale folded in) and row sum l of 2^(score - m).
  auto note = [&](float mx, auto sum) {
    const float m_new = fmaxf(m_run, mx * a.scale_log2e);
    l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_new) + sum(m_new);
    m_run = m_new;
  };
  auto largest = [](const f32x16& s) {
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    return mx;
  };
  auto sum_of = [&](const f32x16& s, float m) {
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(fmaf(s[v], a.scale_log2e, -m));
    return sum;
  };
  // Second pass: normalised weights 2^(score - m) / l, rounded, stored, multiplied with V.  (log2 l is not added to m: the rounding of
  // m is the same in l and cancels, that of the sum would not: rows of scores around 1e6 added up to anything from 0.96 to 1.04.)
  auto weigh = [&](const f32x16& s, const bf16_t* vb, int kb32, int jb) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      u32x4 pw;
#pragma unroll
      for (int w = 0; w < 4; ++w)
        pw[w] = pack_bf16(__builtin_amdgcn_exp2f(fmaf(s[8 * s2 + 2 * w], a.scale_log2e, -m_run)) * inv_l,
                          __builtin_amdgcn_exp2f(fmaf(s[8 * s2 + 2 * w + 1], a.scale_log2e, -m_run)) * inv_l);
      if (keep) {
        if constexpr (PACKED) {   // 256-byte runs either way
          *map_piece(kb32, 2 * s2) = u32x2{pw.x, pw.y};
          *map_piece(kb32, 2 * s2 + 1) = u32x2{pw.z, pw.w};
        } else {
          // The lane halves exchange, so that the lower one has all eight columns of group 2 s2 and the
          // upper one those of the next: rows get 16 instead of 8 bytes at a time (160 x 12 heads of
          // 512 x 128, causal, padded: 582 -> 484 us).
          uint32_t x = pw.x, y = pw.y, z = pw.z, w = pw.w;
          swap_halves(x, z);
          swap_halves(y, w);
          *reinterpret_cast<u32x4*>(map_piece(kb32, 2 * s2 + kh) - kh) = u32x4{x, y, z, w};
        }
      }
      const bf16x8 pop = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
      for (int db = 0; db < D / 32; ++db) acc[db] = mfma_bf16(vop(vb, db, jb, s2), pop, acc[db]);
    }
  };
  // one staged chunk
  auto chunk = [&](const bf16_t* kb, const bf16_t* vb, int c, const bool SECOND)
                   __attribute__((always_inline)) {
    const int nblk = blocks(c);
    for (int jb = 0; jb < nblk; ++jb) {
      const f32x16 s = scores(kb, c, jb);
      if (!SECOND) note(largest(s), [&](float m) { return sum_of(s, m); });
      else weigh(s, vb, 2 * c + jb, jb);
    }
  };
  auto join_halves = [&]() {
    const float m = max_with_other_half(m_run), l = l_run * __builtin_amdgcn_exp2f(m_run - m);
    inv_l = 1.0f / (l + __shfl_xor(l, 32));
    m_run = m;
  };
  // All chunks of the row block, chunk c in stage c & 1; two per trip so that the stages are named statically (the
  // compiler then knows that the copy in flight and the reads of the other stage do not meet).  The second pass takes them
  // from the last to the first: K of the last two is still there, and their V arrives under the end of the first pass.
  auto both_passes = [&]() __attribute__((always_inline)) {
    auto copy_last_v = [&]() {
      if ((n_chunk - 1) & 1) {
        copy_v(vb1, n_chunk - 1);
        copy_v(vb0, n_chunk - 2);
      } else {
        copy_v(vb0, n_chunk - 1);
        if (n_chunk > 1) copy_v(vb1, n_chunk - 2);
      }
    };
    copy_k(kb0, 0);
    publish();
    int c = 0;
    for (; c + 1 < n_chunk; c += 2) {
      copy_k(kb1, c + 1);
      chunk(kb0, vb0, c, false);
      publish();
      if (c + 2 < n_chunk) copy_k(kb0, c + 2);
      else copy_last_v();
      chunk(kb1, vb1, c + 1, false);
      publish();
    }
    if (c < n_chunk) {   // odd count: the last chunk sits in the first stage
      copy_last_v();
      chunk(kb0, vb0, c, false);
      publish();
    }
    join_halves();
    c = n_chunk - 1;
    if (!(c & 1)) {
      chunk(kb0, vb0, c, true);
      if (c >= 2) {
        publish();
        copy_k(kb0, c - 2);
        copy_v(vb0, c - 2);
      }
      --c;
    }
    for (; c > 0; c -= 2) {
      chunk(kb1, vb1, c, true);
      if (n_chunk > 2) publish();
      if (c >= 3) {
        copy_k(kb1, c - 2);
        copy_v(vb1, c - 2);
      }
      chunk(kb0, vb0, c - 1, true);
      if (c >= 3) {
        publish();
        copy_k(kb0, c - 3);
        copy_v(vb0, c - 3);
      }
    }
  };

  if (RESIDENT) {
    copy_k(kb0, 0);
    copy_v(vb0, 0);
    if (n_chunk > 1) {
      copy_k(kb1, 1);
      copy_v(vb1, 1);
    }
    publish();
  }
  const int n_heads = RESIDENT ? g : 1;   // streaming: one unit per wave
  for (int hl = 0; hl < n_heads; ++hl) {
    const int h = kvh * g + (RESIDENT ? hl : min(unit, top) % g);
    const size_t qo = (((size_t)b * a.Lc + l) * a.Hq + h) * (size_t)S * D;
    At = reinterpret_cast<bf16_t*>(a.maps) +
         (((size_t)(keep ? entry : 0) * a.L + (a.layer_begin + l)) * a.Hq + h) * tile_elems;
    if (active) {
      const bf16_t* qrow = reinterpret_cast<const bf16_t*>(a.Q) + qo + (size_t)(r0 + il) * D + 8 * kh;
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) q[ks] = *reinterpret_cast<const u32x4*>(qrow + 16 * ks);
    }
    m_run = kNoScore;
    l_run = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;

    if (RESIDENT) {
      chunk(kb0, vb0, 0, false);
      if (n_chunk > 1) chunk(kb1, vb1, 1, false);
      join_halves();
      chunk(kb0, vb0, 0, true);
      if (n_chunk > 1) chunk(kb1, vb1, 1, true);
    } else {
      both_passes();
    }

    if (active) {
      // Zeros: blocks in the padding, and in a dense causal map those right of the diagonal block
      // (the packed layout does not store them)
      if (keep) {
        const int end = PACKED ? row_blocks : n32;
        for (int kb = min(row_blocks, (len + 31) >> 5); kb < end; ++kb)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) *map_piece(kb, q4) = u32x2{0u, 0u};
      }
      // the result leaves through the wave's small buffer: K and V stay where they are
      bf16_t* Oh = reinterpret_cast<bf16_t*>(a.O) + qo + (size_t)r0 * D;
      store_tile_bf16_small<D>(acc, 1.0f, ost_small + wave * (16 * kSmallOutStride), Oh, lane);
    }
  }
}

// The same for a launch that leaves the chip idle: ALL waves of a workgroup share one unit of 32 rows,
// wave w takes the 32-key blocks w, w + NW, ... of both passes.  The statistics of the waves meet
// between the passes, their partial outputs at the end.
template <int D, bool CAUSAL, bool PACKED>
__global__ __launch_bounds__(kThreads, 2) void insert_bf16_split_kernel(const InsertArgs a) {
  constexpr int NW = kThreads / kWave;
  // the waves' V tiles (half of it), and at the end their partial results
  __shared__ __attribute__((aligned(16))) f32x4 smem[NW * (D / 8) * kWave];
  __shared__ float ms[NW][32], ls[NW][32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int S = a.S, heads = a.n_tiles / a.Hkv * a.Hq, n32 = S >> 5;
  // heaviest row blocks first, neighbouring workgroups (and so the XCDs) on different heads
  const int block = n32 - 1 - blockIdx.x / heads, u = blockIdx.x % heads;   // u: (item, layer, head)
  const int h = u % a.Hq, bl = u / a.Hq, l = bl % a.Lc, b = bl / a.Lc;
  if (a.row_sel && a.row_sel[b] >= 0) return;
  const int len = a.key_len ? min(max(a.key_len[b], 1), S) : S;
  const int entry = a.slot ? a.slot[b] : -1;
  const bool keep = entry >= 0 && entry < a.M;   // anything else: compute O only
  // the item's first workgroup also copies its feature vector into the same slot
  if (a.feat && keep && l == 0 && h == 0 && block == n32 - 1)
    for (int p = tid; p < a.feat_pieces; p += kThreads)
      a.emb[(size_t)entry * a.feat_pieces + p] = a.feat[(size_t)b * a.feat_pieces + p];

  const size_t kv = ((size_t)bl * a.Hkv + h / (a.Hq / a.Hkv)) * (size_t)S * D;
  const size_t at = ((size_t)u * S + 32 * block) * D;
  const size_t tile_elems = PACKED ? (size_t)packed_blocks(S, CAUSAL) * 512 : (size_t)S * S;
  bf16_t* At = reinterpret_cast<bf16_t*>(a.maps) +
               (((size_t)(keep ? entry : 0) * a.L + (a.layer_begin + l)) * a.Hq + h) * tile_elems;
  const int row_blocks = CAUSAL ? block + 1 : n32;
  const int n_keys = min(row_blocks, (len + 31) >> 5);   // key blocks that hold a visible key
  const int r16 = 2 * block + (il >> 4);
  auto map_piece = [&](int kb, int q4) -> u32x2* {   // scores 4 q4 .. 4 q4 + 3 of this lane, key block kb
    if (PACKED) {
      const int blk = (CAUSAL ? packed_prefix(r16) : r16 * n32) + kb;
      return reinterpret_cast<u32x2*>(At + (size_t)blk * 512 + (16 * q4 + (il & 15)) * 8 + 4 * kh);
    }
    return reinterpret_cast<u32x2*>(At + (size_t)(32 * block + il) * S + 32 * kb + 8 * q4 + 4 * kh);
  };
  SplitOperands<D> t(reinterpret_cast<const bf16_t*>(a.K) + kv, reinterpret_cast<const bf16_t*>(a.V) + kv,
                     reinterpret_cast<bf16_t*>(smem) + wave * 32 * D, lane);
  auto hide = [&](f32x16& s, int blk) {
    if ((CAUSAL && blk == block) || 32 * blk + 32 > len) {   // wave-uniform: most blocks skip the tests
      const int limit = (CAUSAL ? min(len - 1, 32 * block + il) : len - 1) - 32 * blk;
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (mfma_row(x, kh) > limit) s[x] = -INFINITY;
    }
  };
  t.load_q(reinterpret_cast<const bf16_t*>(a.Q) + at);
  if (wave < n_keys) {
    t.load_k(wave);
    t.load_v(wave);
  }
  // zeros: blocks in the padding, and in a dense causal map those right of the diagonal block
  if (keep)
    for (int kb = n_keys + wave; kb < (PACKED ? row_blocks : n32); kb += NW)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) *map_piece(kb, q4) = u32x2{0u, 0u};

  float m = -INFINITY, sum = 0.f;
  for (int blk = wave; blk < n_keys; blk += NW) {
    f32x16 s = t.scores();
    t.load_k(blk + NW < n_keys ? blk + NW : wave);   // the last trip: the second pass's first block
    hide(s, blk);
    float mx = s[0];
#pragma unroll
    for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[x]);
    const float m_new = fmaxf(m, max_with_other_half(mx) * a.scale_log2e);
    const float ref = m_new == -INFINITY ? 0.f : m_new;   // no finite score so far
    float part = 0.f;
#pragma unroll
    for (int x = 0; x < 16; ++x) part += __builtin_amdgcn_exp2f(fmaf(s[x], a.scale_log2e, -ref));
    sum = sum * (m_new > m ? __builtin_amdgcn_exp2f(m - m_new) : 1.f) + part;
    m = m_new;
  }
  sum += __shfl_xor(sum, 32);
  if (kh == 0) {
    ms[wave][il] = m;
    ls[wave][il] = sum;
  }
  __syncthreads();
  float top = -INFINITY, total = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) top = fmaxf(top, ms[w][il]);
#pragma unroll
  for (int w = 0; w < NW; ++w)
    total = fmaf(ls[w][il], ms[w][il] < top ? __builtin_amdgcn_exp2f(ms[w][il] - top) : 1.f, total);
  const float inv = 1.0f / total;

  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[db][x] = 0.f;
  for (int blk = wave; blk < n_keys; blk += NW) {
    f32x16 s = t.scores();
    const bool more = blk + NW < n_keys;
    if (more) t.load_k(blk + NW);
    t.stage_v();
    if (more) t.load_v(blk + NW);
    wave_lds_fence();
    hide(s, blk);
#pragma unroll
    for (int x = 0; x < 16; ++x) s[x] = __builtin_amdgcn_exp2f(fmaf(s[x], a.scale_log2e, -top)) * inv;
    u32x4 p[2];
#pragma unroll
    for (int w = 0; w < 8; ++w) p[w >> 2][w & 3] = pack_bf16(s[2 * w], s[2 * w + 1]);
    if (keep)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *map_piece(blk, q4) = q4 & 1 ? u32x2{p[q4 >> 1].z, p[q4 >> 1].w} : u32x2{p[q4 >> 1].x, p[q4 >> 1].y};
    t.weights_v(acc, p);
    wave_lds_fence();   // the tile is read before the next block's rows are written
  }
  __syncthreads();   // V tiles are no longer read
  split_store<D, NW>(acc, 1.0f, 1.0f, smem, reinterpret_cast<bf16_t*>(a.O) + at, wave, lane);
}

template <int D, bool CAUSAL, bool PACKED>
static hipError_t launch_insert_short(const InsertArgs& a, hipStream_t stream);

template <int D, bool CAUSAL, bool PACKED>
static hipError_t launch_insert_t(const InsertArgs& a, dim3 grid, hipStream_t stream) {
  const int g = a.Hq / a.Hkv;
  const size_t units = (size_t)(a.n_tiles / a.Hkv) * a.Hq * (a.S / 32);
  // Up to 128 rows: one pass over the keys (below), but in small launches one unit per workgroup if heads share K and V or there are more than
  // 64 rows, else two passes.  The lines are where the workgroups of those begin a second round.  us per call, split or two passes / one: two heads on one K
  // and V, 32 x 64 (192 units) 4.7 / 4.8, (320) 5.7 / 5.0, 64 x 64 (256) 5.1 / 5.7, (320) 5.9 / 5.7, 64 x 128 (256) 6.6 / 6.8, (320) 9.3 / 7.0, 96 x 128
  // (240) 7.0 / 7.6, (288) 9.2 / 7.7, 128 x 128 (256) 7.5 / 8.6, (320) 9.6 / 8.7, 96 x 64 (480) 6.6 / 6.5, (528) 9.3 / 6.6, 128 x 64 (512) 6.9 / 7.2,
  // (576) 10.7 / 7.3; four and eight alike; one head each, 32 x 64 (768) 5.7 / 5.7, (776) 7.5 / 5.7, 32 x 128 (512) 6.0 / 6.6, (520) 8.9 / 6.7, 64 x 64
  // (1,536) 7.0 / 7.7, (1,552) 9.7 / 7.8, 64 x 128 (1,024) 7.8 / 8.2, (1,040) 11.9 / 9.6, 96 x 128 (768) 8.0 / 7.7, (1,032) 9.5 / 9.2, 128 x 128 (1,024) 9.9 /
  // 9.5, (1,152) 11.3 / 11.5, (1,600) 14.8 / 13.9; 64 x 16 x 32 heads of 32 x 64 (49,152) 295 / 163, of 64 x 64 204 / 170, 32 on 8 of 128 x 128 262 / 249.
  const size_t few = g > 1 ? (a.S >= 96 && D == 64 ? 512 : 256) : a.S <= 64 ? (D == 64 ? 24 : 16) * a.S : 1024;
  // Rows of dense maps, 96 and more of them, are written in shorter runs by the units of one pass than by two passes over a whole tile, which
  // shows where every head has its own K and V (two passes / one: causal, 128 x 64, 512 heads 11.9 / 12.0, 600 13.5 / 16.3, 4,096 84 / 96, 16,384 308 / 385;
  // 96 x 64, 4,096 46.8 / 45.1, 6,000 81 / 85, 16,384 215 / 226; 96 x 128, 1,488 33.7 / 33.4, 6,000 134 / 143, 16,384 352 / 386; 128 x 128, 1,488 44.0 / 42.6, 2,992
  // 96 / 103, 16,384 478 / 528; not causal, 128 x 128, 2,992 94 / 100, 16,384 485 / 513, 128 x 64, 6,000 115 / 114, 32,768 606 / 581, 96 x 64 alike).  With
  // two heads on a K and V: causal, 128 x 64, 512 heads 13.0 / 12.4, 592 15.5 / 16.6, 1,488 23.0 / 26.1, 4,096 55.5 / 57.7, 6,000 118 / 111, 16,384 296 / 281; 64 x
  // 128, 8,192 96 / 96, 32,768 364 / 374, 65,536 719 / 753; four of 128 x 64 2,976 38.7 / 39.8, 5,984 121 / 112, two of 96 x 64 6,000 55.9 / 53.0, of
  // 128 x 128 2,992 82.7 / 79.0.  So do packed maps of 128 x 128, but only in very large launches of one or two heads on a K and V (32,768 heads
  // 852 / 874, 24,576 651 / 639; 16,384 of two 713 / 746, 8,192 361 / 363; of four 1,282 / 1,287, of eight 8,192 1,216 / 1,188).
  const bool slower = PACKED                ? CAUSAL && D == 128 && a.S == 128 && g <= 2 && units > 100000
                      : g == 1 && a.S >= 96 ? (CAUSAL || D == 128) && units > (D == 128 ? 10000 : a.S == 128 ? 2100 : 14000)
                      : g == 2 && D == 64   ? CAUSAL && a.S == 128 && units > 2100 && units <= 20000
                                            : g == 2 && a.S == 64 && units > 50000;
  if (a.S <= kChunk && units > few && !slower) return launch_insert_short<D, CAUSAL, PACKED>(a, stream);
  // Else one unit per workgroup while that leaves room on the chip (beyond, K and V, which only the other kernel shares between rows, cost
  // more).  us per call, split / not: 8 heads of 1024 x 128 causal (256 units) 22.9 / 43.8, 32 of 512 x 128 (512) 19.9 / 25.3, 108 of 160 x 128
  // (540) 13.0 / 11.9, 72 of it dense (360) 12.5 / 11.4, 96 of 288 x 64 (864) 13.2 / 15.4, 64 of 512 x 64 (1,024) 20.4 / 20.9; 64 on 16 K and V of
  // 128 x 128 (256) 7.3 / 22.3, 8 on 8 of 128 x 128 (32) 6.8 / 8.1, 128 on 128 (512) 10.2 / 8.8, 256 on 256 of 32 x 64 (256) 5.0 / 4.4.
  const size_t most = a.S > 128 ? (CAUSAL ? (D == 64 ? 768 : 480) : (D == 64 ? 448 : 320)) : g > 1 ? few : a.S > 64 ? 128 : 0;
  if (units <= most) {
    hipLaunchKernelGGL((insert_bf16_split_kernel<D, CAUSAL, PACKED>), dim3((unsigned)units), dim3(kThreads), 0, stream, a);
    return hipGetLastError();
  }
  if (a.S <= kChunk)
    hipLaunchKernelGGL((insert_bf16_kernel<D, CAUSAL, PACKED, true>), grid, dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((insert_bf16_kernel<D, CAUSAL, PACKED, false>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

// Sequences of up to 128 rows (short_tile.hpp): the scores of a row are all there before its first weight is, so one pass does.
template <int D, bool CAUSAL, bool PACKED, int NRB>
__global__ __launch_bounds__(kThreads, 2) void insert_bf16_short_kernel(const ShortArgs s, const InsertArgs a) {
  constexpr int S = 32 * NRB;
  extern __shared__ __attribute__((aligned(16))) unsigned char short_smem[];
  const int lane = threadIdx.x & 63, il = lane & 31, kh = lane >> 5;
  const size_t tile_elems = PACKED ? (size_t)packed_blocks(S, CAUSAL) * 512 : (size_t)S * S;
  auto slot_of = [&](int b) {   // -1: compute O only
    const int entry = a.slot ? a.slot[b] : -1;
    return entry < a.M ? entry : -1;
  };
  int slots[kShortTiles];   // of the workgroup's tiles
#pragma unroll
  for (int t = 0; t < kShortTiles; ++t) {
    const int tile = short_tile0(s) + t, b = tile / (s.Hkv * s.Lc);
    slots[t] = -1;
    if (t >= s.tiles_per_wg || tile >= s.n_tiles) continue;
    slots[t] = slot_of(b);
    // the item's first workgroup also copies its feature vector into the same slot
    if (a.feat && (blockIdx.x >> s.xcd_bits) % s.parts == 0 && tile % (s.Hkv * s.Lc) == 0 && slots[t] >= 0 && !(a.row_sel && a.row_sel[b] >= 0))
      for (int p = threadIdx.x; p < a.feat_pieces; p += kThreads)
        a.emb[(size_t)slots[t] * a.feat_pieces + p] = a.feat[(size_t)b * a.feat_pieces + p];
  }
  auto slot_at = [&](int t) { return t == 0 ? slots[0] : t == 1 ? slots[1] : t == 2 ? slots[2] : slots[3]; };
  auto map_of = [&](const ShortUnit& w, int entry) {
    const int l = w.tile / s.Hkv % s.Lc;
    return reinterpret_cast<bf16_t*>(a.maps) + (((size_t)entry * a.L + (a.layer_begin + l)) * a.Hq + w.head) * tile_elems;
  };
  // where register group q4 (scores 4 q4 .. 4 q4 + 3 of this lane) of key block kb goes
  auto map_piece = [&](const ShortUnit& w, bf16_t* At, int kb, int q4) -> u32x2* {
    const int r16 = 2 * w.rb + (il >> 4);
    if (PACKED)
      return reinterpret_cast<u32x2*>(At + (size_t)((CAUSAL ? packed_prefix(r16) : r16 * NRB) + kb) * 512 +
                                      (16 * q4 + (il & 15)) * 8 + 4 * kh);
    return reinterpret_cast<u32x2*>(At + (size_t)(32 * w.rb + il) * S + 32 * kb + 8 * q4 + 4 * kh);
  };
  short_attention<D, CAUSAL, NRB, true>(
      s, reinterpret_cast<bf16_t*>(short_smem),
      [&](const ShortUnit& w, int jb, const u32x4 (&p)[2]) {
        const int entry = slot_at(w.t);
        if (entry < 0) return;
        bf16_t* At = map_of(w, entry);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          if constexpr (PACKED) {
            *map_piece(w, At, jb, 2 * s2) = u32x2{p[s2].x, p[s2].y};
            *map_piece(w, At, jb, 2 * s2 + 1) = u32x2{p[s2].z, p[s2].w};
          } else {   // 16 bytes a row, as above
            uint32_t x = p[s2].x, y = p[s2].y, z = p[s2].z, v = p[s2].w;
            swap_halves(x, z);
            swap_halves(y, v);
            *reinterpret_cast<u32x4*>(map_piece(w, At, jb, 2 * s2 + kh) - kh) = u32x4{x, y, z, v};
          }
        }
      },
      [&](const ShortUnit& w, int n) {   // zeros: blocks in the padding and, in a dense causal map, right of the diagonal block
        const int entry = slot_at(w.t);
        if (entry < 0) return;
        bf16_t* At = map_of(w, entry);
        for (int kb = n; kb < (PACKED && CAUSAL ? w.rb + 1 : NRB); ++kb)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) *map_piece(w, At, kb, q4) = u32x2{0u, 0u};
      });
}

template <int D, bool CAUSAL, bool PACKED>
static hipError_t launch_insert_short(const InsertArgs& a, hipStream_t stream) {
  ShortArgs s;
  s.Q = static_cast<const bf16_t*>(a.Q); s.K = static_cast<const bf16_t*>(a.K); s.V = static_cast<const bf16_t*>(a.V);
  s.O = static_cast<bf16_t*>(a.O); s.row_sel = a.row_sel; s.key_len = a.key_len;
  s.Hq = a.Hq; s.Hkv = a.Hkv; s.Lc = a.Lc; s.n_tiles = a.n_tiles; s.scale_log2e = a.scale_log2e;
  const dim3 grid(short_plan(s, a.S, D));
  const size_t lds = short_lds(s, a.S, D);
  auto go = [&](auto nrb) {
    constexpr auto kernel = &insert_bf16_short_kernel<D, CAUSAL, PACKED, decltype(nrb)::value>;
    const hipError_t e = ensure_lds<kernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), lds, stream, s, a);
    return hipGetLastError();
  };
  return a.S == 32   ? go(std::integral_constant<int, 1>{})
         : a.S == 64 ? go(std::integral_constant<int, 2>{})
         : a.S == 96 ? go(std::integral_constant<int, 3>{})
                     : go(std::integral_constant<int, 4>{});
}

template <int D>
static hipError_t launch_insert_d(const InsertArgs& a, dim3 grid, bool causal, bool packed,
                                       hipStream_t stream) {
  if (causal) return packed ? launch_insert_t<D, true, true>(a, grid, stream)
                            : launch_insert_t<D, true, false>(a, grid, stream);
  return packed ? launch_insert_t<D, false, true>(a, grid, stream)
                : launch_insert_t<D, false, false>(a, grid, stream);
}

// Host launcher.  Shapes were validated by the caller (api.hip).
hipError_t launch_insert(const InsertLaunch& p, hipStream_t stream) {
  if (p.B == 0 || p.Lc == 0) return hipSuccess;
  InsertArgs a;
  a.Q = p.Q; a.K = p.K; a.V = p.V; a.O = p.O; a.maps = p.maps;
  a.feat = reinterpret_cast<const u32x4*>(p.feat); a.emb = reinterpret_cast<u32x4*>(p.emb);
  a.feat_pieces = p.emb_row_bytes / 16;
  a.slot = p.slot; a.row_sel = p.row_sel; a.key_len = p.key_len;
  a.B = p.B; a.M = p.M; a.L = p.L; a.layer_begin = p.layer_begin; a.Lc = p.Lc;
  a.Hq = p.Hq; a.Hkv = p.Hkv; a.S = p.S;
  a.n_tiles = p.B * p.Lc * p.Hkv;
  const float scale = p.scale == 0.f ? 1.0f / sqrtf((float)p.D) : p.scale;
  a.scale_log2e = scale * 1.44269504088896340736f;
  const int units = p.S <= kChunk ? 4 : p.Hq / p.Hkv * (p.S / 32);
  const int groups8 = (a.n_tiles + 7) / 8 * 8;   // padded to a multiple of 8
  const dim3 grid((unsigned)((size_t)groups8 * ((units + 3) / 4)));
  return p.D == 64 ? launch_insert_d<64>(a, grid, p.causal, p.packed, stream)
                   : launch_insert_d<128>(a, grid, p.causal, p.packed, stream);
}

}  // namespace ac

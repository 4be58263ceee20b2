// Reuse branch of Algorithm 2: O = A_cached . V, with the cached map read in
// place from the database (the hit index selects the entry; nothing is
// gathered or copied first).
//
// bf16 path (matrix cores).  Three kernels: apply_bf16_short_kernel for up to 128 rows, apply_bf16_long_kernel for more, and
// this one, v_mfma_f32_16x16x32_bf16, for many tiles of 128.  One workgroup = one (query, layer, head group).  The product is formed
// transposed, O^T = V^T A^T, so that
//   - the map operand is eight consecutive bf16 of one map row per lane: a
//     plain 16-byte global load straight into the MFMA operand, no LDS;
//   - the V operand comes from an LDS tile that was transposed while staging;
//   - each lane ends up with four consecutive d of one output row.
// Causal maps are exactly zero above the diagonal: 16-row block r only needs
// its first ceil((r+1)/2) blocks of 32 columns.  A wave owns row blocks w and
// 7-w of the 128-row block, which gives every wave the same five column
// blocks on the diagonal chunk (1+4, 1+4, 2+3, 2+3).
//
// Two storage layouts of a map [S][S]:
//   dense   row-major, as computed;
//   packed  only the needed 16 x 32 blocks, row-block-major, each block (1 KiB)
//           stored in MFMA operand order: element (i, 8q+e) of the block at
//           offset (16 q + i) * 8 + e.  A wave's load of one block is then one
//           contiguous KiB, a tile is one contiguous run of 20 KiB (S = 128)
//           instead of 32 KiB with holes, and no 128-byte line is fetched for
//           only half of its bytes.
// HBM-bound: per (query, layer, head) the kernel moves S(S+32) map bytes
// (causal bf16), V once per head group and O once.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "f32_tile.hpp"
#include "launch.hpp"

namespace ac {

struct ApplyArgs {
  const void* maps;     // [M][L][Hq][tile] (device), or one staged entry
  const int32_t* hit;   // [B] device, or nullptr when q_list is used
  const void* V;
  void* O;
  int32_t M, L, layer_begin, Lc, Hq, Hkv, S;
  int32_t heads_per_wg;  // query heads handled by one workgroup (shares V)
  int32_t n_rblk;        // ceil(S / 128); S <= 128: workgroups that share a tile's units
  int32_t xcd_bits;      // S <= 128: 3 if those get ids equal mod 8 (one XCD, one L2), else 0
  int32_t tiles_per_wg;  // (item, layer, KV head) of one workgroup, S <= 128
  int32_t n_tiles;       // B' * Lc * (Hq / heads_per_wg)
  int32_t tile0;         // first tile of the launch (fp32 path, see launch_apply_f32)
  int32_t fixed_entry;   // >= 0: every listed query uses maps as this single entry
  int32_t n_list;        // number of valid q_list items when fixed_entry >= 0
  int32_t q_list[32];    // queries served by the staged entry
};

__device__ __forceinline__ f32x4 mfma16_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// 128 rows of packed causal maps, 64 columns of V, many tiles (launch_apply).  PREFETCH: the map pieces of the next head are
// requested before the products of the current one, so a workgroup that walks several heads always has loads in flight.
template <bool PREFETCH>
__global__ __launch_bounds__(kThreads, PREFETCH ? 3 : 4) void apply_bf16_kernel(const ApplyArgs a) {
  constexpr int D = 64, S = kChunk, OS = D + 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* vt = reinterpret_cast<bf16_t*>(smem);                 // [D][kVtStride]
  bf16_t* ost_all = vt + D * kVtStride;                          // [4][32][D + 4]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, kq = lane >> 4;
  const int tile = blockIdx.x;
  if (tile >= a.n_tiles) return;
  const int hgroups = a.Hq / a.heads_per_wg;
  const int hg = tile % hgroups;
  const int l = (tile / hgroups) % a.Lc;
  const int bslot = tile / (hgroups * a.Lc);

  int b, entry;
  if (a.fixed_entry >= 0) {
    b = a.q_list[bslot];
    entry = 0;
  } else {
    b = bslot;
    entry = a.hit[b];
    if (entry < 0 || entry >= a.M) return;   // miss (or invalid index): O[b] untouched
  }

  const int g = a.Hq / a.Hkv;
  const int h0 = hg * a.heads_per_wg;
  const int kvh = h0 / g;
  const size_t tile_elems = (size_t)packed_blocks(S, 1) * 512;
  const bf16_t* Vt_src = reinterpret_cast<const bf16_t*>(a.V) +
                         (((size_t)b * a.Lc + l) * a.Hkv + kvh) * (size_t)S * D;
  const bf16_t* A_layer = reinterpret_cast<const bf16_t*>(a.maps) +
                          ((size_t)entry * a.L + (a.layer_begin + l)) * ((size_t)a.Hq * tile_elems);

  const int rA = wave, rB = 7 - wave;                         // the two 16-row blocks of this wave
  const int nA = (rA >> 1) + 1;                               // 32-column blocks the first one needs, of five for both
  auto issue = [&](const bf16_t* At, u32x4 (&am)[5]) {        // this lane's 16-byte operand pieces
#pragma unroll
    for (int t = 0; t < 5; ++t) {
      const bool inA = t < nA;
      am[t] = *reinterpret_cast<const u32x4*>(
          At + (size_t)(packed_prefix(inA ? rA : rB) + (inA ? t : t - nA)) * 512 + lane * 8);
    }
  };

  u32x4 am[5], am_next[5];
  if (PREFETCH) issue(A_layer + (size_t)h0 * tile_elems, am_next);
  for (int hl = 0; hl < a.heads_per_wg; ++hl) {
    const int h = h0 + hl;
    const bf16_t* At = A_layer + (size_t)h * tile_elems;
    f32x4 accA[D / 16], accB[D / 16];
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      accA[db] = f32x4{0.f, 0.f, 0.f, 0.f};
      accB[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // 1. map pieces: requested first, so that they are in flight while V is staged
    if (PREFETCH) {
#pragma unroll
      for (int t = 0; t < 5; ++t) am[t] = am_next[t];
    } else {
      issue(At, am);
    }
    // 2. V^T into LDS (once per workgroup; shared by its heads)
    if (hl == 0) {
      stage_v_transposed<D>(Vt_src, S, vt, tid);
      __syncthreads();
    }
    if (PREFETCH && hl + 1 < a.heads_per_wg) issue(At + tile_elems, am_next);
    // 3. O^T[d][i] += sum_j V^T[d][j] A^T[j][i]
    auto vop = [&](int db, int ks) {
      const u32x2* src = reinterpret_cast<const u32x2*>(vt + (16 * db + i16) * kVtStride + 32 * ks + 8 * kq);
      u32x2 lo = src[0], hi = src[1];
      return u32x4{lo.x, lo.y, hi.x, hi.y};
    };
    auto product = [&](f32x4 (&acc)[D / 16], int t, int ks) {
#pragma unroll
      for (int db = 0; db < D / 16; ++db) acc[db] = mfma16_bf16(vop(db, ks), am[t], acc[db]);
    };
    product(accA, 0, 0);   // (the first row block needs one or two of the five)
    if (nA == 2) product(accA, 1, 1);
    else product(accB, 1, 0);
#pragma unroll
    for (int t = 2; t < 5; ++t) product(accB, t, t - nA);

    // 4. result registers: out[row i16 of the block][d = 16 db + 4 kq + v].  Both row blocks go
    // through a wave-private LDS buffer so that global stores are contiguous 16-byte pieces.
    bf16_t* ost = ost_all + wave * (32 * OS);
#pragma unroll
    for (int db = 0; db < D / 16; ++db) {
      u32x2 wa, wb;
      wa.x = pack_bf16(accA[db][0], accA[db][1]);
      wa.y = pack_bf16(accA[db][2], accA[db][3]);
      wb.x = pack_bf16(accB[db][0], accB[db][1]);
      wb.y = pack_bf16(accB[db][2], accB[db][3]);
      *reinterpret_cast<u32x2*>(ost + i16 * OS + 16 * db + 4 * kq) = wa;
      *reinterpret_cast<u32x2*>(ost + (16 + i16) * OS + 16 * db + 4 * kq) = wb;
    }
    // LDS operations of one wave execute in order; only the compiler must keep the order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    bf16_t* Ot = reinterpret_cast<bf16_t*>(a.O) + ((((size_t)b * a.Lc + l) * a.Hq + h) * S) * D;
    constexpr int PIECES = 32 * D / 8;
#pragma unroll
    for (int it = 0; it < PIECES / kWave; ++it) {
      const int p = it * kWave + lane;
      const int row = p / (D / 8), c8 = p % (D / 8);
      const u32x2* s = reinterpret_cast<const u32x2*>(ost + row * OS + 8 * c8);
      u32x2 x = s[0], y = s[1];
      u32x4 w = {x.x, x.y, y.x, y.y};
      const int lrow = row < 16 ? 16 * rA + row : 16 * rB + row - 16;
      // written once, never re-read by this kernel: streaming store
      __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(Ot + (size_t)lrow * D + 8 * c8));
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// Sequences of up to 128 rows.  With the kernel above a workgroup has one (item, layer, K/V head) and its heads one after the
// other, 128 map rows at a time: of 32 rows two of its four waves would have none, and LDS for 128 keys of 128 columns leaves room for two
// workgroups on a compute unit.  Here a wave takes units of 32 rows of one head, the next unit's map pieces on their way
// during the products of this one, the workgroup as many K/V heads as give its waves a unit each, and LDS holds their V
// and no more.  V is copied and read as in the long kernel below.
// us per call, with 128 rows at a time / so: 118 x 16 x 3 heads on one K/V head of 32 x 128, half of them misses 21.3 / 9.2; 100 x 32 x 8 of 32 x
// 128 160 / 74; 123 x 2 x 16 on 4 of 64 x 64 17.3 / 11.2; 100 x 4 x 24 on 12 of 64 x 128 51.4 / 35.1; 64 x 4 x 32 of 96 x 128 95 / 75;
// 64 x 16 x 32 of 96 x 64 213 / 186 (5.4 TB/s); a small one, 11 x 4 x 3 on one of 96 x 128 11.6 / 5.9.  Bound by the memory where it is large
// (64 x 8 x 32 on 8 of 128 x 128, 161 us, 5.0 TB/s), else by the chain hit -> map, V -> products -> stores.
template <int D, bool CAUSAL, bool PACKED, int NRB>
__global__ __launch_bounds__(kThreads, (D == 64 ? (NRB == 4 ? 3 : 4) : NRB == 4 ? 2 : 3)) void apply_bf16_short_kernel(const ApplyArgs a) {
  constexpr int S = 32 * NRB, PPR = D / 8, NCOPY = S * PPR / kWave / 4;   // copy instructions per wave and tile
  constexpr int kMostTiles = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* vb = reinterpret_cast<bf16_t*>(smem);   // [tiles_per_wg][S][D]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  bf16_t* ost = vb + (size_t)a.tiles_per_wg * S * D + wave * (16 * kSmallOutStride);
  const int g = a.Hq / a.Hkv, per = g * NRB;      // units of a tile
  const unsigned slot = blockIdx.x >> a.xcd_bits, group = slot / a.n_rblk;
  const int part = (int)(slot - group * a.n_rblk);
  const int tile0 = (int)(group << a.xcd_bits | (blockIdx.x & ((1u << a.xcd_bits) - 1))) * a.tiles_per_wg;
  const size_t tile_elems = PACKED ? (size_t)packed_blocks(S, CAUSAL) * 512 : (size_t)S * S;

  // the tiles: query (-1: a miss, past the end or an invalid index) and entry
  int qb[kMostTiles], entry[kMostTiles];
#pragma unroll
  for (int t = 0; t < kMostTiles; ++t) {
    qb[t] = -1;
    entry[t] = 0;
    if (t < a.tiles_per_wg && tile0 + t < a.n_tiles) {
      const int bslot = (tile0 + t) / (a.Hkv * a.Lc);
      if (a.fixed_entry >= 0) {
        qb[t] = a.q_list[bslot];
      } else {
        entry[t] = a.hit[bslot];
        qb[t] = entry[t] >= 0 && entry[t] < a.M ? bslot : -1;
      }
    }
  }
  if (max(max(qb[0], qb[1]), max(qb[2], qb[3])) < 0) return;   // nothing to do
  struct Unit { int t, head, rb; };
  // (rows rotate with the head, so that a causal map's heavy ones fall to all waves in turn)
  auto unit = [&](int u) {
    const int head = u % per / NRB;
    return Unit{u / per, head, (u + head) % NRB};
  };
  auto query = [&](int t) { return t == 0 ? qb[0] : t == 1 ? qb[1] : t == 2 ? qb[2] : qb[3]; };
  auto entry_at = [&](int t) { return t == 0 ? entry[0] : t == 1 ? entry[1] : t == 2 ? entry[2] : entry[3]; };
  auto layer_of = [&](int t) { return (tile0 + t) / a.Hkv % a.Lc; };
  auto head_of = [&](const Unit& w) { return (tile0 + w.t) % a.Hkv * g + w.head; };

  // 16 columns of 32 map rows a step: eight elements of row il
  struct Pieces { u32x4 p[2 * NRB]; };
  auto steps = [&](const Unit& w) { return CAUSAL ? 2 * (w.rb + 1) : 2 * NRB; };
  auto issue = [&](int u) {
    Pieces m;
    const Unit w = unit(u);
    if (query(w.t) < 0) return m;
    const bf16_t* At = reinterpret_cast<const bf16_t*>(a.maps) +
                       (((size_t)entry_at(w.t) * a.L + (a.layer_begin + layer_of(w.t))) * a.Hq + head_of(w)) * tile_elems;
    const int r16 = 2 * w.rb + (il >> 4);
    const unsigned row = PACKED ? (unsigned)((CAUSAL ? packed_prefix(r16) : r16 * NRB) * 512 + (kh * 16 + (il & 15)) * 8)
                                : (unsigned)((32 * w.rb + il) * S + 8 * kh);
#pragma unroll
    for (int ks = 0; ks < 2 * NRB; ++ks)
      if (ks < steps(w)) m.p[ks] = *reinterpret_cast<const u32x4*>(At + ks * (PACKED ? 256 : 16) + row);
    return m;
  };

  const int u_end = a.n_rblk > 1 ? min(4 * part + 4, per) : a.tiles_per_wg * per;
  int u = 4 * part + wave;
  Pieces now;
  if (u < u_end) now = issue(u);
  // copy instruction wave + 4 i of a tile fills its LDS slots [64 k, 64 k + 64), 16-byte piece p of row r at p ^ v_piece_swizzle(r)
  const int slot0 = kWave * wave + lane;
  const unsigned copy_off = (unsigned)((slot0 / PPR) * D + 8 * ((slot0 % PPR) ^ v_piece_swizzle<D>(slot0 / PPR)));
#pragma unroll
  for (int t = 0; t < kMostTiles; ++t)
    if (qb[t] >= 0) {
      const bf16_t* src = reinterpret_cast<const bf16_t*>(a.V) +
                          (((size_t)qb[t] * a.Lc + layer_of(t)) * a.Hkv + (tile0 + t) % a.Hkv) * (size_t)(S * D);
#pragma unroll
      for (int i = 0; i < NCOPY; ++i)
        __builtin_amdgcn_global_load_lds(src + (copy_off + 2048u * i), vb + t * (S * D) + kWave * 8 * (wave + 4 * i), 16, 0, 0);
    }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef short s16x8 __attribute__((ext_vector_type(8)));
  int voff[2][D / 32];   // as in the long kernel
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
      const int t = lane & 15, j = 8 * kh + 4 * half + (t >> 2), d0 = 32 * db + 16 * (il >> 4) + 4 * (t & 3);
      voff[half][db] = j * D + 8 * ((d0 >> 3) ^ v_piece_swizzle<D>(j)) + (d0 & 7);
    }
  for (; u < u_end; u += 4) {
    Pieces next;
    if (u + 4 < u_end) next = issue(u + 4);
    const Unit w = unit(u);
    const int b = query(w.t);
    if (b >= 0) {
      const bf16_t* v = vb + w.t * (S * D);
      f32x16 acc[D / 32];
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc[db][x] = 0.f;
#pragma unroll
      for (int ks = 0; ks < 2 * NRB; ++ks)
        if (ks < steps(w)) {
#pragma unroll
          for (int db = 0; db < D / 32; ++db) {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (s16x4 __attribute__((address_space(3)))*)(v + voff[0][db] + 16 * ks * D));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                (s16x4 __attribute__((address_space(3)))*)(v + voff[1][db] + 16 * ks * D));
            const s16x8 op = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            acc[db] = mfma_bf16(__builtin_bit_cast(bf16x8, op), __builtin_bit_cast(bf16x8, now.p[ks]), acc[db]);
          }
        }
      bf16_t* out = reinterpret_cast<bf16_t*>(a.O) +
                    ((((size_t)b * a.Lc + layer_of(w.t)) * a.Hq + head_of(w)) * S + 32 * w.rb) * (size_t)D;
      store_tile_bf16_small<D>(acc, 1.0f, ost, out, lane);
    }
    now = next;
  }
}

// Long sequences (S > 128).  The 16x16x32 matrix instruction runs at half the rate of 32x32x16 on
// this chip (measured 1.3 vs 2.0 PFLOP/s), which does not matter for one 128-column chunk per
// tile but bounds the reuse product once a workgroup walks many full chunks.  Here a wave owns
// one 32-row block of the 128-row block and uses v_mfma_f32_32x32x16_bf16.  Only the diagonal
// chunk is unbalanced (wave w needs 2 (w + 1) of its 8 column steps).
//
// V is not transposed by the ALUs here.  Each 128-key chunk is copied global -> LDS directly
// (global_load_lds_dwordx4, no data registers), row-major, into one of two LDS buffers, so the
// copy of chunk c+1 and the map pieces of chunk c+1 are in flight while chunk c is multiplied;
// the matrix operand is then fetched with the transposing LDS read (ds_read_b64_tr_b16): in a
// group of 16 lanes, lane i supplies the address of four consecutive d of key j(i/4) and lane
// t receives, for ITS d, the four keys j(0..3) -- exactly the operand layout, no shuffles.
// Rows are stored unpadded; 16-byte piece p of key row r sits at position p ^ v_piece_swizzle(r),
// which spreads the 32 lanes one LDS cycle serves over all banks; the copy applies the
// permutation by choosing which global piece each lane fetches.
constexpr int kOutStride = 64 + 4;   // row stride of the 16 x 64 output staging passes

template <int D, bool CAUSAL, bool PACKED>
__global__ __launch_bounds__(kThreads, 2) void apply_bf16_long_kernel(const ApplyArgs a) {
  constexpr int PPR = D / 8;                       // 16-byte pieces per V row
  constexpr int NCOPY = kChunk * PPR / kWave / 4;  // copy instructions per wave and chunk
  __shared__ __attribute__((aligned(16))) bf16_t vb0[kChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t vb1[kChunk * D];
  // Causal maps at head_dim 64: a workgroup takes a PAIR of row blocks (see below).  Its
  // results then leave through a small wave-private buffer, 16 rows x 64 columns per pass,
  // because the V buffers stay in use.
  constexpr bool PAIRED = CAUSAL && D == 64;
  __shared__ __attribute__((aligned(16))) bf16_t ost_small[PAIRED ? 4 * 16 * kOutStride : 8];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // scalar: branches on it stay uniform
  const int il = lane & 31, kh = lane >> 5;

  const int bid = blockIdx.x;
  // PAIRED: row blocks are handled in pairs (n_rblk - 1 - p, then p): under the causal mask
  // their chunk counts add up to n_rblk + 1 for every p, so all workgroups of a launch carry
  // equal work, and the chunk pipeline runs on across the switch (one fill per workgroup, not
  // two): 61 -> 70 % of HBM peak at S = 1024, D = 64.  At D = 128 the V copies, not the short
  // workgroups, are the limit and pairing gains nothing; dense maps have equal work anyway.
  const int n_pairs = PAIRED ? (a.n_rblk + 1) >> 1 : a.n_rblk;
  const int tile = (bid >> 3) / n_pairs * 8 + (bid & 7);
  const int pair = (bid >> 3) % n_pairs;
  if (tile >= a.n_tiles) return;
  const int h = tile % a.Hq;
  const int l = (tile / a.Hq) % a.Lc;
  const int bslot = tile / (a.Hq * a.Lc);
  int b, entry;
  if (a.fixed_entry >= 0) {
    b = a.q_list[bslot];
    entry = 0;
  } else {
    b = bslot;
    entry = a.hit[b];
    if (entry < 0 || entry >= a.M) return;   // miss (or invalid index): O[b] untouched
  }

  const int S = a.S, g = a.Hq / a.Hkv;
  const int n32 = S >> 5;
  const size_t tile_elems = PACKED ? (size_t)packed_blocks(S, CAUSAL) * 512 : (size_t)S * S;
  const bf16_t* Vsrc = uniform_ptr(reinterpret_cast<const bf16_t*>(a.V) +
                                   (((size_t)b * a.Lc + l) * a.Hkv + h / g) * (size_t)S * D);
  const bf16_t* At = uniform_ptr(reinterpret_cast<const bf16_t*>(a.maps) +
                                 (((size_t)entry * a.L + (a.layer_begin + l)) * a.Hq + h) * tile_elems);

  const int R_hi = a.n_rblk - 1 - pair, R_lo = PAIRED ? pair : R_hi;   // heaviest first
  const int n_hi = CAUSAL ? R_hi + 1 : (S + kChunk - 1) / kChunk;
  const int n_total = n_hi + (R_hi != R_lo ? (CAUSAL ? R_lo + 1 : n_hi) : 0);
  // chunk t of the workgroup's walk: its row block and its chunk index within that block
  auto row_block = [&](int t) { return t < n_hi ? R_hi : R_lo; };
  auto chunk_of = [&](int t) { return t < n_hi ? t : t - n_hi; };

  // 16-byte operand piece of column step ks (16 columns, counted from column 0) for this lane:
  // map row 32 rb32 + il, columns 16 ks + 8 kh .. + 8, rb32 = 4 R + wave being this wave's rows
  // (32-bit element offsets from the tile's base, which is uniform over the workgroup: the
  // loads then take a scalar base and one offset register instead of 64-bit lane addresses)
  auto piece_row_of = [&](int R) {
    const int rb32 = 4 * R + wave;
    return PACKED
      ? (unsigned)((CAUSAL ? packed_prefix(2 * rb32 + (il >> 4)) : (2 * rb32 + (il >> 4)) * n32) * 512 +
                   (kh * 16 + (il & 15)) * 8)
      : (unsigned)((32 * rb32 + il) * S + 8 * kh);
  };
  const unsigned piece_row_hi = piece_row_of(R_hi), piece_row_lo = piece_row_of(R_lo);
  // (the column step is uniform over the wave: it goes into the scalar base, the lane's own
  // offset stays one register per row block whatever the step)
  auto piece = [&](int R, int ks) -> const u32x4* {
    const unsigned piece_row = R == R_hi ? piece_row_hi : piece_row_lo;
    const char* step_base = reinterpret_cast<const char*>(At + (size_t)ks * (PACKED ? 256 : 16));
    return reinterpret_cast<const u32x4*>(step_base + 2u * piece_row);   // 32-bit BYTE offset
  };
  // column steps of chunk c this wave needs
  auto steps = [&](int R, int c) {
    if (32 * (4 * R + wave) >= S) return 0;
    const int nk = min(kChunk, S - c * kChunk) >> 4;
    return (CAUSAL && c == R) ? min(nk, 2 * (wave + 1)) : nk;
  };
  auto full = [&](int R, int c) {   // uniform over the workgroup: every wave takes all 8 steps
    return !(CAUSAL && c == R) && S - c * kChunk >= kChunk && 32 * (4 * R + 3) < S;
  };
  // map pieces of chunk c into am.  Every lane loads 8 pieces whatever it needs: a step beyond
  // the wave's last one repeats that last piece (same cache lines, no extra memory traffic,
  // never multiplied), which keeps the loads free of per-wave control flow.
  auto issue = [&](int R, int c, u32x4 (&am)[8]) {
    const int nks = steps(R, c);
    if (nks == 0) return;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) am[ks] = *piece(R, 8 * c + min(ks, nks - 1));
  };
  // copy key rows [128 c, 128 c + nj) of V into buf: instruction k = wave + 4 i fills LDS slots
  // [64 k, 64 k + 64) (slot = row * PPR + position), i.e. rows [k 64/PPR, (k + 1) 64/PPR).
  // Row and position of a lane's slot differ between instructions only by whole multiples of
  // 2048 elements on both sides, so one 32-bit lane offset serves all of them.  Rows past the
  // end of V (ragged last chunk) repeat the last row: finite values that are never multiplied.
  const int slot0 = kWave * wave + lane;
  const unsigned copy_off = (unsigned)((slot0 / PPR) * D + 8 * ((slot0 % PPR) ^ v_piece_swizzle<D>(slot0 / PPR)));
  const bf16_t* vrun = Vsrc;   // chunk after chunk, in order: a running (scalar) source pointer
  auto copy_v = [&](bf16_t* buf, int c) {
    const int nj = min(kChunk, S - c * kChunk);
    const bf16_t* src = vrun;
    vrun += kChunk * D;
    if (nj == kChunk) {
#pragma unroll
      for (int i = 0; i < NCOPY; ++i)
        __builtin_amdgcn_global_load_lds(src + (copy_off + 2048u * i), buf + kWave * 8 * (wave + 4 * i),
                                         16, 0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < NCOPY; ++i) {
        const int slot = slot0 + 4 * kWave * i;
        const int row = slot / PPR, pos = slot % PPR;
        const int src_piece = pos ^ v_piece_swizzle<D>(row);
        __builtin_amdgcn_global_load_lds(src + (size_t)min(row, nj - 1) * D + 8 * src_piece,
                                         buf + kWave * 8 * (wave + 4 * i), 16, 0, 0);
      }
    }
  };

  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;

  // transposing operand fetch: rows d = 32 db + il of V^T, contraction slots (kh, e) = key
  // 16 ks + 8 kh + e.  Lane i of a 16-lane group names key row 16 ks + 8 kh + i / 4 (+ 4 for
  // the second half) and the four d starting at 32 db + 16 (il / 16) + 4 (i % 4).  The row's
  // permutation only depends on (key & 3), i.e. not on ks: one element offset per (half, db) is
  // kept in a register and ks enters as a constant.
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  int voff[2][D / 32];
  {
    const int t = lane & 15;
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        const int j = 8 * kh + 4 * half + (t >> 2);               // key row for ks = 0
        const int d0 = 32 * db + 16 * (il >> 4) + 4 * (t & 3);     // first of this lane's four d
        voff[half][db] = j * D + 8 * ((d0 >> 3) ^ v_piece_swizzle<D>(j)) + (d0 & 7);
      }
  }
  auto vop = [&](const bf16_t* buf, int db, int ks) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(buf + voff[0][db] + 16 * ks * D));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3)))*)(buf + voff[1][db] + 16 * ks * D));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    s16x8 w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, w);
  };
  // Products of chunk c.  The scheduling fences keep the compiler from hoisting every operand
  // read of a chunk in front of the first product (more registers than the file has).
  auto compute = [&](const bf16_t* buf, int R, int c, const u32x4 (&am)[8]) {
    if (full(R, c)) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
          acc[db] = mfma_bf16(vop(buf, db, ks), __builtin_bit_cast(bf16x8, am[ks]), acc[db]);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      const int nks = steps(R, c);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        if (ks < nks) {
#pragma unroll
          for (int db = 0; db < D / 32; ++db)
            acc[db] = mfma_bf16(vop(buf, db, ks), __builtin_bit_cast(bf16x8, am[ks]), acc[db]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Software pipeline over chunks, unrolled by two so that buffers and register sets alternate
  // without copies: while chunk c is multiplied out of (vb0, am0), the copy of V chunk c + 1
  // into vb1 and the map pieces of chunk c + 1 into am1 are in flight, and vice versa.
  // publish(): this wave's copies and loads have landed (copies are counted like loads), then
  // the barrier makes every wave's part of the V chunk visible and retires the other buffer.
  auto publish = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };
  auto prefetch = [&](bf16_t* buf, int t, u32x4 (&am)[8]) {
    if (t == n_hi) vrun = Vsrc;   // the second row block starts over at the first keys
    copy_v(buf, chunk_of(t));
    issue(row_block(t), chunk_of(t), am);
    __builtin_amdgcn_sched_barrier(0);
  };
  // after the last chunk of a row block: the wave's 32 x D result leaves in 16 x 64 passes
  // through its small private buffer (every global store covers whole 128-byte lines), and
  // the accumulator starts over.  No barrier: the V buffers are not touched.
  auto finish = [&](int t) {
    if (!PAIRED) return;   // one row block per workgroup: stored after the loop, through the V buffers
    if (t + 1 != n_hi && t + 1 != n_total) return;
    const int rb32 = 4 * row_block(t) + wave;
    if (32 * rb32 < S) {
      bf16_t* dst = reinterpret_cast<bf16_t*>(a.O) +
                    ((((size_t)b * a.Lc + l) * a.Hq + h) * S + 32 * rb32) * (size_t)D;
      bf16_t* ost = ost_small + wave * (16 * kOutStride);
#pragma unroll
      for (int rh = 0; rh < 2; ++rh)
#pragma unroll
        for (int dh = 0; dh < D / 64; ++dh) {
          if ((il >> 4) == rh) {
#pragma unroll
            for (int dbp = 0; dbp < 2; ++dbp)
#pragma unroll
              for (int vq = 0; vq < 4; ++vq) {
                const f32x16& r = acc[2 * dh + dbp];
                u32x2 w;
                w.x = pack_bf16(r[4 * vq], r[4 * vq + 1]);
                w.y = pack_bf16(r[4 * vq + 2], r[4 * vq + 3]);
                *reinterpret_cast<u32x2*>(ost + (il & 15) * kOutStride + 32 * dbp + 8 * vq + 4 * kh) = w;
              }
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
          for (int it = 0; it < 2; ++it) {
            const int p = it * kWave + lane;
            const int row = p >> 3, c8 = p & 7;
            const u32x2* sp = reinterpret_cast<const u32x2*>(ost + row * kOutStride + 8 * c8);
            u32x2 lo = sp[0], hi = sp[1];
            __builtin_nontemporal_store(
                u32x4{lo.x, lo.y, hi.x, hi.y},
                reinterpret_cast<u32x4*>(dst + (size_t)(16 * rh + row) * D + 64 * dh + 8 * c8));
          }
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;
  };

  u32x4 am0[8], am1[8];
  prefetch(vb0, 0, am0);
  for (int t = 0; t < n_total; t += 2) {
    publish();
    if (t + 1 < n_total) prefetch(vb1, t + 1, am1);
    compute(vb0, row_block(t), chunk_of(t), am0);
    finish(t);
    if (t + 1 < n_total) {
      publish();
      if (t + 2 < n_total) prefetch(vb0, t + 2, am0);
      compute(vb1, row_block(t + 1), chunk_of(t + 1), am1);
      finish(t + 1);
    }
  }
  if constexpr (!PAIRED) {
    __syncthreads();   // every wave is done with both V buffers: they now stage the output
    const int rb32 = 4 * R_hi + wave;
    if (32 * rb32 < S) {
      bf16_t* dst = reinterpret_cast<bf16_t*>(a.O) +
                    ((((size_t)b * a.Lc + l) * a.Hq + h) * S + 32 * rb32) * (size_t)D;
      bf16_t* ost = ((wave & 2) ? vb1 : vb0) + (wave & 1) * (32 * (D + 4));
      store_tile_bf16<D>(acc, 1.0f, ost, dst, lane);
    }
  }
}

// Dense -> packed conversion of whole tiles (database build).  One workgroup per tile; a
// thread moves 16-byte pieces: piece `lane` of packed block (r, cb) is map row 16 r + lane % 16,
// columns 32 cb + 8 (lane / 16) .. + 8.
__global__ __launch_bounds__(kThreads) void pack_maps_kernel(const bf16_t* __restrict__ dense,
                                                             bf16_t* __restrict__ packed, int S,
                                                             int causal) {
  const int n16 = S >> 4, n32 = S >> 5;
  const int nblk = packed_blocks(S, causal);
  const bf16_t* src = dense + (size_t)blockIdx.x * S * S;
  bf16_t* dst = packed + (size_t)blockIdx.x * nblk * 512;
  const int lane = threadIdx.x & 63;
  const int i16 = lane & 15, kq = lane >> 4;
  for (int r = 0; r < n16; ++r) {
    const int nc = causal ? ((r + 1) + 1) >> 1 : n32;
    const int base = causal ? packed_prefix(r) : r * n32;
    for (int cb = threadIdx.x >> 6; cb < nc; cb += kThreads / kWave) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(src + (size_t)(16 * r + i16) * S + 32 * cb + 8 * kq);
      *reinterpret_cast<u32x4*>(dst + (size_t)(base + cb) * 512 + lane * 8) = v;
    }
  }
}

// fp32 path (binary32 matrix instructions, dense layout, any S, D <= 64 DB).  Four waves of 16 map
// rows each share 32-key stages of V; the map goes from memory straight into the lanes that feed
// the products (a lane reads four consecutive columns of its row; rows of odd lengths are only
// 4-byte aligned, which the load allows).  The next stage's V and map pieces are requested before
// this one is multiplied.  Above the diagonal of a causal map nothing that was read is used.
// 16 queries (12 hits) x 2 layers x 24 heads on 8 V, 94 x 128 causal: 403 us with one thread per
// output and scalar loads, 20.5 us so (48 MB, 9 us at the copy rate; bound by the chain of load,
// stage and product in a workgroup -- 64-key stages or four workgroups per CU measure the same; with map
// pieces behind tests, which the compiler waited for before the products, 22.2 us).
template <int DB, int COLS>
__device__ __forceinline__ void apply_f32_tiles(const ApplyArgs& a, int D, int causal) {
  constexpr int KC = 32, NB = KC / 16;
  typedef F32Stage<DB, KC, COLS> Stage;
  __shared__ __attribute__((aligned(16))) float vl[KC * Stage::LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, kq = lane >> 4;
  const int S = a.S, g = a.Hq / a.Hkv;
  const F32Unit u = f32_unit<true>(blockIdx.x, wave, g, S, a.n_tiles);
  if (u.tile < 0) return;
  const int tile = a.tile0 + u.tile;
  const int h = tile % a.Hkv * g + u.head;
  const int l = (tile / a.Hkv) % a.Lc;
  const int bslot = tile / (a.Hkv * a.Lc);
  int b, entry;
  if (a.fixed_entry >= 0) {
    b = a.q_list[bslot];
    entry = 0;
  } else {
    b = bslot;
    entry = a.hit[b];
    if (entry < 0 || entry >= a.M) return;
  }
  const int row = kF32Rows * max(u.block, 0) + i;
  const float* A_tile = reinterpret_cast<const float*>(a.maps) +
                        (((size_t)entry * a.L + (a.layer_begin + l)) * a.Hq + h) * (size_t)S * S;
  const float* A = A_tile + (size_t)min(row, S - 1) * S;
  bool redo = false;   // wave-uniform
  const float* V = reinterpret_cast<const float*>(a.V) +
                   (((size_t)b * a.Lc + l) * a.Hkv + h / g) * (size_t)S * D;
  const int limit = causal ? min(row + 1, S) : S;   // columns of this row that count
  const int wave_keys = u.block < 0 ? 0 : causal ? min(S, kF32Rows * (u.block + 1)) : S;
  const int wg_keys = causal ? min(S, kF32Rows * (u.last_block + 1)) : S;

  Stage vs;
  f32x4 map[NB];
  // Four columns of the lane's row of each block from jc on (S >= 4).  Past the columns that count the last four of
  // them are read again, at the end of a row shifted, which lane_map undoes: no load behind a test (the compiler
  // waits for such a load where the branches meet), and none past the row.
  const int last_col = max(wave_keys - 4, 0);
  auto load_map = [&](int jc) {
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
      map[bk] = *reinterpret_cast<const f32x4_dw*>(A + min(jc + 16 * bk + 4 * kq, last_col));
  };
  auto lane_map = [&](int j0, f32x4 m) {
    const int by = j0 + 4 * kq - last_col;   // columns the lane read too early (four or more: none counts)
    const bool two = by > 0 && (by & 2), one = by > 0 && (by & 1);
    m = two ? f32x4{m[2], m[3], m[2], m[3]} : m;
    return one ? f32x4{m[1], m[2], m[3], m[3]} : m;
  };
  f32x4 acc[4 * DB];
#pragma unroll
  for (int x = 0; x < 4 * DB; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int last_stage = (wg_keys - 1) / KC * KC;
  vs.load(V, 0, S, D, tid);
  load_map(0);
  for (int jc = 0; jc < wg_keys; jc += KC) {
    vs.template mask<true>(jc, S, D, tid);
    __syncthreads();   // the previous stage has been read by everybody
    vs.commit(vl, tid);
    f32x4 w[NB];
#pragma unroll
    for (int bk = 0; bk < NB; ++bk) {
      const f32x4 m = lane_map(jc + 16 * bk, map[bk]);
#pragma unroll
      for (int x = 0; x < 4; ++x) w[bk][x] = jc + 16 * bk + 4 * kq + x < limit ? m[x] : 0.f;
    }
    __syncthreads();
    // The next stage.  Whole pieces of narrow rows are requested without a test, in the last trip once more and unused:
    // 2 x 8 heads of 600 x 128 36.7 us with the test, 35.4 without.  Wide rows lose by it (16 x 24 heads of 94 x 160, all
    // keys 28.2 / 30.9) and so do rows that end in part of a block (of 94 x 80, causal 13.0 / 14.1).
    if ((COLS == kAllCols && DB <= 2) || jc + KC < wg_keys) {
      const int next = min(jc + KC, last_stage);
      vs.load(V, next, S, D, tid);
      load_map(next);
    }
#pragma unroll
    for (int bk = 0; bk < NB; ++bk)
      if (jc + 16 * bk < wave_keys) {
        const float* v = vl + 16 * bk * Stage::LD;
        if (causal && (jc >> 4) + bk == u.block) redo = f32_block_not_finite<DB>(v, i, kq);
        f32_weights_v<DB>(acc, v, w[bk], i, kq);
      }
  }
  float* O = reinterpret_cast<float*>(a.O) + (((size_t)b * a.Lc + l) * a.Hq + h) * (size_t)S * D;
  if (u.block >= 0 && row < S && !redo) f32_store_row<DB, COLS, false>(O + (size_t)row * D, acc, 1.f, kq, D);
  if (redo) {   // infinite or NaN V near the diagonal: lane = output column, only visible keys are read
    const int first = kF32Rows * u.block, rows = min(kF32Rows, S - first);
#pragma unroll 1
    for (int r = 0; r < rows; ++r)
      for (int d = lane; d < D; d += kWave) {
        const float* Ar = A_tile + (size_t)(first + r) * S;
        float o = 0.f;
        for (int j = 0; j <= first + r; ++j) o = fmaf(Ar[j], V[(size_t)j * D + d], o);
        O[(size_t)(first + r) * D + d] = o;
      }
  }
}

// Three workgroups per compute unit, also of the widest rows (168 registers, two of them spilled): with two, as eight
// registers more had it, 16 x 24 heads of 94 x 160, all keys, take 33.3 us instead of 28.2, 32 x 12 of 128 x 256 37.5 instead of 34.6.
template <int DB>   // D == 64 DB
__global__ __launch_bounds__(kThreads, 3) void apply_f32_kernel(const ApplyArgs a, int causal) {
  apply_f32_tiles<DB, kAllCols>(a, 64 * DB, causal);
}
template <int DB, int COLS>
__global__ __launch_bounds__(kThreads, 3) void apply_f32_kernel_cols(const ApplyArgs a, int D, int causal) {
  apply_f32_tiles<DB, COLS>(a, D, causal);
}

// The same for maps of a few rows, whose time is the chain above and not the work: one workgroup per (query,
// layer, head), a thread per output, sums over ascending columns.  us per call, tiles / this: 256 heads of
// 1 x 256 6.0 / 2.5, of 8 x 64 3.8 / 3.5, of 12 x 40 4.0 / 4.2.  The first workgroup takes (b0, l0, h0): several
// launches may have more (query, layer, head) triples between them than 32 bits count.
__global__ __launch_bounds__(kThreads) void apply_f32_small_kernel(const ApplyArgs a, int D, int causal, int b0, int l0, int h0) {
  const int th = h0 + blockIdx.x, tl = l0 + th / a.Hq, h = th % a.Hq, l = tl % a.Lc, bslot = b0 + tl / a.Lc;
  const int b = a.fixed_entry >= 0 ? a.q_list[bslot] : bslot;
  const int entry = a.fixed_entry >= 0 ? a.fixed_entry : a.hit[b];
  if (a.fixed_entry < 0 && (entry < 0 || entry >= a.M)) return;
  const int S = a.S, g = a.Hq / a.Hkv;
  const float* A = reinterpret_cast<const float*>(a.maps) +
                   (((size_t)entry * a.L + (a.layer_begin + l)) * a.Hq + h) * (size_t)S * S;
  const float* V = reinterpret_cast<const float*>(a.V) + (((size_t)b * a.Lc + l) * a.Hkv + h / g) * (size_t)S * D;
  float* O = reinterpret_cast<float*>(a.O) + (((size_t)b * a.Lc + l) * a.Hq + h) * (size_t)S * D;
  for (int idx = threadIdx.x; idx < S * D; idx += kThreads) {
    const int i = idx / D, d = idx % D;
    const int nj = causal ? i + 1 : S;
    float acc = 0.f;
    for (int j = 0; j < nj; ++j) acc = fmaf(A[(size_t)i * S + j], V[(size_t)j * D + d], acc);
    O[idx] = acc;
  }
}

template <int DB>
static hipError_t launch_apply_f32(ApplyArgs a, int D, int causal, hipStream_t stream) {
  // a launch has fewer than 2^32 threads: very many tiles of narrow heads take several
  const int g = a.Hq / a.Hkv, n_tiles = a.n_tiles;
  const size_t eights = (((size_t)1 << 32) - 1) / kThreads / f32_grid(8, g, a.S);
  const int fit = 8 * (int)std::min<size_t>(std::max<size_t>(eights, 1), 1 << 27);
  for (a.tile0 = 0; a.tile0 < n_tiles; a.tile0 += a.n_tiles) {
    a.n_tiles = std::min(n_tiles - a.tile0, fit);
    const dim3 grid(f32_grid(a.n_tiles, g, a.S));
    if (D == 64 * DB)
      hipLaunchKernelGGL((apply_f32_kernel<DB>), grid, dim3(kThreads), 0, stream, a, causal);
    else if (D % 4 == 0)
      hipLaunchKernelGGL((apply_f32_kernel_cols<DB, kVecCols>), grid, dim3(kThreads), 0, stream, a, D, causal);
    else if (DB == 1 && D < 4)
      hipLaunchKernelGGL((apply_f32_kernel_cols<1, kFewCols>), grid, dim3(kThreads), 0, stream, a, D, causal);
    else
      hipLaunchKernelGGL((apply_f32_kernel_cols<DB, kAnyCols>), grid, dim3(kThreads), 0, stream, a, D, causal);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Up to kShortFew workgroups of four units each take a tile's units side by side, each with its own copy of V, as the launch leaves
// room on the chip; from kShortMany on again, on one XCD: what a large launch reads and writes together then lies closer together, and
// memory gives more (V comes from the L2 after the first time).  us per call with one workgroup a tile / so, packed causal maps of 128 x 128, twice as
// many entries as queries: 4,096 tiles (item, layer, K/V head) of two heads 86.7 / 86.9, 8,192 197 / 180, 16,384 429 / 365, 32,768 886 / 774; of eight heads 1,024 72.2 / 71.0,
// 4,096 347 / 318, 16,384 1,355 / 1,265; dense ones without mask, 32,768 of two 1,015 / 914; 64 x 128, 8,192 of eight 270 / 255; 128 x 64 dense, 8,192 of
// four 294 / 278; of 32 x 64 16,384 of eight 129 / 130.  Six units (two heads of 96 rows) leave two waves without one: 8,192 127 / 135.
// kShortFew is 700 for 128 x 128, which two workgroups of a compute unit hold, if the tiles go round by themselves: 512 tiles of two heads in 512
// workgroups 11.9, in 1,024 16.8; 256 of four 12.7 / 17.8; but 128 of eight 18.8 / 17.1, and 528 workgroups instead of 264 8.7 / 10.1.
constexpr size_t kShortFew = 1024, kShortMany = 16384;

template <bool PREFETCH>
static hipError_t launch_halves(const ApplyArgs& a, hipStream_t stream) {
  constexpr size_t lds = (size_t)(64 * kVtStride + 4 * 32 * (64 + 4)) * sizeof(bf16_t);
  hipLaunchKernelGGL((apply_bf16_kernel<PREFETCH>), dim3((unsigned)a.n_tiles), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool PACKED>
static hipError_t launch_long(const ApplyArgs& a, int tiles8, hipStream_t stream) {
  // causal maps at head_dim 64: a workgroup takes a pair of row blocks (see the kernel)
  const int per_tile = (CAUSAL && D == 64) ? (a.n_rblk + 1) / 2 : a.n_rblk;
  const dim3 grid((unsigned)(tiles8 * per_tile));
  hipLaunchKernelGGL((apply_bf16_long_kernel<D, CAUSAL, PACKED>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_long_d(const ApplyArgs& a, int tiles8, bool causal, bool packed,
                                hipStream_t stream) {
  if (causal) return packed ? launch_long<D, true, true>(a, tiles8, stream)
                            : launch_long<D, true, false>(a, tiles8, stream);
  return packed ? launch_long<D, false, true>(a, tiles8, stream)
                : launch_long<D, false, false>(a, tiles8, stream);
}

static hipError_t launch_short(ApplyArgs a, int D, int S, bool causal, bool packed, int nb, hipStream_t stream) {
  const int units = a.Hq / a.Hkv * (S >> 5);
  a.n_tiles = nb * a.Lc * a.Hkv;
  a.tiles_per_wg = units < 4 ? 4 / units : 1;
  a.n_rblk = 1;
  const size_t apart = (size_t)a.n_tiles * ((units + 3) / 4);
  const bool many = units > 4 && units % 4 == 0 && apart >= kShortMany && apart < (size_t)1 << 23;   // (a grid has 2^32 threads at most)
  const size_t few = D == 128 && S == 128 && a.n_tiles >= 256 ? 700 : kShortFew;
  if (many || (units > 4 && apart <= few)) a.n_rblk = (units + 3) / 4;
  a.xcd_bits = many ? 3 : 0;
  const int wgs = many ? (a.n_tiles + 7) / 8 * 8 : (a.n_tiles + a.tiles_per_wg - 1) / a.tiles_per_wg;
  const dim3 grid((unsigned)wgs * a.n_rblk);
  const size_t lds = ((size_t)a.tiles_per_wg * S * D + 4 * 16 * kSmallOutStride) * sizeof(bf16_t);
  auto go = [&](auto d, auto c, auto pk, auto nrb) {
    hipLaunchKernelGGL((apply_bf16_short_kernel<decltype(d)::value, decltype(c)::value, decltype(pk)::value, decltype(nrb)::value>),
                       grid, dim3(kThreads), lds, stream, a);
    return hipGetLastError();
  };
  auto rows = [&](auto d, auto c, auto pk) {
    return S == 32   ? go(d, c, pk, std::integral_constant<int, 1>{})
           : S == 64 ? go(d, c, pk, std::integral_constant<int, 2>{})
           : S == 96 ? go(d, c, pk, std::integral_constant<int, 3>{})
                     : go(d, c, pk, std::integral_constant<int, 4>{});
  };
  auto layout = [&](auto d, auto c) { return packed ? rows(d, c, std::true_type{}) : rows(d, c, std::false_type{}); };
  auto mask = [&](auto d) { return causal ? layout(d, std::true_type{}) : layout(d, std::false_type{}); };
  return D == 64 ? mask(std::integral_constant<int, 64>{}) : mask(std::integral_constant<int, 128>{});
}

// Host launcher.  Shapes were validated by the caller (api.hip).
hipError_t launch_apply(const ApplyLaunch& p, hipStream_t stream) {
  ApplyArgs a;
  a.maps = p.maps; a.hit = p.hit; a.V = p.V; a.O = p.O;
  a.M = p.M; a.L = p.L; a.layer_begin = p.layer_begin; a.Lc = p.Lc;
  a.Hq = p.Hq; a.Hkv = p.Hkv; a.S = p.S;
  a.fixed_entry = p.fixed_entry; a.n_list = p.n_list; a.tile0 = 0;
  for (int i = 0; i < 32; ++i) a.q_list[i] = i < p.n_list ? p.q_list[i] : 0;
  const int nb = p.fixed_entry >= 0 ? p.n_list : p.B;
  if (nb == 0 || p.Lc == 0) return hipSuccess;

  if (p.is_f32) {
    a.heads_per_wg = 1; a.n_rblk = 1;
    const size_t tiles = (size_t)nb * p.Lc * p.Hq;
    if (p.S <= 5 || (size_t)p.S * p.S * p.D <= 3400) {   // (the other kernel reads rows of four columns or more)
      constexpr size_t kFit = ((size_t)1 << 31) / kThreads;
      for (size_t t0 = 0; t0 < tiles; t0 += kFit) {
        const size_t l0 = t0 / p.Hq;
        hipLaunchKernelGGL(apply_f32_small_kernel, dim3((unsigned)std::min(tiles - t0, kFit)), dim3(kThreads), 0, stream, a, p.D,
                           p.causal, (int)(l0 / p.Lc), (int)(l0 % p.Lc), (int)(t0 % p.Hq));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
      return hipSuccess;
    }
    a.n_tiles = nb * p.Lc * p.Hkv;
    if (p.D <= 64) return launch_apply_f32<1>(a, p.D, p.causal, stream);
    if (p.D <= 128) return launch_apply_f32<2>(a, p.D, p.causal, stream);
    return launch_apply_f32<4>(a, p.D, p.causal, stream);
  }
  // 128 rows of packed causal maps of 64 columns of V, many tiles: the kernel with the two balanced 16-row blocks a wave is 2 to 4 %
  // faster, unless heads share V and a launch is so large that units on one XCD read and write closer together (kShortMany).  us per call,
  // that one / units of 32 rows, K/V heads of one head: 768 5.8 / 6.4, 2,048 17.0 / 17.2, 8,192 61.3 / 63.8, 32,768 290 / 289; of two 1,024 13.4 / 13.7,
  // 4,096 52.5 / 54.3, 8,192 113 / 111, 16,384 248 / 235; of three 4,096 75.7 / 77.2, 8,192 165 / 157; of four 768 18.1 / 18.9, 4,096 96.5 / 100, 8,192
  // 235 / 211, 32,768 1,009 / 923; of eight 2,048 92.5 / 95.1, 4,096 215 / 197; of twelve 768 49.3 / 49.1, 2,048 145 / 146, 4,096 351 / 301.  Up to 512 tiles:
  // 16 x 2 x 32 heads on 8 11.8 / 11.7, 8 x 2 x 32 on 8 11.3 / 6.9.  All others gain: 128 columns, 64 x 8 x 32 heads on 8 170 / 161, 3 x 16
  // on 8, dense 10.1 / 6.3; dense maps, 64 columns, 16 x 6 x 32 on 8 29.0 / 24.0; no mask, 60 x 8 x 24 on 12 80.5 / 72.7.
  const bool halves = p.S == 128 && p.D == 64 && p.causal && p.packed && (size_t)nb * p.Lc * p.Hkv > 512 &&
                      (p.Hq == p.Hkv || (size_t)nb * p.Lc * p.Hq <= 20000);
  if (p.S <= 128 && !halves) return launch_short(a, p.D, p.S, p.causal, p.packed, nb, stream);
  a.n_rblk = (p.S + kChunk - 1) / kChunk;
  const int g = p.Hq / p.Hkv;
  a.heads_per_wg = halves ? g : 1;
  a.n_tiles = nb * p.Lc * (p.Hq / a.heads_per_wg);
  const int tiles8 = (a.n_tiles + 7) / 8 * 8;
  if (!halves)   // long rows: 32-row blocks per wave, full-rate matrix instruction
    return p.D == 64 ? launch_long_d<64>(a, tiles8, p.causal, p.packed, stream)
                     : launch_long_d<128>(a, tiles8, p.causal, p.packed, stream);
  // a workgroup that walks several heads prefetches the next head's map pieces
  return g > 1 ? launch_halves<true>(a, stream) : launch_halves<false>(a, stream);
}

hipError_t launch_pack_maps(const void* dense, void* packed, int64_t n_tiles, int32_t S,
                            int32_t causal, hipStream_t stream) {
  if (n_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_maps_kernel, dim3((unsigned)n_tiles), dim3(kThreads), 0, stream,
                     reinterpret_cast<const bf16_t*>(dense), reinterpret_cast<bf16_t*>(packed), S,
                     causal);
  return hipGetLastError();
}

}  // namespace ac

// Binary32 attention tiles on the matrix cores (v_mfma_f32_16x16x4_f32: full binary32 operands
// and sums, 157 TFLOP/s on the chip, twice the rate of unpacked vector fma): what the exact and
// the reuse kernel of fp32 databases share.
//
// A wave owns 16 rows of one head and forms everything transposed, so that a lane (i = lane % 16,
// kq = lane / 16) only ever deals with row i:
//   scores   S^T = K Q^T   result register v of the lane = key 4 kq + v of a 16-key block;
//   output   O^T = V^T W^T the weights sit where the second product wants them: product v takes
//                          weight register v, whose contraction slot kq is key 4 kq + v.
// The row operands come from LDS as 16-byte reads: the four floats of one read feed four products
// (K: four consecutive contraction indices; V: four consecutive d, i.e. result row i of product t
// is d = 64 b + 4 i + t, which leaves 16 consecutive d of its row in every lane: results go to
// memory as whole 64-byte runs without another trip through LDS).
#pragma once
#include "common.hpp"

namespace ac {

typedef f32x4 f32x4_dw __attribute__((aligned(4)));   // 16-byte load from a 4-byte aligned address

constexpr int kF32Rows = 16;   // rows of a wave, keys of a block

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// What is known of the head dimension when a kernel is compiled.  With all forms in one kernel every piece
// of a row was a load behind tests of its own (16 x 24 heads on 8 K and V, 94 x 128 causal: 24.0 us exact, 21.7 so;
// 16 x 8 heads of 333 x 128 61 / 54).  Rows of any length in single floats behind tests took, exact / reuse, 35.0 / 26.8 us at
// 333 x 33 and 144 / 89 at 333 x 199; in pieces of four that may overlap 31.9 / 21.5 and 128 / 77.
enum F32Cols {
  kAnyCols = 0,   // any D >= 4: rows may start at any 4-byte address
  kVecCols = 1,   // D % 4 == 0: whole 16-byte pieces
  kAllCols = 2,   // D == 64 DB
  kFewCols = 3,   // D < 4: single floats, behind one test
};

// KC rows of up to 64 DB floats on their way from memory through registers to LDS.  LDS rows are four
// floats longer than the data, which spreads the 16-byte reads of 16 consecutive rows over all banks.
// (DB is 1, 2 or 4: from one piece of a thread to its next the row grows by a whole number and
// the column stays, so one lane offset serves all of them.)
template <int DB, int KC, int COLS>
struct F32Stage {
  static constexpr int LD = 64 * DB + 4;
  static constexpr int N = KC * 16 * DB / kThreads, STEP = kThreads / (16 * DB);
  f32x4 r[N];

  // Rows [row0, row0 + KC) of which those from `valid` (> row0) on do not exist.  No load sits behind a
  // test of its own: what does not exist repeats something that does, and mask() takes it out.  The end of a row
  // that is no whole piece is read with what lies before it, and mask() shifts it.
  __device__ __forceinline__ void load(const float* __restrict__ src, int row0, int valid, int D,
                                       int tid) {
    const int row = tid / (16 * DB), c = 4 * (tid % (16 * DB));
    const float* base = src + (size_t)row0 * D;   // uniform
    const int last = valid - 1 - row0;
    if constexpr (COLS == kFewCols) {
#pragma unroll
      for (int n = 0; n < N; ++n) r[n] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (c == 0)
#pragma unroll
        for (int n = 0; n < N; ++n)
#pragma unroll
          for (int t = 0; t < 3; ++t)
            if (t < D) r[n][t] = base[min(row + n * STEP, last) * D + t];
      return;
    }
    const int col = COLS == kAllCols ? c : COLS == kVecCols ? (c < D ? c : 0) : min(c, D - 4);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const float* at = base + (unsigned)(min(row + n * STEP, last) * D + col);
      if constexpr (COLS == kAnyCols) r[n] = *reinterpret_cast<const f32x4_dw*>(at);
      else r[n] = *reinterpret_cast<const f32x4*>(at);
    }
  }
  // Zeros in the rows from `valid` on (hidden keys then carry finite values whatever the padding of a
  // batch holds), if ROWS, and in the columns from D on.
  template <bool ROWS>
  __device__ __forceinline__ void mask(int row0, int valid, int D, int tid) {
    const int row = tid / (16 * DB), c = 4 * (tid % (16 * DB));
    if (COLS == kAnyCols) {
      const int by = c - (D - 4);   // columns that were read too early (four or more: none counts)
      const bool two = by > 0 && (by & 2), one = by > 0 && (by & 1);
#pragma unroll
      for (int n = 0; n < N; ++n) {
        r[n] = two ? f32x4{r[n][2], r[n][3], r[n][2], r[n][3]} : r[n];
        r[n] = one ? f32x4{r[n][1], r[n][2], r[n][3], r[n][3]} : r[n];
      }
    }
    if ((ROWS && row0 + KC > valid) || COLS == kAnyCols || (COLS == kVecCols && D < 64 * DB)) {   // uniform
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const bool in = !ROWS || row0 + row + n * STEP < valid;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const bool col = COLS == kAnyCols ? c + t < D : COLS == kVecCols ? c < D : true;
          r[n][t] = in && col ? r[n][t] : 0.f;
        }
      }
    }
  }
  __device__ __forceinline__ void commit(float* __restrict__ lds, int tid) const {
    float* to = lds + tid / (16 * DB) * LD + 4 * (tid % (16 * DB));
#pragma unroll
    for (int n = 0; n < N; ++n) *reinterpret_cast<f32x4*>(to + n * STEP * LD) = r[n];
  }
};

// acc += W V for one 16-key block: `v` is the block's first row in LDS, w[x] the lane's weight of
// key 4 kq + x (zero where the key is hidden from its row).
template <int DB>
__device__ __forceinline__ void f32_weights_v(f32x4 (&acc)[4 * DB], const float* __restrict__ v,
                                              const f32x4 w, int i, int kq) {
  constexpr int LD = F32Stage<DB, 64, kAllCols>::LD;
  struct Rows { f32x4 b[DB]; };   // this lane's part of key 4 kq + x
  auto read = [&](int x) {
    Rows r;
#pragma unroll
    for (int b = 0; b < DB; ++b)
      r.b[b] = *reinterpret_cast<const f32x4*>(v + (4 * kq + x) * LD + 64 * b + 4 * i);
    return r;
  };
  // the rows of product x + 1 are requested before product x; the fences keep the compiler from
  // requesting all of them at once (registers)
  Rows now = read(0);
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    Rows next = now;
    if (x < 3) next = read(x + 1);
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[4 * b + t] = mfma_f32(now.b[b][t], w[x], acc[4 * b + t]);
    now = next;
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Whether a 16-key block of V holds an infinity or a NaN (in any lane's part of it).  The block on
// the diagonal hides some of its keys from some rows, and a hidden key must not touch a row even
// then: 0 * inf, which a product over all 16 keys cannot avoid.  A wave that finds such a value in
// its diagonal block forms its rows again after the loop, key by key.
__device__ __forceinline__ bool f32_not_finite(const f32x4 r) {
  bool odd = false;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float f = r[t];
    odd |= (~__builtin_bit_cast(uint32_t, f) & 0x7f800000u) == 0u;
  }
  return odd;
}
template <int DB>
__device__ __forceinline__ bool f32_block_not_finite(const float* __restrict__ v, int i, int kq) {
  constexpr int LD = F32Stage<DB, 64, kAllCols>::LD;
  bool odd = false;
#pragma unroll
  for (int x = 0; x < 4; ++x)
#pragma unroll
    for (int b = 0; b < DB; ++b)
      odd |= f32_not_finite(*reinterpret_cast<const f32x4*>(v + (4 * kq + x) * LD + 64 * b + 4 * i));
  return __any(odd);
}

// x / by as the division gives it but for the last bit in rare cases: one reciprocal serves a whole row
// (a division is ten instructions).  Infinities and NaN are those of the product.
__device__ __forceinline__ float f32_divide(float x, float by, float inv) {
  const float q = x * inv, rest = fmaf(-q, by, x);
  return rest == rest ? fmaf(rest, inv, q) : q;
}

// The lane's share of its output row: o points at the row, acc is divided by `by` unless that is known to be 1.
template <int DB, int COLS, bool DIVIDE>
__device__ __forceinline__ void f32_store_row(float* __restrict__ o, const f32x4 (&acc)[4 * DB],
                                              float by, int kq, int D) {
  const float inv = DIVIDE ? 1.f / by : 1.f;
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int d = 64 * b + 16 * kq + 4 * x;
      f32x4 w = {acc[4 * b][x], acc[4 * b + 1][x], acc[4 * b + 2][x], acc[4 * b + 3][x]};
      if (DIVIDE)
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] = f32_divide(w[t], by, inv);
      if constexpr (COLS == kVecCols || COLS == kAllCols) {
        if (COLS == kAllCols || d < D) *reinterpret_cast<f32x4*>(o + d) = w;
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (d + t < D) o[d + t] = w[t];
      }
    }
}

// Which rows a wave owns.  The rows of all g heads that share K and V are cut into units of 16
// rows of one head, numbered row block first, head second; a workgroup takes four consecutive
// units, last ones first.  Its waves then walk (nearly) the same keys, K and V are staged once for
// all of them, and only the lightest workgroup can have idle waves.
struct F32Unit {
  int tile, head, block;   // (item, KV head), head within the group, 16-row block (-1: no unit)
  int last_block;          // the workgroup's last row block
};
// Workgroup order: ids equal mod 8 (one XCD, one L2) share K and V.  A launch that the chip holds
// nearly at once (up to kF32Spread workgroups) takes the heaviest workgroup of EVERY tile first,
// so that no compute unit ends up with several heavy ones (384 heads of 94 x 128 causal, 640
// workgroups: 29.5 -> 25.3 us exact, 25.4 -> 23.1 us reuse); a larger one finishes tile by tile,
// while its K and V are in the L2.  Of the former every second 32 workgroups of an XCD go out in the other order, so
// that the compute units (32 per XCD, filled one after the other) that got the heaviest get the lightest
// next (the same shape 21.7 -> 20.8 and 21.9 -> 21.2 us).  Not where a compute unit holds two workgroups (exact, D > 128):
// the third 32 then wait for the lightest to end, 16 x 24 heads of 94 x 256 43.3 us so, 39.6 in one order.
constexpr int kF32Spread = 2048;
constexpr int kXcdCus = 32;
template <bool MIRROR>
__device__ __forceinline__ F32Unit f32_unit(int bid, int wave, int g, int S, int n_tiles) {
  const int n_units = g * ((S + kF32Rows - 1) / kF32Rows), per_tile = (n_units + 3) >> 2;
  const int tiles8 = (n_tiles + 7) >> 3;
  const bool spread = gridDim.x <= kF32Spread;
  int slot = bid >> 3;
  if (MIRROR && spread && (slot & kXcdCus) && (slot | (kXcdCus - 1)) < (int)(gridDim.x >> 3)) slot ^= kXcdCus - 1;
  F32Unit u;
  u.tile = (spread ? slot % tiles8 : slot / per_tile) * 8 + (bid & 7);
  const int top = n_units - 1 - 4 * (spread ? slot / tiles8 : slot % per_tile), n = top - wave;
  u.last_block = top / g;
  u.block = n >= 0 ? n / g : -1;
  u.head = n >= 0 ? n % g : 0;
  if (u.tile >= n_tiles) u.tile = -1;
  return u;
}
inline unsigned f32_grid(int n_tiles, int g, int S) {
  const size_t per_tile = ((size_t)g * ((S + kF32Rows - 1) / kF32Rows) + 3) / 4;
  return (unsigned)((n_tiles + 7) / 8 * 8 * per_tile);
}

}  // namespace ac

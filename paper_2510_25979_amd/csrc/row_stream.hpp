// Rows times one vector, by one workgroup: sums over a row's columns on the vector ALUs.
#pragma once
#include <algorithm>

#include "common.hpp"

namespace ac {

// Columns [c, c + P) of a row, P = 16 bytes' worth, and their values as binary32.  fp16 rows are
// whole pieces (E % 8 == 0); fp32 rows may end in part of one and need not be 16-byte aligned.
template <typename T>
struct RowPiece;
template <>
struct RowPiece<f16_t> {
  static constexpr int P = 8;
  f16x8 w;
  __device__ __forceinline__ void load(const f16_t* row, int c, int) {
    w = *reinterpret_cast<const f16x8*>(row + c);
  }
  __device__ __forceinline__ float at(int t) const { return (float)w[t]; }
};
template <>
struct RowPiece<float> {
  static constexpr int P = 4;
  f32x4 w;
  __device__ __forceinline__ void load(const float* row, int c, int E) {
    typedef f32x4 f32x4_dw __attribute__((aligned(4)));
    if (c + P <= E) {
      w = *reinterpret_cast<const f32x4_dw*>(row + c);
    } else {
#pragma unroll
      for (int t = 0; t < P; ++t) w[t] = c + t < E ? row[c + t] : 0.f;
    }
  }
  __device__ __forceinline__ float at(int t) const { return w[t]; }
};

// The eight threads of a row add up their parts of eight rows in three exchanges of half of what is left (four, two,
// one value), so that thread part8 ends up with row part8 of its eight: seven exchanges instead of 24, and every
// thread holds one row.
__device__ __forceinline__ float row_of_eight(float (&v)[8], int part8) {
#define AC_HALVE(n, bit, ctrl)                                                                       \
  _Pragma("unroll") for (int u = 0; u < n; ++u) {                                                    \
    const float keep = (part8 & bit) ? v[u + n] : v[u], give = (part8 & bit) ? v[u] : v[u + n];      \
    v[u] = keep + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, give),  \
                                                                     ctrl, 0xf, 0xf, true));         \
  }
  AC_HALVE(4, 4, 0x141)   // row_half_mirror: lane 7 - p of the eight
  AC_HALVE(2, 2, 0x4e)    // quad_perm 2 3 0 1: lane p ^ 2
  AC_HALVE(1, 1, 0xb1)    // quad_perm 1 0 3 2: lane p ^ 1
#undef AC_HALVE
  return v[0];
}

// Every row of a matrix [n_rows][n_cols] against one vector by a workgroup of 1,024 threads, eight threads a row.
// Bound by the latency of its first loads, then by the 64 bytes per clock of a compute unit: a thread has U rows of C
// pieces in flight, U C = 8 (128 KB a workgroup and step, about 1 us), the next ones while these are multiplied.  U is
// taken so that rows and columns fill the steps (stream_unroll).
constexpr int kStreamThreads = 1024;

// stage() puts the vector into vec (LDS; zeros up to the next multiple of 64 columns) while the first rows are on their way.
// done(r, s) has row r's sum: of products, or of -(vec - row)^2 for L2.
template <typename T, bool L2, int U, typename Stage, typename Done>
__device__ __forceinline__ void stream_rows(const T* rows, int n_rows, int n_cols, const float* vec, Stage stage, Done done) {
  typedef RowPiece<T> Piece;
  constexpr int P = Piece::P, RPT = kStreamThreads / 8, C = 8 / U, STEP = 8 * P * C;   // columns of a step
  const int slot = threadIdx.x >> 3, part8 = threadIdx.x & 7, last_piece = (n_cols - 1) / P * P;
  struct Pieces { Piece p[U][C]; };
  auto fetch = [&](int row0, int c0) {   // what lies past the end repeats something that does not
    Pieces f;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T* row = rows + (size_t)min(row0 + RPT * u + slot, n_rows - 1) * n_cols;
#pragma unroll
      for (int i = 0; i < C; ++i) f.p[u][i].load(row, min(c0 + P * (part8 + 8 * i), last_piece), n_cols);
    }
    return f;
  };
  Pieces now = fetch(0, 0);
  stage();
  __syncthreads();
  float acc[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) acc[u] = 0.f;
  int row0 = 0, c0 = 0;
#pragma unroll 1
  while (true) {
    const bool last = c0 + STEP >= n_cols;   // of these rows
    const int next_row = last ? row0 + RPT * U : row0, next_c = last ? 0 : c0 + STEP;
    const bool more = next_row < n_rows;
    Pieces next;
    if (more) next = fetch(next_row, next_c);
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int c = c0 + P * (part8 + 8 * i);
      if (c < n_cols) {
#pragma unroll
        for (int t = 0; t < P; ++t) {
          const float v = vec[c + t];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (L2) {
              const float d = v - now.p[u][i].at(t);
              acc[u] = fmaf(-d, d, acc[u]);
            } else {
              acc[u] = fmaf(v, now.p[u][i].at(t), acc[u]);
            }
          }
        }
      }
    }
    if (last) {
      const float s = row_of_eight(acc, part8);   // thread p of a row's eight: row RPT p + slot of the first U
      const int r = row0 + RPT * part8 + slot;
      if (part8 < U && r < n_rows) done(r, s);
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[u] = 0.f;
    }
    if (!more) break;
    now = next;
    row0 = next_row;
    c0 = next_c;
  }
}

// Steps with U = u, for elements of which P make 16 bytes.
inline long stream_steps(int P, int n_rows, int n_cols, int u) {
  const int rows = kStreamThreads / 8 * u, cols = 64 * P / u;
  return (((long)n_rows + rows - 1) / rows) * ((n_cols + cols - 1) / cols);
}
// The fewest that any U takes.
inline long stream_least(int P, int n_rows, int n_cols) {
  long least = stream_steps(P, n_rows, n_cols, 8);
  for (int u = 4; u >= 1; u /= 2) least = std::min(least, stream_steps(P, n_rows, n_cols, u));
  return least;
}
// The U of the fewest steps (of equals the most rows, whose parts are added up the fewest times).  A single row of each
// thread is a longer step: it has to save a third of them.  Search, us with one row / more: 640 x 256 fp32 (5 / 6 steps)
// 9.6 / 9.0, the best 4 of 300 x 512 fp16 (3 / 4) 11.2 / 9.4, 300 x 512 fp32 (6 / 8) 10.4 / 10.6, 100 x 640 fp16 (2 / 3) 6.2 / 6.7.
inline int stream_unroll(int P, int n_rows, int n_cols) {
  int best = 8;
  for (int u = 4; u >= 2; u /= 2)
    if (stream_steps(P, n_rows, n_cols, u) < stream_steps(P, n_rows, n_cols, best)) best = u;
  return 3 * stream_steps(P, n_rows, n_cols, 1) <= 2 * stream_steps(P, n_rows, n_cols, best) ? 1 : best;
}

}  // namespace ac

// Algorithm 1, search and threshold steps: exact top-k similarity search of a
// batch of query feature vectors against the whole feature-vector database,
// then hit / miss routing.  (The paper uses an approximate graph index; this
// is the exact search that index approximates.)
//
// Two phases.
//  1. score + group maximum.  The database rows are split into contiguous
//     groups (one workgroup each).  The N x B score matrix is never written:
//     a workgroup forms its scores on the matrix cores (fp16 inputs, fp32
//     accumulation) and keeps, per query, only the best (score, row) of the
//     group under the order "higher score, then lower row".
//  2. finalise.  k = 1: the best group maximum is the answer.  k > 1: every
//     member of the exact top-k lies in one of the k groups with the best
//     maxima (each such group holds at least one of the k best elements), so
//     those k groups are re-scored row by row and the k best rows selected.
//     Groups are contiguous and ascend, so among equal maxima the lower group
//     number stands for the lower row and only the score has to be kept.
// fp32 databases (and the L2 metric) use a vector-ALU phase 1 of the same shape, or, for more work, matrix-core
// bounds that tell which rows have to be scored (search_bound_kernel).
// Both phases are one launch, a workgroup per query, for databases of some 100 KB to 1 MB (search_small).
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "row_stream.hpp"

namespace ac {

constexpr int kQPad = 8;            // fp16 elements of padding per staged query row
constexpr int kValuRowsPerWg = 256;
constexpr int kNarrowBytes = 160;   // widest rows of search_row_kernel
constexpr int kIdxNone = 0x7fffffff;
constexpr int kMaxK = 64;           // AC_MAX_K of the C interface
constexpr int kUnsure = -2;         // idx[b][0] between two launches: what the bounds leave open is searched row by row
// Maximum of a group (k > 1) in which no row ranks, every score being NaN.  -infinity is a score like
// any other: a group that holds one comes before a group that holds none.  (Rows past the end count as
// -infinity: they are in the last group only, which no other group has to come after.)
constexpr float kNoRow = __builtin_nanf("");

struct SearchArgs {
  const void* emb;
  const void* q;
  const int32_t* map_of;
  int32_t N, E, B, k, metric;
  int32_t q0, nq;          // queries handled by this launch
  int32_t rows, G;         // group size and count (a group: the rows one partial result covers)
  int32_t wg_rows;         // rows one phase-1 workgroup scans: one group (k = 1) or several
  float threshold;
  float* part_s;           // [B][G] best score of each group (k > 1: kNoRow where no row ranks)
  int32_t* part_i;         // [B][G] its row (k = 1 only)
  float* cand;             // [B][k * rows] scores of the selected groups' rows (k > 1 only)
  int32_t* unsure;         // 1 where a query is left open: the launches that get it search those with idx[b][0] == kUnsure, whose
                           // score[b][0] is the k-th best score found
  int32_t* idx;
  float* score;
  int32_t* hit;
};

// (s1, i1) ranks before (s0, i0): higher score, or equal score and lower row.
__device__ __forceinline__ bool ranks_before(float s1, int i1, float s0, int i0) {
  return s1 > s0 || (s1 == s0 && i1 < i0);
}

// Best (score, row) over a workgroup; result valid in every thread.
__device__ __forceinline__ void block_argmax(float& s, int& i, float* red_s, int* red_i) {
  for (int off = 32; off > 0; off >>= 1) {
    const float so = __shfl_xor(s, off);
    const int io = __shfl_xor(i, off);
    if (ranks_before(so, io, s, i)) { s = so; i = io; }
  }
  const int wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();   // red_* may still be read from a previous call
  if ((threadIdx.x & 63) == 0) { red_s[wave] = s; red_i[wave] = i; }
  __syncthreads();
  s = red_s[0]; i = red_i[0];
  for (int w = 1; w < nw; ++w)
    if (ranks_before(red_s[w], red_i[w], s, i)) { s = red_s[w]; i = red_i[w]; }
}

// Largest x of the wave in every lane: four steps inside rows of 16 lanes, two across.
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
#define AC_DPP_MAX(ctrl, rows) \
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, ctrl, rows, 0xf, false))
  AC_DPP_MAX(0x111, 0xf);   // row_shr:1, 2, 4, 8
  AC_DPP_MAX(0x112, 0xf);
  AC_DPP_MAX(0x114, 0xf);
  AC_DPP_MAX(0x118, 0xf);
  AC_DPP_MAX(0x142, 0xa);   // lane 15 of a row into the next one
  AC_DPP_MAX(0x143, 0xc);   // lane 31 into the upper half: lane 63 has seen them all
#undef AC_DPP_MAX
  return __builtin_amdgcn_readlane(x, 63);
}
// Scores as whole numbers in the same order (no NaN; zeros compare equal); 0 stands for "none".
__device__ __forceinline__ uint32_t score_key(float s) {
  const uint32_t b = __builtin_bit_cast(uint32_t, s + 0.f);   // -0 becomes +0
  return b ^ ((uint32_t)((int32_t)b >> 31) | 0x80000000u);
}
__device__ __forceinline__ float key_score(uint32_t k) {
  return __builtin_bit_cast(float, k ^ (k >> 31 ? 0x80000000u : 0xffffffffu));
}
// What the second phase is handed as the maximum of a group (k > 1): where no row ranks, the NaN whose key
// comes after that of -infinity (it is key_score(0)), so that the selection need not test for it.
__device__ __forceinline__ float group_max(float s) { return s == s ? s : key_score(0u); }

// ---------------------------------------------------------------- phase 1, matrix cores
// KSMAX > 0: a wave keeps its 32 rows whole in registers (E <= 16 KSMAX, E % 16 == 0) and multiplies
// them with one query block after the other.  KSMAX = 0, any E % 8 == 0 whose queries fit in LDS:
// the rows pass through registers 64 columns at a time, every piece feeding all NQB query blocks
// (20,000 x 768, 64 queries: 103 us per call on the vector ALUs, 28 us so).
template <int KSMAX, int NQB, bool TOPK>
__global__ __launch_bounds__(kThreads) void search_f16_kernel(const SearchArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int E = a.E, QS = ((E + 15) & ~15) + kQPad;
  f16_t* qs = reinterpret_cast<f16_t*>(smem);                                 // [32 NQB][QS]
  float* red_s = reinterpret_cast<float*>(smem + (size_t)32 * NQB * QS * 2);  // [4][32 NQB]
  int* red_i = reinterpret_cast<int*>(red_s + 4 * 32 * NQB);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it scalar
  const int il = lane & 31, kh = lane >> 5;
  const int nks = (E + 15) >> 4;
  const int q0 = a.q0 + 32 * NQB * blockIdx.y, nq = min(a.q0 + a.nq - q0, 32 * NQB);   // this workgroup's queries

  // stage the query super-block, zeros beyond nq and beyond an odd last half step
  {
    const int EQ = E >> 3;
    const u32x4* src = reinterpret_cast<const u32x4*>(reinterpret_cast<const f16_t*>(a.q) +
                                                      (size_t)q0 * E);
    for (int p = tid; p < 32 * NQB * 2 * nks; p += kThreads) {
      const int r = p / (2 * nks), c = p % (2 * nks);
      u32x4 w = {0u, 0u, 0u, 0u};
      if (r < nq && c < EQ) w = src[(size_t)r * EQ + c];
      *reinterpret_cast<u32x4*>(qs + r * QS + 8 * c) = w;
    }
  }
  __syncthreads();

  constexpr float none = TOPK ? kNoRow : -INFINITY;
  float best_s[NQB];
  int best_i[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) { best_s[qb] = none; best_i[qb] = kIdxNone; }

  const int row_begin = blockIdx.x * a.wg_rows;
  const int row_end = min(row_begin + a.wg_rows, a.N);
  const f16_t* emb = reinterpret_cast<const f16_t*>(a.emb);
  for (int pass = row_begin; pass < row_end; pass += 128) {   // the same trips for all four waves
    const int rb = pass + 32 * wave;
    // database operand: lane (il, kh) holds emb[rb + il][16 ks + 8 kh .. +8); rows past the
    // end are clamped for the load and masked below
    const int rowc = min(rb + il, a.N - 1);
    const f16_t* erow = emb + (size_t)rowc * E + 8 * kh;
    // acc[v] = <emb[rb + mfma_row(v)], q[32 qb + il]>; rows ascend with v, so a strict
    // comparison keeps the lowest row among equal scores
    auto rank = [&](int qb, const f32x16& acc) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = rb + mfma_row(v, kh);
        const float s = r < a.N ? acc[v] : -INFINITY;
        if (TOPK) {
          best_s[qb] = fmaxf(best_s[qb], s);
        } else if (s > best_s[qb]) {
          best_s[qb] = s;
          best_i[qb] = r;
        }
      }
    };
    if constexpr (KSMAX > 0) {
      f16x8 e[KSMAX];
#pragma unroll
      for (int ks = 0; ks < KSMAX; ++ks)
        if (ks < nks) e[ks] = *reinterpret_cast<const f16x8*>(erow + 16 * ks);
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const f16_t* qrow = qs + (32 * qb + il) * QS + 8 * kh;
#pragma unroll
        for (int ks = 0; ks < KSMAX; ++ks)
          if (ks < nks) acc = mfma_f16(e[ks], *reinterpret_cast<const f16x8*>(qrow + 16 * ks), acc);
        rank(qb, acc);
      }
    } else {
      f32x16 acc[NQB];
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[qb][v] = 0.f;
      struct Four { f16x8 e[4]; };
      auto fetch = [&](int ks0) {   // steps past the end repeat a piece of the row, their products are skipped
        Four f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int c = 16 * (ks0 + t);
          f.e[t] = *reinterpret_cast<const f16x8*>(erow + (c + 8 * kh < E ? c : 0) - (8 * kh < E ? 0 : 8 * kh));
          if (c + 8 * kh >= E) {
#pragma unroll
            for (int x = 0; x < 8; ++x) f.e[t][x] = (f16_t)0.f;
          }
        }
        return f;
      };
      Four now = fetch(0);
      for (int ks0 = 0; ks0 < nks; ks0 += 4) {
        const Four next = fetch(ks0 + 4);
#pragma unroll
        for (int t = 0; t < 4; ++t)
          if (ks0 + t < nks) {
#pragma unroll
            for (int qb = 0; qb < NQB; ++qb)
              acc[qb] = mfma_f16(now.e[t], *reinterpret_cast<const f16x8*>(qs + (32 * qb + il) * QS + 8 * kh + 16 * (ks0 + t)),
                                 acc[qb]);
          }
        now = next;
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) rank(qb, acc[qb]);
    }
    if (TOPK) {   // group maxima leave as soon as a group is complete
      const bool per_wave = a.rows == 32;   // a wave's 32 rows are a group: nothing to merge
      const int gi = (per_wave ? rb : pass) / a.rows;
      if (!per_wave && pass + 128 < row_end && (pass + 128) / a.rows == gi) continue;   // uniform
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const float s = fmaxf(best_s[qb], __shfl_xor(best_s[qb], 32));
        best_s[qb] = none;
        const int t = 32 * qb + il;
        if (!per_wave) {
          if (kh == 0) red_s[wave * 32 * NQB + t] = s;
        } else if (kh == 0 && t < nq && rb < a.N) {
          a.part_s[(size_t)(q0 + t) * a.G + gi] = group_max(s);
        }
      }
      if (!per_wave) {   // one group per pass (or several passes): the four waves meet in LDS
        __syncthreads();
        for (int t = tid; t < nq; t += kThreads)
          a.part_s[(size_t)(q0 + t) * a.G + gi] =
              group_max(fmaxf(fmaxf(red_s[t], red_s[32 * NQB + t]), fmaxf(red_s[64 * NQB + t], red_s[96 * NQB + t])));
        __syncthreads();
      }
    }
  }
  if (TOPK) return;
  // combine the two lane halves
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const float so = __shfl_xor(best_s[qb], 32);
    const int io = __shfl_xor(best_i[qb], 32);
    if (ranks_before(so, io, best_s[qb], best_i[qb])) { best_s[qb] = so; best_i[qb] = io; }
  }
  // one group per workgroup: the four waves meet in LDS
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    if (kh == 0) {
      red_s[wave * 32 * NQB + 32 * qb + il] = best_s[qb];
      red_i[wave * 32 * NQB + 32 * qb + il] = best_i[qb];
    }
  }
  __syncthreads();
  for (int t = tid; t < nq; t += kThreads) {
    float s = red_s[t];
    int i = red_i[t];
    for (int w = 1; w < 4; ++w) {
      const float so = red_s[w * 32 * NQB + t];
      const int io = red_i[w * 32 * NQB + t];
      if (ranks_before(so, io, s, i)) { s = so; i = io; }
    }
    a.part_s[(size_t)(q0 + t) * a.G + blockIdx.x] = s;
    a.part_i[(size_t)(q0 + t) * a.G + blockIdx.x] = i;
  }
}

// ---------------------------------------------------------------- phase 1, query-stationary
// For more than 64 queries, and for large databases at any batch size, the roles are swapped: the QUERIES live in registers (each of the
// four waves keeps QPW blocks of 32 queries as MFMA column operands for the whole kernel) and
// the database rows stream through LDS in chunks of 64 rows.  Every row operand read from LDS
// feeds QPW MFMAs per wave and is shared by the four waves, so LDS traffic is 4x the HBM
// stream instead of 32x, and no cross-wave reduction is needed (a wave owns its queries).
//
// The chunks are copied global -> LDS directly (global_load_lds_dwordx4: no data registers; a
// wave instruction fills 1 KiB of LDS contiguously, lane l at base + 16 l, whatever global
// address lane l names), double-buffered in two separate LDS arrays so that the copy of chunk
// c+1 runs while chunk c is multiplied.  Rows are stored unpadded; piece p (16 bytes) of row r
// sits at position p ^ (r & 15) of its row, which makes the 16-byte operand reads of 32
// consecutive rows conflict-free; the copy obtains the swizzle for free by choosing which
// global piece each lane fetches.
constexpr int kBigRows = 64;   // database rows per LDS chunk

template <int KSMAX, int QPW, bool TOPK>
__global__ __launch_bounds__(kThreads, (KSMAX == 32 ? 1 : 2)) void search_f16_big_kernel(const SearchArgs a) {
  constexpr int E = 16 * KSMAX;               // this kernel is built for E = 128, 256, 512
  constexpr int EQ = E / 8;                   // 16-byte pieces per row
  constexpr int NDMA = kBigRows * EQ / kWave / 4;   // copy instructions per wave and chunk
  __shared__ __attribute__((aligned(16))) f16_t buf0[kBigRows * E];
  __shared__ __attribute__((aligned(16))) f16_t buf1[kBigRows * E];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it scalar
  const int il = lane & 31, kh = lane >> 5;

  // query operands: lane (il, kh) keeps q[q0 + 32 (QPW wave + j) + il][16 ks + 8 kh .. +8)
  f16x8 qop[QPW][KSMAX];
#pragma unroll
  for (int j = 0; j < QPW; ++j) {
    const int qi = 32 * (QPW * wave + j) + il;
    const f16_t* qrow = reinterpret_cast<const f16_t*>(a.q) + (size_t)(a.q0 + min(qi, a.nq - 1)) * E + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < KSMAX; ++ks) {
      qop[j][ks] = *reinterpret_cast<const f16x8*>(qrow + 16 * ks);
      if (qi >= a.nq) {   // padding query: all-zero operand
#pragma unroll
        for (int e = 0; e < 8; ++e) qop[j][ks][e] = (f16_t)0.f;
      }
    }
  }

  const int row_begin = blockIdx.x * a.wg_rows;
  const int row_end = min(row_begin + a.wg_rows, a.N);
  const int n_chunk = (row_end - row_begin + kBigRows - 1) / kBigRows;
  const f16_t* emb = reinterpret_cast<const f16_t*>(a.emb);

  // copy chunk ch into buf: instruction k = wave + 4 i fills LDS slots [64 k, 64 k + 64) of the
  // chunk (slot = row * EQ + position).  The element offset of the global piece a lane fetches
  // with instruction i, relative to the chunk's first row, is fixed for the whole kernel.
  unsigned coff[NDMA];
#pragma unroll
  for (int i = 0; i < NDMA; ++i) {
    const int slot = kWave * (wave + 4 * i) + lane;
    const int row = slot / EQ, pos = slot % EQ;
    coff[i] = (unsigned)(row * E + 8 * (pos ^ (row & 15)));
  }
  auto copy_in = [&](f16_t* buf, int ch) {
    const f16_t* src = emb + (size_t)(row_begin + ch * kBigRows) * E;
#pragma unroll
    for (int i = 0; i < NDMA; ++i) {
      const f16_t* piece = src + coff[i];
      __builtin_amdgcn_global_load_lds(piece, buf + kWave * (wave + 4 * i) * 8, 16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // the same for a chunk that reaches beyond the database: rows past the end repeat the last
  // row (they are masked when compared)
  auto copy_in_clamped = [&](f16_t* buf, int ch) {
    const int first = row_begin + ch * kBigRows;
    const f16_t* src = emb + (size_t)first * E;   // uniform; lanes add a small 32-bit offset
    const int last = a.N - 1 - first;
#pragma unroll
    for (int i = 0; i < NDMA; ++i) {
      const int slot = kWave * (wave + 4 * i) + lane;
      const int row = slot / EQ, pos = slot % EQ;
      const unsigned off = (unsigned)(min(row, last) * E + 8 * (pos ^ (row & 15)));
      const f16_t* piece = src + off;
      __builtin_amdgcn_global_load_lds(piece, buf + kWave * (wave + 4 * i) * 8, 16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  constexpr float none = TOPK ? kNoRow : -INFINITY;
  float best_s[QPW];
  int best_i[QPW];
#pragma unroll
  for (int j = 0; j < QPW; ++j) { best_s[j] = none; best_i[j] = kIdxNone; }

  // RAGGED is a literal at both call sites and the body is inlined: the copy used for complete
  // chunks carries no per-row tests
  // LDS element offset of this lane's operand piece of contraction step ks (row il of a 32-row
  // block; piece 2 ks + kh at position (2 ks + kh) ^ (il & 15)).  The exchange only touches the
  // low four bits of the piece index, so steps ks and ks + 8 lie exactly 16 pieces apart:
  // eight offsets serve every width, the rest is an immediate.
  int eoff[8];
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) eoff[ks] = il * E + 8 * ((2 * ks + kh) ^ (il & 15));
  auto operand = [&](const f16_t* buf, int rb, int ks) {
    return *reinterpret_cast<const f16x8*>(buf + eoff[ks & 7] + 128 * (ks >> 3) + 32 * rb * E);
  };

  // RAGGED is a literal at both call sites and the body is inlined: the copy used for complete
  // chunks carries no per-row tests.  The operand reads run two steps ahead of the products
  // (three operand registers in rotation), the fences keep that order in the instruction stream.
  auto compute = [&](const f16_t* buf, int ch, const bool RAGGED) __attribute__((always_inline)) {
    const int cbase = row_begin + ch * kBigRows;
    constexpr int NRB = kBigRows / 32;
    f16x8 eop[3];
    eop[0] = operand(buf, 0, 0);
    eop[1] = operand(buf, 0, 1);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      f32x16 acc[QPW];
#pragma unroll
      for (int j = 0; j < QPW; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < KSMAX; ++ks) {
        const int t = rb * KSMAX + ks;   // step within the chunk: the reads run on into the next block
        if (ks + 2 < KSMAX) eop[(t + 2) % 3] = operand(buf, rb, ks + 2);
        else if (rb + 1 < NRB) eop[(t + 2) % 3] = operand(buf, rb + 1, ks + 2 - KSMAX);
#pragma unroll
        for (int j = 0; j < QPW; ++j) acc[j] = mfma_f16(eop[t % 3], qop[j][ks], acc[j]);
        __builtin_amdgcn_sched_barrier(0);
      }
      // acc[j][v] = <emb[r], q>.  A new best becomes rare as the scan proceeds, so first only the
      // block maximum is compared; the position is looked up only when some lane improved.
      // Rows ascend with v, rb and ch, so strict comparisons keep the lowest row among equals.
      if (RAGGED) {
        const int rbase = cbase + 32 * rb + 4 * kh;
#pragma unroll
        for (int j = 0; j < QPW; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (rbase + 8 * (v >> 2) + (v & 3) >= row_end) acc[j][v] = -INFINITY;
      }
      // Only WHICH 32-row block holds a lane's best score is remembered (one compare and two
      // selects per block and query block); the row inside that block is found by the
      // finalising kernel, which re-scores the 32 rows of the one winning block per query.
      // Looking the position up here was the expensive part: with 64 lanes and a few dozen
      // blocks per workgroup some lane improves in nearly every block, so a wave-wide
      // "did anyone improve" test almost never skipped the 48-instruction search.
      // Blocks ascend with rb and ch, so the strict comparison keeps the lowest block among equals.
      const int blk = ch * (kBigRows / 32) + rb;
#pragma unroll
      for (int j = 0; j < QPW; ++j) {
        float mx = fmaxf(fmaxf(acc[j][0], acc[j][1]), acc[j][2]);
#pragma unroll
        for (int v = 3; v < 15; v += 2) mx = fmaxf(fmaxf(mx, acc[j][v]), acc[j][v + 1]);
        mx = fmaxf(mx, acc[j][15]);
        if (TOPK) {
          best_s[j] = fmaxf(best_s[j], mx);
        } else {
          const bool up = mx > best_s[j];
          best_s[j] = up ? mx : best_s[j];
          best_i[j] = up ? blk : best_i[j];
        }
      }
      // the next block's products must not start before these comparisons are done: a second
      // live set of result registers does not fit next to the query operands
      __builtin_amdgcn_sched_barrier(0);
    }
    if (TOPK) {   // a group is one or several chunks: its maxima leave with its last chunk
      const int next = cbase + kBigRows, gi = cbase / a.rows;
      if (next >= row_end || next / a.rows != gi) {
#pragma unroll
        for (int j = 0; j < QPW; ++j) {
          const float s = fmaxf(best_s[j], __shfl_xor(best_s[j], 32));
          best_s[j] = none;
          const int qi = 32 * (QPW * wave + j) + il;
          if (kh == 0 && qi < a.nq) a.part_s[(size_t)(a.q0 + qi) * a.G + gi] = group_max(s);
        }
      }
    }
  };
  // own copies landed (they are counted like loads), then everybody's
  auto publish = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };

  // Complete chunks run through the test-free copy of the loop body, two per trip so that the
  // buffers alternate without pointer arithmetic; a last incomplete chunk (end of the group
  // or of the database) goes through the clamped copy and the masked comparison.
  const int n_full = (row_end - row_begin) / kBigRows;
  if (n_full > 0) copy_in(buf0, 0); else copy_in_clamped(buf0, 0);
  publish();
  int ch = 0;
  for (; ch + 1 < n_full; ch += 2) {
    copy_in(buf1, ch + 1);
    compute(buf0, ch, false);
    publish();
    if (ch + 2 < n_full) copy_in(buf0, ch + 2);
    else if (ch + 2 < n_chunk) copy_in_clamped(buf0, ch + 2);
    compute(buf1, ch + 1, false);
    publish();
  }
  for (; ch < n_chunk; ++ch) {   // at most one complete and one incomplete chunk are left
    f16_t* cur = (ch & 1) ? buf1 : buf0;
    f16_t* nxt = (ch & 1) ? buf0 : buf1;
    if (ch + 1 < n_chunk) {
      if (ch + 1 < n_full) copy_in(nxt, ch + 1); else copy_in_clamped(nxt, ch + 1);
    }
    compute(cur, ch, true);
    publish();
  }
  if (TOPK) return;
  // combine the two lane halves; every wave owns its queries, nothing else to merge
#pragma unroll
  for (int j = 0; j < QPW; ++j) {
    if (best_i[j] != kIdxNone)   // block -> its first database row (the stand-in for "the row")
      best_i[j] = row_begin + 32 * best_i[j];
    const float so = __shfl_xor(best_s[j], 32);
    const int io = __shfl_xor(best_i[j], 32);
    if (ranks_before(so, io, best_s[j], best_i[j])) { best_s[j] = so; best_i[j] = io; }
    const int qi = 32 * (QPW * wave + j) + il;
    if (kh == 0 && qi < a.nq) {
      a.part_s[(size_t)(a.q0 + qi) * a.G + blockIdx.x] = best_s[j];
      a.part_i[(size_t)(a.q0 + qi) * a.G + blockIdx.x] = best_i[j];
    }
  }
}

// ------------------------------------------------------------- vector-ALU scoring
// phase 1 for NQ <= 8 queries per workgroup on the vector ALUs: a stream over the rows.  Eight threads
// read a row side by side in 16-byte pieces, a thread has eight rows (32 apart) in flight, the
// queries sit in LDS as binary32; a workgroup takes the 256 rows of a group.  Nothing but the queries
// goes through LDS and no barrier sits in the loop, which is what a memory-bound (or, on a small
// database, latency-bound) search wants: 1M x 128 fp32, one query, 96 us = 5.3 TB/s (165 us with a
// thread per row); 200,000 x 768 fp16, one query, 68 us (210 us through the tiles below).  With many
// queries the tiles win, their rows feed more queries (launch_valu_k).
template <typename T, bool L2, int NQ, bool TOPK>
__global__ __launch_bounds__(kThreads) void search_stream_kernel(const SearchArgs a) {
  typedef RowPiece<T> Piece;
  constexpr int P = Piece::P, U = kValuRowsPerWg / 32;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int Ep = (a.E + 7) & ~7;
  float* qf = reinterpret_cast<float*>(smem);           // [NQ][Ep]
  __shared__ float red_s[4][NQ][TOPK ? 4 : 1];
  __shared__ int red_i[4][NQ];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int slot = tid >> 3, part8 = tid & 7;
  const int row0 = blockIdx.x * kValuRowsPerWg;
  const T* emb = reinterpret_cast<const T*>(a.emb);
  const T* row[U];
#pragma unroll
  for (int u = 0; u < U; ++u) row[u] = emb + (size_t)min(row0 + 32 * u + slot, a.N - 1) * a.E;
  Piece now[U];   // the first pieces are on their way while the queries are staged
  if (P * part8 < a.E) {
#pragma unroll
    for (int u = 0; u < U; ++u) now[u].load(row[u], P * part8, a.E);
  }
  const int q0 = blockIdx.y * NQ;
  const T* q = reinterpret_cast<const T*>(a.q) + (size_t)q0 * a.E;
#pragma unroll
  for (int j = 0; j < NQ; ++j)
    for (int c = tid; c < Ep; c += kThreads)
      qf[j * Ep + c] = q0 + j < a.B && c < a.E ? (float)q[(size_t)j * a.E + c] : 0.f;
  __syncthreads();
  float acc[U][NQ];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < NQ; ++j) acc[u][j] = 0.f;
  for (int c = P * part8; c < a.E; c += 8 * P) {
    Piece next[U];
    const int cn = min(c + 8 * P, a.E - 1) / P * P;   // past the end: any piece of the row, unused
#pragma unroll
    for (int u = 0; u < U; ++u) next[u].load(row[u], cn, a.E);
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      float qv[P];
#pragma unroll
      for (int t = 0; t < P; ++t) qv[t] = qf[j * Ep + c + t];
#pragma unroll
      for (int t = 0; t < P; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (L2) {
            const float d = qv[t] - now[u].at(t);
            acc[u][j] = fmaf(-d, d, acc[u][j]);
          } else {
            acc[u][j] = fmaf(qv[t], now[u].at(t), acc[u][j]);
          }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) now[u] = next[u];
  }
  const int r = row0 + 32 * part8 + slot;
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = acc[u][j];
    const float s = row_of_eight(v, part8);
    if (TOPK) {   // groups of 64 rows: threads 2 p and 2 p + 1 of every eight
      float m = r < a.N ? s : -INFINITY;
#pragma unroll
      for (int off = 1; off < kWave; off = off == 1 ? 8 : 2 * off) m = fmaxf(m, __shfl_xor(m, off));
      if (lane < 8) red_s[wave][j][TOPK ? lane >> 1 : 0] = m;
    } else {
      const bool ranks = r < a.N && s == s;   // a NaN never ranks
      const uint32_t key = ranks ? score_key(s) : 0u, top = wave_max(key);
      const uint32_t low = wave_max(ranks && key == top ? ~(uint32_t)r : 0u);   // lowest row
      if (lane == 0) {
        red_s[wave][j][0] = top ? key_score(top) : -INFINITY;
        red_i[wave][j] = top ? (int)~low : kIdxNone;
      }
    }
  }
  __syncthreads();
  if (tid >= NQ || q0 + tid >= a.B || row0 >= a.N) return;   // (the grid may be padded, see stream_groups)
  const size_t out = (size_t)(q0 + tid) * a.G;
  if (TOPK) {
    float all = kNoRow;
    for (int p = 0; p < U / 2; ++p) {
      const int pp = TOPK ? p : 0;
      const float v = fmaxf(fmaxf(red_s[0][tid][pp], red_s[1][tid][pp]), fmaxf(red_s[2][tid][pp], red_s[3][tid][pp]));
      all = fmaxf(all, v);
      if (a.rows == 64 && row0 + 64 * p < a.N) a.part_s[out + row0 / 64 + p] = group_max(v);
    }
    if (a.rows != 64) a.part_s[out + blockIdx.x] = group_max(all);
  } else {
    float s = red_s[0][tid][0];
    int i = red_i[0][tid];
    for (int w = 1; w < 4; ++w)
      if (ranks_before(red_s[w][tid][0], red_i[w][tid], s, i)) { s = red_s[w][tid][0]; i = red_i[w][tid]; }
    a.part_s[out + blockIdx.x] = s;
    a.part_i[out + blockIdx.x] = i;
  }
}

// phase 1 for narrow rows: a thread per row, a workgroup per group of 256 rows and query.  A row is a few
// pieces, which leave the eight threads of the stream above little to share and the tiles below mostly
// padding.  Every score is one chain of fmas over ascending columns.
template <typename T, bool L2, bool TOPK>
__global__ __launch_bounds__(kThreads) void search_row_kernel(const SearchArgs a) {
  typedef RowPiece<T> Piece;
  constexpr int P = Piece::P;
  __shared__ __attribute__((aligned(16))) float qf[kNarrowBytes / sizeof(T)];
  __shared__ float red_s[4];
  __shared__ int red_i[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y, gidx = blockIdx.x, r = gidx * kValuRowsPerWg + tid;
  if (gidx * kValuRowsPerWg >= a.N) return;   // (padding)
  const T* row = reinterpret_cast<const T*>(a.emb) + (size_t)min(r, a.N - 1) * a.E;
  Piece now;   // on its way while the query is staged
  now.load(row, 0, a.E);
  if (tid < ((a.E + P - 1) & -P))
    qf[tid] = tid < a.E ? (float)reinterpret_cast<const T*>(a.q)[(size_t)b * a.E + tid] : 0.f;
  __syncthreads();
  float s = 0.f;
#pragma unroll 2
  for (int c = 0; c < a.E; c += P) {
    Piece next;
    next.load(row, c + P < a.E ? c + P : c, a.E);
#pragma unroll
    for (int t = 0; t < P; ++t) {
      const float q = qf[c + t];
      const float d = q - now.at(t);
      s = L2 ? fmaf(-d, d, s) : fmaf(q, now.at(t), s);
    }
    now = next;
  }
  const bool ranks = r < a.N && s == s;
  const uint32_t key = ranks ? score_key(s) : 0u, top = wave_max(key);
  if (TOPK && a.rows == kWave) {   // the wave's rows are a group
    if (lane == 0 && r < a.N) a.part_s[(size_t)b * a.G + r / kWave] = key_score(top);
    return;
  }
  const uint32_t low = TOPK ? 0u : wave_max(ranks && key == top ? ~(uint32_t)r : 0u);   // lowest row
  if (lane == 0) {
    red_s[wave] = TOPK || top ? key_score(top) : -INFINITY;
    red_i[wave] = top ? (int)~low : kIdxNone;
  }
  __syncthreads();
  if (tid != 0) return;
  s = red_s[0];
  int i = red_i[0];
  for (int w = 1; w < 4; ++w) {
    if (TOPK) s = fmaxf(s, red_s[w]);
    else if (ranks_before(red_s[w], red_i[w], s, i)) { s = red_s[w]; i = red_i[w]; }
  }
  a.part_s[(size_t)b * a.G + gidx] = TOPK ? group_max(s) : s;
  if (!TOPK) a.part_i[(size_t)b * a.G + gidx] = i;
}

// phase 1 on the vector ALUs (binary32 databases, the Euclidean metric, and the fp16 widths that no
// matrix-core kernel is built for).  A workgroup scores the 256 rows of its group against 4 QW
// queries: rows and queries go through LDS in slices of 32 columns (as binary32; the next
// slice is in registers meanwhile), wave w takes queries QW w .. QW w + QW - 1, a lane four rows
// 64 apart, so one row read feeds QW queries, one (broadcast) query read four rows, and the
// index is read once per 4 QW queries instead of once per query.  Every score is one chain of
// fmas over ascending columns.
// Bound by the vector ALUs: two instructions per element of q - e (Euclidean), one per product.
// 100,000 x 128 fp32, 64 queries, Euclidean: 885 us with one row per thread and one query per
// workgroup, 49 us so (42 us at the full issue rate).  Sixteen queries per workgroup leave some six
// workgroups per compute unit there, so the last, partly filled round costs little.
constexpr int kTileCols = 32;
constexpr int kTileLd = kTileCols + 4;   // 16-byte reads of 16 consecutive rows spread over all banks

// kTileCols columns of `rows` rows, kThreads / 8 rows at a time, on their way to LDS as binary32
template <typename T, int N>
struct TileSlice {
  f32x4 r[N];
  __device__ __forceinline__ void load(const T* __restrict__ src, int row0, int n_rows, int E, int e0,
                                       int tid) {
    const int c = e0 + 4 * (tid & 7);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int row = row0 + (tid >> 3) + n * (kThreads / 8);
      r[n] = f32x4{0.f, 0.f, 0.f, 0.f};   // columns past E add nothing, rows past the end are masked
      if (row < n_rows && c < E) {
        const T* at = src + (size_t)row * E + c;
        if (c + 4 <= E) {
          typedef T T4 __attribute__((ext_vector_type(4)));
          typedef T4 T4_elem __attribute__((aligned(sizeof(T) == 2 ? 8 : 4)));   // odd fp32 widths
          const T4 v = *reinterpret_cast<const T4_elem*>(at);
#pragma unroll
          for (int t = 0; t < 4; ++t) r[n][t] = (float)v[t];
        } else {
#pragma unroll
          for (int t = 0; t < 4; ++t)
            if (c + t < E) r[n][t] = (float)at[t];
        }
      }
    }
  }
  __device__ __forceinline__ void commit(float* lds, int tid) const {
#pragma unroll
    for (int n = 0; n < N; ++n)
      *reinterpret_cast<f32x4*>(lds + ((tid >> 3) + n * (kThreads / 8)) * kTileLd + 4 * (tid & 7)) = r[n];
  }
};

template <typename T, bool L2, int QW, bool TOPK>
__global__ __launch_bounds__(kThreads) void search_valu_kernel(const SearchArgs a) {
  constexpr int R = kValuRowsPerWg / kWave;   // rows of a lane
  __shared__ __attribute__((aligned(16))) float el[kValuRowsPerWg * kTileLd];
  __shared__ __attribute__((aligned(16))) float ql[kThreads / 8 * kTileLd];   // 4 QW <= 32 rows used
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the query blocks of one group get ids equal mod 8: one XCD reads the group's rows once
  const int nqb = (a.nq + 4 * QW - 1) / (4 * QW), slot = blockIdx.x >> 3;
  const int gidx = slot / nqb * 8 + (blockIdx.x & 7), q0 = a.q0 + slot % nqb * (4 * QW);
  if (gidx >= (a.N + kValuRowsPerWg - 1) / kValuRowsPerWg) return;
  const T* emb = reinterpret_cast<const T*>(a.emb);
  const T* qs = reinterpret_cast<const T*>(a.q);
  const int row0 = gidx * kValuRowsPerWg;

  float acc[R][QW];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < QW; ++j) acc[r][j] = 0.f;
  TileSlice<T, kValuRowsPerWg * 8 / kThreads> es;
  TileSlice<T, 1> qt;
  const int q_end = min(a.q0 + a.nq, q0 + 4 * QW);
  es.load(emb, row0, a.N, a.E, 0, tid);
  qt.load(qs, q0, q_end, a.E, 0, tid);
  for (int e0 = 0; e0 < a.E; e0 += kTileCols) {
    __syncthreads();   // the previous slice has been read by everybody
    es.commit(el, tid);
    qt.commit(ql, tid);
    __syncthreads();
    if (e0 + kTileCols < a.E) {
      es.load(emb, row0, a.N, a.E, e0 + kTileCols, tid);
      qt.load(qs, q0, q_end, a.E, e0 + kTileCols, tid);
    }
#pragma unroll
    for (int c = 0; c < kTileCols; c += 4) {
      f32x4 e[R];
#pragma unroll
      for (int r = 0; r < R; ++r)
        e[r] = *reinterpret_cast<const f32x4*>(el + (lane + kWave * r) * kTileLd + c);
#pragma unroll
      for (int j = 0; j < QW; ++j) {
        const f32x4 q = *reinterpret_cast<const f32x4*>(ql + (QW * wave + j) * kTileLd + c);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            if (L2) {
              const float d = q[t] - e[r][t];
              acc[r][j] = fmaf(-d, d, acc[r][j]);
            } else {
              acc[r][j] = fmaf(q[t], e[r][t], acc[r][j]);
            }
          }
      }
    }
  }
  if (TOPK) {   // groups of 64 rows (those of one r) or of all 256
#pragma unroll
    for (int j = 0; j < QW; ++j) {
      const int q = q0 + QW * wave + j;
      float all = kNoRow;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int first = row0 + kWave * r;
        const bool ranks = first + lane < a.N && acc[r][j] == acc[r][j];
        const float s = key_score(wave_max(ranks ? score_key(acc[r][j]) : 0u));
        all = fmaxf(all, s);
        if (a.rows == kWave && lane == 0 && q < q_end && first < a.N)
          a.part_s[(size_t)q * a.G + first / kWave] = s;
      }
      if (a.rows != kWave && lane == 0 && q < q_end) a.part_s[(size_t)q * a.G + gidx] = group_max(all);
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < QW; ++j) {
    float s = -INFINITY;
    int i = kIdxNone;
#pragma unroll
    for (int r = 0; r < R; ++r) {   // rows ascend with r: a strict comparison keeps the lowest
      const int row = row0 + lane + kWave * r;
      if (row < a.N && ranks_before(acc[r][j], row, s, i)) { s = acc[r][j]; i = row; }
    }
    for (int off = 32; off > 0; off >>= 1) {
      const float so = __shfl_xor(s, off);
      const int io = __shfl_xor(i, off);
      if (ranks_before(so, io, s, i)) { s = so; i = io; }
    }
    const int q = q0 + QW * wave + j;
    if (lane == 0 && q < q_end) {
      a.part_s[(size_t)q * a.G + gidx] = s;
      a.part_i[(size_t)q * a.G + gidx] = i;
    }
  }
}

// ---------------------------------------------------------------- phase 1, bounds from the matrix cores
// Binary32 inner products and Euclidean distances of a larger search: the tiles above are bound by the vector ALUs (two
// instructions per element of q - e), a contraction on the matrix cores would lose digits where it cancels.  So the matrix
// cores only say which rows can be among the best: for every (query, group) this kernel writes an upper bound of the score
// that the vector ALUs would compute, less the query's own part, and the second phase scores the rows of the groups with the
// best bounds exactly, then those of every other group whose bound reaches the k-th best score found (finalize_bounds_kernel).
//   bound[q][g] = max over the rows e of g of  2 <q, e> - (1 - c) |e|^2   (Euclidean)   or   <q, e> + c/2 |e|^2   (inner product);
// with (c - 1) |q|^2 or c/2 |q|^2 added no row's computed score lies above it.  Values of a magnitude for
// which this does not hold, and NaN, become +infinity: the group is scored.
// c, relative to (|q|^2 + |e|^2) >= 2 |q| |e| >= 2 sum |q_i e_i|: a binary32 value is taken as the sum of two bf16 (rest 2^-18 of it)
// and the product of the two low parts is left out: 3 * 2^-18 |q| |e|; each of at most 3 (E + 15) additions on the matrix cores
// costs no more than 2^-23 of the sum of magnitudes; |e|^2, in E / 2 steps, E 2^-25 of itself; the exact scores, |q|^2 and the last
// few steps (E + 4) 2^-23: together below 2^-16 + (E + 16) 2^-20.
// The rows are read once for 32 NQB queries, straight into registers as the row-stationary kernel reads them.
__host__ __device__ inline float bound_slack(int E) { return 0x1p-16f + (float)(E + 16) * 0x1p-20f; }
constexpr float kBoundMost = 0x1p100f;   // larger magnitudes of a bound, or of its parts, are not relied on
constexpr float kBoundLeast = 0x1p-90f;  // what products lost below the smallest normal numbers add up to, at most

// What the bound of a row has to reach that may score s with a query of |q|^2 = qq; -infinity where bounds are not relied on.
template <bool L2>
__device__ __forceinline__ float bound_reach(float s, float qq, int E) {
  const float c = bound_slack(E), reach = s - 0x1p-20f * fabsf(s) + (L2 ? (1.f - c) * qq : -0.5f * c * qq) - kBoundLeast;
  return qq < kBoundMost && reach > -kBoundMost ? reach : -INFINITY;
}
__host__ __device__ inline int bound_query(int E) { return ((E + 15) & ~15) + kQPad; }   // 16-bit elements of a staged query

template <typename T> struct BoundParts;   // eight columns of a row or query as operands of the matrix cores
template <>
struct BoundParts<float> {
  static constexpr int N = 2;
  typedef bf16x8 op;
  op p[2];
  // (the low part is what the 16 bits kept above leave: the difference is exact)
  __device__ __forceinline__ void set(const f32x4& a, const f32x4& b) {
    u32x4 high, low;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float x = t < 2 ? a[2 * t] : b[2 * t - 4], y = t < 2 ? a[2 * t + 1] : b[2 * t - 3];
      high[t] = pack_bf16(x, y);
      low[t] = pack_bf16(x - __builtin_bit_cast(float, high[t] << 16), y - __builtin_bit_cast(float, high[t] & 0xffff0000u));
    }
    p[0] = __builtin_bit_cast(bf16x8, high);
    p[1] = __builtin_bit_cast(bf16x8, low);
  }
  static __device__ __forceinline__ f32x16 product(const BoundParts& e, const BoundParts& q, f32x16 acc) {
    acc = mfma_bf16(e.p[0], q.p[0], acc);
    acc = mfma_bf16(e.p[1], q.p[0], acc);
    return mfma_bf16(e.p[0], q.p[1], acc);
  }
};
template <>
struct BoundParts<f16_t> {
  static constexpr int N = 1;
  typedef f16x8 op;
  op p[1];
  static __device__ __forceinline__ f32x16 product(const BoundParts& e, const BoundParts& q, f32x16 acc) {
    return mfma_f16(e.p[0], q.p[0], acc);
  }
};

// Columns of a step of 16 that a lane of half kh holds, as they come from memory: fp16 columns 8 kh .. + 8, fp32 columns
// 4 kh .. + 4 and 8 + 4 kh .. + 4, so that the two lanes of a row read neighbouring 16-byte pieces.  Zeros past E.
template <typename T> struct BoundPiece;
template <>
struct BoundPiece<float> {
  f32x4 a, b;
  __device__ __forceinline__ void load(const float* row, int c0, int kh, int E, bool whole) {
    typedef f32x4 f32x4_dw __attribute__((aligned(4)));
    const int c = c0 + 4 * kh;
    if (whole) {
      a = *reinterpret_cast<const f32x4_dw*>(row + c);
      b = *reinterpret_cast<const f32x4_dw*>(row + c + 8);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        a[t] = c + t < E ? row[c + t] : 0.f;
        b[t] = c + 8 + t < E ? row[c + 8 + t] : 0.f;
      }
    }
  }
  __device__ __forceinline__ void parts(BoundParts<float>& p) const { p.set(a, b); }
  __device__ __forceinline__ void load_whole(const float* row, int c0, int kh) {   // (16-byte aligned)
    a = *reinterpret_cast<const f32x4*>(row + c0 + 4 * kh);
    b = *reinterpret_cast<const f32x4*>(row + c0 + 4 * kh + 8);
  }
  __device__ __forceinline__ void values(f32x4& x, f32x4& y) const { x = a; y = b; }
  __device__ __forceinline__ float squares(float s) const {
#pragma unroll
    for (int t = 0; t < 4; ++t) s = fmaf(a[t], a[t], fmaf(b[t], b[t], s));
    return s;
  }
};
template <>
struct BoundPiece<f16_t> {
  f16x8 a;
  __device__ __forceinline__ void load(const f16_t* row, int c0, int kh, int E, bool whole) {
    if (whole || c0 + 8 * kh < E) {   // (E % 8 == 0)
      a = *reinterpret_cast<const f16x8*>(row + c0 + 8 * kh);
    } else {
#pragma unroll
      for (int t = 0; t < 8; ++t) a[t] = (f16_t)0.f;
    }
  }
  __device__ __forceinline__ void parts(BoundParts<f16_t>& p) const { p.p[0] = a; }
  __device__ __forceinline__ void load_whole(const f16_t* row, int c0, int kh) { a = *reinterpret_cast<const f16x8*>(row + c0 + 8 * kh); }
  __device__ __forceinline__ void values(f32x4& x, f32x4& y) const {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      x[t] = (float)a[t];
      y[t] = (float)a[4 + t];
    }
  }
  __device__ __forceinline__ float squares(float s) const {
#pragma unroll
    for (int t = 0; t < 8; ++t) s = fmaf((float)a[t], (float)a[t], s);
    return s;
  }
};

// The products of rows [row_begin, row_end) with queries [q0, q0 + nq), up to 32 NQB.  done(pass, rb, acc, part, all, same) has those of
// the wave's rows rb .. rb + 31 in each of the passes of 128 rows: acc[qb][v] = <row rb + mfma_row(v, kh), query 32 qb + il>, that
// row's share of the bound in part[v >> 2][v & 3], and whether the block has a row whose bound is not relied on.
// kAgain and kCentred (search_unsure_kernel): bit t > 0 of `same` is set where rows rb + t and rb + t - 1 are the same, and qq[t] is |q|^2
// of query t.  kCentred: row row_begin is subtracted from rows and queries first, which leaves their distance as it is.
// LDS: qs [Parts::N][32 NQB][QS]; own [4][32]; qq [32 NQB] (not kFirst); ref [QS] (kCentred).
enum { kFirst = 0, kAgain = 1, kCentred = 2 };
template <typename T, bool L2, int NQB, int MODE, typename Done>
__device__ __forceinline__ void bound_products(const SearchArgs& a, int row_begin, int row_end, int q0, int nq, uint16_t* qs, float* own,
                                               T* ref, float* qq, int wave, Done done) {
  typedef BoundParts<std::conditional_t<MODE == kCentred, float, T>> Parts;
  typedef BoundPiece<T> Piece;
  typedef typename Parts::op op;
  const int E = a.E, nks = (E + 15) >> 4, QS = 16 * nks + kQPad;   // (bound_query(E))
  const int tid = threadIdx.x, lane = tid & 63;
  const int il = lane & 31, kh = lane >> 5;
  const T* emb = reinterpret_cast<const T*>(a.emb);

  struct Four { Piece p[4]; };
  auto fetch = [&](const T* row, int ks0) {   // steps past the end repeat the last one, their products are skipped
    Four f;
    if (16 * (ks0 + 4) <= E) {
#pragma unroll
      for (int t = 0; t < 4; ++t) f.p[t].load(row, 16 * (ks0 + t), kh, E, true);
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int c = 16 * min(ks0 + t, nks - 1);
        f.p[t].load(row, c, kh, E, c + 16 <= E);
      }
    }
    return f;
  };
  auto row_of = [&](int pass) { return emb + (size_t)min(pass + 32 * wave + il, a.N - 1) * E; };   // past the end: the last row again
  const T* row = row_of(row_begin);
  Four now = fetch(row, 0);   // on its way while the queries are staged

  const T* ref_row = emb + (size_t)row_begin * E;
  if (MODE == kCentred)
    for (int c = tid; c < 16 * nks; c += kThreads) ref[c] = c < E ? ref_row[c] : (T)0.f;
  float own_qq[NQB] = {};
  // eight threads a query; a thread's pieces of all query blocks are in flight together
#pragma unroll 2
  for (int c = tid & 7; c < 2 * nks; c += 8) {   // half step
    Piece w[NQB];
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
      w[qb].load(reinterpret_cast<const T*>(a.q) + (size_t)(q0 + min(32 * qb + (tid >> 3), nq - 1)) * E, 16 * (c >> 1), c & 1, E,
                 16 * (c >> 1) + 16 <= E);
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      Parts p;
      if constexpr (MODE == kFirst) {
        w[qb].parts(p);
      } else {
        f32x4 x, y;
        w[qb].values(x, y);
        if constexpr (MODE == kCentred) {
          Piece r;
          f32x4 rx, ry;
          r.load(ref_row, 16 * (c >> 1), c & 1, E, 16 * (c >> 1) + 16 <= E);
          r.values(rx, ry);
          x -= rx;
          y -= ry;
          p.set(x, y);
        } else {
          w[qb].parts(p);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) own_qq[qb] = fmaf(x[t], x[t], fmaf(y[t], y[t], own_qq[qb]));
      }
#pragma unroll
      for (int n = 0; n < Parts::N; ++n)
        *reinterpret_cast<op*>(qs + (size_t)(32 * NQB * n + 32 * qb + (tid >> 3)) * QS + 8 * c) = p.p[n];
    }
  }
  if (MODE != kFirst) {
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
      for (int off = 1; off < 8; off <<= 1) own_qq[qb] += __shfl_xor(own_qq[qb], off);
      if ((tid & 7) == 0) qq[32 * qb + (tid >> 3)] = own_qq[qb];
    }
  }
  __syncthreads();

  for (int pass = row_begin; pass < row_end; pass += 128) {   // the same trips for all four waves
    const int rb = pass + 32 * wave;
    const bool more = pass + 128 < row_end;
    const T* next_row = row_of(more ? pass + 128 : pass);
    f32x16 acc[NQB];
    float sq = 0.f;
    uint32_t differ = 0;   // bits that the row does not share with the one before it
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[qb][v] = 0.f;
    auto step = [&](const Piece& piece, int ks) {
      Parts e;
      if (MODE != kFirst) {   // (from the lane before it)
        constexpr int W = sizeof(Piece) / 4;
        typedef uint32_t words __attribute__((ext_vector_type(W)));
        const words w = __builtin_bit_cast(words, piece);
#pragma unroll
        for (int t = 0; t < W; ++t) differ |= w[t] ^ (uint32_t)__builtin_amdgcn_update_dpp((int)~w[t], (int)w[t], 0x138, 0xf, 0xf, false);
      }
      if constexpr (MODE == kCentred) {
        f32x4 x, y, rx, ry;
        piece.values(x, y);
        Piece r;
        r.load_whole(ref, 16 * ks, kh);
        r.values(rx, ry);
        x -= rx;
        y -= ry;
        e.set(x, y);
#pragma unroll
        for (int t = 0; t < 4; ++t) sq = fmaf(x[t], x[t], fmaf(y[t], y[t], sq));
      }
      if constexpr (MODE != kCentred) {
        piece.parts(e);
        sq = piece.squares(sq);
      }
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        Parts q;
#pragma unroll
        for (int n = 0; n < Parts::N; ++n)
          q.p[n] = *reinterpret_cast<const op*>(qs + (size_t)(32 * NQB * n + 32 * qb + il) * QS + 16 * ks + 8 * kh);
        acc[qb] = Parts::product(e, q, acc[qb]);
      }
    };
    int ks0 = 0;
    for (; ks0 + 4 <= nks; ks0 += 4) {
      const bool last = ks0 + 4 >= nks;
      Four next;
      if (!last || more) next = fetch(last ? next_row : row, last ? 0 : ks0 + 4);
#pragma unroll
      for (int t = 0; t < 4; ++t) step(now.p[t], ks0 + t);
      now = next;
    }
    if (ks0 < nks) {
      Four next;
      if (more) next = fetch(next_row, 0);
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (ks0 + t < nks) step(now.p[t], ks0 + t);
      now = next;
    }
    row = next_row;
    // acc[qb][v] = <emb[rb + mfma_row(v)], q[32 qb + il]>; lane il has half of that row's |e|^2.  Where all squares stay below
    // kBoundMost so do the products; a block with a row where they don't is scored whatever its other rows are.
    sq += __shfl_xor(sq, 32);
    const bool all = __ballot(!(sq < kBoundMost)) != 0;
    const float c = L2 ? bound_slack(E) - 1.f : 0.5f * bound_slack(E);
    if (kh == 0) own[32 * wave + il] = c * sq;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    f32x4 part[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) part[v] = *reinterpret_cast<const f32x4*>(own + 32 * wave + mfma_row(4 * v, kh));
    if (MODE != kFirst) differ |= __shfl_xor((int)differ, 32);
    done(pass, rb, acc, part, all, MODE == kFirst ? 0u : (uint32_t)__ballot(il > 0 && differ == 0));
  }
}

template <typename T, bool L2, int NQB>
__global__ __launch_bounds__(kThreads) void search_bound_kernel(const SearchArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint16_t* qs = reinterpret_cast<uint16_t*>(smem);
  float* red = reinterpret_cast<float*>(qs + (size_t)BoundParts<T>::N * 32 * NQB * bound_query(a.E));   // [4][32 NQB]
  float* own = red + 4 * 32 * NQB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int q0 = 32 * NQB * blockIdx.y, nq = min(a.B - q0, 32 * NQB);
  const int row_begin = blockIdx.x * a.wg_rows, row_end = min(row_begin + a.wg_rows, a.N);
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *a.unsure = 0;
  auto keep = [&](int pass, int rb, const f32x16 (&acc)[NQB], const f32x4 (&part)[4], bool all, uint32_t) __attribute__((always_inline)) {
    const bool per_wave = a.rows == 32;   // a wave's 32 rows are a group
    const int gi = (per_wave ? rb : pass) / a.rows;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      float best = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float w = part[v >> 2][v & 3];
        best = fmaxf(best, L2 ? fmaf(2.f, acc[qb][v], w) : acc[qb][v] + w);
      }
      const float s = all ? INFINITY : max_with_other_half(best);
      const int t = 32 * qb + il;
      if (!per_wave) {
        if (kh == 0) red[wave * 32 * NQB + t] = s;
      } else if (kh == 0 && t < nq && rb < a.N) {
        a.part_s[(size_t)(q0 + t) * a.G + gi] = s;
      }
    }
    if (!per_wave) {
      __syncthreads();
      if (a.rows == 64) {
        for (int x = tid; x < 2 * 32 * NQB; x += kThreads) {
          const int t = x % (32 * NQB), half = x / (32 * NQB), first = pass + 64 * half;
          if (t < nq && first < a.N)
            a.part_s[(size_t)(q0 + t) * a.G + first / 64] = fmaxf(red[64 * NQB * half + t], red[64 * NQB * half + 32 * NQB + t]);
        }
      } else {
        for (int t = tid; t < nq; t += kThreads)
          a.part_s[(size_t)(q0 + t) * a.G + gi] =
              fmaxf(fmaxf(red[t], red[32 * NQB + t]), fmaxf(red[64 * NQB + t], red[96 * NQB + t]));
      }
      __syncthreads();
    }
  };
  bound_products<T, L2, NQB, kFirst>(a, row_begin, row_end, q0, nq, qs, own, (T*)nullptr, nullptr, wave, keep);
}

// The scores of what bounds have left open: for a query with idx[b][0] == kUnsure every row whose own bound reaches score[b][0], the
// k-th best score found so far, is scored, and the best of each group takes the place of the group's bound (kNoRow: none reaches).
// Rows alike are few of a group, and rows far from the origin are not far from each other, so the bounds are formed again, by
// row and (Euclidean) of the differences to one of the workgroup's rows.  A workgroup takes wg_rows rows (128 or 256) and 32 NQB queries,
// eight threads the score of a row and query; of neighbours that are the same they take the first.  Where more than kUnsurePairs reach, all
// are scored, kUnsureRows rows of an eight by eight queries.  (A thread a row and query, each reading its own lines, took three times as long.)
// Usually nothing is open, so the grid is one that is quickly through.
// us per call, 100,000 x 128 fp32 Euclidean, 64 queries; exact scores of all rows first, / all rows of what is left open in tiles / so: 40 rows
// at random places alike for each query 58 / 75 / 48; all rows of 40 kinds 59 / 77 / 58; rows 100 times their spread from the origin 57 / 73 / 47; all
// rows the same 58 / 75 / 56.  Two kinds in random order, of which every third row reaches, so that all are scored, 57 / 73 / 118 (one row at a time 166; fp16
// 100,000 x 256 118 / 139 / 201, 335): the vector ALUs take 55 of it, on 391 workgroups for 256 compute units.  Five kinds, one in ten 57 / 73 / 91.
constexpr int kUnsurePairs = 2048;   // (twice as many cost fp16 rows of 256 columns the second workgroup of a compute unit)
constexpr int kUnsureRows = 4;
template <typename T, bool L2, int NQB, int MODE>
__global__ __launch_bounds__(kThreads, 2) void search_unsure_kernel(const SearchArgs a) {
  typedef RowPiece<T> Piece;
  constexpr int P = Piece::P, NQ = 32 * NQB, Parts = MODE == kCentred ? 2 : BoundParts<T>::N;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ uint16_t pairs[kUnsurePairs * NQB];   // row of the workgroup << 6 | query
  __shared__ uint32_t top[NQ][8];                  // best of the query's rows 32 t .. 32 t + 31
  __shared__ int n_pairs;
  if (*a.unsure == 0) return;
  uint16_t* qs = reinterpret_cast<uint16_t*>(smem);
  T* ref = reinterpret_cast<T*>(qs + (size_t)Parts * NQ * bound_query(a.E));
  float* own = reinterpret_cast<float*>(ref + bound_query(a.E));
  float* qq = own + 4 * 32;
  T* raw = reinterpret_cast<T*>(smem);             // [NQ][QE], once the products are done
  const T* emb = reinterpret_cast<const T*>(a.emb);
  const int QE = ((a.E + 7) & ~7) + kQPad;         // (no more than bound_query, and no multiple of all banks)
  const int tid = threadIdx.x, lane = tid & 63, il = lane & 31, kh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nqb = (a.B + NQ - 1) / NQ, n_rows = (a.N + a.wg_rows - 1) / a.wg_rows;
  const int64_t units = ((int64_t)n_rows + 7) / 8 * 8 * nqb;   // (the query blocks of the same rows on one XCD)
  for (int64_t unit = blockIdx.x; unit < units; unit += gridDim.x) {
    const int ri = (int)((unit >> 3) / nqb) * 8 + (int)(unit & 7), q0 = (int)((unit >> 3) % nqb) * NQ;
    if (ri >= n_rows) continue;
    const int row0 = ri * a.wg_rows, row_end = min(row0 + a.wg_rows, a.N), nq = min(a.B - q0, NQ);
    const bool open_here = lane < nq && a.idx[(size_t)(q0 + min(lane, nq - 1)) * a.k] == kUnsure;
    const unsigned long long opens = __ballot(open_here);   // the same in all waves
    if (opens == 0) continue;
    for (int x = tid; x < NQ * 8; x += kThreads) top[x >> 3][x & 7] = 0;
    if (tid == 0) n_pairs = 0;
    float least[NQB];   // score to be reached
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) least[qb] = a.score[(size_t)(q0 + min(32 * qb + il, nq - 1)) * a.k];
    auto note = [&](int, int rb, const f32x16 (&acc)[NQB], const f32x4 (&part)[4], bool all, uint32_t same) __attribute__((always_inline)) {
      // rows there are, that are not the row before (whose score the group has)
      const uint32_t rows = (rb >= row_end ? 0u : row_end - rb >= 32 ? ~0u : (1u << (row_end - rb)) - 1) & ~same;
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const float reach = bound_reach<L2>(least[qb], qq[32 * qb + il], a.E);
        uint32_t mask = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float w = part[v >> 2][v & 3], bound = L2 ? fmaf(2.f, acc[qb][v], w) : acc[qb][v] + w;
          if (all || !(bound < reach)) mask |= 1u << mfma_row(v, kh);
        }
        mask &= rows;
        if (((opens >> (32 * qb + il)) & 1) == 0 || mask == 0) continue;
        int at = atomicAdd(&n_pairs, __popc(mask));
        for (; mask; mask &= mask - 1, ++at)
          if (at < kUnsurePairs * NQB) pairs[at] = (uint16_t)((rb - row0 + __ffs(mask) - 1) << 6 | (32 * qb + il));
      }
    };
    // (a barrier between the zeros above and note())
    bound_products<T, L2, NQB, MODE>(a, row0, row_end, q0, nq, qs, own, ref, qq, wave, note);
    __syncthreads();
    const int many = n_pairs, part8 = tid & 7;
    constexpr bool STAGED = std::is_same<T, float>::value;   // pairs take the query from LDS (fp16 ones 153 us so, 135 from the L1)
    if (many > (STAGED ? 0 : kUnsurePairs * NQB)) {          // the queries in place of their parts
#pragma unroll 4
      for (int c = P * part8; c < QE - kQPad; c += 8 * P) {
        Piece w[NQB];
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb)
          w[qb].load(reinterpret_cast<const T*>(a.q) + (size_t)(q0 + min(32 * qb + (tid >> 3), nq - 1)) * a.E, c, a.E);
#pragma unroll
        for (int qb = 0; qb < NQB; ++qb) *reinterpret_cast<decltype(w[qb].w)*>(raw + (32 * qb + (tid >> 3)) * QE + c) = w[qb].w;   // (zeros past E)
      }
      __syncthreads();
    }
    if (many <= kUnsurePairs * NQB) {   // scores of eight rows and queries, thread u of the eight has the u-th
      for (int p = tid & ~7; p < many; p += kThreads) {
        int r[8], t[8];
        float acc[8] = {};
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int pair = pairs[min(p + u, many - 1)];
          r[u] = pair >> 6;
          t[u] = pair & 63;
        }
        auto add = [&](int c) __attribute__((always_inline)) {
          Piece e[8], x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            e[u].load(emb + (size_t)(row0 + r[u]) * a.E, c, a.E);
            if constexpr (STAGED) x[u].w = *reinterpret_cast<const decltype(x[u].w)*>(raw + t[u] * QE + c);   // (zeros past E)
            else x[u].load(reinterpret_cast<const T*>(a.q) + (size_t)(q0 + t[u]) * a.E, c, a.E);
          }
#pragma unroll
          for (int i = 0; i < P; ++i)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              const float y = e[u].at(i), d = x[u].at(i) - y;
              acc[u] = L2 ? fmaf(-d, d, acc[u]) : fmaf(x[u].at(i), y, acc[u]);
            }
        };
        if constexpr (STAGED) {
#pragma unroll 2
          for (int c = P * part8; c < a.E; c += 8 * P) add(c);
        } else {
#pragma unroll 1
          for (int c = P * part8; c < a.E; c += 8 * P) add(c);
        }
        const float s = row_of_eight(acc, part8);
        if (p + part8 < many && s == s) {
          int mr = r[0], mt = t[0];
#pragma unroll
          for (int u = 1; u < 8; ++u) {
            mr = part8 == u ? r[u] : mr;
            mt = part8 == u ? t[u] : mt;
          }
          atomicMax(&top[mt][mr >> 5], score_key(s));
        }
      }
    } else {
      // Rows r0 + 32 j of an eight by eight queries; the sums take the steps of those above.
      const int n = row_end - row0;
      for (int r0 = tid >> 3; r0 < n; r0 += 32 * kUnsureRows) {
        const T* row[kUnsureRows];
#pragma unroll
        for (int j = 0; j < kUnsureRows; ++j) row[j] = emb + (size_t)(row0 + min(r0 + 32 * j, n - 1)) * a.E;
        for (int t0 = 0; t0 < NQ; t0 += 8) {
          if (((opens >> t0) & 0xff) == 0) continue;
          const T* x0 = raw + t0 * QE;
          float acc[kUnsureRows][8] = {};
#pragma unroll 2
          for (int c = P * part8; c < a.E; c += 8 * P) {
            Piece e[kUnsureRows];
#pragma unroll
            for (int j = 0; j < kUnsureRows; ++j) e[j].load(row[j], c, a.E);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              Piece x;
              x.w = *reinterpret_cast<const decltype(x.w)*>(x0 + u * QE + c);   // (zeros past E)
#pragma unroll
              for (int i = 0; i < P; ++i)
#pragma unroll
                for (int j = 0; j < kUnsureRows; ++j) {
                  const float y = e[j].at(i), d = x.at(i) - y;
                  acc[j][u] = L2 ? fmaf(-d, d, acc[j][u]) : fmaf(x.at(i), y, acc[j][u]);
                }
            }
          }
#pragma unroll
          for (int j = 0; j < kUnsureRows; ++j) {
            const float s = row_of_eight(acc[j], part8);
            if (r0 + 32 * j < n && s == s && ((opens >> (t0 + part8)) & 1)) atomicMax(&top[t0 + part8][(r0 >> 5) + j], score_key(s));
          }
        }
      }
    }
    __syncthreads();
    for (int x = tid; x < NQ * 8; x += kThreads) {   // groups of 32, 64 or 128 rows
      const int t = x >> 3, per = a.rows >> 5, first = (x & 7) * a.rows;
      if (((opens >> t) & 1) == 0 || first >= row_end - row0) continue;
      uint32_t best = 0;
      for (int y = (x & 7) * per; y < (x & 7) * per + per; ++y) best = max(best, top[t][y]);
      a.part_s[(size_t)(q0 + t) * a.G + (row0 + first) / a.rows] = key_score(best);
    }
    __syncthreads();
  }
}

constexpr size_t kGridThreads = ((size_t)1 << 32) - 1;   // most threads of a launch in one dimension

template <typename T, bool L2, int QW, bool TOPK>
static hipError_t launch_tiles(SearchArgs a, size_t groups8, hipStream_t stream) {
  // the grid is one-dimensional (groups x query blocks, so that it can choose the XCD): a large index
  // with a large batch takes several launches
  const size_t fit = kGridThreads / kThreads / groups8 * (4 * QW);   // queries of a launch
  for (size_t q0 = 0; q0 < (size_t)a.B; q0 += fit) {
    a.q0 = (int32_t)q0;
    a.nq = (int32_t)((size_t)a.B - q0 < fit ? (size_t)a.B - q0 : fit);
    const size_t tiles = groups8 * ((a.nq + 4 * QW - 1) / (4 * QW));
    hipLaunchKernelGGL((search_valu_kernel<T, L2, QW, TOPK>), dim3((unsigned)tiles), dim3(kThreads), 0, stream, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Groups of the grid: with a multiple of eight one XCD gets a group's rows for every query block, and they come
// from its L2 after the first time.  22,464 x 768 fp16 (88 groups), nine queries, 24 us; 20,000 rows (79 groups) 42
// unpadded.  Not where it would leave more than an eighth of the XCDs' time idle.
static unsigned stream_groups(int32_t N) {
  const unsigned groups = (unsigned)(((size_t)N + kValuRowsPerWg - 1) / kValuRowsPerWg), padded = (groups + 7) / 8 * 8;
  return (padded - groups) * 8 <= groups ? padded : groups;
}

constexpr size_t kStreamLds = 128 * 1024;   // eight queries of 4,096 columns
static size_t stream_lds(int nq, int E) { return (size_t)nq * ((E + 7) & ~7) * 4; }

template <typename T, bool L2, int NQ, bool TOPK>
static hipError_t launch_stream(const SearchArgs& a, hipStream_t stream) {
  const size_t lds = stream_lds(NQ, a.E);
  hipError_t e = ensure_lds<&search_stream_kernel<T, L2, NQ, TOPK>>(lds);
  if (e != hipSuccess) return e;
  const dim3 grid(stream_groups(a.N), (unsigned)((a.B + NQ - 1) / NQ));
  hipLaunchKernelGGL((search_stream_kernel<T, L2, NQ, TOPK>), grid, dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <typename T, bool L2, bool TOPK>
static hipError_t launch_rows(const SearchArgs& a, hipStream_t stream) {
  const dim3 grid(stream_groups(a.N), (unsigned)a.B);
  hipLaunchKernelGGL((search_row_kernel<T, L2, TOPK>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

// Rows so narrow that a thread reads one whole: 16 bytes always; more while the threads' reads, a row
// apart, stay in the caches or the call is short.  (Rows 128 bytes apart fall on the same channels.)
// us per call, this way / the best other one: 300,000 x 8 fp16, 8 queries 11.3 / 21.3; 4,000 x 40, 200
// queries, Euclidean 8.4 / 12.0; 20,000 x 8 fp32, 64 queries 8.2 / 9.9; 20,000 x 32, 8 queries 9.5 / 6.8;
// 20,000 x 37, one query 5.7 / 7.5, 8 queries 12.0 / 9.1.
static bool narrow_rows(int32_t is_f16, int32_t E, int32_t B, int32_t N) {
  const size_t bytes = (size_t)E * (is_f16 ? 2 : 4), pieces = (bytes + 15) / 16;
  const size_t work = (size_t)((N + kValuRowsPerWg - 1) / kValuRowsPerWg) * B;   // workgroups
  if (bytes > kNarrowBytes || bytes % 128 == 0 || B > 65535) return false;   // (B: a dimension of the grid)
  return bytes <= 16 || work * pieces <= 3300 || (bytes <= 32 && work <= 16384) || (bytes <= 48 && work <= 8192) ||
         (N * bytes <= 640 * 1024 && work * pieces <= (is_f16 ? 24000 : 5000));
}

template <typename T, bool L2, bool TOPK>
static hipError_t launch_valu_k(const SearchArgs& a, hipStream_t stream) {
  constexpr bool kF16 = std::is_same<T, f16_t>::value;
  const size_t groups = (size_t)(a.N + kValuRowsPerWg - 1) / kValuRowsPerWg, groups8 = (groups + 7) / 8 * 8;
  if (narrow_rows(kF16, a.E, a.B, a.N)) return launch_rows<T, L2, TOPK>(a, stream);
  auto fits = [&](int nq) { return stream_lds(nq, a.E) <= kStreamLds; };
  if (fits(1)) {
    // One query per workgroup while the chip holds them all (nearly) at once: a short call is a chain
    // of latencies, and the other forms leave most of the chip idle.  1,024 x 128 fp32, four queries:
    // 7.0 us with four per workgroup, 4.9 us with one.  More than eight queries, tiles below / one per
    // workgroup: 64 against 1,000 x 256 fp16 23.6 / 7.7; fp32 64 against 1,000 x 256 17.2 / 9.9, 40 against 5,000 x 128 (800
    // workgroups) 11.4 / 10.6, 200 against 2,000 x 128 (1,600) 12.6 / 14.8.  Very wide fp32 rows of a larger database
    // are better shared: 20,000 x 8,192, four queries (316) 414 / 343 in tiles, but 64 x 4,608, 400 (400) 93 / 374.
    const size_t one = groups <= 32 && kF16 ? 640 : !fits(8) && !kF16 ? (a.B <= 8 ? 256 : 512)
                       : a.B <= 8 ? 512 : kF16 ? 1400 : 1024;
    if (groups * a.B <= one) return launch_stream<T, L2, 1, TOPK>(a, stream);
    // fp16 tiles pay for the conversion of every element in LDS: streams of four queries win while their
    // workgroups are few.  One query each / four / tiles: 400 against 1,000 x 768 (1,600) 33 / 24 / 112; 200 against
    // 4,000 x 264, Euclidean (3,200) 66 / 30 / 49, 400 of them (6,400) 66 / 44 / 73.
    if (kF16 && a.B > 8 && fits(4) && groups * a.B <= 6500) return launch_stream<T, L2, 4, TOPK>(a, stream);
    // Larger databases: a stream per eight queries, as long as it beats the tiles.
    // fp16: 136,118 x 384, 16 queries 103 us in tiles, streams 73; x 256, 32
    // queries 95 / 85, 64 queries 152 / 151; 200,000 x 128, 16 queries 51.6 / 49.0; x 96, 17 queries 58 / 64;
    // 300,000 x 72, 16 queries 45 / 70.  fp32: 136,118 x 384, 9 queries 72 / 80.  Rows that leave LDS room for fewer
    // queries: fp16 20,000 x 8,192, 8 queries 876 / 226 four each; 10,000 x 12,000, 32 queries 1,608 / 508 one each.
    if (a.B == 1 || (a.B <= 8 && (kF16 || fits(8))) || (kF16 && a.B <= (a.E >= 256 ? 64 : a.E >= 96 ? 16 : 8))) {
      if (a.B == 1 || !fits(4)) return launch_stream<T, L2, 1, TOPK>(a, stream);
      // (five to eight queries of a database of few groups: two workgroups each, 20,000 x 768 fp16 29 -> 23 us)
      if (a.B <= 4 || !fits(8) || (a.B <= 8 && groups <= 256)) return launch_stream<T, L2, 4, TOPK>(a, stream);
      return launch_stream<T, L2, 8, TOPK>(a, stream);
    }
  }
  // queries per wave: as many as leave some four workgroups per compute unit
  auto blocks = [&](int qw) { return (size_t)((a.B + 4 * qw - 1) / (4 * qw)); };
  const int qw = groups * blocks(4) >= 1024 ? 4 : groups * blocks(2) >= 1024 ? 2 : 1;
  return qw == 1   ? launch_tiles<T, L2, 1, TOPK>(a, groups8, stream)
         : qw == 2 ? launch_tiles<T, L2, 2, TOPK>(a, groups8, stream)
                   : launch_tiles<T, L2, 4, TOPK>(a, groups8, stream);
}

template <typename T>
static hipError_t launch_valu(const SearchArgs& a, hipStream_t stream) {
  if (a.k > 1) return a.metric ? launch_valu_k<T, true, true>(a, stream) : launch_valu_k<T, false, true>(a, stream);
  return a.metric ? launch_valu_k<T, true, false>(a, stream) : launch_valu_k<T, false, false>(a, stream);
}

// ------------------------------------------------------------------- phase 2
__device__ __forceinline__ int entry_of(const SearchArgs& a, int row) { return a.map_of ? a.map_of[row] : row; }
__device__ __forceinline__ void write_entry(const SearchArgs& a, int b, float s0, int entry) {
  float sim = s0;
  if (a.metric == 1) sim = 1.0f - sqrtf(-s0);
  a.hit[b] = (sim >= a.threshold) ? entry : -1;
}
__device__ __forceinline__ void write_hit(const SearchArgs& a, int b, float s0, int i0) {
  if (i0 == kIdxNone) a.hit[b] = -1;   // no row ranked at all (every score of the query is NaN): a miss
  else write_entry(a, b, s0, entry_of(a, i0));
}

// k = 1: best of the group maxima.
__global__ __launch_bounds__(kThreads) void finalize_top1_kernel(const SearchArgs a) {
  __shared__ float red_s[4];
  __shared__ int red_i[4];
  const int b = blockIdx.x;
  float s = -INFINITY;
  int i = kIdxNone;
  for (int gi = threadIdx.x; gi < a.G; gi += kThreads) {
    const float so = a.part_s[(size_t)b * a.G + gi];
    const int io = a.part_i[(size_t)b * a.G + gi];
    if (ranks_before(so, io, s, i)) { s = so; i = io; }
  }
  block_argmax(s, i, red_s, red_i);
  if (threadIdx.x == 0) {
    a.idx[b] = i == kIdxNone ? -1 : i;
    a.score[b] = s;
    write_hit(a, b, s, i);
  }
}

// k = 1 after the query-stationary kernel: the partial results name the first row of the
// 32-row block that holds a group's maximum.  Best group first (lowest block on ties), then
// the 32 rows of that one block are scored again (eight threads per row, fp32) and the best of
// them (lowest row on ties) is the answer; the score reported is the matrix-core one of phase 1.
__global__ __launch_bounds__(kThreads) void finalize_top1_block_kernel(const SearchArgs a) {
  __shared__ float red_s[4];
  __shared__ int red_i[4];
  const int b = blockIdx.x, tid = threadIdx.x;
  float s = -INFINITY;
  int i = kIdxNone;
  for (int gi = tid; gi < a.G; gi += kThreads) {
    const float so = a.part_s[(size_t)b * a.G + gi];
    const int io = a.part_i[(size_t)b * a.G + gi];
    if (ranks_before(so, io, s, i)) { s = so; i = io; }
  }
  block_argmax(s, i, red_s, red_i);
  const f16_t* q = reinterpret_cast<const f16_t*>(a.q) + (size_t)b * a.E;
  const int row = i + (tid >> 3), part = tid & 7;
  float rs = -INFINITY;
  int ri = kIdxNone, entry = -1;
  if (i != kIdxNone && row < a.N) {
    entry = entry_of(a, row);   // (with the row: of the winner later it would be a round trip to memory more)
    const f16_t* e = reinterpret_cast<const f16_t*>(a.emb) + (size_t)row * a.E;
    float acc = 0.f;
    for (int c = 8 * part; c < a.E; c += 64) {   // 16-byte pieces, eight threads side by side
      const f16x8 ev = *reinterpret_cast<const f16x8*>(e + c);
      const f16x8 qv = *reinterpret_cast<const f16x8*>(q + c);
#pragma unroll
      for (int t = 0; t < 8; ++t) acc = fmaf((float)ev[t], (float)qv[t], acc);
    }
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    rs = acc;
    ri = row;
  }
  block_argmax(rs, ri, red_s, red_i);
  if (tid == 0) {
    a.idx[b] = ri == kIdxNone ? -1 : ri;
    a.score[b] = s;
    if (ri == kIdxNone) a.hit[b] = -1;
  }
  if (row == ri && part == 0) write_entry(a, b, s, entry);
}

// An item of a selection: score and number in one word that orders like them (higher score, then
// lower number); 0 stands for "none".
__device__ __forceinline__ uint64_t item_key(float s, int i) {
  return (uint64_t)score_key(s) << 32 | (uint32_t)~i;
}

constexpr int kCountPerDraw = 16;   // items per rank sought that are all compared with each other straight away
constexpr int kRankMost = 384;      // items that are compared with each other after the bound has been applied
// Few ranks are drawn, the best again and again: up to eight of 256 items by one wave without a barrier, up to two of more
// by all waves with a barrier each.  us per call, by bound and comparison / so: 1,895 x 256, two queries, k = 2 (60
// groups, 64 rows) 13.2 / 9.7; 5,000 x 256, 64 queries, k = 8 17.9 / 16.6; 117,042 x 64, three, k = 2 (1,829 groups) 14.9 /
// 13.6; 82,156 x 256 fp32, one, k = 2 27.6 / 26.1.  A draw costs what comparing 14 items does, and two less of them than
// there are: 16 queries, the best 8 of 40 rows compared 5.2, drawn 6.0, of 64 5.5 / 6.0, of 128 6.4 / 6.0; the best 4 of
// 20 5.0 / 5.0, of 64 5.5 / 5.0.
constexpr int kDrawRanks = 8, kDrawItems = 14;

// x of the lane that the DPP control names (a lane without one keeps its own).
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint64_t dpp64(uint64_t x) {
  const int lo = (int)(uint32_t)x, hi = (int)(uint32_t)(x >> 32);
  return (uint64_t)(uint32_t)__builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false) << 32 |
         (uint32_t)__builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
}

// The best item of the lane's four, of its sixteen.
__device__ __forceinline__ uint64_t quad_best(uint64_t x) {
  x = max(x, dpp64<0xb1>(x));          // quad_perm 1 0 3 2
  return max(x, dpp64<0x4e>(x));       // quad_perm 2 3 0 1
}
__device__ __forceinline__ uint64_t row_best(uint64_t x) {
  x = quad_best(x);
  x = max(x, dpp64<0x141>(x));         // row_half_mirror
  return max(x, dpp64<0x140>(x));      // row_mirror
}
// The best item of the wave, in every lane.
__device__ __forceinline__ uint64_t wave_best(uint64_t x) {
  x = row_best(x);
  x = max(x, dpp64<0x142, 0xa>(x));    // lane 15 of a row into the next one
  x = max(x, dpp64<0x143, 0xc>(x));    // lane 31 into the upper half: lane 63 has seen them all
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(x >> 32), 63) << 32 |
         (uint32_t)__builtin_amdgcn_readlane((uint32_t)x, 63);
}

// The k best of n items under the total order "higher score, then lower number", in rank order.
// get(x) is item x as item_key (0: it does not rank, e.g. a NaN score); put(r, s, i) is called once
// for every rank r < k, with kIdxNone where fewer than k items rank.
// An item's rank is the number of items before it, and few items need to be compared: the k-th best of the
// maxima of 64 parts is a bound that k items reach and, in unordered data, some 2 k to 4 k.  Drawing the best k times in
// every wave, then again among what the waves drew, took 36 KB of code and 30.7 us per call of 100,000 x 256, 64 queries,
// k = 8, 141 at k = 64; 23.6 and 57 so.
// Where the best items are neighbours (a database ordered by similarity) they share few parts and any number of items may
// reach the bound.  Then they are counted in 256 equal ranges of keys up to the best one, which raises the bound to where
// at most kRankMost reach it, whatever the data (the same call at k = 64 with runs of 1,000 rows alike: 58 us; k rounds of a
// workgroup-wide arg-max 220).
// Few items for that many ranks are compared straight away, and few ranks drawn (above).
// NT threads, list[NT]: the items that are ranked, before them the best item of every part or the counts, behind them
// the best item, two numbers (items that reach the bound, and how many of them there were counted) and the bound.
template <int NT, typename Get, typename Put>
__device__ __forceinline__ void select_best(int n, int k, Get get, Put put, uint64_t* list) {
  typedef uint32_t __attribute__((may_alias)) word;
  constexpr int MOST = kRankMost < NT - 3 ? kRankMost : NT - 3, BINS = 256;
  uint64_t& top = list[NT - 3];
  word& count = *reinterpret_cast<word*>(list + NT - 2);
  word& reach = *(reinterpret_cast<word*>(list + NT - 2) + 1);
  uint64_t& least = list[NT - 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto item_at = [&](int x) {
    const uint64_t it = get(min(x, n - 1));   // (no load behind a test)
    return x < n ? it : 0;
  };
  // list[0, m) is there: ranks of the items in it that rank at all
  auto rank = [&](int m) {
    uint64_t mine = tid < m ? list[tid] : 0;
    const int ranked = __syncthreads_count(mine != 0);
    if (wave * kWave < m) {
      typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
      int before = 0;
#pragma unroll 4
      for (int x = 0; x + 1 < m; x += 2) {
        const u64x2 o = *reinterpret_cast<const u64x2*>(list + x);
        before += (o.x > mine) + (o.y > mine);
      }
      if (m & 1) before += list[m - 1] > mine;
      if (mine != 0 && before < k) put(before, key_score((uint32_t)(mine >> 32)), (int)~(uint32_t)mine);
    }
    if (tid >= ranked && tid < k) put(tid, -INFINITY, kIdxNone);
    __syncthreads();
  };
  // The bound rises until at most MOST items reach it, k of them at least.  Fewer than k items lie above `top`, so each
  // pass leaves those and one range, and the last one, whose ranges are single keys, no more than k.
  auto raise = [&]() {
    word* bins = reinterpret_cast<word*>(list);
    do {
      const uint64_t low = least, high = top;
      const int shift = max(64 - 8 - (int)__clzll(high - low), 0);
      if (tid < BINS) bins[tid] = 0;
      __syncthreads();
#pragma unroll 1
      for (int x = tid; x < n; x += NT) {
        const uint64_t it = get(x);
        if (it >= low) atomicAdd(&bins[(uint32_t)((min(it, high) - low) >> shift)], 1u);
      }
      __syncthreads();
      if (wave == 0) {
        uint32_t own[4], sum = 0;   // a lane: four neighbouring ranges
#pragma unroll
        for (int t = 0; t < 4; ++t) sum += own[t] = bins[4 * lane + t];
        uint32_t above = sum;
        for (int off = 1; off < kWave; off <<= 1) {
          const uint32_t next = __shfl_down(above, off);
          above += lane + off < kWave ? next : 0;
        }
        above -= sum;   // items of the lanes behind this one
        if (above < (uint32_t)k && above + sum >= (uint32_t)k) {   // one lane
          int bin = 0;
#pragma unroll
          for (int t = 3; t >= 0; --t)
            if (above < (uint32_t)k) {
              above += own[t];
              bin = 4 * lane + t;
            }
          const uint64_t from = low + ((uint64_t)bin << shift);
          least = from;
          top = min(high, from + ((1ull << shift) - 1));
          reach = above;
        }
        if (lane == 0) count = 0;
      }
      __syncthreads();
    } while (reach > (uint32_t)MOST);
  };
  // list := the items that reach the bound.  A thread's first four items stay in registers, others are fetched again.
  auto collect = [&]() {
    uint64_t it[4], best = 0;
    auto fetch = [&](int x) {
#pragma unroll
      for (int t = 0; t < 4; ++t) it[t] = item_at(x + t * NT);
    };
    auto best_of = [&]() {
#pragma unroll
      for (int t = 0; t < 4; ++t) best = max(best, it[t]);
    };
    if (n > 4 * NT) {
#pragma unroll 1
      for (int x = 4 * NT + tid; x < n; x += 4 * NT) {
        fetch(x);
        best_of();
      }
    }
    fetch(tid);
    best_of();
    // parts: NT / 64 neighbouring lanes, or whole waves where there are two of them for every rank and as many as ranks
    // have items (with fewer no bound is found and all items are compared: 295 x 64 fp32, 271 queries, k = 8 27.0 / 19.9)
    const bool waves = 2 * k <= NT / kWave && k * kWave <= n;   // uniform
    const int parts = waves ? NT / kWave : kWave;
    if (waves) {
      best = wave_best(best);
      if (lane == 0) list[wave] = best;
    } else {
      best = NT == 1024 ? row_best(best) : quad_best(best);
      if (tid % (NT / kWave) == 0) list[tid / (NT / kWave)] = best;
    }
    if (tid == 0) count = 0;
    __syncthreads();
    if (wave == 0) {
      const uint64_t mine = lane < parts ? list[lane] : 0;
      int before = 0;
#pragma unroll 4
      for (int x = 0; x < parts; ++x) before += list[x] > mine;
      if (__popcll(__ballot(mine != 0)) < k) {
        if (lane == 0) least = 1;   // fewer parts than that hold an item: all of them count
      } else if (mine != 0 && before == k - 1) {
        least = mine;
      }
      if (mine != 0 && before == 0) top = mine;
    }
    __syncthreads();
#pragma unroll 1
    for (;;) {
      const uint64_t bound = least;
#pragma unroll 1
      for (int x0 = wave * kWave;;) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const bool in = it[t] >= bound;
          const unsigned long long who = __ballot(in);
          if (who == 0) continue;   // (wave-uniform: most)
          int at = 0;
          if (lane == 0) at = (int)atomicAdd(&count, (uint32_t)__popcll(who));
          at = __builtin_amdgcn_readfirstlane(at) + __popcll(who & ((1ull << lane) - 1));
          if (in && at < MOST) list[at] = it[t];
        }
        if ((x0 += 4 * NT) >= n) break;
        fetch(x0 + lane);
      }
      __syncthreads();
      // (256 threads select among up to 1,024 items with k <= 8 or among 256: k of 64 parts hold at most 128)
      if (NT == 256 || __builtin_expect(count <= (uint32_t)MOST, 1)) break;
      raise();
      fetch(tid);
    }
  };
  int m = n;
  const bool many = n > 4 * kWave;   // uniform
  auto draw = [&](auto all_waves) {
    const bool all = all_waves;
    if (!all && wave != 0) return;
    uint64_t it[4], last = ~0ull;
#pragma unroll
    for (int t = 0; t < 4; ++t) it[t] = item_at(t * (all ? NT : kWave) + tid);
#pragma unroll 1
    for (int r = 0; r < k; ++r) {
      uint64_t best = 0;
#pragma unroll
      for (int t = 0; t < 4; ++t) best = max(best, it[t] < last ? it[t] : 0);
      last = wave_best(best);
      if (all) {
        if (lane == 0) list[16 * r + wave] = last;
        __syncthreads();
        last = list[16 * r + (lane & (NT / kWave - 1))];
        last = NT == 1024 ? row_best(last) : quad_best(last);
      }
      if (tid == 0) put(r, last ? key_score((uint32_t)(last >> 32)) : -INFINITY, last ? (int)~(uint32_t)last : kIdxNone);
    }
  };
  if (k <= (many ? 2 : kDrawRanks) && n <= 4 * NT && n > kDrawItems * (k - 2)) {
    // One loop for both, or two: 3,000 x 128, 64 queries, k = 8 14.1 / 13.7 us (256 threads), but the second loop's code costs
    // every larger call, 100,000 x 256, k = 8 24.1 / 24.3 (1,024 threads).
    if (NT > 256) draw(many);
    else if (many) draw(std::true_type{});
    else draw(std::false_type{});
    __syncthreads();
    return;
  }
  if (n <= NT && n <= kCountPerDraw * k) {
    list[tid] = item_at(tid);
    __syncthreads();
  } else {
    collect();
    m = (int)count;
  }
  rank(m);
}

// Groups that a query's own workgroup scores beside the first, 0.4 us for one of 16 KB and 1.0 for one of 64: up to what
// search_unsure_kernel takes (100,000 x 128 fp32, 64 queries, 20 such groups each: 49 us per call there, 40 here; of 64: 48 and 75).
constexpr int kMoreGroups = 24;
constexpr size_t kMoreBytes = 3 << 19;
// k > 1: pick the k best groups, re-score their rows, pick the k best rows.  One workgroup per
// query.  Rows are re-scored by eight threads each, reading 16-byte pieces side by side, four rows
// in flight per thread.  100,000 x 256, 64 queries, k = 8: 70 us with 256-row groups, a row per
// thread read two bytes at a time, and k rounds of a workgroup-wide arg-max; 10 us so.  Bound by the serial
// chain of a selection among 1,563 groups, 512 rows (260 KB through one compute unit's 64 bytes per clock) and
// a selection among those, on as many compute units as queries.
// kBounds: the groups' values are those of search_bound_kernel.  The groups with the best bounds are scored, usually holding
// the answer: then no other group's bound reaches the k-th best score found, and that is all.  Groups whose bound does are scored
// as well, while they are few; of a query with more of them (rows alike in many groups, or values far from the origin) idx[b][0] is set to
// kUnsure, and the two launches that follow search it: search_unsure_kernel and this one as kUnsureOnly.
enum { kPlain = 0, kBounds = 1, kUnsureOnly = 2 };
template <typename T, int NT, bool L2, int KIND>
__global__ __launch_bounds__(NT) void finalize_topk_kernel(const SearchArgs a, int cand_in_lds) {   // (rows that fit in LDS, or 0)
  typedef RowPiece<T> Piece;
  constexpr bool BOUNDS = KIND == kBounds;
  constexpr int P = Piece::P, RPT = NT / 8;   // rows per step
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint64_t* lists = reinterpret_cast<uint64_t*>(smem);        // [NT] for the selections
  int* sel = reinterpret_cast<int*>(lists + NT);              // [kMaxK] selected groups
  float* qf = reinterpret_cast<float*>(sel + kMaxK);          // [E rounded up to 4]
  const int b = a.q0 + blockIdx.x, tid = threadIdx.x;
  float* cand = cand_in_lds ? qf + ((a.E + 3) & ~3) : a.cand + (size_t)b * a.k * a.rows;
  __shared__ uint64_t found[BOUNDS ? kMaxK : 1];    // the best so far
  __shared__ int more[BOUNDS ? kMoreGroups : 1];    // groups still to be scored
  __shared__ int n_more;
  if (KIND == kUnsureOnly && (*a.unsure == 0 || a.idx[(size_t)b * a.k] != kUnsure)) return;
  const T* q = reinterpret_cast<const T*>(a.q) + (size_t)b * a.E;
  for (int e = tid; e < ((a.E + 3) & ~3); e += NT) qf[e] = e < a.E ? (float)q[e] : 0.f;

  // 1. the min(k, G) groups with the best maxima
  const float* part = a.part_s + (size_t)b * a.G;
  const int ng = min(a.k, a.G);
  select_best<NT>(
      a.G, ng, [&](int x) { return item_key(part[x], x); }, [&](int r, float, int i) { sel[r] = i; }, lists);

  // 2. the scores of their rows
  const int shift = __builtin_ctz(a.rows);   // group sizes are powers of two
  int n_rows = ng * a.rows;
  const int part8 = tid & 7;
  // (the last RPT rows or fewer alone: the other three of every thread would be repeats.  The large form
  // does without this and with less unrolling above: every call pays for the code it brings in, 0.3 us of 32
  // at 100,000 x 256, 64 queries, k = 8.)
  auto score_rows = [&](auto rows_in_flight, int slot0) {
    constexpr int U = decltype(rows_in_flight)::value;
    const T* row[U];
    bool live[U];
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int slot = min(slot0 + u * RPT, n_rows - 1);
      const int g = sel[slot >> shift];
      const int r = g == kIdxNone ? a.N : (g << shift) + (slot & (a.rows - 1));
      live[u] = slot0 + u * RPT < n_rows && r < a.N;
      row[u] = reinterpret_cast<const T*>(a.emb) + (size_t)(r < a.N ? r : 0) * a.E;
      acc[u] = 0.f;
    }
#pragma unroll L2 ? 2 : 4   // (Euclidean, twice the instructions: 3,000 x 768 fp16, 40 queries, k = 2 20.1 / 23.1 us)
    for (int c = P * part8; c < a.E; c += 8 * P) {
      Piece e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) e[u].load(row[u], c, a.E);
#pragma unroll
      for (int t = 0; t < P; ++t) {
        const float qv = qf[c + t];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!L2) {
            acc[u] = fmaf(qv, e[u].at(t), acc[u]);
          } else {
            const float d = qv - e[u].at(t);
            acc[u] = fmaf(-d, d, acc[u]);
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] += __shfl_xor(acc[u], 1);
      acc[u] += __shfl_xor(acc[u], 2);
      acc[u] += __shfl_xor(acc[u], 4);
      if (part8 == 0 && slot0 + u * RPT < n_rows)
        cand[slot0 + u * RPT] = live[u] ? acc[u] : __builtin_nanf("");   // never ranks
    }
  };
  auto score_all = [&] {
    for (int first = 0; first < n_rows; first += 4 * RPT) {
      if ((NT > 256 && !BOUNDS) || n_rows - first > RPT) score_rows(std::integral_constant<int, 4>{}, first + (tid >> 3));
      else score_rows(std::integral_constant<int, 1>{}, first + (tid >> 3));
    }
    __syncthreads();
  };
  auto item = [&](int x) {
    const float s = cand[x];
    return s == s ? item_key(s, (sel[x >> shift] << shift) + (x & (a.rows - 1))) : 0;
  };
  auto write = [&](int r, float s, int i) {
    a.idx[(size_t)b * a.k + r] = i == kIdxNone ? -1 : i;
    a.score[(size_t)b * a.k + r] = s;
    if (r == 0) write_hit(a, b, s, i);
  };

  // 3. the k best rows among them
  if (!BOUNDS) {
    score_all();
    select_best<NT>(n_rows, a.k, item, write, lists);
    return;
  }
  int had = 0, done = 0, many = 0;   // best rows in found; groups of `more` scored, of how many
  const int g_last = min(sel[ng - 1], a.G - 1);
  const uint64_t last = item_key(part[g_last], g_last);   // of the groups scored first
  do {
    score_all();
    select_best<NT>(
        n_rows + had, a.k, [&](int x) { return x < n_rows ? item(x) : found[x - n_rows]; },
        [&](int r, float s, int i) { found[r] = i == kIdxNone ? 0 : item_key(s, i); }, lists);
    __syncthreads();
    if (had == 0) {   // 4. the groups that may hold a better row than the last of them
      had = a.k;
      float qq = 0.f;
      for (int e = tid & 63; e < a.E; e += kWave) qq = fmaf(qf[e], qf[e], qq);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) qq += __shfl_xor(qq, off);
      const uint64_t kth = found[a.k - 1];
      const float s = kth ? key_score((uint32_t)(kth >> 32)) : -INFINITY, reach = bound_reach<L2>(s, qq, a.E);
      if (tid == 0) n_more = 0;
      __syncthreads();
      for (int x = tid; x < a.G && qq == qq; x += NT)   // (of a query with NaN no row ranks)
        if (part[x] >= reach && item_key(part[x], x) < last) {
          const int at = atomicAdd(&n_more, 1);
          if (at < kMoreGroups) more[at] = x;
        }
      __syncthreads();
      many = n_more;
      if (many > kMoreGroups || (size_t)many * a.rows * a.E * sizeof(T) > kMoreBytes) {
        if (tid == 0) {
          a.idx[(size_t)b * a.k] = kUnsure;
          a.score[(size_t)b * a.k] = s;
          *a.unsure = 1;
        }
        return;
      }
    }
    const int now = min(many - done, max(cand_in_lds / a.rows, min(a.k, kMaxK)));
    if (now > 0) {
      if (tid < now) sel[tid] = more[done + tid];
      n_rows = now * a.rows;
      __syncthreads();
    }
    done += now;
    many = now > 0 ? many : -1;
  } while (many >= 0);
  if (tid < a.k)
    write(tid, found[tid] ? key_score((uint32_t)(found[tid] >> 32)) : -INFINITY, found[tid] ? (int)~(uint32_t)found[tid] : kIdxNone);
}

// k = 1 after search_bound_kernel: the same in fewer steps.  The group with the best bound is scored, eight threads a row, then
// every other group whose bound reaches the best score, of three and more four at a time.  UNSURE: after search_unsure_kernel, which leaves the best
// scores of the groups in place of their bounds, so the first group holds the answer.
template <typename T, bool L2, bool UNSURE>
__global__ __launch_bounds__(1024) void finalize_bound1_kernel(const SearchArgs a) {
  constexpr int NT = 1024, KEEP = 4;   // bounds of a thread that stay in registers
  typedef RowPiece<T> Piece;
  constexpr int P = Piece::P;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* qf = reinterpret_cast<float*>(smem);   // [E rounded up to 8]
  __shared__ uint64_t wave_top[2][NT / kWave];
  __shared__ int more[kMoreGroups], n_more;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, part8 = tid & 7;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (UNSURE && (*a.unsure == 0 || a.idx[b] != kUnsure)) return;
  const float* part = a.part_s + (size_t)b * a.G;
  const T* q = reinterpret_cast<const T*>(a.q) + (size_t)b * a.E;
  float u[KEEP];
#pragma unroll
  for (int t = 0; t < KEEP; ++t) u[t] = part[min(tid + t * NT, a.G - 1)];
  for (int e = tid; e < ((a.E + 7) & ~7); e += NT) qf[e] = e < a.E ? (float)q[e] : 0.f;
  if (tid == 0) n_more = 0;
  uint64_t best = 0;
#pragma unroll
  for (int t = 0; t < KEEP; ++t) best = max(best, item_key(u[t], min(tid + t * NT, a.G - 1)));
  for (int x = tid + KEEP * NT; x < a.G; x += NT) best = max(best, item_key(part[x], x));
  auto block_best = [&](uint64_t x, int which) {   // in every lane
    x = wave_best(x);
    if (lane == 0) wave_top[which][wave] = x;
    __syncthreads();
    return row_best(wave_top[which][lane & (NT / kWave - 1)]);
  };
  // Best of the thread's rows of U groups of 128 rows at most; 0 where none ranks.  A row's sum takes the same steps whatever U is.
  auto score_groups = [&](auto groups, auto group) {
    constexpr int U = decltype(groups)::value;
    const T* row[U];
    int r[U];
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      r[u] = group(u) * a.rows + (tid >> 3);
      if ((tid >> 3) >= a.rows || r[u] >= a.N) r[u] = -1;   // (all eight threads of a row)
      row[u] = reinterpret_cast<const T*>(a.emb) + (size_t)max(r[u], 0) * a.E;
      acc[u] = 0.f;
    }
    auto add = [&](int c) __attribute__((always_inline)) {
      Piece e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) e[u].load(row[u], c, a.E);
#pragma unroll
      for (int t = 0; t < P; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const float d = qf[c + t] - e[u].at(t);
          acc[u] = L2 ? fmaf(-d, d, acc[u]) : fmaf(qf[c + t], e[u].at(t), acc[u]);
        }
    };
    if constexpr (U == 1) {   // (as many loads in flight as of four groups)
#pragma unroll 4
      for (int c = P * part8; c < a.E; c += 8 * P) add(c);
    } else {
#pragma unroll 2
      for (int c = P * part8; c < a.E; c += 8 * P) add(c);
    }
    uint64_t top = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      acc[u] += __shfl_xor(acc[u], 1);
      acc[u] += __shfl_xor(acc[u], 2);
      acc[u] += __shfl_xor(acc[u], 4);
      if (r[u] >= 0 && acc[u] == acc[u]) top = max(top, item_key(acc[u], r[u]));
    }
    return top;
  };
  best = block_best(best, 0);   // (qf is there, too)
  const int first = (int)~(uint32_t)best;
  const int own_row = min(first * a.rows + (tid >> 3), a.N - 1), own_entry = part8 == 0 ? entry_of(a, own_row) : -1;   // (with the rows)
  const uint64_t own = score_groups(std::integral_constant<int, 1>{}, [&](int) { return first; });
  best = own;
  float qq = 0.f;
  for (int e = lane; e < a.E; e += kWave) qq = fmaf(qf[e], qf[e], qq);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) qq += __shfl_xor(qq, off);
  best = block_best(best, 1);
  int many = 0;
  if (!UNSURE) {
    const float s = best ? key_score((uint32_t)(best >> 32)) : -INFINITY, reach = bound_reach<L2>(s, qq, a.E);
    auto look = [&](float bound, int x) {
      if (bound >= reach && x < a.G && x != first && qq == qq) {   // (of a query with NaN no row ranks)
        const int at = atomicAdd(&n_more, 1);
        if (at < kMoreGroups) more[at] = x;
      }
    };
#pragma unroll
    for (int t = 0; t < KEEP; ++t) look(u[t], tid + t * NT);
    for (int x = tid + KEEP * NT; x < a.G; x += NT) look(part[x], x);
    __syncthreads();
    many = n_more;
    if (many > kMoreGroups || (size_t)many * a.rows * a.E * sizeof(T) > kMoreBytes) {
      if (tid == 0) {
        a.idx[b] = kUnsure;
        a.score[b] = s;
        *a.unsure = 1;
      }
      return;
    }
    if (many > 0) {
      if (many < 3)   // (as fours 64 queries of 100,000 x 128 fp32, most with one or none, take 7.4 us for 5.8)
        for (int x = 0; x < many; ++x) best = max(best, score_groups(std::integral_constant<int, 1>{}, [&](int) { return more[x]; }));
      else
        for (int x = 0; x < many; x += 4)   // (past the last one: that one again)
          best = max(best, score_groups(std::integral_constant<int, 4>{}, [&](int u) { return more[min(x + u, many - 1)]; }));
      best = block_best(best, 0);
    }
  }
  if (tid == 0) {
    const float top = best ? key_score((uint32_t)(best >> 32)) : -INFINITY;
    const int i = best ? (int)~(uint32_t)best : kIdxNone;
    a.idx[b] = i == kIdxNone ? -1 : i;
    a.score[b] = top;
    if (many > 0 || best == 0) write_hit(a, b, top, i);
  }
  if (many == 0 && part8 == 0 && own == best && best != 0) write_entry(a, b, key_score((uint32_t)(best >> 32)), own_entry);
}

// ------------------------------------------------------------- both phases in one launch
// For a database so small that one compute unit reads all of it in about the time that a second launch takes: one
// workgroup per query scores every row, eight threads a row as in the stream above, and picks the best k itself.
// us per call, the two launches before / this: four queries on 1,024 x 128 fp32 6.9 / 6.5, on 512 x 128 6.8 / 4.9, on
// 256 x 512 fp16 10.4 / 5.4, the best 8 of that 17.2 / 7.3, and one launch less on the host (2.7).
constexpr int kSmallThreads = kStreamThreads;
template <typename T, bool L2, bool TOPK, int U>
__global__ __launch_bounds__(kSmallThreads) void search_small_kernel(const SearchArgs a) {
  constexpr int NT = kSmallThreads;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  uint64_t* lists = reinterpret_cast<uint64_t*>(smem);                  // [NT] for the selection
  const int Ep = (a.E + 63) & ~63;
  float* qf = reinterpret_cast<float*>(lists + NT);                     // [Ep]
  float* cand = qf + Ep;                                                // [N], TOPK only
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* emb = reinterpret_cast<const T*>(a.emb);
  const T* q = reinterpret_cast<const T*>(a.q) + (size_t)b * a.E;
  uint64_t best = 0;
  stream_rows<T, L2, U>(
      emb, a.N, a.E, qf,
      [&] {
        for (int c = tid; c < Ep; c += NT) qf[c] = c < a.E ? (float)q[c] : 0.f;
      },
      [&](int r, float s) {
        if (TOPK) cand[r] = s;
        else if (s == s) best = max(best, item_key(s, r));   // a NaN never ranks
      });
  if (TOPK) {
    __syncthreads();
    select_best<NT>(
        a.N, a.k, [&](int x) { return cand[x] == cand[x] ? item_key(cand[x], x) : 0; },
        [&](int r, float s, int i) {
          a.idx[(size_t)b * a.k + r] = i == kIdxNone ? -1 : i;
          a.score[(size_t)b * a.k + r] = s;
          if (r == 0) write_hit(a, b, s, i);
        },
        lists);
    return;
  }
  best = wave_best(best);
  if (lane == 0) lists[wave] = best;
  __syncthreads();
  if (wave != 0) return;
  best = row_best(lists[lane & (NT / kWave - 1)]);
  if (lane == 0) {
    const float s = best ? key_score((uint32_t)(best >> 32)) : -INFINITY;
    const int i = best ? (int)~(uint32_t)best : kIdxNone;
    a.idx[b] = i == kIdxNone ? -1 : i;
    a.score[b] = s;
    write_hit(a, b, s, i);
  }
}

// ------------------------------------------------------------------- host side
enum { kModeValu = 0, kModeMfma = 1, kModeMfmaBig = 2, kModeMfmaWide = 3 };
constexpr int kBigBatch = 64;   // above this many queries the query-stationary kernel is used
constexpr int kBigRowsMin = 50000;   // and from this many database rows on, whatever the batch
constexpr int kSmallBatch = 256;     // queries of a single-launch search: a compute unit each, one round

// What the workspace is sized for: 8 bytes per (query, group), and for k > 1 the rows of k groups.
static void search_plan(int32_t N, int32_t mode, int32_t k, int32_t* rows_per_group, int32_t* G) {
  int rpg;
  if (mode == kModeMfma && k > 1 && N <= 32 * 1024) {
    rpg = 32;   // the rows of one wave
  } else if (mode == kModeMfma) {
    // 128 rows per pass of a workgroup; more passes per workgroup for large databases so that
    // the query tile staged in LDS is amortised, while keeping >= ~1000 workgroups
    long c = ((long)N + 128L * 1024 - 1) / (128L * 1024);
    if (c < 1) c = 1;
    if (c > 8) c = 8;
    rpg = 128 * (int)c;
  } else if (mode == kModeMfmaBig) {
    // chunks of 64 rows.  Loading the queries into registers and filling the copy pipeline
    // costs a workgroup as much as five chunks (measured), so a workgroup takes as many chunks
    // as leave about 480 workgroups: just under two per compute unit, all resident at once.
    // (k > 1: at most 16, so that the workspace for the rows of k groups stays small.)
    long c = ((long)N + 64L * 480 - 1) / (64L * 480);
    if (c < 1) c = 1;
    if (c > (k > 1 ? 16 : 64)) c = k > 1 ? 16 : 64;
    rpg = kBigRows * (int)c;
  } else {
    rpg = kValuRowsPerWg;
  }
  *rows_per_group = rpg;
  *G = (N + rpg - 1) / rpg;
}

// Groups of a top-k search.  k = 1 keeps one group per workgroup (search_plan).  For k > 1 the second phase
// re-scores k whole groups per query, so the groups are the smallest that one phase-1 step can hand
// out (the 32 rows of a wave, a chunk of 64, 64 lanes) or a power of two of it, as long as their
// maxima and the rows of k of them fit the space that search_plan stands for, which per query is
// 8 G + 4 k rows bytes (a position needs no row number: 4 instead of 8 bytes).  The largest power of two
// within search_plan's own group always fits.  A workgroup scans whole groups.
// 100,000 x 256, 64 queries, k = 8: 2,048 rows to re-score per query become 512.
static void topk_plan(int32_t N, int32_t mode, int32_t k, int32_t* rows, int32_t* G, int32_t* wg_rows) {
  int32_t rpg, g0;
  search_plan(N, mode, k, &rpg, &g0);
  const size_t space = (size_t)8 * g0 + (size_t)4 * k * rpg;
  auto fits = [&](int32_t r) {
    return (size_t)4 * ((N + r - 1) / r) + (size_t)4 * k * r <= space;
  };
  int32_t r = mode == kModeMfma || mode == kModeMfmaWide ? 32 : kBigRows, scan = rpg;
  if (mode == kModeMfma || mode == kModeMfmaWide) {
    if (!fits(r)) {   // otherwise whole passes of 128 rows
      r = 128;
      while (2 * r <= rpg && !fits(r)) r *= 2;
    }
    // (a group of 256 rows need not be scanned by one workgroup when the groups are smaller)
    if (scan < 128 || (mode == kModeMfmaWide && N <= 128 * 1024)) scan = 128;
  } else if (mode == kModeMfmaBig) {
    while (2 * r <= rpg && !fits(r)) r *= 2;
  } else {
    if (!fits(r)) r = rpg;   // 64 lanes or all 256 rows
  }
  *rows = r;
  *G = (N + r - 1) / r;
  *wg_rows = r > scan ? r : (scan + r - 1) / r * r;
}

static bool use_mfma(int32_t is_f16, int32_t metric, int32_t E) {
  return is_f16 && metric == 0 && E % 16 == 0 && E <= 512;
}

static size_t f16_lds_bytes(int nqb, int E) {
  return (size_t)32 * nqb * (((E + 15) & ~15) + kQPad) * 2 + (size_t)4 * 32 * nqb * 8;
}
constexpr size_t kF16Lds = 150 * 1024;

static int search_mode(int32_t is_f16, int32_t metric, int32_t E, int32_t B, int32_t N, int32_t k) {
  if (!use_mfma(is_f16, metric, E)) {
    // Inner products of other fp16 widths: up to eight queries are a stream over the rows, which
    // the vector ALUs follow; more are matrix work while a block of 32 queries fits in LDS and there
    // are workgroups (256 rows and up to 128 queries each) to go round.  us per call, matrix cores /
    // streams of one query / of four: 300 x 520, 64 queries 18.3 / 9.2 / 15.7; 1,000 x 520, 200 queries
    // 38.9 / 20.2 / 15.6, 400 queries 30.9 / 34 / 20.6; 4,000 x 520, 16 queries 11.8 / 10.2 / 15.6, 32 queries 12.3 / 13.8 / 15.6,
    // 200 queries 40 / 61 / 32; 7,500 x 1,536, 64 queries 37 / - / 49; 4,000 x 264, 400 queries 21.5 / 62 / 32; 20,000 x 136, 9 queries 8.1 / 13.5 / 10.3.
    const size_t groups = (size_t)(N + kValuRowsPerWg - 1) / kValuRowsPerWg;
    if (!is_f16 || metric != 0 || B <= 8 || f16_lds_bytes(1, E) > kF16Lds) return kModeValu;
    if (k > 1) return kModeMfmaWide;   // whose groups of 32 rows leave less to re-score: 4,000 x 520, 64 queries, k = 4 22.2 / 37 / 29.8
    if (groups * B <= 448 || (B > 32 && groups * ((B + 127) / 128) <= (B > 128 ? 32 : 16))) return kModeValu;
    return groups <= 32 && narrow_rows(is_f16, E, B, N) ? kModeValu : kModeMfmaWide;
  }
  const bool big_shape = E == 128 || E == 256 || E == 512;   // instantiated widths
  // the query-stationary kernel streams a large database faster at any batch size (1M x 256:
  // 94 us against 105-126 us for 4..64 queries); below kBigRowsMin rows both are latency-bound
  // and the row-stationary kernel starts up faster
  return (big_shape && (B > kBigBatch || N >= kBigRowsMin)) ? kModeMfmaBig : kModeMfma;
}

size_t search_workspace_bytes(int32_t N, int32_t E, int32_t B, int32_t k, int32_t is_f16) {
  // the metric is not known here: size for the larger of the paths this (dtype, E, B) can take
  size_t need = 0;
  for (int metric = 0; metric < 2; ++metric) {
    int32_t rpw, G;
    search_plan(N, search_mode(is_f16, metric, E, B, N, k), k, &rpw, &G);
    size_t bytes = ((size_t)B * G * 8 + 255) / 256 * 256;
    if (k > 1) bytes += (size_t)B * k * rpw * 4;
    if (bytes > need) need = bytes;
  }
  return need + 256;
}

// The same for any batch of up to max_batch queries.  Within a mode the size grows with the batch; the one
// change of mode that changes the groups is at kBigBatch, where more queries can need less.
size_t search_workspace_bytes_up_to(int32_t N, int32_t E, int32_t max_batch, int32_t k, int32_t is_f16) {
  const size_t own = search_workspace_bytes(N, E, max_batch, k, is_f16);
  if (max_batch <= kBigBatch) return own;
  const size_t below = search_workspace_bytes(N, E, kBigBatch, k, is_f16);
  return own > below ? own : below;
}

template <int KSMAX, int QPW>
static hipError_t launch_f16_big(const SearchArgs& a, dim3 grid, hipStream_t stream) {
  if (a.k > 1)
    hipLaunchKernelGGL((search_f16_big_kernel<KSMAX, QPW, true>), grid, dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((search_f16_big_kernel<KSMAX, QPW, false>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int KSMAX, int NQB, bool TOPK>
static hipError_t launch_f16_one(const SearchArgs& a, dim3 grid, size_t lds, hipStream_t stream) {
  hipError_t e = ensure_lds<&search_f16_kernel<KSMAX, NQB, TOPK>>(lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((search_f16_kernel<KSMAX, NQB, TOPK>), grid, dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <int KSMAX, int NQB>
static hipError_t launch_f16_k(const SearchArgs& a, dim3 grid, size_t lds, hipStream_t stream) {
  return a.k > 1 ? launch_f16_one<KSMAX, NQB, true>(a, grid, lds, stream)
                 : launch_f16_one<KSMAX, NQB, false>(a, grid, lds, stream);
}

template <int KSMAX>
static hipError_t launch_f16_phase1(const SearchArgs& a, int nqb, dim3 grid, size_t lds,
                                    hipStream_t stream) {
  switch (nqb) {
    case 1: return launch_f16_k<KSMAX, 1>(a, grid, lds, stream);
    case 2: return launch_f16_k<KSMAX, 2>(a, grid, lds, stream);
    case 4: return launch_f16_k<KSMAX, 4>(a, grid, lds, stream);
    default: return launch_f16_k<KSMAX, 8>(a, grid, lds, stream);
  }
}

// A query's second phase is one workgroup.  1,024 threads shorten it when there are many groups to
// pick from, or many or very wide rows to re-score (those of k groups, or of all there are); below that the barriers of
// sixteen waves cost more.  Time with them over time without, 8 queries: 256 rows of 1,024 bytes 1.10,
// 512 of them 0.84; 64 rows of 4,800 bytes 0.90, 256 of them 1.18; 128 rows of 9,600 bytes 0.83, 256 0.89.
template <typename T, int NT, bool L2, int KIND>
static hipError_t launch_topk_n(SearchArgs a, hipStream_t stream) {
  const size_t lists = (size_t)NT * 8 + kMaxK * 4, query = (size_t)((a.E + 3) & ~3) * 4;
  const size_t cand = (size_t)(KIND == kBounds && a.k < 4 ? 4 : a.k) * a.rows * 4;
  const int in_lds = lists + query + cand <= 62 * 1024 ? (int)(cand / 4) : 0;   // the rows' scores: in LDS, else in the workspace
  const size_t lds = lists + query + (in_lds ? cand : 0);
  hipError_t e = ensure_lds<&finalize_topk_kernel<T, NT, L2, KIND>>(lds);
  if (e != hipSuccess) return e;
  constexpr int kFit = (int)(kGridThreads / NT);   // queries of a launch
  for (a.q0 = 0; e == hipSuccess && a.q0 < a.B; a.q0 += a.nq) {
    a.nq = a.B - a.q0 < kFit ? a.B - a.q0 : kFit;
    hipLaunchKernelGGL((finalize_topk_kernel<T, NT, L2, KIND>), dim3((unsigned)a.nq), dim3(NT), lds, stream, a, in_lds);
    e = hipGetLastError();
  }
  return e;
}

static bool topk_large(const SearchArgs& a, size_t esz) {
  return a.G > 1024 || (a.k < a.G ? a.k : a.G) * a.rows > 256 || a.E * esz > 6000;
}
template <typename T>
static hipError_t launch_topk(const SearchArgs& a, hipStream_t stream) {
  const bool large = topk_large(a, sizeof(T));
  if (a.metric) return large ? launch_topk_n<T, 1024, true, kPlain>(a, stream) : launch_topk_n<T, 256, true, kPlain>(a, stream);
  return large ? launch_topk_n<T, 1024, false, kPlain>(a, stream) : launch_topk_n<T, 256, false, kPlain>(a, stream);
}
template <typename T, bool L2, bool UNSURE>
static hipError_t launch_bound1(const SearchArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL((finalize_bound1_kernel<T, L2, UNSURE>), dim3((unsigned)a.B), dim3(1024), ((size_t)a.E + 7) / 8 * 32, stream, a);
  return hipGetLastError();
}
template <typename T, bool L2>
static hipError_t launch_bounded_finish(const SearchArgs& a, hipStream_t stream) {
  if (a.k > 1) return launch_topk_n<T, 1024, L2, kBounds>(a, stream);
  return launch_bound1<T, L2, false>(a, stream);
}

// ---- bounds, exact scores of what they leave, bounds by row for what they leave open
static size_t bound_lds(int nqb, int E, size_t parts) {
  return (size_t)32 * nqb * bound_query(E) * 2 * parts + (size_t)4 * 32 * nqb * 4 + 4 * 32 * 4;
}
constexpr size_t kBoundLds = 150 * 1024;

// Where bounds first are faster than exact scores of all rows: four launches (two of which usually find nothing to do) and a
// second phase that reads whole groups of wide rows, against work that grows with N B E.  us per call (graph), all rows / bounds:
//   fp32 Euclidean, k = 1   32,000 x 256, 9 queries 20.6 / 19.7, 16 21.0 / 20.1; 100,000 x 32, 24 14.6 / 15.8, 40 19.9 / 17.0; 100,000 x 128, 9 23.9 / 22.4, 64
//                           57 / 24; 32,000 x 128, 40 23.5 / 16.5; 2,000 x 128, 400 20.6 / 21.1; 2,000 x 256, 400 33.0 / 26.8
//   fp32 inner, k = 1       100,000 x 32, 24 queries 13.7 / 15.9, 64 21.9 / 17.1; 2,000 x 128, 400 18.9 / 21.2; 32,000 x 256, 16 19.7 / 19.9; 8,000 x 128, 128
//                           19.6 / 17.8; 300,000 x 64, 9 27.4 / 28.6; 500,000 x 256, 9 110 / 113 (both bound by the stream)
//   fp16 Euclidean, k = 1   2,000 x 64, 400 queries 14.2 / 16.4; 32,000 x 64, 24 12.2 / 11.9; 100,000 x 64, 9 15.3 / 13.8; 32,000 x 256, 9 14.7 / 15.6;
//                           8,000 x 256, 40 16.8 / 15.0; 128,000 x 256, 64 147 / 27
//   k = 8                   fp32 Euclidean 100,000 x 32, 40 queries 25.0 / 25.4; 8,000 x 256, 64 31.8 / 31.8; 32,000 x 64, 64 27.2 / 21.9; inner 100,000 x 64, 24
//                           23.7 / 27.9; 8,000 x 256, 64 29.8 / 31.3; 32,000 x 128, 40 30.1 / 27.4; fp16 2,000 x 64, 400 26.1 / 29.4; 8,000 x 256, 64 24.7 / 25.2;
//                           32,000 x 512, 16 40.8 / 39.5, 40 69 / 41
// Of 106 sizes just past these lines (9 to 400 queries, 2,000 to 300,000 rows of 32 to 1,024 columns) nine take longer than all rows, up to 1.06 times as long
// (8,000 x 256, 64 queries, inner products 19.0 / 20.1; fp16 Euclidean, k = 8 24.2 / 25.6), and all together 0.83.
// Up to eight queries are streams, which follow the memory.  Rows below 64 columns (inner products 128) leave the bounds' kernel little
// work a row with up to 16 queries: 500,000 x 32 fp32, 16 queries 33.4 / 35.2, 40 69 / 37.
// What the bounds cannot tell apart costs the launches that follow as well (search_unsure_kernel).
static bool use_bounds(int32_t is_f16, int32_t metric, int32_t E, int32_t B, int32_t N, int32_t k) {
  if (B <= 8 || B > 1 << 20 || (is_f16 && !metric) || bound_lds(1, E, is_f16 ? 1 : 2) > kBoundLds) return false;
  // (so many rows and queries that tiles of them take several launches have not been measured, and stay there)
  if (((size_t)N + 8 * kValuRowsPerWg - 1) / (8 * kValuRowsPerWg) * 8 * ((B + 15) / 16) > kGridThreads / kThreads) return false;
  const double work = (double)N * B * E, bytes = (double)N * E * (is_f16 ? 2 : 4);
  if (B <= 16 && !is_f16 && (E < (metric ? 64 : 128) || (!metric && bytes > 256e6))) return false;
  const double least = is_f16 ? (E <= 64 ? 5.5e7 : k == 1 ? 8e7 : 1.1e8) : metric ? (k == 1 ? 1.1e8 : 1.3e8) : k == 1 ? 1.3e8 : 1.6e8;
  return work >= least && work >= (k > 1 && is_f16 ? 5e5 : 2.8e5) * E;
}

// Groups of the bounds: as small as the workspace of search_plan allows (8 bytes for each 256 rows of a query and, for
// k > 1, 4 for each row of k of those groups).
static void bound_plan(int32_t N, int32_t k, int32_t* rows, int32_t* G) {
  const size_t space = (size_t)8 * ((N + kValuRowsPerWg - 1) / kValuRowsPerWg) + (k > 1 ? (size_t)4 * k * kValuRowsPerWg : 0);
  int32_t r = 32;
  while ((size_t)4 * ((N + r - 1) / r) + (k > 1 ? (size_t)4 * k * r : 0) > space) r *= 2;   // 128 always fits
  *rows = r;
  *G = (N + r - 1) / r;
}

template <typename T, bool L2, int NQB>
static hipError_t launch_bound_n(const SearchArgs& a, hipStream_t stream) {
  const size_t lds = bound_lds(NQB, a.E, BoundParts<T>::N);
  hipError_t e = ensure_lds<&search_bound_kernel<T, L2, NQB>>(lds);
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)((a.N + a.wg_rows - 1) / a.wg_rows), (unsigned)((a.B + 32 * NQB - 1) / (32 * NQB)));
  hipLaunchKernelGGL((search_bound_kernel<T, L2, NQB>), grid, dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

constexpr size_t kUnsureGrid = 512;   // workgroups: two a compute unit

static size_t unsure_lds(int nqb, int E, size_t parts, size_t esz) {
  return ((size_t)32 * nqb * parts * 2 + esz) * bound_query(E) + (4 * 32 + 32 * nqb) * 4;
}

template <typename T, bool L2, int NQB, int MODE>
static hipError_t launch_unsure_n(const SearchArgs& a, hipStream_t stream) {
  const size_t lds = unsure_lds(NQB, a.E, MODE == kCentred ? 2 : BoundParts<T>::N, sizeof(T));
  hipError_t e = ensure_lds<&search_unsure_kernel<T, L2, NQB, MODE>>(lds);
  if (e != hipSuccess) return e;
  const size_t units = ((size_t)(a.N + a.wg_rows - 1) / a.wg_rows + 7) / 8 * 8 * ((a.B + 32 * NQB - 1) / (32 * NQB));
  hipLaunchKernelGGL((search_unsure_kernel<T, L2, NQB, MODE>), dim3((unsigned)(units < kUnsureGrid ? units : kUnsureGrid)), dim3(kThreads),
                     lds, stream, a);
  return hipGetLastError();
}
template <typename T, bool L2>
static hipError_t launch_unsure(const SearchArgs& a, hipStream_t stream) {
  constexpr size_t most = 160 * 1024 - 5500;   // (the rest is for pairs; rows that use_bounds takes leave room for 32 queries, but fp16
                                               // ones of more than 1,170 columns not for their two parts)
  constexpr int kBest = L2 ? kCentred : kAgain;
  constexpr size_t parts = L2 ? 2 : BoundParts<T>::N;
  hipError_t e;
  if (a.B > 32 && unsure_lds(2, a.E, parts, sizeof(T)) <= most - 5500) e = launch_unsure_n<T, L2, 2, kBest>(a, stream);
  else if (std::is_same<T, float>::value || unsure_lds(1, a.E, parts, sizeof(T)) <= most) e = launch_unsure_n<T, L2, 1, kBest>(a, stream);
  else e = launch_unsure_n<T, L2, 1, kAgain>(a, stream);
  if (e != hipSuccess) return e;
  if (a.k > 1) return launch_topk_n<T, 1024, L2, kUnsureOnly>(a, stream);
  return launch_bound1<T, L2, true>(a, stream);
}

template <typename T, bool L2>
static hipError_t launch_bounded(SearchArgs a, hipStream_t stream) {
  bound_plan(a.N, a.k, &a.rows, &a.G);
  // a second pass shares the staged queries, while there are workgroups for all compute units: 100,000 x 128 fp32, 64 queries 18.5 us
  // with one pass, 15.9 with two, 21 with four; 20,000 x 768, 32 queries 21.8, 33, 59
  a.wg_rows = a.N > 65536 ? 256 : 128;
  const size_t used = ((size_t)a.B * a.G * 4 + 255) / 256 * 256;
  unsigned char* ws = reinterpret_cast<unsigned char*>(a.part_s);
  a.cand = reinterpret_cast<float*>(ws + used);
  auto fits = [&](int nqb) { return bound_lds(nqb, a.E, BoundParts<T>::N) <= kBoundLds; };
  hipError_t e = a.B > 32 && fits(2) ? (a.B > 64 && fits(4) ? launch_bound_n<T, L2, 4>(a, stream) : launch_bound_n<T, L2, 2>(a, stream))
                                     : launch_bound_n<T, L2, 1>(a, stream);
  if (e == hipSuccess) e = launch_bounded_finish<T, L2>(a, stream);
  return e == hipSuccess ? launch_unsure<T, L2>(a, stream) : e;
}

// Where one launch is faster than two.  A step of 128 KB costs 1 us (fp16 Euclidean, which converts and subtracts
// vector by vector, 1.7), the launch and the sums 3 us (top-k 5.5); the two launches cost 5 us and what their rows'
// length adds, which is why the limits grow with E.  us per call, four queries, two launches / one:
//   fp32 inner, k = 1    64 columns: 2 steps 6.1 / 4.5, 4 steps 6.0 / 6.6; 128: 4 steps 6.9 / 6.5, 8 steps 7.0 / 10.6;
//                        512: 8 steps 12.3 / 10.8
//   fp16 inner, k = 1    128 columns: 2 steps 6.3 / 4.8, 4 steps 6.4 / 7.1; 256: 4 steps 7.7 / 7.0; 512: 8 steps 10.6 / 10.8
//   fp16 Euclidean, k = 1   128 columns: 2 steps 6.15 / 6.1, 4 steps 6.1 / 9.6; 512: 2 steps 8.8 / 6.3, 4 steps 8.9 / 9.9
//   short rows, k = 1    2,000 x 15 fp32 (whose rows end in part of a piece) 5.6 / 6.7, 64 queries 6.2 / 7.2, 179 on
//                        1,644 x 22 9.4 / 7.6; 2,000 x 16 5.3 / 4.8; 250 x 8 fp16 Euclidean 5.0 / 5.2, 250 x 16 5.0 / 4.6
//   fp16 inner, k = 8    128 columns: 2 steps 11.2 / 6.8, 8 steps 12.2 / 13.0; 512: 8 steps 17.6 / 12.8
// The lines hold for one query to 256: of 3,605 drawn calls that they send here six take more than 1.02 times the two
// launches' time, 1.06 at most, and all together 0.56.  More queries than compute units take a second round here, and the matrix cores more queries at a time: 4,096 queries,
// 96 x 825 fp16 15.0 / 61.7.
static bool search_small(bool f16, int32_t metric, int32_t E, int32_t B, int32_t N, int32_t k) {
  if (B > kSmallBatch) return false;
  const int P = f16 ? 8 : 4;
  const long steps = stream_least(P, N, E);
  if (k > 1) {
    const long limit = !f16 ? 3 + E / 64 : (metric ? 1 : 2) + (E < 96 ? 0 : 1 + E / 192);
    return steps <= (limit < 8 ? limit : 8);
  }
  if (!f16) return steps <= (E < 32 && E % 4 && B <= 64 ? 1 : E < 384 ? 2 + E / 64 : 8);
  if (metric && E < 16) return false;
  const int limit = metric ? 1 + (E + 128) / 256 : E < 256 ? 2 : 4;
  return steps <= (limit < 4 ? limit : 4);
}

template <typename T, bool L2, bool TOPK>
static hipError_t launch_small_k(const SearchArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)kSmallThreads * 8 + (size_t)((a.E + 63) & ~63) * 4 + (TOPK ? (size_t)a.N * 4 : 0);
  const dim3 grid((unsigned)a.B), block(kSmallThreads);
  switch (stream_unroll(RowPiece<T>::P, a.N, a.E)) {
    case 1: hipLaunchKernelGGL((search_small_kernel<T, L2, TOPK, 1>), grid, block, lds, stream, a); break;
    case 2: hipLaunchKernelGGL((search_small_kernel<T, L2, TOPK, 2>), grid, block, lds, stream, a); break;
    case 4: hipLaunchKernelGGL((search_small_kernel<T, L2, TOPK, 4>), grid, block, lds, stream, a); break;
    default: hipLaunchKernelGGL((search_small_kernel<T, L2, TOPK, 8>), grid, block, lds, stream, a);
  }
  return hipGetLastError();
}
template <typename T>
static hipError_t launch_small(const SearchArgs& a, hipStream_t stream) {
  if (a.metric) return a.k > 1 ? launch_small_k<T, true, true>(a, stream) : launch_small_k<T, true, false>(a, stream);
  return a.k > 1 ? launch_small_k<T, false, true>(a, stream) : launch_small_k<T, false, false>(a, stream);
}

hipError_t launch_search(const SearchLaunch& p, hipStream_t stream) {
  if (p.B == 0) return hipSuccess;
  SearchArgs a;
  a.unsure = nullptr;
  a.emb = p.emb; a.q = p.q; a.map_of = p.map_of;
  a.N = p.N; a.E = p.E; a.B = p.B; a.k = p.k; a.metric = p.metric;
  a.threshold = p.threshold;
  a.idx = p.idx; a.score = p.score; a.hit = p.hit;
  a.q0 = 0; a.nq = p.B;
  if (search_small(p.is_f16, p.metric, p.E, p.B, p.N, p.k))
    return p.is_f16 ? launch_small<f16_t>(a, stream) : launch_small<float>(a, stream);
  const int mode = search_mode(p.is_f16, p.metric, p.E, p.B, p.N, p.k);
  const bool mfma = mode == kModeMfma || mode == kModeMfmaWide;
  if (p.k > 1) {
    topk_plan(p.N, mode, p.k, &a.rows, &a.G, &a.wg_rows);
  } else {
    search_plan(p.N, mode, p.k, &a.rows, &a.G);
    a.wg_rows = a.rows;
  }
  unsigned char* ws = reinterpret_cast<unsigned char*>(p.ws);
  const size_t part_bytes = ((size_t)p.B * a.G * (p.k > 1 ? 4 : 8) + 255) / 256 * 256;
  a.part_s = reinterpret_cast<float*>(ws);
  a.part_i = p.k > 1 ? nullptr : reinterpret_cast<int32_t*>(ws + (size_t)p.B * a.G * 4);
  a.cand = reinterpret_cast<float*>(ws + part_bytes);

  if (mode == kModeMfmaBig) {
    // query super-blocks of 128 * QPW queries (4 waves x QPW blocks of 32); two blocks per wave
    // only while the query operands fit in the register file (E <= 256)
    const int ksmax = p.E <= 128 ? 8 : (p.E <= 256 ? 16 : 32);
    const int qpw_max = p.E <= 256 ? 2 : 1;
    const dim3 grid((unsigned)((p.N + a.wg_rows - 1) / a.wg_rows));
    for (int q0 = 0; q0 < p.B; q0 += 128 * qpw_max) {
      a.q0 = q0;
      a.nq = p.B - q0 < 128 * qpw_max ? p.B - q0 : 128 * qpw_max;
      const int qpw = a.nq > 128 ? 2 : 1;
      hipError_t e;
      if (ksmax == 8) e = qpw == 2 ? launch_f16_big<8, 2>(a, grid, stream) : launch_f16_big<8, 1>(a, grid, stream);
      else if (ksmax == 16) e = qpw == 2 ? launch_f16_big<16, 2>(a, grid, stream) : launch_f16_big<16, 1>(a, grid, stream);
      else e = launch_f16_big<32, 1>(a, grid, stream);
      if (e != hipSuccess) return e;
    }
  } else if (mfma) {
    // query super-blocks of 32 * nqb queries; the staged tile must fit in LDS
    const int ksmax = mode == kModeMfmaWide ? 0 : p.E <= 128 ? 8 : (p.E <= 256 ? 16 : 32);
    int max_nqb = mode == kModeMfmaWide ? 4 : 8;
    while (max_nqb > 1 && f16_lds_bytes(max_nqb, p.E) > kF16Lds) max_nqb >>= 1;
    // the full super-blocks are one launch (one after the other they left a small database with a
    // handful of workgroups at a time), the rest of the queries one of their own size
    const int full = p.B / (32 * max_nqb) * (32 * max_nqb);
    for (a.q0 = 0; a.q0 < p.B; a.q0 += a.nq) {
      a.nq = a.q0 < full ? full : p.B - a.q0;
      int nqb = a.q0 < full ? max_nqb : 1;
      while (32 * nqb < a.nq && a.q0 >= full) nqb <<= 1;
      const size_t lds = f16_lds_bytes(nqb, p.E);
      const dim3 grid((unsigned)((p.N + a.wg_rows - 1) / a.wg_rows), (unsigned)((a.nq + 32 * nqb - 1) / (32 * nqb)));
      hipError_t e;
      if (ksmax == 0) e = nqb == 1 ? launch_f16_k<0, 1>(a, grid, lds, stream)
                        : nqb == 2 ? launch_f16_k<0, 2>(a, grid, lds, stream) : launch_f16_k<0, 4>(a, grid, lds, stream);
      else if (ksmax == 8) e = launch_f16_phase1<8>(a, nqb, grid, lds, stream);
      else if (ksmax == 16) e = launch_f16_phase1<16>(a, nqb, grid, lds, stream);
      else e = launch_f16_phase1<32>(a, nqb, grid, lds, stream);
      if (e != hipSuccess) return e;
    }
  } else if (use_bounds(p.is_f16, p.metric, p.E, p.B, p.N, p.k)) {
    // the last 256 bytes of the workspace are behind what the searches use
    a.unsure = reinterpret_cast<int32_t*>(ws + search_workspace_bytes(p.N, p.E, p.B, p.k, p.is_f16) - 256);
    return p.is_f16   ? launch_bounded<f16_t, true>(a, stream)
           : p.metric ? launch_bounded<float, true>(a, stream)
                      : launch_bounded<float, false>(a, stream);
  } else {
    const hipError_t e = p.is_f16 ? launch_valu<f16_t>(a, stream) : launch_valu<float>(a, stream);
    if (e != hipSuccess) return e;
  }

  if (p.k == 1 && mode == kModeMfmaBig) {
    hipLaunchKernelGGL(finalize_top1_block_kernel, dim3((unsigned)p.B), dim3(kThreads), 0, stream, a);
  } else if (p.k == 1) {
    hipLaunchKernelGGL(finalize_top1_kernel, dim3((unsigned)p.B), dim3(kThreads), 0, stream, a);
  } else {
    return p.is_f16 ? launch_topk<f16_t>(a, stream) : launch_topk<float>(a, stream);
  }
  return hipGetLastError();
}

}  // namespace ac

// Feature projector (AttnCache Algorithm 1, f = feature_projector(h); Sec. 3.1
// "Feature Projector": two MLP layers that lower the dimension of the input
// embedding).  Four small kernels, all in binary32 (small sizes: two, see further down):
//
//   pool_kernel     x[b][i]  = mean over the sentence's tokens of h[b][t][i]      HBM-bound
//   dense_kernel    P1[z]    = partial products of x with W1 over K-slice z       fp32 matrix cores
//   dense_kernel    P2[z]    = partial products of relu(b1 + sum_z P1[z]) with W2
//   finish_kernel   f[b]     = b2 + sum_z P2[z], optionally scaled to unit norm, cast
//
// The two layers are dense contractions, so they run on the matrix cores
// (v_mfma_f32_32x32x2_f32: full binary32 operands, same peak as the vector
// ALUs but no staging through LDS: operands go from global memory straight
// into the lanes that feed the instruction).  With 64 queries a layer has only
// a few dozen 32 x 32 output tiles, so the contraction index is split over
// workgroups and the slices are added, in slice order, by whoever reads them
// next: the result does not depend on scheduling.  Most of the split happens
// inside a workgroup (up to 16 waves, partial tiles added through LDS), so few
// partial results travel through global memory.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "row_stream.hpp"

namespace ac {

constexpr int kPoolWaves = 8;

// Intermediate activations (pooled input, partial layer outputs) are stored as
// [index / 4][query][4]: the 16-byte piece a lane of the dense kernel wants
// (four consecutive contraction indices of its query) sits next to the pieces
// of the neighbouring queries, so one load instruction of a wave touches 8
// cache lines instead of 32 (a row-major [query][index] array made the dense
// kernel's load phase 2.5 times longer).
__device__ __forceinline__ size_t granule_at(int index4, int b, int B) {
  return ((size_t)index4 * B + b) * 4;
}

// ---- pooling ---------------------------------------------------------------
// grid (ceil(dm / (64 * VEC)), B), kPoolWaves waves.  Wave w adds tokens w,
// w + kPoolWaves, ...; a lane owns VEC consecutive columns (one 16-byte load
// per token).  The waves' partial sums meet in LDS and are added in wave order.
template <typename T> struct PoolVec;
template <> struct PoolVec<bf16_t> { static constexpr int VEC = 8; };
template <> struct PoolVec<float> { static constexpr int VEC = 4; };

template <int VEC>
__device__ __forceinline__ void pool_add(float (&acc)[VEC], u32x4 w);
template <>
__device__ __forceinline__ void pool_add<8>(float (&acc)[8], u32x4 w) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {   // a bf16 is the upper half of the binary32 of the same value
    acc[2 * p] += __builtin_bit_cast(float, w[p] << 16);
    acc[2 * p + 1] += __builtin_bit_cast(float, w[p] & 0xffff0000u);
  }
}
template <>
__device__ __forceinline__ void pool_add<4>(float (&acc)[4], u32x4 w) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const uint32_t bits = w[p];   // a copy: the cast wants an object, not a vector element
    acc[p] += __builtin_bit_cast(float, bits);
  }
}

template <typename T>
__global__ __launch_bounds__(kPoolWaves * kWave) void pool_kernel(const T* __restrict__ h,
                                                        const int32_t* __restrict__ seq_len,
                                                        float* __restrict__ x, int S, int dm,
                                                        int B) {
  constexpr int VEC = PoolVec<T>::VEC;
  constexpr int UNROLL = 16;
  __shared__ float part[kPoolWaves][kWave * VEC];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = blockIdx.y;
  const int col = (blockIdx.x * kWave + lane) * VEC;
  int s = seq_len ? seq_len[b] : S;
  s = min(max(s, 1), S);
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
  if (col < dm) {
    const T* src = h + (size_t)b * S * dm + col;
    // every load of a round is issued before the first sum: one memory round trip per round
    for (int t = wave; t < s; t += kPoolWaves * UNROLL) {
      u32x4 w[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int tt = t + kPoolWaves * u;   // wave-uniform, so the test costs no lanes
        w[u] = u32x4{0u, 0u, 0u, 0u};
        if (tt < s)
          w[u] = __builtin_nontemporal_load(
              reinterpret_cast<const u32x4*>(src + (size_t)tt * dm));
      }
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) pool_add<VEC>(acc, w[u]);
    }
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) part[wave][lane * VEC + v] = acc[v];
  __syncthreads();
  if (wave == 0 && col < dm) {
    const float fs = (float)s;
    float out[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      float sum = part[0][lane * VEC + v];
#pragma unroll
      for (int w = 1; w < kPoolWaves; ++w) sum += part[w][lane * VEC + v];
      out[v] = sum / fs;
    }
#pragma unroll
    for (int v = 0; v < VEC; v += 4) {
      f32x4 o = {out[v], out[v + 1], out[v + 2], out[v + 3]};
      *reinterpret_cast<f32x4*>(x + granule_at((col + v) >> 2, b, B)) = o;
    }
  }
}

// ---- one dense layer, split over the contraction index ----------------------
// out[z][b][j] = sum over k in slice z of  W[j][k] * in(b, k),
// in(b, k) = act(bias_in[k] + sum_{zi < NZ_IN} in_part[zi][b][k]),
// act = max(0, .) when RELU (the input and activation of a layer are compile-time
// cases so that no branch sits between the loads).
// grid (ceil(J / 32), ceil(B / 32), nz), up to 16 waves per workgroup.  The
// workgroup owns a 32 (j) x 32 (b) tile and K-slice z; its waves split that
// slice further, each forms its own 32 x 32 partial tile on the matrix core,
// and the partial tiles are added through LDS in wave order.
// v_mfma_f32_32x32x2_f32 takes from lane l one element of row l % 32 at
// contraction slot l / 32; a lane loads four consecutive k of its row in one
// 16-byte load (k = k0 + 4 (l / 32) + t feeds product t), which is a valid
// assignment of indices to slots because W and the input use the same one.
// K, the per-wave slice length and J are multiples of 8.
constexpr int kDenseWaves = 16;

struct DenseArgs {
  const float* W;        // [J][K]
  const float* in_part;  // [NZ_IN][K / 4][B][4]
  const float* bias_in;  // [K] or nullptr
  float* out;            // [nz][J / 4][B][4]
  int B, J, K, slice;    // slice: contraction indices per wave
};

// Loads of one step of a lane (eight contraction indices of the tile, four of
// them this lane's): its piece of W, of each of the NZ_IN partial inputs and
// of the bias.  Requested together; combined only after a scheduling fence so
// that a step costs one memory round trip, not one per operand.
template <int NZ_IN>
struct DenseRaw {
  f32x4 w, part[NZ_IN], bias;
};

template <int NZ_IN, bool BIAS>
__device__ __forceinline__ DenseRaw<NZ_IN> dense_load(const DenseArgs& a, const float* wrow, int b,
                                                      int k, int kh) {
  DenseRaw<NZ_IN> r;
  r.w = *reinterpret_cast<const f32x4*>(wrow + k);
  const size_t at = granule_at((k >> 2) + kh, b, a.B);
  const size_t zstride = (size_t)a.B * a.K;
#pragma unroll
  for (int z = 0; z < NZ_IN; ++z)
    r.part[z] = *reinterpret_cast<const f32x4*>(a.in_part + z * zstride + at);
  if (BIAS) r.bias = *reinterpret_cast<const f32x4*>(a.bias_in + k + 4 * kh);
  return r;
}

template <int NZ_IN, bool BIAS, bool RELU>
__device__ __forceinline__ f32x4 dense_input(const DenseRaw<NZ_IN>& r) {
  f32x4 v = r.part[0];
#pragma unroll
  for (int z = 1; z < NZ_IN; ++z) v += r.part[z];
  if (BIAS) v += r.bias;
  if (RELU) {
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = fmaxf(v[t], 0.f);
  }
  return v;
}

template <int NZ_IN, bool BIAS, bool RELU>
__global__ __launch_bounds__(kDenseWaves * kWave) void dense_kernel(DenseArgs a) {
  // one tile per wave of the launch: a fixed 64 KiB left room for two workgroups per compute unit,
  // however few waves they had (191 x 60 tokens, 4096 -> 1024 -> 128: 58.3 -> 52.0 us per call)
  extern __shared__ float red_lds[];
  float (*red)[16][kWave] = reinterpret_cast<float (*)[16][kWave]>(red_lds);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n_waves = blockDim.x >> 6;
  const int r = lane & 31, kh = lane >> 5;
  const int j0 = 32 * blockIdx.x, b0 = 32 * blockIdx.y;
  const int k_begin = min((blockIdx.z * n_waves + wave) * a.slice, a.K);
  const int k_end = min(k_begin + a.slice, a.K);
  // rows past the edge repeat the last one; their products are never stored
  const int jr = min(j0 + r, a.J - 1), br = min(b0 + r, a.B - 1);
  const float* wrow = a.W + (size_t)jr * a.K + 4 * kh;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  int k = k_begin;
  for (; k + 32 <= k_end; k += 32) {
    DenseRaw<NZ_IN> raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) raw[u] = dense_load<NZ_IN, BIAS>(a, wrow, br, k + 8 * u, kh);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const f32x4 x = dense_input<NZ_IN, BIAS, RELU>(raw[u]);
#pragma unroll
      for (int t = 0; t < 4; ++t)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(raw[u].w[t], x[t], acc, 0, 0, 0);
    }
  }
  for (; k < k_end; k += 8) {
    const DenseRaw<NZ_IN> raw = dense_load<NZ_IN, BIAS>(a, wrow, br, k, kh);
    const f32x4 x = dense_input<NZ_IN, BIAS, RELU>(raw);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(raw.w[t], x[t], acc, 0, 0, 0);
  }
  // a lane holds query b0 + r; its register v holds output j0 + mfma_row(v, kh)
#pragma unroll
  for (int v = 0; v < 16; ++v) red[wave][v][lane] = acc[v];
  __syncthreads();
  // 256 items per tile: (vq, lane) -> four consecutive outputs of one query
  for (int item = tid; item < 4 * kWave; item += blockDim.x) {
    const int vq = item >> 6, l = item & 63;
    const int b = b0 + (l & 31), j = j0 + 8 * vq + 4 * (l >> 5);
    f32x4 o = {0.f, 0.f, 0.f, 0.f};
    for (int w = 0; w < n_waves; ++w)
#pragma unroll
      for (int t = 0; t < 4; ++t) o[t] += red[w][4 * vq + t][l];
    if (b < a.B && j < a.J)
      *reinterpret_cast<f32x4*>(a.out + (size_t)blockIdx.z * a.B * a.J + granule_at(j >> 2, b, a.B)) = o;
  }
}

// ---- bias, unit norm, cast ---------------------------------------------------
// grid B, 256 threads; thread t owns outputs t, t + 256, ...
template <typename OUT>
__global__ __launch_bounds__(kThreads) void finish_kernel(const float* __restrict__ part, int nz,
                                                          const float* __restrict__ bias,
                                                          OUT* __restrict__ feat, int B, int E,
                                                          int normalize) {
  __shared__ float wsum[kThreads / kWave];
  const int b = blockIdx.x, tid = threadIdx.x;
  constexpr int kMaxOwn = 8;   // E <= 2048
  float val[kMaxOwn];
  float sq = 0.f;
#pragma unroll
  for (int o = 0; o < kMaxOwn; ++o) {
    const int e = tid + o * kThreads;
    float v = 0.f;
    if (e < E) {
      v = bias ? bias[e] : 0.f;
      for (int z = 0; z < nz; ++z) v += part[(size_t)z * B * E + granule_at(e >> 2, b, B) + (e & 3)];
    }
    val[o] = v;
    sq += v * v;
  }
  float mul = 1.f;
  if (normalize) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off);
    if ((tid & 63) == 0) wsum[tid >> 6] = sq;
    __syncthreads();
    const float total = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    if (total > 0.f) mul = 1.f / sqrtf(total);
  }
#pragma unroll
  for (int o = 0; o < kMaxOwn; ++o) {
    const int e = tid + o * kThreads;
    if (e < E) feat[(size_t)b * E + e] = (OUT)(val[o] * mul);
  }
}

// ---- small projections in two or three launches -----------------------------
// Where the four launches above take longer than their work, pooling and the first layer are one launch and the second
// layer, bias, norm and cast another (or two, fused_plan).
//
// pool_dense_kernel: grid (ceil(dm / 128), ceil(B / Q), ceil(hid / rows)), 16 waves.  A workgroup pools 128 columns of Q
// queries (the waves share the queries, so that one query alone still has 16 waves on its tokens) and forms the partial
// products of these 128 contraction indices with its rows of W1: eight threads a row, a sum per query each.  The first rows
// of W1 are on their way while the tokens are added up.  Bound by the latency of the two round trips to memory, then by
// the 64 bytes per clock of a compute unit and its vector ALUs.
//   out[z][b][j] = sum over k in [128 z, 128 z + 128) of W1[j][k] x[b][k]
constexpr int kFusedCols = 128, kFusedThreads = 1024, kFusedRows = 256;   // rows: two of each thread
constexpr int32_t kFusedBatch = 256;

// The eight threads of a row add up their parts for Q queries: thread p ends up with query p % Q.
template <int Q>
__device__ __forceinline__ float query_of_eight(float (&v)[Q], int part8) {
  auto from = [](float x, auto ctrl) {
    const int bits = __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true);
    return __builtin_bit_cast(float, bits);
  };
  const std::integral_constant<int, 0x141> mirror;    // lane 7 - p of the eight
  const std::integral_constant<int, 0x4e> swap2;      // lane p ^ 2
  const std::integral_constant<int, 0xb1> swap1;      // lane p ^ 1
#pragma unroll
  for (int q = 0; q < Q; ++q) v[q] += from(v[q], mirror);
  if (Q == 4) {   // half of the queries each
#pragma unroll
    for (int q = 0; q < Q / 2; ++q) {
      const float keep = (part8 & 2) ? v[q + Q / 2] : v[q], give = (part8 & 2) ? v[q] : v[q + Q / 2];
      v[q] = keep + from(give, swap2);
    }
  } else {
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] += from(v[q], swap2);
  }
  if (Q == 1) return v[0] + from(v[0], swap1);
  const float keep = (part8 & 1) ? v[Q > 1] : v[0], give = (part8 & 1) ? v[0] : v[Q > 1];
  return keep + from(give, swap1);
}

template <typename T, int Q>
__global__ __launch_bounds__(kFusedThreads) void pool_dense_kernel(const T* __restrict__ h, const int32_t* __restrict__ seq_len,
                                                                   const float* __restrict__ W1, float* __restrict__ out, int S,
                                                                   int dm, int hid, int B, int rows) {
  constexpr int VEC = PoolVec<T>::VEC, LPR = kFusedCols / VEC, RPW = kWave / LPR;   // lanes per row, rows per wave and load
  constexpr int NW = kFusedThreads / kWave, RPT = kFusedThreads / 8, UNROLL = 8, I = kFusedRows / RPT, C = kFusedCols / 32;
  __shared__ float ps[NW][kFusedCols];
  __shared__ __attribute__((aligned(16))) float xs[Q][kFusedCols];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slot = tid >> 3, part8 = tid & 7;
  const int c0 = kFusedCols * blockIdx.x, b0 = Q * blockIdx.y, j_begin = rows * blockIdx.z, j_end = min(j_begin + rows, hid);
  f32x4 w[I][C];
  auto fetch = [&](int i, int j0) {   // rows and columns past the end repeat what does not lie there (dm is a multiple of 8)
    const float* row = W1 + (size_t)min(j0 + RPT * i + slot, hid - 1) * dm;
#pragma unroll
    for (int c = 0; c < C; ++c) w[i][c] = *reinterpret_cast<const f32x4*>(row + min(c0 + 32 * c + 4 * part8, dm - 4));
  };
#pragma unroll
  for (int i = 0; i < I; ++i) fetch(i, j_begin);
  // pooling: NW / Q waves a query, RPW tokens a wave and load
  constexpr int per = NW / Q;
  const int nq = min(Q, B - b0);
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
  const int mine = wave / per;   // the query
  if (mine < nq) {
    const int s = min(max(seq_len ? seq_len[b0 + mine] : S, 1), S);
    const int t0 = (wave % per) * RPW, sub = lane / LPR;
    const int col = min(c0 + VEC * (lane % LPR), dm - VEC);   // (columns past the end are zeroed below)
    const T* src = h + (size_t)(b0 + mine) * S * dm + col;
    for (int t = t0; t < s; t += UNROLL * per * RPW) {
      u32x4 v[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int first = t + u * per * RPW;   // wave-uniform
        v[u] = u32x4{0u, 0u, 0u, 0u};
        if (first < s) v[u] = *reinterpret_cast<const u32x4*>(src + (size_t)min(first + sub, s - 1) * dm);
      }
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        if (t + u * per * RPW + sub >= s) v[u] = u32x4{0u, 0u, 0u, 0u};
        pool_add<VEC>(acc, v[u]);
      }
    }
  }
  // the RPW lanes of a column piece add up
#pragma unroll
  for (int off = 32; off >= LPR; off /= 2)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] += __shfl_xor(acc[v], off);
  if (lane < LPR)
#pragma unroll
    for (int v = 0; v < VEC; ++v) ps[wave][VEC * lane + v] = acc[v];
  __syncthreads();
  if (tid < Q * kFusedCols) {
    const int q = tid / kFusedCols, c = tid % kFusedCols;   // q: wave-uniform
    float x = 0.f;
    if (q < nq && c0 + c < dm) {
#pragma unroll
      for (int w = 0; w < per; ++w) x += ps[q * per + w][c];
      x /= (float)min(max(seq_len ? seq_len[b0 + q] : S, 1), S);
    }
    xs[q][c] = x;
  }
  __syncthreads();
  f32x4 x[Q][C];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int c = 0; c < C; ++c) x[q][c] = *reinterpret_cast<const f32x4*>(&xs[q][32 * c + 4 * part8]);
  float* dst = out + ((size_t)blockIdx.x * B + b0 + part8) * hid;   // thread p of a row's eight writes query p
  const bool whole = c0 + kFusedCols <= dm;
#pragma unroll 1
  for (int j0 = j_begin; j0 < j_end; j0 += RPT * I) {
#pragma unroll
    for (int i = 0; i < I; ++i) {
      if (!whole)   // (a product of a zero with a weight of another column would be NaN where that is infinite)
#pragma unroll
        for (int c = 0; c < C; ++c)
          if (c0 + 32 * c + 4 * part8 >= dm) w[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
      float sum[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        float v = 0.f;
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int t = 0; t < 4; ++t) v = fmaf(w[i][c][t], x[q][c][t], v);
        sum[q] = v;
      }
      if (j0 + RPT * I < j_end) fetch(i, j0 + RPT * I);
      const float v = query_of_eight<Q>(sum, part8);
      const int j = j0 + RPT * i + slot;
      if (part8 < nq && j < j_end) dst[j] = v;
    }
  }
}

// dense_finish_kernel: grid (B, parts).  A workgroup adds up the partial products of its query (in slice order within a group
// of threads, then over the groups), activates them and streams its rows of W2 past them.  With all rows in one workgroup
// (PARTS = false) norm and cast follow as above, otherwise the sums are left to finish_kernel: part[E / 4][B][4].
template <typename OUT, int U, bool PARTS>
__global__ __launch_bounds__(kStreamThreads) void dense_finish_kernel(const float* __restrict__ part, int nz,
                                                                      const float* __restrict__ b1, const float* __restrict__ W2,
                                                                      const float* __restrict__ b2, OUT* __restrict__ feat, int B,
                                                                      int hid, int E, int rows, int normalize) {
  constexpr int NT = kStreamThreads;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f32x4* red = reinterpret_cast<f32x4*>(smem);            // [NT]
  float* x = reinterpret_cast<float*>(red + NT);          // [hid], zeros to the next multiple of 64
  float* y = x + ((hid + 63) & ~63);                      // [E]
  __shared__ float wsum[NT / kWave];
  const int b = blockIdx.x, tid = threadIdx.x, e0 = PARTS ? rows * blockIdx.y : 0;
  const int n4 = hid >> 2, groups = NT / n4, g = tid / n4, i = tid - g * n4;   // n4 <= NT
  stream_rows<float, false, U>(
      W2 + (size_t)e0 * hid, PARTS ? min(rows, E - e0) : E, hid, x,
      [&] {
        if (g < groups) {
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
          const f32x4* src = reinterpret_cast<const f32x4*>(part + (size_t)b * hid) + i;
#pragma unroll 4
          for (int z = g; z < nz; z += groups) v += src[(size_t)z * B * n4];
          red[tid] = v;
        }
        __syncthreads();
        if (tid < n4) {
          f32x4 v = red[tid];
          for (int k = 1; k < min(groups, nz); ++k) v += red[tid + k * n4];
          if (b1) v += *reinterpret_cast<const f32x4*>(b1 + 4 * tid);
#pragma unroll
          for (int t = 0; t < 4; ++t) x[4 * tid + t] = fmaxf(v[t], 0.f);
        }
        for (int c = hid + tid; c < ((hid + 63) & ~63); c += NT) x[c] = 0.f;
      },
      [&](int e, float s) {
        if (PARTS) feat[granule_at((e0 + e) >> 2, b, B) + ((e0 + e) & 3)] = s;
        else y[e] = s;
      });
  if (PARTS) return;
  __syncthreads();
  float sq = 0.f;
  for (int e = tid; e < E; e += NT) {
    const float v = b2 ? b2[e] + y[e] : y[e];
    y[e] = v;
    sq += v * v;
  }
  float mul = 1.f;
  if (normalize) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sq += __shfl_xor(sq, off);
    if ((tid & 63) == 0) wsum[tid >> 6] = sq;
    __syncthreads();
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) total += wsum[w];
    if (total > 0.f) mul = 1.f / sqrtf(total);
  }
  for (int e = tid; e < E; e += NT) feat[(size_t)b * E + e] = (OUT)(y[e] * mul);
}

static int ceil_div(int a, int b) { return (a + b - 1) / b; }

// How one layer's contraction index is split: waves per workgroup, workgroups
// along K (= partial results in global memory) and indices per wave.  Aim: about
// one wave per SIMD of the chip (1024), at least 32 indices per wave.
struct DenseSplit { int n_waves, nz, slice; };
static DenseSplit dense_split(int32_t B, int32_t J, int32_t K) {
  const int tiles = ceil_div(B, 32) * ceil_div(J, 32);
  // waves per tile: about two per SIMD of the chip in total, 32 indices each at least
  const int want = std::min(std::max(1, 2048 / tiles), std::min(std::max(1, K / 32), 64));
  // Spread them over workgroups first (more compute units share the load phase), up to the
  // four partial results the next kernel reads, then over the waves of a workgroup.
  DenseSplit d;
  d.nz = std::min(want, 4);
  if (d.nz == 3) d.nz = 2;
  d.n_waves = std::min(ceil_div(want, d.nz), kDenseWaves);
  d.slice = ceil_div(ceil_div(K, d.n_waves * d.nz), 8) * 8;
  return d;   // slices past K are empty and contribute zeros
}

static size_t dense_lds(const DenseSplit& s) { return sizeof(float) * s.n_waves * 16 * kWave; }   // <= 64 KiB

// How a small projection is split, and whether it is small.  us per call in a graph, four launches / so (bf16 in, 256 out):
//   dm 512, hid 128      8 x 500 tokens 20.2 / 8.9, 256 x 16 16.2 / 9.9
//   dm 1024, hid 256     1 x 16 13.2 / 9.1, 128 x 100 19.0 / 13.5, 256 x 16 (512 workgroups) 20.4 / 17.2
//   dm 2048, hid 512     16 x 90 18.1 / 14.1, 64 x 128 padded 21.6 / 18.3, 128 x 16 (512 workgroups) 21.6 / 23.3
//   dm 4096, hid 1024    1 x 1024 38.0 / 18.0, 8 x 16 21.2 / 17.7, 32 x 16 (256 workgroups) 22.4 / 23.7
// so the partial products (workgroups of four queries x hidden units, a query and unit of each workgroup being 128
// products) are what the line is drawn at.  Of 19,500 drawn sizes those with dm and hid multiples of 32 gain 1.10 times on
// average from half of that line to three quarters, 1.08 from there to the line, 0.97 up to a quarter beyond, 0.95 further
// on.  Many rows of W2 for each of many queries lose, every query streams all of W2 past itself.
//
// Rows of W1 and W2 that do not start on 128-byte lines cost extra lines in every slice of 128 columns, and hidden layers
// that leave a step over W2 half empty cost whole steps.  For such widths the gain is estimated, fitted to the same sizes, in us:
//   6 for the launches, less 2.6 per 1,024 hidden units, 1.1 per 1,024 rows of W1 times queries that a compute unit works
//   off, 1.4 more per 1,024 rows off the lines, 0.3 per step off the lines, 1 for the third launch and 0.03 per MB of
//   tokens that several workgroups pool again; and 0.4 per 128 tokens where the pooling launch leaves the chip idle.
// us per call, four / fused, and what is taken: 20 x 83 tokens, 3432 -> 856 -> 256 24.5 / 30.7, four; 130 x 169, 1384 -> 344 ->
// 512 33.0 / 39.6, four; 4 x 30, 2872 -> 712 -> 128 20.3 / 16.2, fused.  Of the drawn sizes 16,390 are fused: 1.46 times on
// average, 0.84 at worst, 127 below 0.98 (by the line alone 293, 0.78 at worst); those that this refuses 0.96 on average.
struct FusedPlan { bool fits, use; int nz, Q, rows, parts, rows2; };

static double fused_gain(const FusedPlan& f, int32_t B, int32_t S, int32_t dm, int32_t hid, bool f32) {
  const int z = ceil_div(hid, f.rows), bytes = f32 ? 4 : 2;
  const double kilo_rows = (double)ceil_div(f.nz * ceil_div(B, f.Q) * z, 256) * f.rows / 1024;   // rows of W1 a compute unit reads
  const double steps2 = (double)ceil_div(B * f.parts, 256) * stream_least(4, f.rows2, hid);
  const int pools = ceil_div(dm, kWave * (f32 ? PoolVec<float>::VEC : PoolVec<bf16_t>::VEC)) * B;   // workgroups of pool_kernel
  double us = 6 - 2.6 * hid / 1024 - 1.1 * kilo_rows * f.Q;
  if (dm % 32) us -= 1.4 * kilo_rows;
  if (hid % 32) us -= 0.3 * steps2;
  if (f.parts > 1) us -= 1;
  us -= 0.03e-6 * bytes * dm * B * S * (z - 1);
  us += 0.4 * std::max(S / 128. - 1, 0.) * std::min(1., 256. / pools);
  return us;
}

static FusedPlan fused_plan(int32_t B, int32_t S, int32_t dm, int32_t hid, int32_t E, bool f32) {
  FusedPlan f = {false, false, ceil_div(dm, kFusedCols), 4, 0, 1, E};
  if (B > kFusedBatch || hid > 1024) return f;
  const long wgs4 = (long)f.nz * ceil_div(B, 4), steps = stream_least(4, E, hid);
  if (steps > 16 || steps * B > 1024 || wgs4 > 512 || wgs4 * hid > 128 * 1024) return f;
  f.fits = true;   // (whatever the length of the sentences, which the size of the workspace does not know)
  long least = 0;
  for (int Q = 1; Q <= 4; Q *= 2) {
    const int wgs = f.nz * ceil_div(B, Q);
    if (wgs > 256 && Q < 4) continue;
    const int rows = ceil_div(ceil_div(hid, std::max(1, 256 / wgs)), kFusedRows) * kFusedRows;
    // a compute unit each where there are so few: bytes of W1, vector instructions in bytes of the same time, bytes of tokens
    const long cost = 512L * rows + 180L * rows * Q + (long)Q * S * kFusedCols * (f32 ? 4 : 2);
    if (least == 0 || cost < least) { least = cost; f.Q = Q; f.rows = rows; }
  }
  if (steps > 4) {   // 128 rows at least: fewer leave threads without one
    f.rows2 = ceil_div(ceil_div(E, std::min((int)(steps + 1) / 2, std::max(1, 256 / B))), 128) * 128;
    f.parts = ceil_div(E, f.rows2);
    if (f.parts == 1) f.rows2 = E;
  }
  f.use = (dm % 32 == 0 && hid % 32 == 0) || fused_gain(f, B, S, dm, hid, f32) > 0;
  return f;
}
static size_t fused_bytes(const FusedPlan& f, int32_t B, int32_t hid, int32_t E) {
  return f.fits ? sizeof(float) * ((size_t)f.nz * B * hid + (f.parts > 1 ? (size_t)B * E : 0)) : 0;
}

template <typename T>
static void launch_pool_dense(const ProjectLaunch& p, const FusedPlan& f, float* part, hipStream_t stream) {
  const dim3 grid(f.nz, ceil_div(p.B, f.Q), ceil_div(p.hid, f.rows));
  auto go = [&](auto q) {
    pool_dense_kernel<T, decltype(q)::value><<<grid, kFusedThreads, 0, stream>>>(static_cast<const T*>(p.h), p.seq_len, p.W1, part,
                                                                                 p.S, p.dm, p.hid, p.B, f.rows);
  };
  if (f.Q == 1) go(std::integral_constant<int, 1>{});
  else if (f.Q == 2) go(std::integral_constant<int, 2>{});
  else go(std::integral_constant<int, 4>{});
}

template <typename OUT, bool PARTS>
static void launch_dense_finish(const ProjectLaunch& p, const FusedPlan& f, const float* part, OUT* out, hipStream_t stream) {
  const size_t lds = 16 * kStreamThreads + sizeof(float) * (size_t)(((p.hid + 63) & ~63) + (PARTS ? 0 : p.E));
  auto go = [&](auto u) {
    dense_finish_kernel<OUT, decltype(u)::value, PARTS><<<dim3(p.B, f.parts), kStreamThreads, lds, stream>>>(
        part, f.nz, p.b1, p.W2, p.b2, out, p.B, p.hid, p.E, f.rows2, p.normalize);
  };
  switch (stream_unroll(RowPiece<float>::P, f.rows2, p.hid)) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    default: go(std::integral_constant<int, 8>{});
  }
}

static void launch_finish(const ProjectLaunch& p, const float* part, int nz, hipStream_t stream) {
  if (p.feat_is_f16)
    finish_kernel<f16_t><<<p.B, kThreads, 0, stream>>>(part, nz, p.b2, static_cast<f16_t*>(p.feat), p.B, p.E, p.normalize);
  else
    finish_kernel<float><<<p.B, kThreads, 0, stream>>>(part, nz, p.b2, static_cast<float*>(p.feat), p.B, p.E, p.normalize);
}

size_t project_workspace_least(int32_t B, int32_t dm, int32_t hid, int32_t E) {
  const DenseSplit s1 = dense_split(B, hid, dm), s2 = dense_split(B, E, hid);
  return sizeof(float) * ((size_t)B * dm + (size_t)s1.nz * B * hid + (size_t)s2.nz * B * E);
}

size_t project_workspace_bytes(int32_t B, int32_t dm, int32_t hid, int32_t E) {
  size_t bytes = project_workspace_least(B, dm, hid, E);
  for (int32_t b = std::min(B, kFusedBatch); b >= 1; --b)   // a smaller batch may want more
    bytes = std::max(bytes, fused_bytes(fused_plan(b, 1, dm, hid, E, false), b, hid, E));
  return bytes;
}

hipError_t launch_project(const ProjectLaunch& p, hipStream_t stream) {
  const FusedPlan f = fused_plan(p.B, p.S, p.dm, p.hid, p.E, p.h_is_f32);
  if (f.use && p.ws_bytes >= fused_bytes(f, p.B, p.hid, p.E)) {
    float* part = static_cast<float*>(p.ws);
    if (p.h_is_f32) launch_pool_dense<float>(p, f, part, stream);
    else launch_pool_dense<bf16_t>(p, f, part, stream);
    if (f.parts > 1) {
      float* y = part + (size_t)f.nz * p.B * p.hid;
      launch_dense_finish<float, true>(p, f, part, y, stream);
      launch_finish(p, y, 1, stream);
    } else if (p.feat_is_f16) {
      launch_dense_finish<f16_t, false>(p, f, part, static_cast<f16_t*>(p.feat), stream);
    } else {
      launch_dense_finish<float, false>(p, f, part, static_cast<float*>(p.feat), stream);
    }
    return hipGetLastError();
  }
  const DenseSplit s1 = dense_split(p.B, p.hid, p.dm), s2 = dense_split(p.B, p.E, p.hid);
  float* x = static_cast<float*>(p.ws);
  float* p1 = x + (size_t)p.B * p.dm;
  float* p2 = p1 + (size_t)s1.nz * p.B * p.hid;

  if (p.h_is_f32) {
    dim3 grid(ceil_div(p.dm, kWave * 4), p.B);
    pool_kernel<float><<<grid, kPoolWaves * kWave, 0, stream>>>(static_cast<const float*>(p.h),
                                                                p.seq_len, x, p.S, p.dm, p.B);
  } else {
    dim3 grid(ceil_div(p.dm, kWave * 8), p.B);
    pool_kernel<bf16_t><<<grid, kPoolWaves * kWave, 0, stream>>>(static_cast<const bf16_t*>(p.h),
                                                                 p.seq_len, x, p.S, p.dm, p.B);
  }
  DenseArgs l1{p.W1, x, nullptr, p1, p.B, p.hid, p.dm, s1.slice};
  dense_kernel<1, false, false><<<dim3(ceil_div(p.hid, 32), ceil_div(p.B, 32), s1.nz),
                                  s1.n_waves * kWave, dense_lds(s1), stream>>>(l1);
  DenseArgs l2{p.W2, p1, p.b1, p2, p.B, p.E, p.hid, s2.slice};
  const dim3 grid2(ceil_div(p.E, 32), ceil_div(p.B, 32), s2.nz);
  const int threads2 = s2.n_waves * kWave;
  auto layer2 = [&](auto nz_in) {
    constexpr int NZ = decltype(nz_in)::value;
    if (p.b1)
      dense_kernel<NZ, true, true><<<grid2, threads2, dense_lds(s2), stream>>>(l2);
    else
      dense_kernel<NZ, false, true><<<grid2, threads2, dense_lds(s2), stream>>>(l2);
  };
  switch (s1.nz) {
    case 1: layer2(std::integral_constant<int, 1>{}); break;
    case 2: layer2(std::integral_constant<int, 2>{}); break;
    default: layer2(std::integral_constant<int, 4>{}); break;
  }
  launch_finish(p, p2, s2.nz, stream);
  return hipGetLastError();
}

}  // namespace ac

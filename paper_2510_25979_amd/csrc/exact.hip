// Recompute branch of Algorithm 2: O = softmax(scale * Q K^T) V, causal or
// dense, without ever writing the S x S map (flash-style online softmax).
//
// bf16 path (matrix cores, v_mfma_f32_32x32x16_bf16), one kernel in two variants and two more:
//   * short (S <= 128): K and V of one or several K/V heads in LDS, a wave takes units of 32 query rows of one head
//     (short_tile.hpp);
//   * resident (S <= 128, routed launches of many tiles): one workgroup = one (batch item, KV head); both 64-key chunks of K
//     and V are copied into LDS once and the workgroup walks all g query heads that share
//     them; after the one barrier behind the copy its four waves never meet again;
//   * streaming (S > 128): one workgroup = four units of 32 query rows of the heads that share K
//     and V, which streams 64-key chunks of them through two LDS stages.
//   * split (launches of few rows): the waves of a workgroup share 32 query rows and deal out its
//     key blocks.
// Otherwise a wave owns 32 query rows and walks the key blocks up to its diagonal.
// Both products are formed transposed:
//   S^T = K Q^T   -> a lane holds 16 keys of ONE query column, so the row
//                    maximum and row sum are in-lane reductions plus one
//                    exchange between the two lane halves;
//   O^T = V^T P^T -> the probabilities sit in exactly the register layout
//                    the second product wants as its column operand, so P
//                    goes from the first MFMA to the second without leaving
//                    registers (the contraction slots are matched by reading
//                    V^T from LDS in the same key order).
// Softmax runs in the log2 domain with the scale folded into one FMA per
// score; the accumulator is rescaled only when some row maximum has moved far.
#include "common.hpp"
#include "f32_tile.hpp"
#include "launch.hpp"
#include "short_tile.hpp"
#include "split_tile.hpp"
#include <type_traits>

namespace ac {

constexpr int kOPass = 64; // output columns staged per pass (16 rows at a time)
constexpr int kOStride = kOPass + 4;
// Online softmax: weights are 2^(score - m); m moves (and the accumulator is rescaled) only when
// a row maximum has outgrown it by more than this many bits (see the chunk step below).
constexpr float kRescaleSlack = 8.0f;

struct ExactArgs {
  const void *Q, *K, *V;
  void* O;
  const int32_t* row_sel;
  const int32_t* key_len;   // real tokens per batch item of a right-padded batch, or nullptr
  int32_t B, Hq, Hkv, S;
  int32_t n_rblk;
  int32_t n_kvtiles;
  float scale_log2e;
};

// How K and V reach the matrix cores:
//   * each chunk of K and of V is copied global -> LDS directly (global_load_lds_dwordx4, no
//     data registers, no ALU work), row-major, into one of two stages, so the copy of chunk
//     c + 1 is in flight while chunk c is multiplied and one barrier per chunk suffices;
//   * rows are unpadded; the copy permutes the 16-byte pieces of a row (a lane picks which
//     global piece lands in its LDS slot) so that the operand reads spread over all banks:
//     K piece p of row r sits at p ^ k_piece_swizzle(r), V piece p of row r at p ^ v_piece_swizzle(r);
//   * the V^T operand is fetched with the transposing LDS read (ds_read_b64_tr_b16): in a
//     group of 16 lanes, lane i names four consecutive d of key j(i / 4) and lane t receives,
//     for its own d, the four keys j(0..3);
//   * the two 32-key blocks of a chunk take their softmax steps in an order that lets matrix
//     and vector work of one wave overlap (see the chunk step below).
constexpr int kLChunk = 64;

template <int D, bool CAUSAL, bool RESIDENT>
__global__ __launch_bounds__(kThreads, (D == 64 ? 3 : 2)) void exact_bf16_kernel(const ExactArgs a) {
  constexpr int PPR = D / 8;                          // 16-byte pieces per row
  constexpr int NCOPY = kLChunk * PPR / kWave / 4;    // copy instructions per wave, tensor, chunk
  __shared__ __attribute__((aligned(16))) bf16_t kb0[kLChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t vb0[kLChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t kb1[kLChunk * D];
  __shared__ __attribute__((aligned(16))) bf16_t vb1[kLChunk * D];
  // wave-private output staging of the resident mode (16 rows x 64 columns per pass)
  __shared__ __attribute__((aligned(16))) bf16_t ost_small[4 * 16 * kOStride];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it scalar
  const int il = lane & 31, kh = lane >> 5;
  const int S = a.S, g = a.Hq / a.Hkv;
  // The scale as a scalar register written by a vector instruction: a register that comes
  // straight from a scalar load makes the compiler wait for "all scalar and LDS traffic" before
  // its first use in a loop iteration, which drains the operand reads in flight.
  const float scale_log2e = __builtin_bit_cast(
      float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.scale_log2e) + (lane & 0)));
  // Sequences of up to 128 keys are RESIDENT: both 64-key chunks of K and V sit in the two
  // stages for the whole tile, the workgroup walks all g query heads that share
  // them, and between the one barrier after the copy and the end of the tile the four waves
  // never meet again.  Longer sequences stream chunks through the stages, one 32-row unit per wave.

  // per tile (the helpers below read these by reference)
  int u = 0, h = 0, b = 0, r0 = 0, n_chunk = 0;
  int Sk = S;   // keys this tile's queries may see at all: the sentence's length in a padded batch
  bool active = false;
  const bf16_t* Ksrc = nullptr;
  const bf16_t* Vsrc = nullptr;

  // ---- copies: instruction k = wave + 4 i fills LDS slots [64 k, 64 k + 64), slot = row * PPR +
  // position.  From one instruction to the next, row grows by 256 / PPR (which leaves both
  // permutations unchanged) and both addresses by 2048 elements: one lane offset per tensor.
  const int slot0 = kWave * wave + lane;
  const int crow = slot0 / PPR, cpos = slot0 % PPR;
  const int kpiece = cpos ^ k_piece_swizzle<D>(crow);   // global piece that lands in this lane's slot
  const int vpiece = cpos ^ v_piece_swizzle<D>(crow);
  // Running source pointers, one per tensor, advanced by one chunk after each use (cheaper
  // than rebuilding 64-bit addresses from the chunk index every time).
  const bf16_t* kptr = nullptr;   // set per tile
  const bf16_t* vptr = nullptr;
  auto prefetch = [&](bf16_t* kb, bf16_t* vb, int c) {
    const int nj = min(kLChunk, S - c * kLChunk);
    if (nj == kLChunk) {
#pragma unroll
      for (int i = 0; i < NCOPY; ++i) {
        __builtin_amdgcn_global_load_lds(kptr + 2048 * i, kb + kWave * 8 * (wave + 4 * i), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(vptr + 2048 * i, vb + kWave * 8 * (wave + 4 * i), 16, 0, 0);
      }
      kptr += kLChunk * D;
      vptr += kLChunk * D;
    } else {
      // ragged last chunk: rows past the end repeat the last row (finite, and masked later)
      const bf16_t* ksrc = Ksrc + (size_t)c * kLChunk * D;
      const bf16_t* vsrc = Vsrc + (size_t)c * kLChunk * D;
#pragma unroll
      for (int i = 0; i < NCOPY; ++i) {
        const int rr = min(crow + (256 / PPR) * i, nj - 1);
        __builtin_amdgcn_global_load_lds(ksrc + (size_t)rr * D + 8 * kpiece,
                                         kb + kWave * 8 * (wave + 4 * i), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(vsrc + (size_t)rr * D + 8 * vpiece,
                                         vb + kWave * 8 * (wave + 4 * i), 16, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- operand addresses (elements, relative to a stage; the 32-key block enters as a constant)
  // K operand of column step ks: row il of the block, piece 2 ks + kh
  int koff[D / 16];
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) koff[ks] = il * D + 8 * ((2 * ks + kh) ^ k_piece_swizzle<D>(il));
  // V^T operand: contraction slot e of lane half kh, step s2, is key 16 s2 + 8 (e / 4) + 4 kh +
  // e % 4 of the block, which is where the first product left the scores in the registers.
  // Lane i of a 16-lane group names key 4 kh + 8 half + i / 4 and the four d from
  // 32 db + 16 (il / 16) + 4 (i % 4).
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
  f32x16 acc[D / 32];
  float m_run = -INFINITY, l_run = 0.f;
  // this wave's 32 query rows of head h as the column operand of the first product, and a
  // fresh accumulator.  (A wave whose rows lie beyond a ragged end works on a copy of the last
  // row and stores nothing: the streaming loop then needs no per-wave branch, whose merge
  // would cost a copy of the accumulator per chunk.)
  auto begin_head = [&]() {
    const bf16_t* qrow = reinterpret_cast<const bf16_t*>(a.Q) +
                         (((size_t)b * a.Hq + h) * S + min(r0 + il, S - 1)) * D + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) q[ks] = *reinterpret_cast<const u32x4*>(qrow + 16 * ks);
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[db][v] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };

  // ---- pieces of one chunk step (32-key block jb of the stage)
  // scores^T of block jb: 32 keys x 32 query rows, this lane: query row il, 16 of the keys
  auto qk = [&](const bf16_t* kb, int jb) {
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      s = mfma_bf16(*reinterpret_cast<const bf16x8*>(kb + koff[ks] + 32 * jb * D),
                    __builtin_bit_cast(bf16x8, q[ks]), s);
    return s;
  };
  // hide the keys this query row must not see (beyond the diagonal or the end of the sentence)
  auto hide = [&](f32x16& s, int c, int jb) {
    const int limit = (CAUSAL ? min(r0 + il, Sk - 1) : Sk - 1) - c * kLChunk - 32 * jb - 4 * kh;
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (8 * (v >> 2) + (v & 3) > limit) s[v] = -INFINITY;
  };
  // largest score of the query row: in-lane over 16 keys, then across the two lane halves
  auto row_max = [&](const f32x16& s) {
    float m01 = fmaxf(fmaxf(s[0], s[1]), s[2]);
    float m02 = fmaxf(fmaxf(s[3], s[4]), s[5]);
    float m03 = fmaxf(fmaxf(s[6], s[7]), s[8]);
    float m04 = fmaxf(fmaxf(s[9], s[10]), s[11]);
    float m05 = fmaxf(fmaxf(s[12], s[13]), s[14]);
    float mx = fmaxf(fmaxf(fmaxf(m01, m02), m03), fmaxf(fmaxf(m04, m05), s[15]));
    return max_with_other_half(mx);
  };
  // probabilities 2^(score * scale_log2e - m) as the packed bf16 operand of the second product;
  // their sum is taken over the ROUNDED values (the ones that are multiplied with V), two per
  // instruction, so numerator and denominator of the softmax see the same weights
  typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
  auto probs = [&](const f32x16& s, float m, u32x4 (&pw)[2], float& sum) {
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(s[8 * s2 + 2 * w], scale_log2e, -m));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(s[8 * s2 + 2 * w + 1], scale_log2e, -m));
        const uint32_t pk = pack_bf16(e0, e1);
        pw[s2][w] = pk;
        sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), ones, sum, false);
      }
  };
  auto pv = [&](const bf16_t* vb, int jb, const u32x4 (&pw)[2]) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
        acc[db] = mfma_bf16(vop(vb, db, jb, s2), __builtin_bit_cast(bf16x8, pw[s2]), acc[db]);
  };
  auto rescale = [&](float m_new) {
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[db][v] *= alpha;
  };

  // One chunk = two 32-key blocks, each with its own online-softmax step, ordered so that
  // matrix and vector work of ONE wave can overlap (the matrix pipe runs asynchronously, but a
  // wave issues in order): the scores of block 1 are requested before the exponentials of
  // block 0 are taken, the second product of block 0 before the exponentials of block 1.
  // The reference point m of a row (weights are 2^(score - m)) follows the row maximum lazily:
  // it moves, and the accumulator is rescaled, only when some row of the wave has outgrown
  // its reference by more than kRescaleSlack, so weights stay below 2^kRescaleSlack and almost
  // every step skips the rescaling (a new maximum turns up in nearly every block of random
  // scores, a jump by 2^8 hardly ever); the final division by the row sum makes the result
  // independent of m.  For block 1 the rescaling happens after the second product of block 0
  // has been added (those weights refer to the old m).
  // MASKED is the variant for chunks that touch the diagonal or the ragged end (nblk of the
  // two blocks exist for this wave, some of their keys may be hidden); the other variant has no
  // per-element tests.  The flag is a literal at every call site and the body is inlined.
  auto step = [&](const bf16_t* kb, const bf16_t* vb, int c, int nblk, const bool MASKED)
      __attribute__((always_inline)) {
    const bool two = !MASKED || nblk > 1;
    f32x16 s0 = qk(kb, 0);
    if (MASKED) hide(s0, c, 0);
    float m0 = m_run;
    {
      const float cand = fmaxf(m_run, row_max(s0) * scale_log2e);
      if (__any(cand > m_run + kRescaleSlack)) {
        rescale(cand);
        m0 = cand;
      }
    }
    m_run = m0;
    f32x16 s1;
    if (two) s1 = qk(kb, 1);
    u32x4 p0[2];
    float sum0 = 0.f;
    probs(s0, m0, p0, sum0);
    l_run += sum0;
    if (two) {
      if (MASKED) hide(s1, c, 1);
      const float cand1 = fmaxf(m0, row_max(s1) * scale_log2e);
      const bool moved = __any(cand1 > m0 + kRescaleSlack);
      const float m1 = moved ? cand1 : m0;
      pv(vb, 0, p0);
      u32x4 p1[2];
      float sum1 = 0.f;
      probs(s1, m1, p1, sum1);
      if (moved) rescale(m1);
      m_run = m1;
      l_run += sum1;
      pv(vb, 1, p1);
    } else {
      pv(vb, 0, p0);
    }
  };
  // chunk c through the masked variant (exact for every chunk, only slower)
  auto tail_step = [&](const bf16_t* kb, const bf16_t* vb, int c) {
    if (!active) return;
    const int nj = min(kLChunk, Sk - c * kLChunk);
    int nblk = (nj + 31) >> 5;
    if (CAUSAL) nblk = min(nblk, (r0 >> 5) + 1 - 2 * c);
    if (nblk > 0) step(kb, vb, c, nblk, true);
  };
  // this wave's copies have landed (they are counted like loads), then everybody's; the
  // barrier also retires the stage that the next copy overwrites
  auto publish = [&]() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  };

  // the 32 x D result of this wave in 16 x 64 passes through its small private buffer (the
  // stages still hold K and V for the next head); every global store covers whole 128-byte lines
  auto store_small = [&](bf16_t* Oh, float inv) {
    bf16_t* ost = ost_small + wave * (16 * kOStride);
#pragma unroll
    for (int rh = 0; rh < 2; ++rh)
#pragma unroll
      for (int dh = 0; dh < D / 64; ++dh) {
        if ((il >> 4) == rh) {
#pragma unroll
          for (int dbp = 0; dbp < 2; ++dbp)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
              const f32x16& t = acc[2 * dh + dbp];
              u32x2 w;
              w.x = pack_bf16(t[4 * vq] * inv, t[4 * vq + 1] * inv);
              w.y = pack_bf16(t[4 * vq + 2] * inv, t[4 * vq + 3] * inv);
              *reinterpret_cast<u32x2*>(ost + (il & 15) * kOStride + 32 * dbp + 8 * vq + 4 * kh) = w;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int it = 0; it < 2; ++it) {
          const int p = it * kWave + lane;
          const int row = p >> 3, c8 = p & 7;
          const u32x2* sp = reinterpret_cast<const u32x2*>(ost + row * kOStride + 8 * c8);
          u32x2 lo = sp[0], hi = sp[1];
          __builtin_nontemporal_store(
              u32x4{lo.x, lo.y, hi.x, hi.y},
              reinterpret_cast<u32x4*>(Oh + (size_t)(16 * rh + row) * D + 64 * dh + 8 * c8));
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
  };

  if constexpr (RESIDENT) {
    // A fixed number of workgroups, each taking every gridDim.x-th tile: the copies of the next
    // tile's K and V are started before the last head of the current tile is written out, so
    // stores and loads of one workgroup overlap, and a tile whose batch item was served by the
    // reuse branch costs no workgroup launch.  Which of its tiles have work a workgroup finds
    // out 64 candidates at a time: lane i tests candidate i (one vector load of the routing
    // flags, one round trip to memory for all of them) and the votes form a wave-uniform bit
    // mask that the walk below consumes with scalar bit operations.
    int cand_base = 0;          // candidates cand_base .. cand_base + 63 are in `live`
    unsigned long long live = 0;
    auto scan = [&](int base) {
      // (tile numbers stay below 2^31 + 64 gridDim.x: unsigned 32-bit arithmetic is enough)
      const unsigned t = blockIdx.x + (unsigned)(base + lane) * gridDim.x;
      const bool work = t < (unsigned)a.n_kvtiles && !(a.row_sel && a.row_sel[(int)t / a.Hkv] >= 0);
      cand_base = base;
      live = __ballot(work);
    };
    // first tile with work among this workgroup's candidates number `from` and up, or -1
    auto locate = [&](int from) {
      while (true) {
        const int shift = from - cand_base;
        const unsigned long long rest = shift < 64 ? (live >> shift) : 0ull;
        if (rest) {
          const int i = from + __builtin_ctzll(rest);
          return (int)(blockIdx.x + (unsigned)i * gridDim.x);
        }
        const int next = cand_base + 64;
        if (blockIdx.x + (unsigned)next * gridDim.x >= (unsigned)a.n_kvtiles) return -1;
        scan(next);
        from = next;
      }
    };
    scan(0);
    int h_first = 0;
    auto enter = [&](int t) {       // tile variables, and its K and V on their way
      u = t;
      h_first = (u % a.Hkv) * g;
      b = u / a.Hkv;
      Ksrc = reinterpret_cast<const bf16_t*>(a.K) + (size_t)u * S * D;
      Vsrc = reinterpret_cast<const bf16_t*>(a.V) + (size_t)u * S * D;
      kptr = Ksrc + crow * D + 8 * kpiece;
      vptr = Vsrc + crow * D + 8 * vpiece;
      Sk = a.key_len ? min(max(a.key_len[b], 1), S) : S;
      n_chunk = (Sk + kLChunk - 1) / kLChunk;
      prefetch(kb0, vb0, 0);
      if (n_chunk > 1) prefetch(kb1, vb1, 1);
    };
    int t = locate(0);
    if (t < 0) return;   // e.g. a batch served entirely by the reuse branch
    enter(t);
    while (true) {
      publish();
      const int rot = (t >> 3) & 3;
      for (int hl = 0; hl < g; ++hl) {
        h = h_first + hl;
        // causal work grows with the row block and wave i always runs on SIMD i: rotating the
        // wave -> row block assignment lets every SIMD see the same mix
        r0 = 32 * ((wave + rot + hl) & 3);
        active = r0 < S;
        begin_head();
        for (int c = 0; c < n_chunk; ++c) tail_step(c ? kb1 : kb0, c ? vb1 : vb0, c);
        if (hl + 1 == g) break;   // the last head is written after the next copies start
        if (active) {
          const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32));
          store_small(reinterpret_cast<bf16_t*>(a.O) + (((size_t)b * a.Hq + h) * S + r0) * (size_t)D, inv);
        }
      }
      const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32));
      bf16_t* Olast = reinterpret_cast<bf16_t*>(a.O) + (((size_t)b * a.Hq + h) * S + r0) * (size_t)D;
      const bool act = active;
      const int tn = locate((t - (int)blockIdx.x) / (int)gridDim.x + 1);
      __syncthreads();          // every wave has finished reading the stages
      if (tn >= 0) enter(tn);
      if (act) store_small(Olast, inv);   // registers and the wave's own small buffer only
      if (tn < 0) break;
      t = tn;
    }
  } else {
    // Units of 32 query rows of one head, numbered row block first, head second; a workgroup
    // takes four consecutive ones of a K/V tile, one per wave (g = 4: the same rows of
    // all four heads), the heaviest workgroup first.  Its waves see (nearly) the same keys and a chunk is
    // copied once for all of them.  The fours are counted from the first rows, where chunks of 64 keys
    // begin with the units, and what is left over are the last rows, by themselves: counted from the end, a workgroup had
    // more chunks on its diagonals (320 heads, 192 x 128, causal 19.0 us, 17.3 so; 448 x 64 26.8 / 24.2).
    // 128 rows of one head per workgroup before: 64 x 32 heads on 8 K and V, 288 x 128, causal 141 -> 105 us; 16 x 32 on 8,
    // 1024 x 128 214 -> 195 us; with one head per K and V it is the same split.
    const int bid = blockIdx.x;
    const int slot = bid >> 3;
    const int n_units = g * (S >> 5), per_u = (n_units + 3) >> 2;
    u = (slot / per_u) * 8 + (bid & 7);   // ids equal mod 8 (one XCD) share K, V in its L2
    if (u >= a.n_kvtiles) return;
    const int low = 4 * (per_u - 1 - slot % per_u), top = min(low + 3, n_units - 1), unit = low + 3 - wave;
    h = (u % a.Hkv) * g + min(unit, top) % g;
    b = u / a.Hkv;
    if (a.row_sel && a.row_sel[b] >= 0) return;
    Ksrc = reinterpret_cast<const bf16_t*>(a.K) + (size_t)u * S * D;
    Vsrc = reinterpret_cast<const bf16_t*>(a.V) + (size_t)u * S * D;
    kptr = Ksrc + crow * D + 8 * kpiece;
    vptr = Vsrc + crow * D + 8 * vpiece;
    Sk = a.key_len ? min(max(a.key_len[b], 1), S) : S;
    const int last_key = CAUSAL ? min(Sk, 32 * (top / g + 1)) : Sk;
    n_chunk = (last_key + kLChunk - 1) / kLChunk;
    r0 = 32 * (min(unit, top) / g);
    active = unit <= top;
    begin_head();
    // Chunks below c_split are complete and fully visible to every wave of the workgroup
    // (they lie left of the diagonal blocks of all its rows, and before a ragged end): the
    // main loop runs only the test-free variant, two chunks per trip so that stages
    // alternate without pointer arithmetic.  The few chunks from c_split on go through the
    // masked variant.
    const int c_split = CAUSAL ? min(32 * (low / g) / kLChunk, Sk / kLChunk) : Sk / kLChunk;
    prefetch(kb0, vb0, 0);
    int c = 0;
    for (; c + 1 < c_split; c += 2) {
      publish();
      prefetch(kb1, vb1, c + 1);
      step(kb0, vb0, c, 2, false);
      publish();
      if (c + 2 < n_chunk) prefetch(kb0, vb0, c + 2);
      step(kb1, vb1, c + 1, 2, false);
    }
    // (one copy of the masked code: the stage is picked at run time, which only costs the
    // compiler its proof that copy and reads touch different arrays, i.e. some overlap)
    for (; c < n_chunk; ++c) {
      publish();
      bf16_t* kcur = (c & 1) ? kb1 : kb0;
      bf16_t* vcur = (c & 1) ? vb1 : vb0;
      if (c + 1 < n_chunk) prefetch((c & 1) ? kb0 : kb1, (c & 1) ? vb0 : vb1, c + 1);
      tail_step(kcur, vcur, c);
    }
    __syncthreads();   // every wave is done with both stages: they now stage the output
    if (active) {
      const float inv = 1.0f / (l_run + __shfl_xor(l_run, 32));
      bf16_t* Oh = reinterpret_cast<bf16_t*>(a.O) + (((size_t)b * a.Hq + h) * S + r0) * (size_t)D;
      bf16_t* ost = wave == 0 ? kb0 : wave == 1 ? vb0 : wave == 2 ? kb1 : vb1;
      store_tile_bf16<D>(acc, inv, ost, Oh, lane);
    }
  }
}

// The same for a launch that leaves the chip idle: ALL waves of a workgroup share 32 query rows of
// one head, wave w takes the 32-key blocks w, w + NW, ..., and the partial results meet in LDS at the
// end.  The chain of a row gets NW times shorter; the price is that nothing of K and V is shared.
template <int D, bool CAUSAL, int NW>
__global__ __launch_bounds__(NW * kWave, 2) void exact_bf16_split_kernel(const ExactArgs a) {
  // the waves' V tiles (half of it), and at the end their partial results
  __shared__ __attribute__((aligned(16))) f32x4 smem[NW * (D / 8) * kWave];
  __shared__ float ms[NW][32], ls[NW][32];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int il = lane & 31, kh = lane >> 5;
  const int S = a.S, heads = a.B * a.Hq;
  // heaviest row blocks first, neighbouring workgroups (and so the XCDs) on different heads
  const int block = (S >> 5) - 1 - blockIdx.x / heads, bh = blockIdx.x % heads, b = bh / a.Hq;
  if (a.row_sel && a.row_sel[b] >= 0) return;
  const int tile = b * a.Hkv + bh % a.Hq / (a.Hq / a.Hkv);
  const int Sk = a.key_len ? min(max(a.key_len[b], 1), S) : S;
  const size_t at = ((size_t)bh * S + 32 * block) * D;
  const int n_keys = CAUSAL ? min((Sk + 31) >> 5, block + 1) : (Sk + 31) >> 5;   // key blocks
  SplitOperands<D> t(reinterpret_cast<const bf16_t*>(a.K) + (size_t)tile * S * D,
                     reinterpret_cast<const bf16_t*>(a.V) + (size_t)tile * S * D,
                     reinterpret_cast<bf16_t*>(smem) + wave * 32 * D, lane);
  t.load_q(reinterpret_cast<const bf16_t*>(a.Q) + at);
  if (wave < n_keys) {
    t.load_k(wave);
    t.load_v(wave);
  }
  f32x16 acc[D / 32];
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[db][x] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int blk = wave; blk < n_keys; blk += NW) {
    f32x16 s = t.scores();
    const bool more = blk + NW < n_keys;
    if (more) t.load_k(blk + NW);
    t.stage_v();
    if (more) t.load_v(blk + NW);
    wave_lds_fence();
    if ((CAUSAL && blk == block) || 32 * blk + 32 > Sk) {
      const int limit = (CAUSAL ? min(32 * block + il, Sk - 1) : Sk - 1) - 32 * blk - 4 * kh;
#pragma unroll
      for (int x = 0; x < 16; ++x)
        if (8 * (x >> 2) + (x & 3) > limit) s[x] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int x = 1; x < 16; ++x) mx = fmaxf(mx, s[x]);
    const float cand = fmaxf(m, max_with_other_half(mx) * a.scale_log2e);
    if (__any(cand > m + kRescaleSlack)) {
      const float alpha = cand > m ? __builtin_amdgcn_exp2f(m - cand) : 1.f;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int x = 0; x < 16; ++x) acc[db][x] *= alpha;
      m = cand;
    }
    const float ref = m == -INFINITY ? 0.f : m;   // no finite score so far: all weights are zero
    typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
    u32x4 p[2];
#pragma unroll
    for (int w = 0; w < 8; ++w) {   // the sum is over the rounded weights, which V is multiplied with
      const float e0 = __builtin_amdgcn_exp2f(fmaf(s[2 * w], a.scale_log2e, -ref));
      const float e1 = __builtin_amdgcn_exp2f(fmaf(s[2 * w + 1], a.scale_log2e, -ref));
      const uint32_t pk = pack_bf16(e0, e1);   // a copy: the cast wants an object, not a vector element
      p[w >> 2][w & 3] = pk;
      l = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pk), ones, l, false);
    }
    t.weights_v(acc, p);
    wave_lds_fence();   // the tile is read before the next block's rows are written
  }
  l += __shfl_xor(l, 32);
  if (kh == 0) {
    ms[wave][il] = m;
    ls[wave][il] = l;
  }
  __syncthreads();   // statistics are there, V tiles are no longer read
  float top = -INFINITY, sum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) top = fmaxf(top, ms[w][il]);
  auto factor = [&](float mw) { return mw < top ? __builtin_amdgcn_exp2f(mw - top) : 1.f; };
#pragma unroll
  for (int w = 0; w < NW; ++w) sum = fmaf(ls[w][il], factor(ms[w][il]), sum);
  split_store<D, NW>(acc, factor(m), 1.0f / sum, smem, reinterpret_cast<bf16_t*>(a.O) + at, wave, lane);
}

// A row next to infinite or NaN V on its diagonal block, key by key: lane = output column, only visible
// keys are read.  m and l are the row's largest score and the sum of its weights.
__device__ __forceinline__ void f32_row_by_key(const ExactArgs& a, const float* K, const float* V, size_t at,
                                               int keys, float m, float l, float scale, int D, int lane) {
  const float* Q = reinterpret_cast<const float*>(a.Q) + at;
  for (int d0 = 0; d0 < D; d0 += kWave) {
    float o = 0.f;
    for (int j = 0; j < keys; ++j) {
      float s = 0.f;
      for (int d = lane; d < D; d += kWave) s = fmaf(Q[d], K[(size_t)j * D + d], s);
      for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
      const float p = expf(s * scale - (m == -INFINITY ? 0.f : m));
      if (d0 + lane < D) o = fmaf(p, V[(size_t)j * D + d0 + lane], o);
    }
    if (d0 + lane < D) reinterpret_cast<float*>(a.O)[at + d0 + lane] = o / l;
  }
}

// fp32 path (binary32 matrix instructions, any S, D <= 64 DB): four waves of 16 query rows each
// share 32-key stages of K and V; the next stage's rows are in registers while this one is
// multiplied.  Online softmax: every lane keeps the running maximum and ITS keys' share of the row
// sum, the accumulator is rescaled when a maximum of the wave moves.
// 16 x 24 heads on 8 K and V, 94 x 128 causal: 805 us with one wave per query row on the vector
// ALUs, 20.8 us so (7 us of matrix instructions at the peak rate, which the vector instructions do not overlap
// here, 10 us of memory at the copy rate; the rest is the load -> stage -> score -> weight chain of 640
// workgroups that start together).  Four workgroups per CU need 128 registers and spill (38 us).
template <int DB, int COLS>
__global__ __launch_bounds__(kThreads, DB <= 2 ? 3 : 2) void exact_f32_kernel(
    const ExactArgs a, int D, int causal, float scale) {
  constexpr int KC = 32;
  typedef F32Stage<DB, KC, COLS> Stage;
  if (COLS == kAllCols) D = 64 * DB;
  __shared__ __attribute__((aligned(16))) float kl[KC * Stage::LD];
  __shared__ __attribute__((aligned(16))) float vl[KC * Stage::LD];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, kq = lane >> 4;
  const int S = a.S, g = a.Hq / a.Hkv;
  const F32Unit u = f32_unit<(DB <= 2)>(blockIdx.x, wave, g, S, a.n_kvtiles);
  if (u.tile < 0) return;
  const int b = u.tile / a.Hkv, h = u.tile % a.Hkv * g + u.head;
  if (a.row_sel && a.row_sel[b] >= 0) return;
  const int len = a.key_len ? min(max(a.key_len[b], 1), S) : S;   // keys beyond it are padding
  const float* K = reinterpret_cast<const float*>(a.K) + (size_t)u.tile * S * D;
  const float* V = reinterpret_cast<const float*>(a.V) + (size_t)u.tile * S * D;

  const int row = kF32Rows * max(u.block, 0) + i;
  const size_t at = (((size_t)b * a.Hq + h) * S + min(row, S - 1)) * (size_t)D;
  f32x4 q[4 * DB];
#pragma unroll
  for (int kk = 0; kk < 4 * DB; ++kk) {
    const int c = 16 * kk + 4 * kq;
    const float* src = reinterpret_cast<const float*>(a.Q) + at + c;
    if constexpr (COLS == kAnyCols || COLS == kFewCols) {
      q[kk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (c + t < D) q[kk][t] = src[t];
    } else {
      q[kk] = *reinterpret_cast<const f32x4*>(COLS == kAllCols || c < D ? src : src - c);
      if (COLS == kVecCols)
#pragma unroll
        for (int t = 0; t < 4; ++t) q[kk][t] = c < D ? q[kk][t] : 0.f;
    }
  }
  f32x4 acc[4 * DB];
#pragma unroll
  for (int x = 0; x < 4 * DB; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  bool redo = false;   // wave-uniform
  const int limit = causal ? min(row + 1, len) : len;                                // keys this row sees
  const int wave_keys = u.block < 0 ? 0 : causal ? min(len, kF32Rows * (u.block + 1)) : len;
  const int wg_keys = causal ? min(len, kF32Rows * (u.last_block + 1)) : len;

  Stage ks, vs;
  ks.load(K, 0, len, D, tid);
  vs.load(V, 0, len, D, tid);
  for (int jc = 0; jc < wg_keys; jc += KC) {
    ks.template mask<false>(jc, len, D, tid);   // (scores of hidden keys are replaced)
    vs.template mask<true>(jc, len, D, tid);
    __syncthreads();   // the previous stage has been read by everybody
    ks.commit(kl, tid);
    vs.commit(vl, tid);
    __syncthreads();
    if (jc + KC < wg_keys) {
      ks.load(K, jc + KC, len, D, tid);
      vs.load(V, jc + KC, len, D, tid);
    }
    const int left = wave_keys - jc;
    if (left <= 0) continue;
    f32x4 s[2];
#pragma unroll
    for (int bk = 0; bk < 2; ++bk) {
      s[bk] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (16 * bk < left) {
        const float* krow = kl + (16 * bk + i) * Stage::LD + 4 * kq;
        f32x4 k = *reinterpret_cast<const f32x4*>(krow);
#pragma unroll
        for (int kk = 0; kk < 4 * DB; ++kk) {
          if (COLS == kAllCols || 16 * kk < D) {   // uniform
            const f32x4 next = *reinterpret_cast<const f32x4*>(krow + 16 * ((kk + 1) & (4 * DB - 1)));
#pragma unroll
            for (int t = 0; t < 4; ++t) s[bk] = mfma_f32(k[t], q[kk][t], s[bk]);
            k = next;
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
    float mx = -INFINITY;
    bool seen[2][4];
#pragma unroll
    for (int bk = 0; bk < 2; ++bk)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        seen[bk][x] = jc + 16 * bk + 4 * kq + x < limit;
        s[bk][x] *= scale;
        mx = seen[bk][x] ? fmaxf(mx, s[bk][x]) : mx;
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx);
    if (__any(m_new > m)) {
      const float alpha = m_new > m ? expf(m - m_new) : 1.f;
      l *= alpha;
#pragma unroll
      for (int x = 0; x < 4 * DB; ++x) acc[x] *= alpha;
      m = m_new;
    }
    const float ref = m == -INFINITY ? 0.f : m;   // no finite score so far: all weights are zero
#pragma unroll
    for (int bk = 0; bk < 2; ++bk) {
      if (16 * bk < left) {
        f32x4 p;
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          p[x] = seen[bk][x] ? expf(s[bk][x] - ref) : 0.f;
          l += p[x];
        }
        const float* v = vl + 16 * bk * Stage::LD;
        if (causal && (jc >> 4) + bk == u.block) redo = f32_block_not_finite<DB>(v, i, kq);
        f32_weights_v<DB>(acc, v, p, i, kq);
      }
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (u.block >= 0 && row < S && !redo)
    f32_store_row<DB, COLS, true>(reinterpret_cast<float*>(a.O) + at, acc, l, kq, D);
  if (redo) {
    const int rows = min(kF32Rows, S - kF32Rows * u.block);
    for (int r = 0; r < rows; ++r)
      f32_row_by_key(a, K, V, __shfl(at, r), __shfl(limit, r), __shfl(m, r), __shfl(l, r), scale, D, lane);
  }
}

// The same rows for a launch that leaves the chip idle: ALL waves of a workgroup share one unit of 16
// rows, wave w takes the 16-key blocks w, w + NW, ... straight from memory to the lanes that
// multiply them (nothing is shared, so nothing goes through LDS and no barrier sits in the loop; a
// block's successor is requested as its registers fall free), and the partial results meet in LDS
// at the end.  The chain of a row gets NW times shorter and the launch has four times the
// workgroups.
template <int DB, int NW, bool FULL>   // FULL: D == 64 DB
__global__ __launch_bounds__(NW * kWave, DB <= 2 ? 2 : 1) void exact_f32_split_kernel(
    const ExactArgs a, int D, int causal, float scale) {
  __shared__ __attribute__((aligned(16))) f32x4 part[NW][4 * DB][kWave];
  __shared__ float ms[NW][kF32Rows], ls[NW][kF32Rows];
  __shared__ int odd;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, kq = lane >> 4;
  const int S = a.S, heads = a.B * a.Hq;
  // heaviest row blocks first, neighbouring workgroups (and so the XCDs) on different heads
  const int n_blk = (S + kF32Rows - 1) / kF32Rows, block = n_blk - 1 - blockIdx.x / heads;
  const int bh = blockIdx.x % heads, b = bh / a.Hq;
  if (a.row_sel && a.row_sel[b] >= 0) return;
  const int tile = b * a.Hkv + bh % a.Hq / (a.Hq / a.Hkv);
  const int len = a.key_len ? min(max(a.key_len[b], 1), S) : S;   // keys beyond it are padding
  const float* K = reinterpret_cast<const float*>(a.K) + (size_t)tile * S * D;
  const float* V = reinterpret_cast<const float*>(a.V) + (size_t)tile * S * D;
  const int keys = causal ? min(len, kF32Rows * (block + 1)) : len;
  const int n_keys = (keys + kF32Rows - 1) / kF32Rows;   // key blocks

  // No load sits behind a lane's own test: rows past the end of the sentence and columns past D (a
  // multiple of 16) repeat valid ones.  A hidden key's score is replaced, its V row zeroed (the last
  // block of a sentence only); columns past D end up in results that nobody stores.
  f32x4 k[4 * DB], v[4][DB];
  auto col = [&](int c) { return FULL || c < D ? c : 0; };
  auto load_k = [&](int blk) {
    const float* src = K + (size_t)min(kF32Rows * blk + i, len - 1) * D + 4 * kq;
#pragma unroll
    for (int kk = 0; kk < 4 * DB; ++kk) k[kk] = *reinterpret_cast<const f32x4*>(src + col(16 * kk));
  };
  auto load_v = [&](int blk) {
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const int key = kF32Rows * blk + 4 * kq + x;
      const float* src = V + (size_t)min(key, len - 1) * D;
#pragma unroll
      for (int db = 0; db < DB; ++db) v[x][db] = *reinterpret_cast<const f32x4*>(src + col(64 * db + 4 * i));
    }
  };
  const int row = kF32Rows * block + i;
  const size_t at = ((size_t)bh * S + min(row, S - 1)) * (size_t)D;
  const float* Q = reinterpret_cast<const float*>(a.Q) + at;
  f32x4 q[4 * DB];
#pragma unroll
  for (int kk = 0; kk < 4 * DB; ++kk) q[kk] = *reinterpret_cast<const f32x4*>(Q + col(16 * kk) + 4 * kq);
  if (wave < n_keys) {
    load_k(wave);
    load_v(wave);
  }
  if (tid == 0) odd = 0;
  f32x4 acc[4 * DB];
#pragma unroll
  for (int x = 0; x < 4 * DB; ++x) acc[x] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  bool redo = false;
  const int limit = causal ? min(row + 1, len) : len;   // keys this row sees
  for (int blk = wave; blk < n_keys; blk += NW) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4 * DB; ++kk)
      if (FULL || 16 * kk < D)
#pragma unroll
        for (int t = 0; t < 4; ++t) s = mfma_f32(k[kk][t], q[kk][t], s);
    if (blk + NW < n_keys) load_k(blk + NW);
    float mx = -INFINITY;
    bool seen[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      seen[x] = kF32Rows * blk + 4 * kq + x < limit;
      s[x] *= scale;
      mx = seen[x] ? fmaxf(mx, s[x]) : mx;
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m, mx);
    if (__any(m_new > m)) {
      const float alpha = m_new > m ? expf(m - m_new) : 1.f;
      l *= alpha;
#pragma unroll
      for (int x = 0; x < 4 * DB; ++x) acc[x] *= alpha;
      m = m_new;
    }
    const float ref = m == -INFINITY ? 0.f : m;   // no finite score so far: all weights are zero
    f32x4 p;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      p[x] = seen[x] ? expf(s[x] - ref) : 0.f;
      l += p[x];
    }
    if (kF32Rows * (blk + 1) > len) {
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int db = 0; db < DB; ++db)
          if (kF32Rows * blk + 4 * kq + x >= len) v[x][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (causal && blk == block) {
      bool any = false;
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int db = 0; db < DB; ++db) any |= f32_not_finite(v[x][db]);
      redo = __any(any);
    }
#pragma unroll
    for (int x = 0; x < 4; ++x)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[4 * db + t] = mfma_f32(v[x][db][t], p[x], acc[4 * db + t]);
    if (blk + NW < n_keys) load_v(blk + NW);
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (lane < kF32Rows) {
    ms[wave][lane] = m;
    ls[wave][lane] = l;
  }
  __syncthreads();   // (also: `odd` has been cleared)
  if (redo && lane == 0) odd = 1;
  float top = -INFINITY, sum = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) top = fmaxf(top, ms[w][i]);
  auto factor = [&](float mw) { return mw < top ? expf(mw - top) : 1.f; };
#pragma unroll
  for (int w = 0; w < NW; ++w) sum = fmaf(ls[w][i], factor(ms[w][i]), sum);
  const float mine = factor(m);
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int x = 0; x < 4; ++x)
      part[wave][4 * db + x][lane] = f32x4{acc[4 * db][x], acc[4 * db + 1][x], acc[4 * db + 2][x], acc[4 * db + 3][x]} * mine;
  __syncthreads();
  if (!odd) {
    float* o = reinterpret_cast<float*>(a.O) + at;
    for (int n = wave; n < 4 * DB; n += NW) {   // columns 64 (n / 4) + 16 kq + 4 (n % 4) and three more
      f32x4 r = part[0][n][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) r += part[w][n][lane];
      r = f32x4{r[0] / sum, r[1] / sum, r[2] / sum, r[3] / sum};
      const int d = 64 * (n >> 2) + 16 * kq + 4 * (n & 3);
      if (row < S && d < D) *reinterpret_cast<f32x4*>(o + d) = r;
    }
  } else {
    const int rows = min(kF32Rows, S - kF32Rows * block);
    for (int r = wave; r < rows; r += NW)
      f32_row_by_key(a, K, V, __shfl(at, r), __shfl(limit, r), __shfl(top, r), __shfl(sum, r), scale, D, lane);
  }
}

template <int DB>
static hipError_t launch_exact_f32(const ExactArgs& a, int D, int causal, float scale,
                                   hipStream_t stream) {
  const size_t units = (size_t)a.B * a.Hq * ((a.S + kF32Rows - 1) / kF32Rows);
  // One unit per workgroup while the chip has room for its chains side by side: beyond these lines K
  // and V, which only the other kernel shares between rows, cost more than the chains save.  us per
  // call, four waves on one unit / on four: 8 heads of 400 x 128 (200 units) 15.6 / 50.1, 64 heads of
  // 400 x 64 (1,600) 26.2 / 34.4, 128 of 94 x 128 (768) 12.4 / 17.1, 168 (1,008) 19.9 / 18.8, 192 of
  // 128 x 128 (1,536) 24.7 / 24.6, 512 of 32 x 64 (1,024) 7.7 / 6.7, 128 of 32 x 64 (256) 4.8 / 5.9.
  const size_t most = a.S <= 64 ? 512 : a.S < 128 ? 768 : 1536;
  if (D % 16 == 0 && units <= most) {
    constexpr int NW = 4;   // eight: 64 heads of 94 x 128 13.5 us, four 9.9
    if (D == 64 * DB)
      hipLaunchKernelGGL((exact_f32_split_kernel<DB, NW, true>), dim3((unsigned)units), dim3(NW * kWave), 0, stream, a, D,
                         causal, scale);
    else
      hipLaunchKernelGGL((exact_f32_split_kernel<DB, NW, false>), dim3((unsigned)units), dim3(NW * kWave), 0, stream, a, D,
                         causal, scale);
    return hipGetLastError();
  }
  const unsigned grid = f32_grid(a.n_kvtiles, a.Hq / a.Hkv, a.S);
  if (D == 64 * DB)
    hipLaunchKernelGGL((exact_f32_kernel<DB, kAllCols>), dim3(grid), dim3(kThreads), 0, stream, a, D, causal, scale);
  else if (D % 4 == 0)
    hipLaunchKernelGGL((exact_f32_kernel<DB, kVecCols>), dim3(grid), dim3(kThreads), 0, stream, a, D, causal, scale);
  else if (DB == 1 && D < 4)
    hipLaunchKernelGGL((exact_f32_kernel<1, kFewCols>), dim3(grid), dim3(kThreads), 0, stream, a, D, causal, scale);
  else
    hipLaunchKernelGGL((exact_f32_kernel<DB, kAnyCols>), dim3(grid), dim3(kThreads), 0, stream, a, D, causal, scale);
  return hipGetLastError();
}

template <int D, bool CAUSAL, bool RESIDENT>
static hipError_t launch_exact_bf16_r(const ExactArgs& a, dim3 grid, hipStream_t stream) {
  // resident launch: at most 32 workgroups per compute unit walk the tiles (enough of them for
  // the hardware to even out an uneven mix of hits and misses -- fewer, longer-lived workgroups
  // measured 2-5 % slower; a multiple of 8 keeps a workgroup's tiles on its own XCD)
  // The resident variant walks its tiles with a fixed number of workgroups.  Dispatching a
  // workgroup takes time even when it finds nothing to do (some 420 workgroups start per
  // microsecond: 8,192 of them cost the 19 us that a launch on a batch without misses used to
  // take), so a routed launch, which may find little or nothing, gets half as many.  Fewer
  // still would help that case more (2,048: 7 instead of 9 us) but costs a launch with many
  // misses its load balance (64 of 128 items at the 8B shape: 4-9 % slower, the hardware
  // balances many short-lived workgroups better than few long-lived ones); 4,096 costs nothing
  // measurable there.
  if (RESIDENT) {
    const unsigned cap = a.row_sel ? 4096u : 8192u;
    if (grid.x > cap) grid.x = cap;
  }
  hipLaunchKernelGGL((exact_bf16_kernel<D, CAUSAL, RESIDENT>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <int D, bool CAUSAL>
static hipError_t launch_exact_bf16(const ExactArgs& a, dim3 grid, hipStream_t stream) {
  return a.n_rblk == 1 ? launch_exact_bf16_r<D, CAUSAL, true>(a, grid, stream)
                       : launch_exact_bf16_r<D, CAUSAL, false>(a, grid, stream);
}

// Sequences of up to 128 keys (short_tile.hpp); us per call, the resident kernel / this one: 64 x 12 heads
// of 64 x 64, padded 7.6 / 7.4; 128 x 12 of 32 x 64 9.9 / 7.4; 192 x 8 of 32 x 128 (1,536 units) 17.4 / 11.2; 100 x 32 of 64 x 128 44 / 36; 51 x 8 on 2
// of 96 x 64 10.8 / 7.2; 48 x 8 on one of 128 x 64 (1,536 units) 21.5 / 7.9; 64 x 512 of 128 x 64, causal 399 / 357 (6.0 TB/s), half of them
// routed away 197 / 187, all 5.5 / 23.  Bound by the memory where it is large, else by the chain of Q, K and V -> scores -> weights -> products -> stores.
template <int D, bool CAUSAL, int NRB>
__global__ __launch_bounds__(kThreads, 2) void exact_bf16_short_kernel(const ShortArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char short_smem[];
  short_attention<D, CAUSAL, NRB, false>(
      a, reinterpret_cast<bf16_t*>(short_smem), [](const ShortUnit&, int, const u32x4 (&)[2]) {}, [](const ShortUnit&, int) {});
}

static ShortArgs exact_short_args(const ExactLaunch& p, float scale_log2e) {
  ShortArgs a;
  a.Q = static_cast<const bf16_t*>(p.Q); a.K = static_cast<const bf16_t*>(p.K); a.V = static_cast<const bf16_t*>(p.V);
  a.O = static_cast<bf16_t*>(p.O); a.row_sel = p.row_sel; a.key_len = p.key_len;
  a.Hq = p.Hq; a.Hkv = p.Hkv; a.Lc = 1; a.n_tiles = p.B * p.Hkv; a.scale_log2e = scale_log2e;
  return a;
}
static hipError_t launch_exact_short(const ExactLaunch& p, const ShortArgs& a, unsigned grid, hipStream_t stream) {
  const size_t lds = short_lds(a, p.S, p.D);
  auto go = [&](auto d, auto c, auto nrb) {
    constexpr auto kernel = &exact_bf16_short_kernel<decltype(d)::value, decltype(c)::value, decltype(nrb)::value>;
    const hipError_t e = ensure_lds<kernel>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads), lds, stream, a);
    return hipGetLastError();
  };
  auto rows = [&](auto d, auto c) {
    return p.S == 32   ? go(d, c, std::integral_constant<int, 1>{})
           : p.S == 64 ? go(d, c, std::integral_constant<int, 2>{})
           : p.S == 96 ? go(d, c, std::integral_constant<int, 3>{})
                       : go(d, c, std::integral_constant<int, 4>{});
  };
  auto mask = [&](auto d) { return p.causal ? rows(d, std::true_type{}) : rows(d, std::false_type{}); };
  return p.D == 64 ? mask(std::integral_constant<int, 64>{}) : mask(std::integral_constant<int, 128>{});
}

constexpr int kSplitWaves = 4;   // eight: 8 heads of 1024 x 128 16.1 us, four 14.0
template <int D, bool CAUSAL>
static hipError_t launch_exact_split(const ExactArgs& a, size_t units, hipStream_t stream) {
  hipLaunchKernelGGL((exact_bf16_split_kernel<D, CAUSAL, kSplitWaves>), dim3((unsigned)units), dim3(kSplitWaves * kWave), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_exact(const ExactLaunch& p, hipStream_t stream) {
  if (p.B == 0) return hipSuccess;
  ExactArgs a;
  a.Q = p.Q; a.K = p.K; a.V = p.V; a.O = p.O; a.row_sel = p.row_sel; a.key_len = p.key_len;
  a.B = p.B; a.Hq = p.Hq; a.Hkv = p.Hkv; a.S = p.S;
  a.n_rblk = (p.S + kChunk - 1) / kChunk;
  a.n_kvtiles = p.B * p.Hkv;
  const float scale = p.scale == 0.f ? 1.0f / sqrtf((float)p.D) : p.scale;
  a.scale_log2e = scale * 1.44269504088896340736f;
  if (p.is_f32) {   // D <= 256, by the number of 64-wide output blocks
    if (p.D <= 64) return launch_exact_f32<1>(a, p.D, p.causal, scale, stream);
    if (p.D <= 128) return launch_exact_f32<2>(a, p.D, p.causal, scale, stream);
    return launch_exact_f32<4>(a, p.D, p.causal, scale, stream);
  }
  const size_t units = (size_t)p.B * p.Hq * (p.S / 32);
  // One unit per workgroup while that leaves room on the chip (as above).  us per call, split / not: 8 heads of 1024 x 128 causal
  // (256 units) 14.0 / 23.7, 64 of 288 x 128 (576) 12.2 / 10.2, 64 of 288 x 64 (576) 7.6 / 7.9, 24 of 512 x 64 dense (384) 9.0 / 9.7, 64
  // of 512 x 64 (1,024) 14.0 / 11.3.  Up to 128 keys: 64 heads of 128 x 128 (256) 7.5 / 8.2, 96 (384) 8.7 / 8.3; 256 of 32 x 64 (256)
  // 5.1 / 5.6, 384 5.7 / 5.8, 192 pairs (384) 5.6 / 5.5, 192 of 64 x 64, causal (384) 5.9 / 6.0, 256 (512) 6.2 / 6.4, 96 of 128 x 64, causal (384)
  // 6.4 / 6.7, 128 (512) 6.7 / 6.8, not causal (384) 7.4 / 6.4.
  const int g = p.Hq / p.Hkv;
  const size_t most = p.S > 128 ? (p.D == 64 ? 576 : 320) / (p.causal ? 1 : 2)
                      : p.D == 64 && p.causal && (p.S == 128 || (g == 1 && p.S <= 64)) ? 512 : p.D == 64 ? 320 : 256;
  if (units <= most) {
    if (p.D == 64) return p.causal ? launch_exact_split<64, true>(a, units, stream) : launch_exact_split<64, false>(a, units, stream);
    return p.causal ? launch_exact_split<128, true>(a, units, stream) : launch_exact_split<128, false>(a, units, stream);
  }
  if (p.S <= 128) {
    // A routed launch of many tiles may find few of them to do: the resident kernel tests 64 at a time, here each costs the launch
    // of a workgroup (32,768 tiles, none to do, 5.5 us and 23).  Very large causal launches of 128 x 128 of two heads on a K and V
    // are faster there too: 1,024 x 32 heads on 16 (131,072 units) 586 / 620 us, 2,048 1,198 / 1,259, 512 298 / 296; not of four, 2,048 x 64 on 16
    // 1,970 / 1,981, 1,024 989 / 995.
    const bool slower = p.causal && p.D == 128 && p.S == 128 && g == 2 && units > 100000;
    ShortArgs sa = exact_short_args(p, a.scale_log2e);
    const unsigned wgs = short_plan(sa, p.S, p.D);
    if (!slower && (!p.row_sel || wgs <= 2048)) return launch_exact_short(p, sa, wgs, stream);
  }
  const int u8 = (a.n_kvtiles + 7) / 8 * 8;
  const int per_u = a.n_rblk == 1 ? 1 : (g * (p.S / 32) + 3) / 4;   // workgroups of a K/V tile
  const dim3 grid((unsigned)((size_t)u8 * per_u));
  if (p.D == 64)
    return p.causal ? launch_exact_bf16<64, true>(a, grid, stream)
                    : launch_exact_bf16<64, false>(a, grid, stream);
  return p.causal ? launch_exact_bf16<128, true>(a, grid, stream)
                  : launch_exact_bf16<128, false>(a, grid, stream);
}

}  // namespace ac

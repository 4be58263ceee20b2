// Operands of a wave that works alone on one 32-row unit and some of its 32-key blocks (bf16): what
// the exact and the insert kernel of small launches share.  K comes straight from memory to the
// lanes that multiply it, V through a wave-private LDS tile (the transposing read wants it there),
// both one block ahead, and no barrier is needed.
#pragma once
#include "common.hpp"

namespace ac {

// LDS operations of one wave execute in order: only the compiler has to keep them so.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int D>
struct SplitOperands {
  static constexpr int PPR = D / 8, NV = 32 * PPR / kWave;   // V pieces per lane and block
  const bf16_t *K, *V;   // of the (item, KV head)
  bf16_t* vt;            // the wave's 32 x D tile in LDS
  int lane, il, kh;
  u32x4 q[D / 16], k[D / 16], v[NV];

  __device__ __forceinline__ SplitOperands(const bf16_t* K, const bf16_t* V, bf16_t* vt, int lane)
      : K(K), V(V), vt(vt), lane(lane), il(lane & 31), kh(lane >> 5) {}
  // the unit's rows as the column operand, K rows as the row operand: row il, piece 2 ks + kh
  __device__ __forceinline__ void load_q(const bf16_t* rows) {
    const bf16_t* src = rows + (size_t)il * D + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) q[ks] = *reinterpret_cast<const u32x4*>(src + 16 * ks);
  }
  __device__ __forceinline__ void load_k(int blk) {
    const bf16_t* src = K + (size_t)(32 * blk + il) * D + 8 * kh;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) k[ks] = *reinterpret_cast<const u32x4*>(src + 16 * ks);
  }
  __device__ __forceinline__ void load_v(int blk) {   // whole rows, side by side
    const bf16_t* src = V + (size_t)(32 * blk) * D + 8 * lane;
#pragma unroll
    for (int n = 0; n < NV; ++n) v[n] = *reinterpret_cast<const u32x4*>(src + 8 * kWave * n);
  }
  __device__ __forceinline__ void stage_v() const {   // then wave_lds_fence()
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      const int r = (n * kWave + lane) / PPR, c = lane % PPR;
      *reinterpret_cast<u32x4*>(vt + r * D + 8 * (c ^ v_piece_swizzle<D>(r))) = v[n];
    }
  }
  // scores^T of the loaded K block: 32 keys x 32 rows, this lane: row il, keys mfma_row(x, kh)
  __device__ __forceinline__ f32x16 scores() const {
    f32x16 s;
#pragma unroll
    for (int x = 0; x < 16; ++x) s[x] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      s = mfma_bf16(__builtin_bit_cast(bf16x8, k[ks]), __builtin_bit_cast(bf16x8, q[ks]), s);
    return s;
  }
  // acc += V^T P^T for the staged V block.  Contraction slot e of lane half kh, step s2, is key
  // 16 s2 + 8 (e / 4) + 4 kh + e % 4, where the first product left the scores; lane i of a group of
  // 16 names key 4 kh + 8 half + i / 4 and four d from 32 db + 16 (il / 16) + 4 (i % 4).
  __device__ __forceinline__ void weights_v(f32x16 (&acc)[D / 32], const u32x4 (&p)[2]) const {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef short s16x8 __attribute__((ext_vector_type(8)));
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int db = 0; db < D / 32; ++db) {
        s16x4 w[2];
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          const int t = lane & 15, j = 16 * s2 + 4 * kh + 8 * half + (t >> 2);
          const int d0 = 32 * db + 16 * (il >> 4) + 4 * (t & 3);
          w[half] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(
              vt + j * D + 8 * ((d0 >> 3) ^ v_piece_swizzle<D>(j)) + (d0 & 7)));
        }
        const s16x8 vop = {w[0][0], w[0][1], w[0][2], w[0][3], w[1][0], w[1][1], w[1][2], w[1][3]};
        acc[db] = mfma_bf16(__builtin_bit_cast(bf16x8, vop), __builtin_bit_cast(bf16x8, p[s2]), acc[db]);
      }
  }
};

// The sum of the NW waves' accumulators (acc * mine) leaves as the unit's output rows, divided into
// column pieces among the waves.  part: NW (D / 8) kWave vectors of LDS that nobody else uses;
// o: the unit's first row.  Every wave of the workgroup takes part.
template <int D, int NW>
__device__ __forceinline__ void split_store(const f32x16 (&acc)[D / 32], float mine, float inv, f32x4* part,
                                            bf16_t* o, int wave, int lane) {
  static_assert(D / 8 % NW == 0, "the pieces are dealt to the waves");
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int vq = 0; vq < 4; ++vq)
      part[(wave * (D / 8) + 4 * db + vq) * kWave + lane] =
          f32x4{acc[db][4 * vq], acc[db][4 * vq + 1], acc[db][4 * vq + 2], acc[db][4 * vq + 3]} * mine;
  __syncthreads();
  o += (size_t)(lane & 31) * D + 4 * (lane >> 5);
#pragma unroll
  for (int n0 = 0; n0 < D / 8; n0 += NW) {   // columns 8 n + 4 kh and three more of row il
    const int n = n0 + wave;
    f32x4 r = part[n * kWave + lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) r += part[(w * (D / 8) + n) * kWave + lane];
    *reinterpret_cast<u32x2*>(o + 8 * n) = u32x2{pack_bf16(r[0] * inv, r[1] * inv), pack_bf16(r[2] * inv, r[3] * inv)};
  }
}

}  // namespace ac

// Decode unit on the matrix cores, for groups of four or more q heads per kv
// head (decode_body.hpp chooses).
//
// Decode is memory-bandwidth bound (Sec. 1 and 2.1 of the paper): every key
// and value of the context is read once per kv head and used by only G q
// heads, so the unit is organised around streaming the paged blocks at full
// HBM rate and keeping the vector work per byte small: both products run on
// the matrix cores (v_mfma_f32_16x16x32_bf16, the q heads as the 16 columns,
// those past G zero), although G columns of them fill only a part.  With
// v_dot2 the vector work grows with G and bound the unit at G = 8, and it
// competed with the tiles' softmax beside it: 40 rows of 234 MB at G = 8
// alone 68 -> 54 us, with 4,056 tokens of prefill tiles 137 -> 115-125 us; at
// G = 4 1,338k keys alone 1101 -> 1081 us.
//
// The range is walked in tiles of 32 keys (one 32-key block or two 16-key
// ones), wave w taking tiles w, w+4, ..., with the next tile's loads issued
// before the current one is used.  Per tile and wave, lane l = 16 g + i:
//   S^T (2 x 16 keys x 16 heads) = K . Q^T.  Row i of key half b is key
//     8 (i / 4) + 4 b + i % 4 of the tile, so that lane (g, i) ends up with
//     head i's scores of keys 8 g .. 8 g + 7: exactly the B operand of the
//     second product, so the weights never leave the lane.
//   O^T (D x 16 heads) += V^T . P^T: lane (g, i) reads 8 consecutive keys of
//     feature rows 16 dt + i, the A operand as the [D][B] blocks store it.
// Every load instruction reads contiguous memory: of V a kilobyte (two half
// ones for 16-key blocks), of K four keys' rows, which pass through a
// wave-private LDS slice to become operands (16 bytes of 16 rows per lane
// group; chunk c of row i at c ^ i, so both sides are conflict-free).  Loaded
// as operands from memory, in 64-byte pieces of 16 rows, K's stream cost
// 7 % of the rate (512-token budget mix 148 -> 159 us).
// Online softmax runs in base 2 with a lazily updated running max per head.
// The 4 waves' (max, sum, output) states are combined through LDS; a unit
// covering the whole context writes the bf16 output, a split unit writes its
// normalised fp32 output and log2-sum-exp for the merge pass.
#pragma once

#include "decode_lds.hpp"
#include "device.hpp"

namespace cpattn {

namespace decode_impl {

constexpr int kMfmaKeys = 32;  // keys per tile

// LDS of one unit, in bytes: a slice per wave that holds 16 keys' rows during
// the loop and the wave's output [G][D] fp32 after it, and 2 x [4][G] fp32.
template <int D, int G>
struct MfmaLds {
  static constexpr int kWaves = kDecodeWaves;
  static constexpr int SLICE = 16 * D * 2;
  static_assert(G * D * 4 <= SLICE, "wave slice");
  static constexpr int O_BYTES = kWaves * SLICE;
  static constexpr int ML_BYTES = kWaves * G * 4;
  static constexpr int SMALL_BYTES = 2 * ML_BYTES;
};

__device__ __forceinline__ f32x4_t mfma16x16x32(uint4 a, uint4 b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

}  // namespace decode_impl

template <int D, int B, int G>
__device__ __forceinline__ void decode_unit_mfma(
    const DecodeItem& it, int kvh, bool active, int tid, const uint16_t* __restrict__ q,
    const uint16_t* __restrict__ k_cache, const uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ bt, uint16_t* __restrict__ out, float* __restrict__ part_o,
    float* __restrict__ part_lse, int hq, int hkv, int mbr, float scale_log2,
    decode_impl::DecodeLdsPtrs lds) {
  using namespace decode_impl;
  using Lds = MfmaLds<D, G>;
  constexpr int TK = kMfmaKeys;
  constexpr int NKS = D / 32;  // k-steps of a score
  constexpr int NDT = D / 16;  // 16-feature blocks of the output
  constexpr int kWaves = Lds::kWaves;
  static_assert(G <= 16 && (B == 16 || B == TK), "tile geometry");

  constexpr int OW = Lds::SLICE / 4;
  float* red_o = lds.o;                                                // [kWaves][OW]
  float* red_m = reinterpret_cast<float*>(lds.small);                  // [kWaves][G]
  float* red_l = reinterpret_cast<float*>(lds.small + Lds::ML_BYTES);  // [kWaves][G]

  const int part = it.part < 0 ? -1 : it.part + kvh * it.part_kvh_stride;
  const int lane = tid & 63;
  // wave-uniform in a scalar register, so that the tile loop, its branches
  // and the block-table reads are scalar and leave the vector memory counter
  // to the K/V loads (the prefetched tile stays in flight during a tile)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15;
  const int g = lane >> 4;

  uint4 qv[NKS];  // head i's features [32 ks + 8 g, +8)
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) qv[ks] = make_uint4(0, 0, 0, 0);
  if (active && i < G) {
    const uint16_t* qb = q + ((int64_t)it.tok * hq + kvh * G + i) * D + g * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qv[ks] = ld_global16(qb + ks * 32);
  }
  __builtin_amdgcn_sched_barrier(0);  // query loads stay older than the tile loads

  float m_run = -INFINITY, l_run = 0.f;  // head i's running max; this lane's share of its sum
  f32x4_t o[NDT];
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int64_t head_elems = (int64_t)B * D;
  const int32_t* bt_row = bt + (int64_t)it.req * mbr;
  const int n_tiles = (it.kv_end - it.kv_begin + TK - 1) / TK;
  const int lb_last = (it.kv_end - 1) / B;
  // V: lane offset inside a block, and (16-key blocks) whether the lane's
  // keys lie in the tile's second block
  const int voff = i * B + (8 * g) % B;
  const bool v_second = 8 * g >= B;
  // K: load (b, j) reads the contiguous KPL rows of half b from row KPL j on,
  // this lane 16 bytes of row KPL j + krow
  constexpr int CH = D / 8, KPL = 64 / CH;  // 16-byte chunks per row, rows per load
  constexpr int NKL = 16 / KPL;             // loads per half
  const int krow = lane / CH, kchunk = lane % CH;
  const int koff = (8 * (krow >> 2) + (krow & 3)) * D + kchunk * 8;
  uint8_t* slice = reinterpret_cast<uint8_t*>(lds.o) + wave * Lds::SLICE;
  // Each K/V byte is read by one workgroup only, so the loads are
  // non-temporal (streamed past the caches instead of displacing lines other
  // workgroups reuse).
  auto load_tile = [&](int t, u32x4_t (&kr)[2][NKL], uint4 (&vr)[NDT]) {
    const int lb = it.kv_begin / B + t * (TK / B);
    const int64_t b0 = ((int64_t)bt_row[lb] * hkv + kvh) * head_elems;
    int64_t b1 = b0;
    // past the range its last block again: those keys are masked
    if constexpr (B < TK) b1 = ((int64_t)bt_row[min(lb + 1, lb_last)] * hkv + kvh) * head_elems;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < NKL; ++j) {
        const int key0 = 2 * KPL * j + 4 * b;  // the load's first key
        kr[b][j] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(
            k_cache + (key0 < B ? b0 : b1) + (key0 % B) * D + koff));
      }
    const uint16_t* vp = v_cache + (v_second ? b1 : b0) + voff;
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) vr[dt] = ld_global16_nt(vp + dt * 16 * B);
  };
  auto slot = [](int row, int chunk) {
    return row * (D * 2) + ((chunk ^ (CH == 16 ? row & 15 : (row >> 1) & 7)) * 16);
  };

  // one tile: scores, online softmax, weighted values
  auto step = [&](const u32x4_t (&kr)[2][NKL], uint4 (&vr)[NDT], int t) {
    const int valid = it.kv_end - it.kv_begin - t * TK;  // keys of the range in this tile
    f32x4_t s[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      // a wave's LDS accesses complete in order: no wait but for the data
#pragma unroll
      for (int j = 0; j < NKL; ++j)
        *reinterpret_cast<u32x4_t*>(slice + slot(KPL * j + krow, kchunk)) = kr[b][j];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
        s[b] = mfma16x16x32(*reinterpret_cast<const uint4*>(slice + slot(i, 4 * ks + g)), qv[ks], s[b]);
      __builtin_amdgcn_wave_barrier();
    }
    if (valid < TK) {  // keys past the range: no weight, and their values may hold NaN
      const int k0 = 8 * g;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k0 + 4 * b + r >= valid) s[b][r] = -INFINITY;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        uint32_t* w = reinterpret_cast<uint32_t*>(&vr[dt]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t lo = (k0 + 2 * e) < valid ? 0x0000ffffu : 0u;
          const uint32_t hi = (k0 + 2 * e + 1) < valid ? 0xffff0000u : 0u;
          w[e] &= (lo | hi);
        }
      }
    }
    float x = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                    fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3]))) * scale_log2;
    if (__builtin_amdgcn_ballot_w64(x > m_run + kRescaleThreshold)) {
      // the four lanes of a head share its max
      x = fmaxf(x, shfl_xor_f(x, 16));
      x = fmaxf(x, shfl_xor_f(x, 32));
      const float mnew = fmaxf(m_run, x);
      const float alpha = m_run == -INFINITY ? 0.f : exp2f(m_run - mnew);
      m_run = mnew;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) o[dt] *= alpha;
    }
    uint32_t p[4];  // keys 8 g + 2 e, + 1
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float p0 = exp2f(__builtin_fmaf(s[e >> 1][2 * (e & 1)], scale_log2, -m_run));
      const float p1 = exp2f(__builtin_fmaf(s[e >> 1][2 * (e & 1) + 1], scale_log2, -m_run));
      p[e] = pack_bf16x2(p0, p1);
      l_run = dot2_bf16(p[e], 0x3f803f80u, l_run);  // the rounded weights
    }
    const uint4 pv = make_uint4(p[0], p[1], p[2], p[3]);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) o[dt] = mfma16x16x32(vr[dt], pv, o[dt]);
  };

  // Two register sets in turn: the loads of a wave's next tile are in flight
  // while it works on the current one.  The prefetch is unconditional (past
  // the range it re-reads the range's last tile, which is unused) so that
  // the compiler's wait counts stay exact and never drain the prefetch.
  // (Three sets at D = 64, whose tiles are half as large: 2 % slower.)
  if (active) {
    u32x4_t ka[2][NKL], kb[2][NKL];
    uint4 va[NDT], vb[NDT];
    const int last = n_tiles - 1;  // units are never empty
    int t = wave;
    load_tile(min(t, last), ka, va);
    for (; t < n_tiles; t += 2 * kWaves) {
      load_tile(min(t + kWaves, last), kb, vb);
      step(ka, va, t);
      if (t + kWaves >= n_tiles) break;
      load_tile(min(t + 2 * kWaves, last), ka, va);
      step(kb, vb, t + kWaves);
    }
  }

  // ---- this wave's state: lane (g, i) holds features 16 dt + 4 g .. + 3 of head i
  l_run += shfl_xor_f(l_run, 16);
  l_run += shfl_xor_f(l_run, 32);
  if (i < G) {
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
      *reinterpret_cast<f32x4_t*>(red_o + wave * OW + i * D + dt * 16 + 4 * g) = o[dt];
    if (g == 0) {
      red_m[wave * G + i] = m_run;
      red_l[wave * G + i] = l_run;
    }
  }
  __syncthreads();
  if (!active) return;

  // ---- combine the waves and write
  for (int x = tid; x < G * D; x += 256) {
    const int h = x / D;
    const int d = x % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) M = fmaxf(M, red_m[w * G + h]);
    float L = 0.f, O = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const float mw = red_m[w * G + h];
      const float f = mw == -INFINITY ? 0.f : exp2f(mw - M);
      L += f * red_l[w * G + h];
      O += f * red_o[w * OW + h * D + d];
    }
    const float val = L > 0.f ? O / L : 0.f;
    if (part < 0) {
      out[((int64_t)it.tok * hq + kvh * G + h) * D + d] = to_bf16(val);
    } else {
      part_o[(int64_t)(part + h) * D + d] = val;
      if (d == 0) part_lse[part + h] = L > 0.f ? M + __log2f(L) : -INFINITY;
    }
  }
}

}  // namespace cpattn

// bf16 GEMMs for the projections of the decoder layer around the attention
// step (include/cp_layer.h, cpl_gemm):
//     C[M][N] = A[M][K] . W[N][K]^T (+ R[M][N]),   fp32 accumulation, bf16 out.
// Both operands are K-contiguous rows, which is how the matrix cores take
// them: with v_mfma_f32_16x16x32_bf16 lane l holds 16 bytes (8 consecutive k)
// of row l % 16.  The products are formed transposed, D^T (16 n x 16 m) =
// W_blk . A_blk^T, so a lane's accumulators hold 4 consecutive n of one m.
//
// A workgroup of 8 waves (WM x WN) computes a BM x BN tile of C.  K is walked
// in stages of 64 (128-byte row pieces, whole cache lines), copied straight
// from global memory into a ring of NS LDS slots (global_load_lds_dwordx4, no
// register staging).  The copies are written as the instruction itself: the
// compiler does not track them, and the explicit vmcnt waits are the only
// ones.  A row's 16-byte chunk c is stored at chunk c ^ ((row >> 1) & 7), so
// the 16 lanes of a phase of an operand read hit 16 distinct bank groups.
//
// Two kernels share that layout and differ in how a stage is worked off:
//
// * gemm_tile_kernel, for tiles whose MFMAs take longer than their copies
//   (large batches).  Two waves share a SIMD; waves 0-3 and 4-7 run half a
//   stage out of step, so that while one reads operands from LDS the other
//   keeps the matrix pipe busy.
// * gemm_stream_kernel, for the short tiles of decode-sized batches, which
//   are bound by the weight stream: one barrier per stage, the next stage's
//   operands read while the current one is multiplied.
//
// Split over K: a grid too small to fill the GPU is multiplied by S slices of
// K; slice s writes its fp32 partial tile to ws[s][M][N] and a second kernel
// adds the S partials (and R) and rounds.
//
// Workgroup order: workgroup g runs on XCD g mod 8, and each XCD takes a
// contiguous run of tiles, ordered in groups of 4 row blocks with the row
// block fastest, so that the ~32 tiles resident on an XCD share their A and W
// panels in its L2.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include "cp_layer.h"

namespace {

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kXcds = 8;
constexpr int kCus = 256;
constexpr int kRowGroup = 4;             // row blocks per group of the tile order
constexpr int kStageK = 64;              // k per stage
constexpr int kRow = kStageK * 2;        // bytes of a staged row
constexpr int kMaxLds = 160 * 1024;
constexpr int kMaxSplit = 8;
constexpr int kGridX = 1 << 20;          // workgroups in a full row of the grid

__device__ __forceinline__ f32x4_t mfma(uint4 a, uint4 b, f32x4_t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// 16 bytes per lane from base + off into LDS at dst + 16 * lane (base and dst
// wave-uniform).  `stream`: non-temporal, for weights that one workgroup
// reads.  (The register constraints exist only in the device pass.)
__device__ __forceinline__ void copy16_to_lds(const char* base, uint32_t off, uint32_t dst,
                                              bool stream) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (stream)
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "{m0}"(dst)
                 : "memory");
  else
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(dst)
                 : "memory");
#endif
}
// The same with a 64-bit address per lane.
__device__ __forceinline__ void copy16_to_lds_far(const char* src, uint32_t dst, bool stream) {
#if defined(__HIP_DEVICE_COMPILE__)
  if (stream)
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "{m0}"(dst) : "memory");
  else
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "{m0}"(dst) : "memory");
#endif
}

// s_waitcnt with vmcnt <= N, the other counters unconstrained (gfx9 encoding)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt");
  __builtin_amdgcn_s_waitcnt((N & 15) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}
// s_waitcnt lgkmcnt(0): this wave's LDS reads have returned
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// waits until at most `later` (<= MAX) stages' copies, L each, are pending
template <int L, int MAX>
__device__ __forceinline__ void wait_stages(int later) {
  if constexpr (MAX > 0) {
    if (later >= MAX) {
      wait_vmcnt<MAX * L>();
      return;
    }
    wait_stages<L, MAX - 1>(later);
  } else {
    wait_vmcnt<0>();
  }
}

// Workgroup barrier without the memory fence of __syncthreads, which would
// also wait for the copies of later stages (the waits above are explicit);
// nothing is moved across it.
__device__ __forceinline__ void barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ uint16_t to_bf16(float a) {
  return __builtin_bit_cast(uint16_t, (__bf16)a);  // nearest even
}
__device__ __forceinline__ uint32_t pack(float a, float b) {
  return (uint32_t)to_bf16(a) | ((uint32_t)to_bf16(b) << 16);
}
__device__ __forceinline__ float lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

struct GemmArgs {
  const uint16_t* a;
  const uint16_t* w;
  const uint16_t* r;   // residual or NULL
  uint16_t* c;
  float* part;         // split partials, or NULL: C is written directly
  int m, n, k;
  int split;
  bool stream_w;       // copy W non-temporally
  bool rotate;         // stream kernel: XCDs start at different stages
};

// The tile and K slice of a workgroup.
struct Tile {
  int m0, n0;    // first row and column
  int slice;
  int st0, nk;   // first stage and stages
};

// false: no tile for this workgroup (the grid is rounded up to the XCDs)
template <int BM, int BN>
__device__ __forceinline__ bool pick_tile(const GemmArgs& g, Tile& t) {
  const int mb = (g.m + BM - 1) / BM, nb = g.n / BN, tiles = mb * nb * g.split;
  const int per = (tiles + kXcds - 1) / kXcds;
  const unsigned wg = blockIdx.y * kGridX + blockIdx.x;
  int i = (int)(wg % kXcds) * per + (int)(wg / kXcds);
  if (i >= tiles || (int)(wg / kXcds) >= per) return false;
  t.slice = i / (mb * nb);
  i -= t.slice * mb * nb;
  const int group = i / (kRowGroup * nb);
  i -= group * kRowGroup * nb;
  const int rows = min(kRowGroup, mb - group * kRowGroup);
  t.n0 = i / rows * BN;
  t.m0 = (group * kRowGroup + i % rows) * BM;
  const int stages = (g.k + kStageK - 1) / kStageK;
  t.st0 = (int)((int64_t)t.slice * stages / g.split);
  t.nk = (int)((int64_t)(t.slice + 1) * stages / g.split) - t.st0;
  return true;
}

// One 1 KiB piece of a staged tile: 8 rows of `src` [limit][K] from `row` (rows past the
// last read the last: their products are discarded).
// FAR: K rows so long that 7 of them pass 32 bits.
template <bool FAR>
struct Offset {
  typedef uint32_t type;
};
template <>
struct Offset<true> {
  typedef uint64_t type;
};
template <bool FAR>
struct Piece {
  const char* base;                  // wave-uniform
  typename Offset<FAR>::type off;    // this lane's byte offset from it (7 rows of K at most)
  uint32_t dst;                      // LDS address in slot 0
};
template <bool FAR = false>
__device__ __forceinline__ Piece<FAR> piece(const uint16_t* src, int k, int row0, int limit, int row,
                                            int st0, uint32_t lds, int lane) {
  typedef typename Offset<FAR>::type offset_t;
  const int rr = row + (lane >> 3);
  const int first = min(row0 + row, limit - 1);
  const int chunk = (lane & 7) ^ ((rr >> 1) & 7);
  Piece<FAR> p;
  p.base = reinterpret_cast<const char*>(src + (int64_t)first * k + (int64_t)st0 * kStageK);
  p.off = (offset_t)(min(row0 + rr, limit - 1) - first) * (offset_t)k * 2 + (offset_t)chunk * 16;
  p.dst = lds + row * kRow;
  return p;
}

// Byte offset inside a 16-row operand block of lane l's chunk, k-half h of a
// stage (row l % 16, logical chunk 4 h + l / 16).
__device__ __forceinline__ uint32_t operand_offset(int h, int lane) {
  const int r = lane & 15;
  return (uint32_t)(r * kRow + (((4 * h + (lane >> 4)) ^ ((r >> 1) & 7)) * 16));
}
__device__ __forceinline__ uint4 lds16(const uint8_t* p) { return *reinterpret_cast<const uint4*>(p); }

// acc[i][j] register e holds m = m1 + 16 i + lane % 16, n = n1 + 16 j + 4 (lane / 16) + e.
// Partials go out as they are (16 bytes per lane).  bf16 rows pass through a
// wave-private LDS slice, so that they leave in 16-byte pieces, consecutive
// lanes along a row; every wave is past its last operand read (a barrier
// before the call).
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const GemmArgs& g, int slice, int m1, int n1,
                                           f32x4_t (&acc)[TM][TN], uint8_t* lds, int lane) {
  if (g.part) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int m = m1 + 16 * i + (lane & 15);
      if (m >= g.m) continue;
      float* row = g.part + ((int64_t)slice * g.m + m) * g.n + n1 + 4 * (lane >> 4);
#pragma unroll
      for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4_t*>(row + 16 * j) = acc[i][j];
    }
    return;
  }
  constexpr int PITCH = TN * 32 + 16;  // bytes of a staged row
  constexpr int CH = TN * 2;           // its 16-byte chunks
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int j = 0; j < TN; ++j)
      *reinterpret_cast<uint2*>(lds + (lane & 15) * PITCH + j * 32 + (lane >> 4) * 8) =
          make_uint2(pack(acc[i][j][0], acc[i][j][1]), pack(acc[i][j][2], acc[i][j][3]));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int x0 = 0; x0 < 16 * CH; x0 += 64) {
      const int x = x0 + lane;
      const int m = m1 + 16 * i + x / CH;
      if (x < 16 * CH && m < g.m)
        *reinterpret_cast<uint4*>(g.c + (int64_t)m * g.n + n1 + (x % CH) * 8) =
            lds16(lds + (x / CH) * PITCH + (x % CH) * 16);
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Adds the residual in place of the accumulators' layout (8 bytes per lane and block).
template <int TM, int TN>
__device__ __forceinline__ void add_residual(const GemmArgs& g, int m1, int n1,
                                             f32x4_t (&acc)[TM][TN], int lane) {
  if (g.part || !g.r) return;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = m1 + 16 * i + (lane & 15);
    if (m >= g.m) continue;
    const uint16_t* row = g.r + (int64_t)m * g.n + n1 + 4 * (lane >> 4);
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const uint2 r = *reinterpret_cast<const uint2*>(row + 16 * j);
      acc[i][j][0] += lo(r.x), acc[i][j][1] += hi(r.x);
      acc[i][j][2] += lo(r.y), acc[i][j][3] += hi(r.y);
    }
  }
}

// Large tiles.  The row blocks of a wave are worked off in two parts, the
// first T0 and the other T1, each as a read phase (operands from LDS to
// registers) and an MFMA phase; W's operands stay in registers over both.
// Waves 0-3 start one phase ahead of waves 4-7 (the latter pass one more
// barrier first), and SIMD s holds waves s and s + 4, so in every phase one
// of them reads while the other multiplies.  With phases 4k.. for stage k of
// the first group:
//     first group   read 0 | mfma 0 | read 1 | mfma 1
//     second group  mfma 1 of stage k-1 | read 0 | mfma 0 | read 1
// Slot k % NS is refilled as soon as both groups have read it: its W rows in
// read 1 of stage k (W of stage k + NS), its A rows in read 0 of stage k + 1.
// A group copies only the A rows that it reads itself, so each copy has about
// four to six phases (2-3k cycles at 256 x 256) to land with two slots.
//
// A 256 x 256 x 64 stage takes 2,048 matrix-pipe cycles per SIMD, 64 KiB of
// copies and 192 KiB of operand reads per CU.  Measured against the earlier
// 128 x 128 tiles (one barrier and one wait per stage, two workgroups per
// CU): 2048 x 6144 x 4096 142 -> 84 us (1.23 PFLOP/s), 4096 x 24576 x 4096
// 847 -> 594 us (1.39 PFLOP/s; a loop of these MFMAs and barriers without
// copies or reads takes 458 us at the clock that the power limit leaves).
// Tried and left out: a single wait and K-half phases (640 us), deeper rings
// of 32-k stages (664), prefetching lines to L2 (+10 %), s_setprio around
// the MFMAs (+1-3 %), other pairings of the groups (750).
template <int WM, int WN, int TM, int TN, int NS>
__global__ __launch_bounds__(512, 2) void gemm_tile_kernel(GemmArgs g) {
  constexpr int BM = WM * TM * 16, BN = WN * TN * 16, SB = (BM + BN) * kRow;
  constexpr int T0 = TM / 2, T1 = TM - T0;
  constexpr int GP = BM / 16, GP0 = (WM / 2) * T0 * 2;  // a group's A pieces, those of the T0 parts
  constexpr int NA = (GP + 3) / 4, NA0 = (GP0 + 3) / 4; // per wave
  constexpr int PW = BN / 8, NW = (PW + 7) / 8;
  constexpr int L = NA + NW;
  static_assert(WM * WN == 8 && WM % 2 == 0 && T0 > 0, "waves");
  static_assert(SB * NS <= kMaxLds && (NS - 1) * L < 64, "ring");
  static_assert(8 * 16 * (TN * 32 + 16) <= SB * NS, "store slices");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[SB * NS];
  Tile t;
  if (!pick_tile<BM, BN>(g, t)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN, group = wave >> 2;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  const bool stream = g.stream_w;
  const int nk = t.nk;

  // the group's A pieces, the T0 parts first, dealt in turn to its 4 waves;
  // W's to all 8 (where they do not divide, the last piece is copied twice)
  Piece<false> pa[NA], pw[NW];
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int x = min(j * 4 + (wave & 3), GP - 1);
    const bool first = x < GP0;
    const int y = first ? x : x - GP0, per = (first ? T0 : T1) * 2;
    const int row = group * (BM / 2) + (y / per) * TM * 16 + (first ? 0 : T0 * 16) + (y % per) * 8;
    pa[j] = piece(g.a, g.k, t.m0, g.m, row, t.st0, lds0, lane);
  }
#pragma unroll
  for (int j = 0; j < NW; ++j)
    pw[j] = piece(g.w, g.k, t.n0, g.n, min(j * 8 + wave, PW - 1) * 8, t.st0, lds0 + BM * kRow, lane);
  auto issue_a = [&](int st, int slot) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
      copy16_to_lds(pa[j].base + (int64_t)st * kRow, pa[j].off, pa[j].dst + slot * SB, false);
  };
  auto issue_w = [&](int st, int slot) {
#pragma unroll
    for (int j = 0; j < NW; ++j)
      copy16_to_lds(pw[j].base + (int64_t)st * kRow, pw[j].off, pw[j].dst + slot * SB, stream);
  };

  const uint32_t ofs[2] = {operand_offset(0, lane), operand_offset(1, lane)};
  const uint8_t* a_lds = smem + wm * TM * 16 * kRow;
  const uint8_t* w_lds = smem + (BM + wn * TN * 16) * kRow;
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // copies are issued in the order W0 A0 W1 A1 ..., here up to W of stage
  // NS - 1; each wait below allows those issued after what it waits for, and
  // near the end, where fewer follow, waits for all
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nk) {
      issue_w(s, s);
      if (s < NS - 1) issue_a(s, s);
    }
  if (nk >= NS)
    wait_vmcnt<(NS - 1) * L - NA>();
  else
    wait_vmcnt<0>();
  barrier();
  if (group) barrier();
  int slot = 0;
  for (int k = 0; k < nk; ++k) {
    const uint8_t* as = a_lds + slot * SB;
    const uint8_t* ws = w_lds + slot * SB;
    uint4 wv[2][TN], av[2][T1];
    // read 0
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int j = 0; j < TN; ++j) wv[h][j] = lds16(ws + ofs[h] + j * 16 * kRow);
#pragma unroll
      for (int i = 0; i < T0; ++i) av[h][i] = lds16(as + ofs[h] + i * 16 * kRow);
    }
    const bool more_a = k + NS - 1 < nk, more_w = k + NS < nk;
    if (more_a) issue_a(k + NS - 1, slot == 0 ? NS - 1 : slot - 1);
    wait_lds();
    barrier();
    // mfma 0
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < T0; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma(wv[h][j], av[h][i], acc[i][j]);
    if (more_a)  // this stage's other A rows
      wait_vmcnt<(NS - 1) * L>();
    else
      wait_vmcnt<0>();
    barrier();
    // read 1
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < T1; ++i) av[h][i] = lds16(as + ofs[h] + (T0 + i) * 16 * kRow);
    if (more_w) issue_w(k + NS, slot);
    wait_lds();
    if (more_w)  // the next stage's W
      wait_vmcnt<(NS - 1) * L>();
    else
      wait_vmcnt<0>();
    barrier();
    // mfma 1
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < T1; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[T0 + i][j] = mfma(wv[h][j], av[h][i], acc[T0 + i][j]);
    if (more_w) wait_vmcnt<(NS - 1) * L - NA0>();  // the next stage's first A rows
    barrier();
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  if (!group) barrier();
  const int m1 = t.m0 + wm * TM * 16, n1 = t.n0 + wn * TN * 16;
  add_residual<TM, TN>(g, m1, n1, acc, lane);
  store_tile<TM, TN>(g, t.slice, m1, n1, acc, smem + wave * 16 * (TN * 32 + 16), lane);
}

// Short tiles.  One barrier per stage: behind it a wave issues the copies of
// stage k + NS into the slot that every wave has just finished reading, the
// LDS reads of stage k + 1, and the MFMAs of stage k from registers.  HALF:
// K is an odd number of 32s, and the last stage's second half is left out
// (its copies re-read the first half, so nothing past a row is touched).
//
// Bound by the weight stream: with W's copies non-temporal and the ring
// holding 16-48 KiB of W in flight per CU, 24 rows x 24576 x 4096 take 37.7
// us (5.3 TB/s; 42.7 with ordinary copies), 24 x 4096 x 12288 20.5 us.
//
// With `rotate`, XCD x walks the stages from x / 8 of them on, around the end.
// All workgroups read the same k at about the same time, and weight rows a
// power of two apart then fall on few memory channels: 24 rows x 24576 x 4096
// 38.7 -> 36.3 us, 96 rows 46.5 -> 42.2, 128 rows 49.0 -> 44.6; no difference
// at K = 12288 or where the weights are small.
template <int WM, int WN, int TM, int TN, int NS, bool HALF = false, bool FAR = false>
__global__ __launch_bounds__(512, 2) void gemm_stream_kernel(GemmArgs g) {
  constexpr int BM = WM * TM * 16, BN = WN * TN * 16, SB = (BM + BN) * kRow;
  constexpr int PA = BM / 8, PW = BN / 8, NA = (PA + 7) / 8, NW = (PW + 7) / 8, L = NA + NW;
  static_assert(WM * WN == 8 && SB * NS <= kMaxLds && (NS - 1) * L < 64, "ring");
  static_assert(8 * 16 * (TN * 32 + 16) <= SB * NS, "store slices");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[SB * NS];
  Tile t;
  if (!pick_tile<BM, BN>(g, t)) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)smem;
  const bool stream = g.stream_w;
  const int nk = t.nk;
  // the slice's last stage when it holds only 32 k, else past the end
  const int half = HALF && g.k % kStageK && t.st0 + nk == (g.k + kStageK - 1) / kStageK ? nk - 1 : nk;

  Piece<FAR> pa[NA], pw[NW];
#pragma unroll
  for (int j = 0; j < NA; ++j)
    pa[j] = piece<FAR>(g.a, g.k, t.m0, g.m, min(j * 8 + wave, PA - 1) * 8, t.st0, lds0, lane);
#pragma unroll
  for (int j = 0; j < NW; ++j)
    pw[j] = piece<FAR>(g.w, g.k, t.n0, g.n, min(j * 8 + wave, PW - 1) * 8, t.st0, lds0 + BM * kRow, lane);
  const int turn = !HALF && g.rotate ? (int)(blockIdx.x % kXcds) * nk / kXcds : 0;
  auto issue = [&](int st, int slot) {
    st += turn;
    if (st >= nk) st -= nk;
    // chunks 4-7 of a half stage read chunks 0-3 (a K row's chunk offset is
    // below 128 bytes, and K a multiple of 64 bytes: bit 6 is the half)
    auto copy = [&](const Piece<FAR>& p, int row, bool nt) {
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      const auto off = HALF && st == half && chunk >= 4 ? p.off - 64 : p.off;
      if constexpr (FAR)
        copy16_to_lds_far(p.base + (int64_t)st * kRow + off, p.dst + slot * SB, nt);
      else
        copy16_to_lds(p.base + (int64_t)st * kRow, off, p.dst + slot * SB, nt);
    };
#pragma unroll
    for (int j = 0; j < NW; ++j) copy(pw[j], min(j * 8 + wave, PW - 1) * 8 + (lane >> 3), stream);
#pragma unroll
    for (int j = 0; j < NA; ++j) copy(pa[j], min(j * 8 + wave, PA - 1) * 8 + (lane >> 3), false);
  };

  const uint32_t ofs[2] = {operand_offset(0, lane), operand_offset(1, lane)};
  const uint8_t* a_lds = smem + wm * TM * 16 * kRow;
  const uint8_t* w_lds = smem + (BM + wn * TN * 16) * kRow;
  f32x4_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  struct Operands {
    uint4 w[2][TN], a[2][TM];
  };
  auto read = [&](Operands& o, int slot) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int j = 0; j < TN; ++j) o.w[h][j] = lds16(w_lds + slot * SB + ofs[h] + j * 16 * kRow);
#pragma unroll
      for (int i = 0; i < TM; ++i) o.a[h][i] = lds16(a_lds + slot * SB + ofs[h] + i * 16 * kRow);
    }
  };
  auto multiply = [&](const Operands& o, int k) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (HALF && h == 1 && k == half) break;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = mfma(o.w[h][j], o.a[h][i], acc[i][j]);
    }
  };

#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nk) issue(s, s);
  wait_stages<L, NS - 1>(min(NS - 1, nk - 1));
  barrier();
  Operands even, odd;
  read(even, 0);
  int slot = 0;
  auto step = [&](int k, Operands& cur, Operands& next) {
    const int nslot = slot + 1 == NS ? 0 : slot + 1;
    wait_lds();  // this wave's reads of stage k, before the slot is refilled
    wait_stages<L, NS - 2>(min(NS - 2, nk - 2 - k));  // stage k + 1 is in
    barrier();
    if (k + NS < nk) issue(k + NS, slot);
    read(next, nslot);
    __builtin_amdgcn_sched_barrier(0);
    multiply(cur, k);
    slot = nslot;
  };
  int k = 0;
  for (; k + 2 < nk; k += 2) {
    step(k, even, odd);
    step(k + 1, odd, even);
  }
  if (k + 1 < nk) {
    step(k, even, odd);
    multiply(odd, k + 1);
  } else {
    multiply(even, k);
  }
  barrier();  // the stores' slices overlap the ring
  const int m1 = t.m0 + wm * TM * 16, n1 = t.n0 + wn * TN * 16;
  add_residual<TM, TN>(g, m1, n1, acc, lane);
  store_tile<TM, TN>(g, t.slice, m1, n1, acc, smem + wave * 16 * (TN * 32 + 16), lane);
}

// C = sum over S slices of part (+ R), 4 elements per thread; all loads are
// issued before the first add.
template <int S>
__global__ __launch_bounds__(256) void split_sum_kernel(const float* __restrict__ part,
                                                        const uint16_t* R, uint16_t* C,
                                                        int64_t mn4) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= mn4) return;
  f32x4_t p[S];
#pragma unroll
  for (int s = 0; s < S; ++s) p[s] = reinterpret_cast<const f32x4_t*>(part)[(int64_t)s * mn4 + i];
  uint2 r = make_uint2(0, 0);
  if (R) r = reinterpret_cast<const uint2*>(R)[i];
  f32x4_t v = p[0];
#pragma unroll
  for (int s = 1; s < S; ++s) v += p[s];
  if (R) v[0] += lo(r.x), v[1] += hi(r.x), v[2] += lo(r.y), v[3] += hi(r.y);
  reinterpret_cast<uint2*>(C)[i] = make_uint2(pack(v[0], v[1]), pack(v[2], v[3]));
}

template <int S>
void launch_sum(const GemmArgs& g, hipStream_t s) {
  if constexpr (S > 1) {
    if (g.split != S) {
      launch_sum<S - 1>(g, s);
      return;
    }
    const int64_t mn4 = (int64_t)g.m * g.n / 4;
    hipLaunchKernelGGL((split_sum_kernel<S>), dim3((unsigned)((mn4 + 255) / 256)), dim3(256), 0, s,
                       g.part, g.r, g.c, mn4);
  }
}

using Kernel = void (*)(GemmArgs);
struct Cfg {
  int bm, bn;
  float stage_us, tile_us;
  Kernel kernel;
};
template <int WM, int WN, int TM, int TN, int NS>
constexpr Cfg tile_cfg(float stage_us, float tile_us) {
  return {WM * TM * 16, WN * TN * 16, stage_us, tile_us, gemm_tile_kernel<WM, WN, TM, TN, NS>};
}
template <int WM, int WN, int TM, int TN, int NS, bool HALF = false, bool FAR = false>
constexpr Cfg stream_cfg(float stage_us, float tile_us) {
  return {WM * TM * 16, WN * TN * 16, stage_us, tile_us,
          gemm_stream_kernel<WM, WN, TM, TN, NS, HALF, FAR>};
}

// Tile configurations (CPL_GEMM_CFG selects one by its index), each with the
// microseconds that a stage of 64 k takes and that a tile takes besides, as
// fitted over 4,600 timings (rows 17-2,048 by the layer's projections at
// hidden 2,048 and 4,096 and its LM head, weights from HBM; 7-14 % rms).
constexpr Cfg kCfgs[] = {
    tile_cfg<2, 4, 8, 4, 2>(1.086f, 12.4f),  // 0: 256 x 256
    tile_cfg<2, 4, 8, 3, 2>(0.987f, 10.3f),  // 1: 256 x 192
    tile_cfg<2, 4, 6, 4, 2>(0.887f, 10.8f),  // 2: 192 x 256
    tile_cfg<4, 2, 4, 4, 3>(0.734f, 8.5f),   // 3: 256 x 128
    tile_cfg<2, 4, 9, 2, 3>(0.820f, 9.2f),   // 4: 288 x 128
    tile_cfg<2, 4, 5, 3, 3>(0.729f, 9.8f),   // 5: 160 x 192
    tile_cfg<2, 4, 4, 3, 3>(0.670f, 8.8f),   // 6: 128 x 192
    tile_cfg<2, 4, 5, 2, 4>(0.604f, 7.4f),   // 7: 160 x 128
    stream_cfg<2, 4, 4, 2, 4>(0.520f, 6.3f), // 8: 128 x 128
    stream_cfg<4, 2, 2, 3, 5>(0.481f, 5.7f), // 9: 128 x 96
    stream_cfg<2, 4, 3, 2, 5>(0.454f, 6.0f), // 10: 96 x 128
    stream_cfg<4, 2, 2, 2, 6>(0.366f, 4.4f), // 11: 128 x 64
    stream_cfg<2, 4, 2, 2, 3>(0.393f, 5.2f), // 12: 64 x 128
    stream_cfg<2, 4, 3, 1, 4>(0.311f, 4.1f), // 13: 96 x 64
    stream_cfg<2, 4, 2, 1, 5>(0.250f, 3.7f), // 14: 64 x 64
    stream_cfg<2, 4, 1, 2, 4>(0.327f, 4.1f), // 15: 32 x 128
    stream_cfg<2, 4, 1, 1, 6>(0.213f, 3.5f), // 16: 32 x 64
};
constexpr int kNumCfgs = sizeof(kCfgs) / sizeof(kCfgs[0]);
// for K an odd number of 32s (times as of the same tiles above)
constexpr Cfg kHalf64 = stream_cfg<2, 4, 2, 2, 3, true>(0.393f, 5.2f);
constexpr Cfg kHalf128 = stream_cfg<2, 4, 4, 2, 4, true>(0.520f, 6.3f);
// for any K, of which 7 rows and a row's chunk may pass 32 bits of byte offset
constexpr int kMaxNearK = (int)((0xffffffffu - kRow) / 14);
constexpr Cfg kFar = stream_cfg<2, 4, 2, 2, 3, true, true>(0.393f, 5.2f);

int env_int(const char* name, int dflt) {
  const char* s = getenv(name);
  return s ? atoi(s) : dflt;
}

// Estimated microseconds of a tile and split: whole rounds of 256 workgroups
// (a CU works off two small ones no faster than one after the other), no less
// than the operands take from HBM (5.8 TB/s, less with idle CUs), plus the
// partials' way through memory and the adding launch.  Where two
// configurations are bound by memory, the shorter compute time wins.  Large
// batches run under the power limit and take longer than this (2048 x 24576 x
// 4096: 258 us here, 280-295 measured), all tiles of them alike.
float estimate(const Cfg& f, int M, int N, int K, int S) {
  const int tiles = (M + f.bm - 1) / f.bm * (N / f.bn) * S;
  const int stages = ((K + kStageK - 1) / kStageK + S - 1) / S;
  const float compute = (float)((tiles + kCus - 1) / kCus) * (stages * f.stage_us + f.tile_us);
  const float mn = (float)M * N;
  float memory = ((float)N * K + (float)M * K + mn) * 2.f / 5.8e6f;
  if (tiles < kCus) memory *= sqrtf((float)kCus / tiles);
  float t = fmaxf(compute, memory + 3.f) + 0.05f * compute;
  if (S > 1) t += 2.5f + S * mn * 4.f / 4.5e6f;
  return t;
}

// Tile configuration and K split for a shape: the cheapest by the estimate
// among those whose columns divide N and whose partials fit the workspace
// (over the timings above, 1 % slower than the best on average, 11 % at
// most).  Slices are at least 6 stages long, and the grid is split no
// further than two workgroups per CU.
void choose(int M, int N, int K, size_t ws_floats, const Cfg** cfg, int* split) {
  const int stages = (K + kStageK - 1) / kStageK;
  const int forced_cfg = env_int("CPL_GEMM_CFG", -1), forced_split = env_int("CPL_GEMM_SPLIT", 0);
  const Cfg* best = nullptr;
  int best_split = 1;
  float best_us = 0.f;
  auto fits = [&](int s) { return s <= 1 || (size_t)s * (size_t)M * (size_t)N <= ws_floats; };
  auto consider = [&](const Cfg& f) {
    const int64_t tiles = (int64_t)((M + f.bm - 1) / f.bm) * (N / f.bn);
    for (int s = 1; s <= kMaxSplit; ++s) {
      if (forced_split > 0) {
        if (s > 1 && (s > forced_split || s > stages || !fits(s))) break;
      } else if (s > 1 && (tiles * s > 2 * kCus || stages / s < 6 || !fits(s))) {
        break;
      }
      const float us = estimate(f, M, N, K, s);
      // a forced split: the largest allowed up to it
      const bool better = !best || (forced_split > 0 && best == &f) || us < best_us;
      if (better) best = &f, best_split = s, best_us = us;
    }
  };
  if (K > kMaxNearK) {
    consider(kFar);
  } else if (K % kStageK != 0) {
    consider(M <= 64 ? kHalf64 : kHalf128);
  } else {
    for (int c = 0; c < kNumCfgs; ++c) {
      if (N % kCfgs[c].bn != 0) continue;
      if (forced_cfg >= 0 && forced_cfg < kNumCfgs && c != forced_cfg &&
          N % kCfgs[forced_cfg].bn == 0)
        continue;
      consider(kCfgs[c]);
    }
  }
  *cfg = best;
  *split = best_split;
}

}  // namespace

extern "C" {

size_t cpl_gemm_workspace_bytes(int32_t m, int32_t n, int32_t k) {
  if (m < 1 || n < 128 || n % 128 != 0 || k < 32 || k % 32 != 0) return 0;
  const Cfg* cfg;
  int s;
  choose(m, n, k, (size_t)-1 / 8, &cfg, &s);
  return s > 1 ? (size_t)s * m * n * sizeof(float) : 0;
}

int cpl_gemm(const void* a, const void* w, const void* r, void* c, int32_t m, int32_t n,
             int32_t k, void* ws, size_t ws_bytes, void* stream) {
  if (m < 1 || n < 128 || n % 128 != 0 || k < 32 || k % 32 != 0) return CP_ERR_INVALID_ARG;
  if (!a || !w || !c || a == c || w == c) return CP_ERR_INVALID_ARG;
  auto al16 = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  if (!al16(a) || !al16(w) || !al16(c) || (r && !al16(r)) || (ws && !al16(ws)))
    return CP_ERR_INVALID_ARG;
  if ((int64_t)m * k >= ((int64_t)1 << 40) || (int64_t)n * k >= ((int64_t)1 << 40) ||
      (int64_t)m * n >= ((int64_t)1 << 40))
    return CP_ERR_INVALID_ARG;
  const Cfg* cfg;
  int split;
  choose(m, n, k, ws ? ws_bytes / sizeof(float) : 0, &cfg, &split);
  GemmArgs g;
  g.a = (const uint16_t*)a;
  g.w = (const uint16_t*)w;
  g.r = (const uint16_t*)r;
  g.c = (uint16_t*)c;
  g.part = split > 1 ? (float*)ws : nullptr;
  g.m = m, g.n = n, g.k = k, g.split = split;
  const int row_blocks = (m + cfg->bm - 1) / cfg->bm;
  // Weights too large to stay in the 256 MB last-level cache beside the
  // layer's others, read by at most two row blocks, bypass it: 24 rows x
  // 24576 x 4096 42.7 -> 37.7 us, 96 rows 48.3 -> 44.9, 261 rows x 4096 x
  // 12288 43.9 -> 41.2.  With more row blocks (1000 x 6144 x 4096 52.9 ->
  // 56.2 us) or fewer weights (96 x 6144 x 4096 19.9 -> 20.4) it loses.
  g.stream_w = row_blocks <= 2 && (int64_t)n * k >= (int64_t)32 << 20;
  const int tiles = row_blocks * (n / cfg->bn) * split;
  // (over more rounds the XCDs drift apart by themselves: 24 rows x 151936 x
  // 4096, 1,187 tiles, 194 -> 203 us)
  g.rotate = tiles <= 2 * kCus;
  (void)hipGetLastError();
  hipStream_t s = (hipStream_t)stream;
  // a launch takes fewer than 2^32 threads in x: larger grids are laid out in rows
  const int wgs = (tiles + kXcds - 1) / kXcds * kXcds, grid_x = wgs < kGridX ? wgs : kGridX;
  hipLaunchKernelGGL(cfg->kernel, dim3(grid_x, (wgs + grid_x - 1) / grid_x), dim3(512), 0, s, g);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && split > 1) {
    launch_sum<kMaxSplit>(g, s);
    e = hipGetLastError();
  }
  return e == hipSuccess ? CP_OK : CP_ERR_HIP;
}

}  // extern "C"

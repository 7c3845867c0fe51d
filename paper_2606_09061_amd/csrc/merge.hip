// Merge of split key ranges.  Each split of a row left its normalised output
// O_s and L_s = log2(sum of its unnormalised weights) in base-2 units; the
// full-range output is
//     O = sum_s 2^(L_s - M) O_s / sum_s 2^(L_s - M),   M = max_s L_s,
// which is exact for any partition of the keys (softmax is shift invariant).
#include "device.hpp"
#include "kernels.hpp"

namespace cpattn {

// A row takes D / 4 threads, 4 features each, and the workgroup's 256 / (D / 4)
// such slots are shared by its rows: with P slots per row, slot p combines
// splits p, p + P, ..., eight loads in flight, and the P partial sums meet in
// LDS.  The kernel moves little and is bound by its chain of dependent loads:
// one slot per row walked the splits one after the other, their L_s first
// (8 decode rows of 40 splits 6.6 -> 2.9 us; a launch cannot do under ~2.4).
template <int D>
__global__ __launch_bounds__(256) void merge_kernel(const MergeGroup* __restrict__ groups,
                                                    const float* __restrict__ part_o,
                                                    const float* __restrict__ part_lse,
                                                    uint16_t* __restrict__ out, int hq, int G) {
  constexpr int DQ = D / 4;        // threads per row and slot
  constexpr int SLOTS = 256 / DQ;  // at least the rows of a group
  constexpr int U = 8;             // splits whose loads are in flight together
  __shared__ float4 s_acc[SLOTS][DQ];
  __shared__ float s_m[SLOTS], s_w[SLOTS];
  const MergeGroup mg = groups[blockIdx.x];
  // this workgroup's rows of the group
  const int per = (mg.n_rows + (int)gridDim.z - 1) / (int)gridDim.z;
  const int first = (int)blockIdx.z * per;
  const int n = min(per, mg.n_rows - first);
  if (n <= 0) return;
  const int slot = threadIdx.x / DQ, dq = threadIdx.x % DQ;
  const int P = min(SLOTS / n, mg.n_split);
  const int rl = slot % n, p = slot / n;
  const int rows = mg.n_tok * G;
  const int kvh = blockIdx.y;
  const int r = mg.row0 + first + rl;
  const int64_t base = (int64_t)mg.part0 + (int64_t)kvh * mg.n_split * rows + r;
  float M = -INFINITY, wsum = 0.f;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (p < P) {
    for (int s0 = p; s0 < mg.n_split; s0 += P * U) {
      float ls[U];
      float4 o[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // past the last split: it again, weight 0
        const int s = s0 + u * P;
        const int64_t pr = base + (int64_t)min(s, mg.n_split - 1) * rows;
        ls[u] = part_lse[pr];
        o[u] = *reinterpret_cast<const float4*>(part_o + pr * D + dq * 4);
        if (s >= mg.n_split) ls[u] = -INFINITY;
      }
      float m = M;
#pragma unroll
      for (int u = 0; u < U; ++u) m = fmaxf(m, ls[u]);
      const float keep = M == -INFINITY ? 0.f : exp2f(M - m);
      M = m;
      wsum *= keep;
      acc.x *= keep, acc.y *= keep, acc.z *= keep, acc.w *= keep;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = s0 + u * P < mg.n_split;
        const float w = ls[u] == -INFINITY ? 0.f : exp2f(ls[u] - m);
        if (in) {
          wsum += w;
          acc.x += w * o[u].x;
          acc.y += w * o[u].y;
          acc.z += w * o[u].z;
          acc.w += w * o[u].w;
        }
      }
    }
  }
  if (P > 1) {  // uniform
    if (p < P) {
      s_acc[slot][dq] = acc;
      if (dq == 0) s_m[slot] = M, s_w[slot] = wsum;
    }
    __syncthreads();
    if (p > 0) return;
    for (int k = 1; k < P; ++k) M = fmaxf(M, s_m[k * n + rl]);
    wsum = 0.f;
    acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < P; ++k) {
      const float mk = s_m[k * n + rl];
      const float w = mk == -INFINITY ? 0.f : exp2f(mk - M);
      const float4 a = s_acc[k * n + rl][dq];
      wsum += w * s_w[k * n + rl];
      acc.x += w * a.x;
      acc.y += w * a.y;
      acc.z += w * a.z;
      acc.w += w * a.w;
    }
  } else if (p > 0) {
    return;
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  const int tok = mg.tok0 + r / G;
  const int h = kvh * G + r % G;
  uint2 w2;
  w2.x = pack_bf16x2(acc.x * inv, acc.y * inv);
  w2.y = pack_bf16x2(acc.z * inv, acc.w * inv);
  *reinterpret_cast<uint2*>(out + ((int64_t)tok * hq + h) * D + dq * 4) = w2;
}

hipError_t launch_merge(int D, int G, const AttnArgs& a, hipStream_t s) {
  // few groups (decode rows): their rows spread over up to 8 workgroups each,
  // so that every row gets more slots; from about 4 workgroups per CU on that
  // only adds workgroups
  const int64_t groups = (int64_t)a.n_merge * a.hkv;
  const int z = groups <= 128 ? 8 : groups <= 256 ? 4 : groups <= 512 ? 2 : 1;
  const dim3 grid(a.n_merge, a.hkv, z);
  if (D == 128)
    hipLaunchKernelGGL(merge_kernel<128>, grid, dim3(256), 0, s, a.merge, a.part_o, a.part_lse,
                       a.out, a.hq, G);
  else if (D == 64)
    hipLaunchKernelGGL(merge_kernel<64>, grid, dim3(256), 0, s, a.merge, a.part_o, a.part_lse,
                       a.out, a.hq, G);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace cpattn

// Split-K decode attention for one (row, block range, kv head) unit, run by
// four waves: the body of the decode kernel, and of the decode blocks that
// the prefill kernel runs beside its tiles when a step's decode rows are
// overlapped with its prefill chunks.
#pragma once

#include <type_traits>

#include "decode_dot2.hpp"
#include "decode_mfma.hpp"

namespace cpattn {

namespace decode_impl {

// Groups of four or more q heads run on the matrix cores; with one or two,
// v_dot2 is little work, and its smaller registers keep four workgroups per
// CU instead of two (30 rows at G = 1, 220 MB: 42.2 against 44.2 us).  The
// planner sizes the units accordingly (kDecodeMfmaMinGroup).
template <int G>
constexpr bool kOnMfma = G >= kDecodeMfmaMinGroup;

template <int D, int G>
using DecodeLds = std::conditional_t<kOnMfma<G>, MfmaLds<D, G>, Dot2Lds<D, G>>;

}  // namespace decode_impl

// Runs one decode unit with the four waves whose workgroup-local thread ids
// are `tid` in [0, 256).  Every wave of the workgroup must call this the
// same number of times, with active == false for a group that has no unit:
// the unit synchronises the whole workgroup (one or two barriers).
template <int D, int B, int G>
__device__ __forceinline__ void decode_unit(
    const DecodeItem& it, int kvh, bool active, int tid, const uint16_t* __restrict__ q,
    const uint16_t* __restrict__ k_cache, const uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ bt, uint16_t* __restrict__ out, float* __restrict__ part_o,
    float* __restrict__ part_lse, int hq, int hkv, int mbr, float scale_log2,
    decode_impl::DecodeLdsPtrs lds) {
  if constexpr (decode_impl::kOnMfma<G>)
    decode_unit_mfma<D, B, G>(it, kvh, active, tid, q, k_cache, v_cache, bt, out, part_o, part_lse,
                              hq, hkv, mbr, scale_log2, lds);
  else
    decode_unit_dot2<D, B, G>(it, kvh, active, tid, q, k_cache, v_cache, bt, out, part_o, part_lse,
                              hq, hkv, mbr, scale_log2, lds);
}

}  // namespace cpattn

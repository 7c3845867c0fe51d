// LDS pointers of a decode unit.
#pragma once

#include <stdint.h>

namespace cpattn {
namespace decode_impl {

// `o` holds O_BYTES; `small` SMALL_BYTES, 16-byte aligned (DecodeLds).
struct DecodeLdsPtrs {
  float* o;
  uint8_t* small;
};

}  // namespace decode_impl
}  // namespace cpattn

// Where the register-staged GEMM's loads lie in a row (host and device; no HIP, so
// that a host program can check it).
#pragma once

namespace gl {

// A row of rowb bytes (a multiple of 16) is staged in stages of `step` bytes; the
// 16-byte slot `slot` of stage s lies at slot + this in the row.  Slots past the row
// load its first 16 bytes, which are zeroed when they are stored: also where the row
// is shorter than a stage, so that the last row's loads end with the tensor.
constexpr int gemm_slot_offset(int s, int step, int slot, int rowb) {
  return s * step + slot < rowb ? s * step : -slot;
}

}  // namespace gl

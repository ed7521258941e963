// Which instances can write their outputs through to the memory-side cache instead of storing them non-temporally: asked by the
// kernels (addrms_body, addrms_span_body, silumul_body) and by the rule that has a launch do it (launch_write_through).
#pragma once

// chunks: per thread, 0 for forms that do not count them.  Beyond six chunks, and with one element per chunk, the second kind of
// store takes registers that some instances do not have without giving up a wave per SIMD.
constexpr bool write_through_instance(int vec, int chunks) { return vec > 1 && chunks <= 6; }
// Output pieces of a thread that are: of up to 16 bytes.  (Residuals of fp16+fp32 with eight elements per chunk are two stores, and
// stay non-temporal.)
constexpr bool write_through_piece(int bytes) { return bytes <= 16; }

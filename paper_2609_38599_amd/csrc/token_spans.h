// The fp32 partial sums of the calibration products: spans of at most
// kSumTokens tokens.  Plain C++, so that the walk can be checked on the host.
#pragma once

namespace jarq {

constexpr int kSumTokens = 256;   // tokens per fp32 partial sum

// End of the span that starts at token t0 < m; no intermediate value passes m
// (chunks of tokens reach almost to the largest int).
constexpr int span_end(int t0, int m) {
  return m - t0 < kSumTokens ? m : t0 + kSumTokens;
}

}  // namespace jarq

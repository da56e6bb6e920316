// Positions of a matrix's entries, in host and device code.
#pragma once

#include <cstdint>

#ifdef __HIPCC__
#define AIRG_HD __host__ __device__ __forceinline__
#else
#define AIRG_HD inline
#endif

namespace airg {

// A matrix holds up to 2^31 - 1 entries.  A loop over a row looks up to a stride
// or a chunk past its end, and a search adds two positions: both pass 2^31, so
// positions that are computed with are unsigned.
typedef uint32_t epos;

AIRG_HD epos middle(epos lo, epos hi) { return (lo + hi) >> 1; }
// aligned pairs of entries that hold those before e
AIRG_HD epos pairs_before(epos e) { return (e + 1) >> 1; }

// the entry of column j among the ascending columns lo .. hi - 1, or -1
AIRG_HD int find_col(const int32_t* col, epos lo, epos hi, int j) {
  while (lo < hi) {
    const epos mid = middle(lo, hi);
    const int c = col[mid];
    if (c == j) return (int)mid;
    if (c < j) lo = mid + 1;
    else hi = mid;
  }
  return -1;
}
// the first of them at or past column w0, hi where none is
AIRG_HD epos first_from(const int32_t* col, epos lo, epos hi, int64_t w0) {
  while (lo < hi) {
    const epos mid = middle(lo, hi);
    if (col[mid] < w0) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}
// the end of the chunk of len entries that starts at p, in a row that ends at e
AIRG_HD epos chunk_end(epos p, epos e, epos len) { return p + len < e ? p + len : e; }

}  // namespace airg

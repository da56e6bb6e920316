// Launch shapes of the products and the shape an operator gets without the
// tuner.  Plain host code, so that the rule is tested without a device.
#pragma once

#include <cstdint>

namespace airg {

// Launch shape of a product: lanes per row in bits 0-7 (0: row-block kernel),
// the XCD mapping in bit 8, the LDS-staged kernel in bit 9, the
// entry-staged kernel (256 consecutive rows per workgroup, one lane per row)
// in bit 10.
constexpr int kShapeXcd = 1 << 8;
constexpr int kShapeLds = 1 << 9;
constexpr int kShapeEntries = 1 << 10;
// Several columns take the XCD mapping whatever bit 8 says (untuned operators): an
// element of x is then a cache line or more that neighbouring rows share.  Solves
// of 4 to 64 columns of FV 300^2 to 2048^2 are 0.2-1.6% faster with it on every
// operator; 20 columns of FV 1000^2 (FP32) 22.4 -> 22.0 ms.
constexpr int kShapeColumnsXcd = 1 << 11;

enum class OpRole { Plain, CPoint, Restrict, Steps, Formed, Top, Coarsest };

// What the rule looks at: the operator's size, the bytes of a stored value and
// of a vector element, and with compressed columns the widest 64-row window.
struct OpShape {
  int64_t rows, nnz;
  int vbytes, xbytes;
  bool windows;
  int64_t max_span;
};

// A matrix past three quarters of the 256 MB cache is read from HBM by every
// product; below that it mostly comes from the caches.
constexpr double kCachedBytes = 192e6;

// Lanes per row, with the XCD mapping (each XCD takes a contiguous eighth of the
// rows) where xcd allows it.  Measured over every operator of 31 systems (FV
// 64^2 to 8192^2, DG 1024^2, FD 1803^2 to 3606^2 with all up-smooths, 500 x
// 26000, batches of 16 and 48, in FP64, FP32 and BF16), the mean time of the
// shape over the best one's in brackets.
//
// From the caches: two lanes from 3.5 entries a row (1.06; one 1.16), 4 from 10
// (1.01; 2 lanes 1.08), 8 from 24 (1.02; 4 lanes 1.09), 16 from 50 (1.01; 8 lanes
// 1.05, from 80 on 1.15), 32 from 160 (equal there).  Eighths of the rows gain up
// to 20% on short rows and lose from about 100 entries a row on, where a row's
// gathers reach far anyway (130-170 entries: 16 lanes 1.08 with, 1.00 without).
//
// From HBM the mapping only spreads the traffic over more pages (FV 8192^2, 1.2 GB
// of B: 222.8 us with, 213.8 without) and lanes are needed earlier, to keep as
// many gathers in flight (FV 4096^2, 22.5 entries a row: 188 us with 4 lanes, 174
// with 8; FV 8192^2, 72.9: 109 with 8, 95.5 with 16).
//
// Short operators take more lanes while the launch has fewer than 400,000: up to
// 8 (from 10 to 24 entries 1.02, 4 lanes 1.10), below 16,384 rows up to 32, and a
// wavefront a row for rows of 256 and more (733 dense rows: 4.9 us with 32, 3.9
// with 64).
inline int default_lanes(int64_t rows, int64_t nnz, double bytes, bool xcd) {
  const double avg = rows > 0 ? (double)nnz / (double)rows : 0.0;
  if (bytes > kCachedBytes)
    return avg <= 3.5 ? 1 : avg <= 10.0 ? 2 : avg <= 16.0 ? 4 : avg <= 40.0 ? 8 : avg <= 160.0 ? 16 : 32;
  int lanes = avg <= 3.5 ? 1 : avg <= 10.0 ? 2 : avg <= 24.0 ? 4 : avg <= 50.0 ? 8 : avg <= 160.0 ? 16 : 32;
  const int most = rows >= 16384 ? 8 : rows >= 4096 || avg < 256.0 ? 32 : 64;
  while (lanes < most && rows * lanes < 400000 && avg >= 4.0 * lanes) lanes <<= 1;
  return lanes | (xcd && avg <= 100.0 ? kShapeXcd : 0);
}

inline int default_shape(const OpShape& A, OpRole role) {
  const double avg = A.rows > 0 ? (double)A.nnz / (double)A.rows : 0.0;
  // the top matrix's rows are so short that their pointers weigh as an index does
  const double bytes = (double)(A.vbytes + (A.windows && role != OpRole::Top ? 2 : 4)) * (double)A.nnz;
  // The entry-staged kernel loads the entries of 256 rows at consecutive
  // addresses, so more gathers are in flight than one lane a row keeps; below
  // four workgroups of it a CU the device is not full and a row's entries in
  // turn are the whole time (FV 64^2 level 1: 8.3 us, 2.8 with 4 lanes a row;
  // 173,000 rows of 2 entries 3.8 and 3.1, 236,000 of 5 entries 6.1 and 5.2).
  const bool entries = A.rows >= (int64_t)1 << 18;
  bool xcd = true;
  switch (role) {
    case OpRole::CPoint:
      // the rows of A_cf and A_cc lie block after block of the nested order, so
      // eighths of them sweep the domain at once and share nothing (FD 3606^2
      // level 1, 2.3 entries a row: 82.7 us with the mapping, 61.4 without)
      xcd = false;
      break;
    case OpRole::Restrict:
      // rows of about 3 entries that gather all over a level's F block (level 1
      // of FV 2048^2: 18.5 us with one lane a row, 15.9); where rows are longer
      // two lanes are even or better (level 2: 15.2, 15.8)
      if (entries && avg > 2.4 && avg <= 3.5) return 1 | kShapeEntries | kShapeXcd;
      break;
    case OpRole::Steps:
      // A_ff where the smoother takes its steps: as the restrictors, rows of 3
      // entries only (FD 3606^2 level 2: 22.0 -> 20.5 us; 1.8 entries 22.1, 24.6;
      // 3.9 entries on FV 4096^2 level 2 with two lanes 30.6, 36.3)
      if (entries && avg > 2.4 && avg <= 3.5) return 1 | kShapeEntries | kShapeXcd;
      break;
    case OpRole::Formed:
      // q(A_ff), whose rows gather further.  FV 2048^2 levels 0 and 1 (1.7 and 4.1
      // entries a row): 17.6 -> 15.1 and 16.6 -> 15.7 us, FV 4096^2 78.4 -> 63.7 and
      // 71.2 -> 62.1; a diagonal (1 entry) and rows of 9 are better with lanes, and so
      // are rows of 4 where an entry is 6 bytes (FV 2048^2 level 1 in FP32: 13.8, 13.7)
      if (entries && avg > 1.2 && avg <= (A.vbytes == 8 ? 5.5 : 3.5)) return 1 | kShapeEntries | kShapeXcd;
      break;
    case OpRole::Top:
      // read from HBM in consecutive addresses: 5 entries a row gain from 250 MB
      // on (DG 1024^2: 82.8 us, 82.0), 3 far above it (FV 8192^2, 2.4 GB: 855,
      // 790; FV 4096^2, 604 MB: 212, 211; batch of 229 MB: 80.6, 87.3)
      if (avg <= 8.0 && bytes > (avg > 4.0 ? kCachedBytes : 1e9)) return 1 | kShapeEntries;
      break;
    case OpRole::Coarsest:
      // ordered for narrow windows of x, which a workgroup of 64 rows stages in
      // LDS where it reads each element twice or more (FD 3606^2 with degree 100,
      // 1.3 times: 112 us staged, 102 with 32 lanes) and two workgroups fit a CU.
      // In FP64 16 lanes, or 8 where the matrix stays in the caches (FV 2048^2
      // 16.7 us, 32 lanes unstaged 18.3; FV 4096^2, 139 MB, 26.5, 29.1, with 16
      // lanes 28.8; the batch of 48, 188 MB, 36.1 with 16, 38.2 with 8, unstaged
      // 38.9; FV 8192^2, 408 MB, 87, 110, 122), and unstaged below 32,768 rows (25,111
      // rows 8.2 and 8.6); in FP32 and BF16 from 8192 rows on (13,463 rows 5.5 us,
      // unstaged 6.2).  The XCD mapping, which leaves a step's result where the next
      // step reads it, pays while the vectors are short: staged below 40,000 rows
      // (solves in ms without and with it: 13,382 rows 5.12 and 5.09, 28,842 in BF16
      // 9.39 and 9.14, 36,168 6.65 and 6.54; 16,771 3.75 and 3.83; a batch's 42,409
      // 5.45 and 5.60, 139,245 41.8 and 43.8), unstaged below 8192 (7,926 rows 2.12
      // and 2.06).
      if (A.windows && avg >= 48.0 && A.max_span * A.xbytes <= 64 * 1024 && 64.0 * avg >= 2.0 * (double)A.max_span &&
          A.rows >= (A.xbytes == 8 ? 32768 : 8192))
        return (A.xbytes == 8 && bytes <= 160e6 ? 8 : 16) | kShapeLds | (A.rows < 40000 ? kShapeXcd : 0);
      // Unstaged, 32 lanes pay from 80 entries a row, and from 16,384 rows on, where
      // 16 lanes are enough wavefronts, from 256 (whole solves in ms with 16 and 32
      // lanes: 6 problems of 256^2, 66 entries, 2.54 and 2.68; FV 1300^2, 15,514 rows
      // of 172 entries, 6.60 and 6.46; FD 2000^2, 19,704 of 249, 16.62 and 17.06; FD
      // 3606^2, 26,974 of 345, 26.49 and 26.37).
      if (A.rows >= 8192 && bytes <= kCachedBytes && avg > 50.0 && avg <= (A.rows >= 16384 ? 256.0 : 80.0))
        return 16;
      xcd = A.rows < 8192;
      break;
    case OpRole::Plain: break;
  }
  return default_lanes(A.rows, A.nnz, bytes, xcd);
}

}  // namespace airg

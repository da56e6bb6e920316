// Sparse products and structural kernels of the setup (paper Eqs. z,
// fixed_sparsity, prolong and the coarse product R A P).
//
// C = A B is formed row by row: a group of lanes takes a row of A, visits its
// entries k in stored (ascending) order one after the other and adds
// a_ik * (row k of B), whose columns are distinct, into a table of columns in
// LDS.  Every c_ij is so accumulated over k ascending from 0.0 and does not
// depend on scheduling.  Exact zeros are dropped afterwards.
#include <algorithm>
#include <cmath>
#include <vector>

#include "kernels.hpp"
#include "rows.hpp"

namespace airg {

// What a counting pass hands to the host besides its row lengths: their total
// and three words the kernels set (zeroed here), all read in one copy.
struct RowStat {
  DBuf<int64_t> d;
  int64_t h[4] = {0, 0, 0, 0};
  explicit RowStat(hipStream_t s) : d(4, s) { launch_zero_bytes(d.get(), 4 * sizeof(int64_t), s); }
  int32_t* flag(int k) const { return reinterpret_cast<int32_t*>(d.get() + 1 + k); }
  int32_t value(int k) const { return (int32_t)h[1 + k]; }
};

// Row pointers (int32) from row lengths; returns their total (the pointers are
// of use up to 2^31 - 1) and leaves st's words on the host.
constexpr int64_t kMaxNnz = 2147483647;
static int64_t count_rows(const DBuf<int32_t>& cnt, int64_t n, DBuf<int32_t>& rowptr, RowStat& st,
                          hipStream_t s) {
  rowptr.alloc(n + 1, s);
  DBuf<int64_t> work(rowptr_work_size(n), s);
  launch_rowptr_scan(cnt.get(), n, rowptr.get(), st.d.get(), work.get(), s);
  read_back(st.h, st.d.get(), sizeof(st.h), s);
  return st.h[0];
}
static void check_nnz(int64_t nnz) {
  if (nnz > kMaxNnz) fail(AIRG_ERR_NOMEM, "sparse matrix exceeds 2^31 nonzeros");
}
static int64_t counts_to_rowptr(const DBuf<int32_t>& cnt, int64_t n, DBuf<int32_t>& rowptr,
                                hipStream_t s) {
  RowStat st(s);
  const int64_t nnz = count_rows(cnt, n, rowptr, st, s);
  check_nnz(nnz);
  return nnz;
}

// ------------------------------------------------------------------ exact zeros
__global__ void nonzero_count_kernel(CSRView A, int32_t* count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  int32_t c = 0;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p) c += (A.val[p] != 0.0);
  count[i] = c;
}
__global__ void nonzero_fill_kernel(CSRView A, const int32_t* rowptr, int32_t* col, double* val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  int64_t o = rowptr[i];
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p)
    if (A.val[p] != 0.0) {
      col[o] = A.col[p];
      val[o] = A.val[p];
      ++o;
    }
}

// Drop the explicit zeros of `in` into `out`.
static void drop_zeros(const CSR& in, CSR& out, hipStream_t s) {
  const int64_t n = in.rows;
  DBuf<int32_t> cnt(n, s);
  unsigned nb = blocks_for(n, kBlock);
  if (n > 0) {
    nonzero_count_kernel<<<nb, kBlock, 0, s>>>(view(in), cnt.get());
    AIRG_CHECK_LAUNCH();
  }
    out.rows = n;
  out.cols = in.cols;
  out.nnz = counts_to_rowptr(cnt, n, out.rowptr, s);
  out.col.alloc(out.nnz, s);
  out.val.alloc(out.nnz, s);
  if (n > 0) {
    nonzero_fill_kernel<<<nb, kBlock, 0, s>>>(view(in), out.rowptr.get(), out.col.get(),
                                              out.val.get());
    AIRG_CHECK_LAUNCH();
  }
}

// ------------------------------------------------------------------ merged rows
// A stable insertion sort of entries s .. e-1 by column, by one thread.
__device__ __forceinline__ void insertion_sort(int s, int e, int32_t* col, double* val) {
  for (int p = s + 1; p < e; ++p) {
    int c = col[p];
    double v = val[p];
    int q = p - 1;
    while (q >= s && col[q] > c) {
      col[q + 1] = col[q];
      val[q + 1] = val[q];
      --q;
    }
    col[q + 1] = c;
    val[q + 1] = v;
  }
}

// Position of each of the lane's entries (the t-th is entry lane + G t, of
// column c[t]) among a row's len columns in LDS when sorted by column, equal
// columns in entry order: the entries before it are counted, four columns a
// read.  sc is padded with INT_MAX to a multiple of 4.
template <int G, int T>
__device__ __forceinline__ void rank_entries(const int32_t* sc, int len, const int (&c)[T], int lane,
                                             int (&r)[T]) {
#pragma unroll
  for (int t = 0; t < T; ++t) r[t] = 0;
  for (int j = 0; j < len; j += 4) {
    const int4 o = *reinterpret_cast<const int4*>(sc + j);
#pragma unroll
    for (int t = 0; t < T; ++t) {
      if (G * t >= len) break;
      const int i = lane + G * t;
      r[t] += (o.x < c[t] || (o.x == c[t] && j < i)) + (o.y < c[t] || (o.y == c[t] && j + 1 < i)) +
              (o.z < c[t] || (o.z == c[t] && j + 2 < i)) + (o.w < c[t] || (o.w == c[t] && j + 3 < i));
    }
  }
}

// A row gathered from up to two rows with mapped columns, entries whose mapped
// column is negative left out, sorted by column (stable) and equal columns
// summed left to right.  Two uses:
//   FC:  B = A_fc + A_ff W with W the one-point prolongation: row i of A_fc
//        (columns kept), then of A_ff (column j becomes cmap[j]);
//   !FC: A P with P one-point, cmap[j] the coarse column of node j or -1: the
//        sums start from 0.0 and exact zeros are dropped, as in a product
//        formed over k ascending (P's entries are 1).
// A group of G lanes ranks the row's entries in LDS, places them, and the
// first entry of each run of equal columns adds its run; the result goes to
// tcol / tval at the sum of the source rows' offsets, its length to cnt.
// As permuted rows, bound by one pass over the matrix; one thread per row with
// insertion in global memory took 21.2 ms for the B of a setup at FV 2048^2,
// and the k-way merges of A P 20 ms.  Rows longer than CAP are ranked from memory.
template <int G, int CAP, bool FC>
__global__ __launch_bounds__(256) void merge_rows_kernel(CSRView A1, CSRView A2,
                                                         const int32_t* __restrict__ cmap,
                                                         int32_t* __restrict__ tcol,
                                                         double* __restrict__ tval,
                                                         int32_t* __restrict__ cnt) {
  constexpr int T = CAP / G;
  __shared__ int4 sc4[256 / G][CAP / 4];
  __shared__ double sv8[256 / G][CAP];
  const int lane = threadIdx.x & (G - 1), g = threadIdx.x / G;
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + g;
  if (i >= A1.rows) return;
  const int s1 = A1.rowptr[i], len1 = A1.rowptr[i + 1] - s1;
  const int s2 = FC ? A2.rowptr[i] : 0, len = len1 + (FC ? A2.rowptr[i + 1] - s2 : 0);
  const int o = s1 + s2;
  auto entry = [&](int k, int& c, double& v) {
    if (!FC || k >= len1) {
      const int p = FC ? s2 + k - len1 : s1 + k;
      c = cmap[FC ? A2.col[p] : A1.col[p]];
      v = FC ? A2.val[p] : A1.val[p];
    } else {
      c = A1.col[s1 + k];
      v = A1.val[s1 + k];
    }
  };
  if (len > CAP) {
    // the same from the source rows instead of LDS; the runs by one lane
    int e = o;
    for (int k0 = 0; k0 < len; k0 += G) {
      const int k = k0 + lane;
      int c = -1, r = 0;
      double v = 0.0;
      if (k < len) entry(k, c, v);
      if (c >= 0) {
        for (int j = 0; j < len; ++j) {
          int cj;
          double vj;
          entry(j, cj, vj);
          r += cj >= 0 && (cj < c || (cj == c && j < k));
        }
        tcol[o + r] = c;
        tval[o + r] = v;
      }
      e += (int)__popcll(group_ballot<G>(c >= 0));
    }
    __threadfence_block();
    wave_order();
    if (lane == 0) {
      int w = o;
      for (int p = o; p < e;) {
        const int c = tcol[p];
        double v = FC ? tval[p] : 0.0 + tval[p];
        for (++p; p < e && tcol[p] == c; ++p) v = v + tval[p];
        if (FC || v != 0.0) {
          tcol[w] = c;
          tval[w] = v;
          ++w;
        }
      }
      cnt[i] = w - o;
    }
    return;
  }
  int32_t* sc = reinterpret_cast<int32_t*>(sc4[g]);
  double* sv = sv8[g];
  int c[T], r[T];
  double v[T];
  int m = 0;  // entries kept
#pragma unroll
  for (int t = 0; t < T; ++t) {
    c[t] = 0x7fffffff;
    v[t] = 0.0;
    if (G * t < len) {
      const int k = lane + G * t;
      bool in = k < len;
      if (in) {
        entry(k, c[t], v[t]);
        in = c[t] >= 0;
        if (!in) c[t] = 0x7fffffff;
      }
      m += (int)__popcll(group_ballot<G>(in));
    }
    if (G * t < len + 3) sc[lane + G * t] = c[t];
  }
  wave_order();
  rank_entries<G, T>(sc, len, c, lane, r);
  wave_order();
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (lane + G * t < len) {
      sc[r[t]] = c[t];
      sv[r[t]] = v[t];
    }
  wave_order();
  int w = 0;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if (G * t >= m) break;
    const int p = lane + G * t;
    bool keep = p < m && (p == 0 || sc[p - 1] != sc[p]);
    double x = 0.0;
    if (keep) {
      x = FC ? sv[p] : 0.0 + sv[p];
      for (int q = p + 1; q < m && sc[q] == sc[p]; ++q) x = x + sv[q];
      keep = FC || x != 0.0;
    }
    const unsigned long long b = group_ballot<G>(keep);
    if (keep) {
      const int at = o + w + bits_below(b, lane);
      tcol[at] = sc[p];
      tval[at] = x;
    }
    w += (int)__popcll(b);
  }
  if (lane == 0) cnt[i] = w;
}
// rows of cnt entries at the sums of two row pointers (the second may be null)
template <int G>
__global__ __launch_bounds__(256) void compact_rows_kernel(int64_t rows, const int32_t* __restrict__ o1,
                                                           const int32_t* __restrict__ o2,
                                                           const int32_t* __restrict__ rowptr,
                                                           const int32_t* __restrict__ tcol,
                                                           const double* __restrict__ tval,
                                                           int32_t* __restrict__ col,
                                                           double* __restrict__ val) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
  if (i >= rows) return;
  const int64_t t0 = (int64_t)o1[i] + (o2 ? o2[i] : 0);
  const int p0 = rowptr[i], len = rowptr[i + 1] - p0;
  for (int k = lane; k < len; k += G) {
    col[p0 + k] = tcol[t0 + k];
    val[p0 + k] = tval[t0 + k];
  }
}
template <bool FC>
static void launch_merge_rows(const CSR& A1, const CSR& A2, const int32_t* cmap, int32_t* tcol,
                              double* tval, int32_t* cnt, hipStream_t s) {
  const double avg = (double)(A1.nnz + (FC ? A2.nnz : 0)) / (double)A1.rows;
#define AIRG_CALL(G, CAP)                                                                             \
  merge_rows_kernel<G, CAP, FC><<<blocks_for(A1.rows, 256 / G), 256, 0, s>>>(view(A1), view(A2), cmap, \
                                                                            tcol, tval, cnt)
  AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
  AIRG_CHECK_LAUNCH();
}

// ------------------------------------------------------------------ hash product
// The row-by-row product with the row of C in an LDS table of T columns (a
// power of two; open addressing, linear probing): first pass (NUMERIC false)
// counts each row's columns, second pass adds the products, packs the table,
// ranks its columns and writes the row in ascending order.  A group of G lanes
// takes the entries of one row of B at consecutive addresses; those columns
// are distinct, so no two lanes add to one slot at a time, and the next row's
// first entries are loaded while this row's are added.  A group stops at
// T - G columns (*overflow: the host takes a larger table, past the largest
// the row goes to window_product_kernel).
//
// Bound by the latency of the rows of B (one memory round trip each, about as
// many in flight as the tables leave wavefronts).  The form it replaced took
// one column of C per wavefront-wide minimum over all pending rows of B:
// R (A P) of level 6 at FV 2048^2 (70,391 rows, 32 rows of B each, 152 columns)
// took 0.9 + 3.4 ms, the products of a whole setup 85 ms.
template <int G, bool NUMERIC>
__global__ __launch_bounds__(256) void hash_product_kernel(
    CSRView A, const int32_t* __restrict__ bptr, const int32_t* __restrict__ bcol,
    const double* __restrict__ bval, int T, int shift, const int32_t* __restrict__ rowptr,
    int32_t* __restrict__ col, double* __restrict__ val, int32_t* __restrict__ cnt, int32_t* overflow,
    int32_t* longest, int32_t* zeros) {
  extern __shared__ __align__(16) unsigned char hash_lds[];
  const int gpb = blockDim.x / G, g = threadIdx.x / G, lane = threadIdx.x & (G - 1);
  double* hv = reinterpret_cast<double*>(hash_lds) + (size_t)(NUMERIC ? g : 0) * T;
  int32_t* hk = reinterpret_cast<int32_t*>(hash_lds + (NUMERIC ? (size_t)gpb * T * sizeof(double) : 0)) +
                (size_t)g * T;
  const int64_t i = (int64_t)blockIdx.x * gpb + g;
  if (i >= A.rows) return;
  for (int k = lane; k < T; k += G) {
    hk[k] = -1;
    if (NUMERIC) hv[k] = 0.0;
  }
  wave_order();
  const epos s = A.rowptr[i], e = A.rowptr[i + 1];
  int n = 0;  // columns in the table, the same in every lane of the group
  bool full = false;
  for (epos p0 = s; p0 < e && !full; p0 += G) {
    // the next G entries of the row: their rows of B, one per lane
    const int np = (int)min((epos)G, e - p0);
    int b0 = 0, b1 = 0;
    double a = 0.0;
    if (lane < np) {
      const int k = A.col[p0 + lane];
      b0 = bptr[k];
      b1 = bptr[k + 1];
      if (NUMERIC) a = A.val[p0 + lane];
    }
    epos q0 = __shfl(b0, 0, G), q1 = __shfl(b1, 0, G);
    int c = -1;
    double v = 0.0;
    if (q0 + lane < q1) {
      c = bcol[q0 + lane];
      if (NUMERIC) v = bval[q0 + lane];
    }
    for (int t = 0; t < np; ++t) {
      const double at = NUMERIC ? __shfl(a, t, G) : 0.0;
      // the first entries of the next row
      epos r0 = 0, r1 = 0;
      int cn = -1;
      double vn = 0.0;
      if (t + 1 < np) {
        r0 = __shfl(b0, t + 1, G);
        r1 = __shfl(b1, t + 1, G);
        if (r0 + lane < r1) {
          cn = bcol[r0 + lane];
          if (NUMERIC) vn = bval[r0 + lane];
        }
      }
      for (epos q = q0; q < q1; q += G) {
        if (n + G > T) {
          full = true;
          break;
        }
        if (q > q0) {
          c = -1;
          if (q + lane < q1) {
            c = bcol[q + lane];
            if (NUMERIC) v = bval[q + lane];
          }
        }
        bool fresh = false;
        if (c >= 0) {
          unsigned h = ((unsigned)c * 0x9E3779B1u) >> shift;
          for (;;) {
            const int old = atomicCAS(&hk[h], -1, c);
            if (old == -1) fresh = true;
            if (old == -1 || old == c) break;
            h = (h + 1) & (unsigned)(T - 1);
          }
          if (NUMERIC) hv[h] = hv[h] + at * v;
        }
        n += (int)__popcll(group_ballot<G>(fresh));
        wave_order();
      }
      if (full) break;
      q0 = r0;
      q1 = r1;
      c = cn;
      v = vn;
    }
  }
  if constexpr (!NUMERIC) {
    if (lane == 0) {
      cnt[i] = full ? -1 : n;
      if (full) atomicOr(overflow, 1);
      // most rows find a longer one counted already and need no atomic
      if (n > __hip_atomic_load(longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(longest, n);
    }
    return;
  }
  if (full) return;  // left to window_product_kernel
  // pack the table to its front (a slot moves down, past slots already read)
  int m = 0;
  for (int k0 = 0; k0 < T; k0 += G) {
    const int k = k0 + lane;
    const int key = k < T ? hk[k] : -1;
    const double x = key >= 0 ? hv[k] : 0.0;
    wave_order();
    const unsigned long long b = group_ballot<G>(key >= 0);
    if (key >= 0) {
      const int at = m + bits_below(b, lane);
      hk[at] = key;
      hv[at] = x;
    }
    m += (int)__popcll(b);
    wave_order();
  }
  if (lane < 3 && m + lane < T) hk[m + lane] = 0x7fffffff;
  wave_order();
  const int o = rowptr[i];
  bool zero = false;
  for (int k = lane; k < m; k += G) {
    const int key = hk[k];
    int r = 0;
    for (int j = 0; j < m; j += 4) {
      const int4 w = *reinterpret_cast<const int4*>(hk + j);
      r += (w.x < key) + (w.y < key) + (w.z < key) + (w.w < key);
    }
    const double x = hv[k];
    col[o + r] = key;
    val[o + r] = x;
    zero = zero || x == 0.0;
  }
  if (zero) atomicOr(zeros, 1);
}

// Largest table (48 KB with its values): a row of C of up to 4096 - 64 columns.
constexpr int kHashMax = 4096;

template <bool NUMERIC>
static void launch_hash_product(const CSR& A, const CSR& B, int G, int T, const int32_t* rowptr,
                                int32_t* col, double* val, int32_t* cnt, const RowStat& st, hipStream_t s) {
  // as many rows per workgroup as fit 64 KB of tables
  const size_t table = (size_t)T * (NUMERIC ? 12 : 4);
  int threads = 256;
  while (threads > 64 && (size_t)(threads / G) * table > 64 * 1024) threads >>= 1;
  const size_t lds = (size_t)(threads / G) * table;
  int shift = 32;
  for (int t = T; t > 1; t >>= 1) --shift;
  const unsigned nb = blocks_for(A.rows, threads / G);
#define AIRG_CALL(GG)                                                                                 \
  case GG:                                                                                            \
    hash_product_kernel<GG, NUMERIC><<<nb, threads, lds, s>>>(view(A), B.rowptr.get(), B.col.get(),   \
                                                              B.val.get(), T, shift, rowptr, col, val, \
                                                              cnt, st.flag(0), st.flag(1), st.flag(2)); \
    break
  switch (G) {
    AIRG_CALL(4);
    AIRG_CALL(8);
    AIRG_CALL(16);
    AIRG_CALL(32);
    AIRG_CALL(64);
    default: fail(AIRG_ERR_INTERNAL, "bad lanes per row of a product");
  }
#undef AIRG_CALL
  AIRG_CHECK_LAUNCH();
}

static int pow2_at_least(double x) {
  int p = 1;
  while (p < x && p < (1 << 30)) p <<= 1;
  return p;
}

// Rows of C too long for a table, one wavefront each: the columns are taken in
// windows of kWindow, a window's sums in LDS at their column (the entries of a
// sorted row of B inside a window start where a binary search says), and come
// out ascending.  The order of every sum is that of hash_product_kernel.
constexpr int kWindow = 4096;
__global__ void overflow_rows_kernel(const int32_t* cnt, int64_t n, int32_t* list, int32_t* nlist) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n && cnt[i] < 0) list[atomicAdd(nlist, 1)] = (int32_t)i;
}
template <bool NUMERIC>
__global__ __launch_bounds__(64) void window_product_kernel(CSRView A, CSRView B, int64_t cols,
                                                            const int32_t* __restrict__ list,
                                                            const int32_t* __restrict__ rowptr,
                                                            int32_t* __restrict__ col,
                                                            double* __restrict__ val,
                                                            int32_t* __restrict__ cnt, int32_t* zeros) {
  __shared__ double acc[NUMERIC ? kWindow : 1];
  __shared__ uint32_t hit[kWindow / 32];
  const int lane = threadIdx.x;
  const int64_t i = list[blockIdx.x];
  const int s = A.rowptr[i], e = A.rowptr[i + 1];
  int n = NUMERIC ? rowptr[i] : 0;
  bool zero = false;
  for (int64_t w0 = 0; w0 < cols; w0 += kWindow) {
    const int64_t w1 = w0 + kWindow;
    for (int k = lane; k < kWindow / 32; k += 64) hit[k] = 0;
    if (NUMERIC)
      for (int k = lane; k < kWindow; k += 64) acc[k] = 0.0;
    wave_order();
    for (int p = s; p < e; ++p) {
      const int k = A.col[p];
      const epos end = B.rowptr[k + 1], lo = first_from(B.col, B.rowptr[k], end, w0);
      const double a = A.val[p];
      for (epos q = lo + lane; q < end; q += 64) {
        const int c = B.col[q];
        if (c >= w1) break;
        const int t = (int)(c - w0);
        atomicOr(&hit[t >> 5], 1u << (t & 31));
        if (NUMERIC) acc[t] = acc[t] + a * B.val[q];
      }
      wave_order();
    }
    for (int k0 = 0; k0 < kWindow; k0 += 64) {
      const int t = k0 + lane;
      const bool in = (hit[t >> 5] >> (t & 31)) & 1u;
      const unsigned long long b = __ballot(in);
      if (NUMERIC && in) {
        const int at = n + bits_below(b, lane);
        col[at] = (int32_t)(w0 + t);
        val[at] = acc[t];
        zero = zero || acc[t] == 0.0;
      }
      n += (int)__popcll(b);
    }
    wave_order();
  }
  if (!NUMERIC && lane == 0) cnt[i] = n;
  if (NUMERIC && zero) atomicOr(zeros, 1);
}

void spgemm(const CSR& A, const CSR& B, CSR& C, hipStream_t s) {
  if (!spgemm(A, B, C, s, kMaxNnz)) check_nnz(kMaxNnz + 1);
}
bool spgemm(const CSR& A, const CSR& B, CSR& C, hipStream_t s, int64_t max_nnz) {
  C = CSR();
  if (A.cols != B.rows) fail(AIRG_ERR_INTERNAL, "spgemm shape mismatch");
  const int64_t n = A.rows;
  CSR full;
  full.rows = n;
  full.cols = B.cols;
  if (n <= 0 || A.nnz <= 0 || B.nnz <= 0) {  // no entries
    full.rowptr.alloc(std::max<int64_t>(n, 0) + 1, s);
    launch_fill_i32(full.rowptr.get(), std::max<int64_t>(n, 0) + 1, 0, s);
    C = std::move(full);
    return true;
  }
  const double la = (double)A.nnz / (double)n, lb = (double)B.nnz / (double)B.rows;
  // lanes: a row of B per step.  First table: room for six rows of C that see
  // no column twice; long rows see most of theirs many times, so not above 1024
  // until one overflows.
  int G = std::min(64, std::max(4, pow2_at_least(lb)));
  int T = std::min(1024, pow2_at_least(6.0 * la * lb + 2.0 * G));
  DBuf<int32_t> cnt(n, s), list;
  int nlist = 0;
  for (;;) {
    while (G < 64 && T / G > 32) G <<= 1;
    T = std::max(T, 2 * G);
    RowStat st(s);
    launch_hash_product<false>(A, B, G, T, nullptr, nullptr, nullptr, cnt.get(), st, s);
    full.nnz = count_rows(cnt, n, full.rowptr, st, s);  // of use unless a row overflowed
    if (!st.value(0)) {
      T = std::min(kHashMax, std::max(2 * G, pow2_at_least(1.5 * st.value(1) + G)));
      break;
    }
    if (T >= kHashMax) {
      DBuf<int32_t> found(1, s);
      launch_fill_i32(found.get(), 1, 0, s);
      list.alloc(n, s);
      overflow_rows_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(cnt.get(), n, list.get(), found.get());
      AIRG_CHECK_LAUNCH();
      nlist = fetch(found.get(), s);
      window_product_kernel<false><<<nlist, 64, 0, s>>>(view(A), view(B), B.cols, list.get(), nullptr,
                                                        nullptr, nullptr, cnt.get(), nullptr);
      AIRG_CHECK_LAUNCH();
      RowStat all(s);
      full.nnz = count_rows(cnt, n, full.rowptr, all, s);
      break;  // the second pass with the same G and T leaves the same rows
    }
    T = std::min(kHashMax, 4 * T);
  }
  if (!nlist) {
    while (G < 64 && T / G > 32) G <<= 1;
    T = std::max(T, 2 * G);
  }
  if (full.nnz > std::min(max_nnz, kMaxNnz)) return false;
  full.col.alloc(full.nnz, s);
  full.val.alloc(full.nnz, s);
  RowStat st(s);
  launch_hash_product<true>(A, B, G, T, full.rowptr.get(), full.col.get(), full.val.get(), nullptr, st, s);
  if (nlist) {
    window_product_kernel<true><<<nlist, 64, 0, s>>>(view(A), view(B), B.cols, list.get(),
                                                     full.rowptr.get(), full.col.get(), full.val.get(),
                                                     nullptr, st.flag(2));
    AIRG_CHECK_LAUNCH();
  }
  read_back(st.h, st.d.get(), sizeof(st.h), s);
  if (st.value(2)) drop_zeros(full, C, s);
  else C = std::move(full);
  return true;
}

// A P for the one-point P given by pmap (pmap[j]: the coarse column of node j,
// or -1): a relabelled, sorted and summed copy of A (merge_rows_kernel).
void one_point_product(const CSR& A, const int32_t* pmap, int64_t nc, CSR& AP, hipStream_t s) {
  const int64_t n = A.rows;
  DBuf<int32_t> cnt(n, s), tcol(A.nnz, s);
  DBuf<double> tval(A.nnz, s);
  if (n > 0) launch_merge_rows<false>(A, A, pmap, tcol.get(), tval.get(), cnt.get(), s);
  AP.rows = n;
  AP.cols = nc;
  AP.nnz = counts_to_rowptr(cnt, n, AP.rowptr, s);
  AP.col.alloc(AP.nnz, s);
  AP.val.alloc(AP.nnz, s);
  if (n > 0) {
    compact_rows_kernel<16><<<blocks_for(n, 16), 256, 0, s>>>(n, A.rowptr.get(), nullptr, AP.rowptr.get(),
                                                              tcol.get(), tval.get(), AP.col.get(),
                                                              AP.val.get());
    AIRG_CHECK_LAUNCH();
  }
}

// ------------------------------------------------------------------ fixed sparsity
// T_out[p] = sum over q in row i (ascending) of T_in[q] * Aff[col(q), col(p)],
// i.e. (T_in Aff) restricted to the pattern of Aff.
// One thread per output entry p (its row i from the entry's row index): the
// entry sums over the row's entries q in ascending order.
__global__ void masked_power_entry_kernel(CSRView Aff, const int32_t* __restrict__ row_of,
                                          int64_t nnz, const double* tin, double* tout) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  const int i = row_of[p];
  const int s = Aff.rowptr[i], e = Aff.rowptr[i + 1];
  const int j = Aff.col[p];
  double acc = 0.0;
  for (int q = s; q < e; ++q) {
    const int k = Aff.col[q];
    int r = find_col(Aff.col, Aff.rowptr[k], Aff.rowptr[k + 1], j);
    if (r >= 0) acc = acc + tin[q] * Aff.val[r];
  }
  tout[p] = acc;
}
__global__ void row_of_entry_kernel(CSRView A, int32_t* row_of) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p) row_of[p] = (int32_t)i;
}

// v = alpha_0 [i == j]; v = v + alpha_k T_k  (k = 1..d, left to right)
__global__ void poly_init_kernel(CSRView Aff, double a0, double a1, int has_a1, double* v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Aff.rows) return;
  for (int p = Aff.rowptr[i]; p < Aff.rowptr[i + 1]; ++p) {
    double x = (Aff.col[p] == i) ? a0 : 0.0;
    if (has_a1) x = x + a1 * Aff.val[p];
    v[p] = x;
  }
}
__global__ void poly_add_kernel(int64_t nnz, double a, const double* t, double* v) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < nnz) v[p] = v[p] + a * t[p];
}

// All masked powers and their sum, a group of G lanes per row: row i of
// T_k = mask(T_{k-1} Aff) depends on row i of T_{k-1} alone, so the powers stay
// in LDS and only their sum is written.  The row's columns go into a table of
// positions; the rows of Aff that the row's entries name are taken one after
// the other (ascending, so every sum keeps its order), their entries across
// the lanes, the next row's loaded while this one's are looked up.  Bound by
// the latency of those rows, d - 1 times each.  A thread per entry with a
// binary search in every row took 11.8 ms a setup at FV 2048^2 and wrote every
// power to memory.  *too_long is set where a row exceeds CAP entries (the
// caller then takes that form), *zeros where a sum is exactly 0.
struct PolyCoeffs {
  double a[65];
  int n;
};
template <int G, int CAP>
__global__ __launch_bounds__(256) void masked_poly_kernel(CSRView A, PolyCoeffs c, double* __restrict__ out,
                                                          int32_t* too_long, int32_t* zeros) {
  constexpr int T = CAP / G, kTable = 2 * CAP;
  constexpr int kShift = 32 - __builtin_ctz(kTable);
  __shared__ double s_t[256 / G][2][CAP];
  __shared__ int32_t s_key[256 / G][kTable];
  __shared__ int16_t s_pos[256 / G][kTable];
  const int lane = threadIdx.x & (G - 1), g = threadIdx.x / G;
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + g;
  if (i >= A.rows) return;
  const int s = A.rowptr[i], len = A.rowptr[i + 1] - s;
  if (len > CAP) {
    if (lane == 0) atomicOr(too_long, 1);
    return;
  }
  int32_t* key = s_key[g];
  int16_t* pos = s_pos[g];
  for (int k = lane; k < kTable; k += G) key[k] = -1;
  wave_order();
  double v[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    v[t] = 0.0;
    const int k = lane + G * t;
    if (k < len) {
      const int j = A.col[s + k];
      const double x = A.val[s + k];
      s_t[g][0][k] = x;
      double y = j == i ? c.a[0] : 0.0;
      if (c.n > 1) y = y + c.a[1] * x;
      v[t] = y;
      unsigned h = ((unsigned)j * 0x9E3779B1u) >> kShift;
      while (atomicCAS(&key[h], -1, j) != -1) h = (h + 1) & (kTable - 1);
      pos[h] = (int16_t)k;
    }
  }
  wave_order();
  int cur = 0;
  for (int k = 2; k < c.n; ++k, cur ^= 1) {
    const double* tin = s_t[g][cur];
    double* tout = s_t[g][cur ^ 1];
    for (int q = lane; q < len; q += G) tout[q] = 0.0;
    wave_order();
    for (int p0 = 0; p0 < len; p0 += G) {
      const int np = min(G, len - p0);
      int b0 = 0, b1 = 0;
      if (lane < np) {
        const int j = A.col[s + p0 + lane];
        b0 = A.rowptr[j];
        b1 = A.rowptr[j + 1];
      }
      epos q0 = __shfl(b0, 0, G), q1 = __shfl(b1, 0, G);
      int cc = -1;
      double x = 0.0;
      if (q0 + lane < q1) {
        cc = A.col[q0 + lane];
        x = A.val[q0 + lane];
      }
      for (int t = 0; t < np; ++t) {
        epos r0 = 0, r1 = 0;
        int cn = -1;
        double xn = 0.0;
        if (t + 1 < np) {
          r0 = __shfl(b0, t + 1, G);
          r1 = __shfl(b1, t + 1, G);
          if (r0 + lane < r1) {
            cn = A.col[r0 + lane];
            xn = A.val[r0 + lane];
          }
        }
        const double w = tin[p0 + t];
        for (epos q = q0; q < q1; q += G) {
          if (q > q0) {
            cc = -1;
            if (q + lane < q1) {
              cc = A.col[q + lane];
              x = A.val[q + lane];
            }
          }
          if (cc >= 0) {
            unsigned h = ((unsigned)cc * 0x9E3779B1u) >> kShift;
            int found = key[h];
            while (found != cc && found != -1) {
              h = (h + 1) & (kTable - 1);
              found = key[h];
            }
            if (found == cc) {
              const int at = pos[h];
              tout[at] = tout[at] + w * x;
            }
          }
          wave_order();
        }
        q0 = r0;
        q1 = r1;
        cc = cn;
        x = xn;
      }
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
      if (lane + G * t < len) v[t] = v[t] + c.a[k] * tout[lane + G * t];
    wave_order();
  }
  bool zero = false;
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (lane + G * t < len) {
      out[s + lane + G * t] = v[t];
      zero = zero || v[t] == 0.0;
    }
  if (zero) atomicOr(zeros, 1);
}

static bool masked_poly(const CSR& Aff, const std::vector<double>& alpha, CSR& full, CSR& out,
                        hipStream_t s) {
  PolyCoeffs c;
  if (alpha.size() > sizeof(c.a) / sizeof(c.a[0])) return false;
  c.n = (int)alpha.size();
  std::copy(alpha.begin(), alpha.end(), c.a);
  const double avg = (double)Aff.nnz / (double)Aff.rows;
  // 28 KB of LDS per workgroup where rows may be 2.5 times the average or more
  // (five workgroups a CU), 56 KB for the longest; a longer row takes the next
  int form = avg <= 2.5 ? 0 : avg <= 6.0 ? 1 : avg <= 20.0 ? 2 : avg <= 50.0 ? 3 : avg <= 100.0 ? 4 : 5;
  for (; form < 6; ++form) {
    RowStat st(s);
#define AIRG_CALL(G, CAP)                                                   \
  masked_poly_kernel<G, CAP><<<blocks_for(Aff.rows, 256 / G), 256, 0, s>>>( \
      view(Aff), c, full.val.get(), st.flag(0), st.flag(2));                \
  break
    switch (form) {
      case 0: AIRG_CALL(4, 16);
      case 1: AIRG_CALL(8, 32);
      case 2: AIRG_CALL(16, 64);
      case 3: AIRG_CALL(32, 128);
      case 4: AIRG_CALL(32, 256);
      default: AIRG_CALL(64, 512);
    }
#undef AIRG_CALL
    AIRG_CHECK_LAUNCH();
    read_back(st.h, st.d.get(), sizeof(st.h), s);
    if (st.value(0)) continue;
    if (st.value(2)) drop_zeros(full, out, s);
    else out = std::move(full);
    return true;
  }
  return false;
}

void fixed_sparsity_inverse(const CSR& Aff, const std::vector<double>& alpha, CSR& out,
                            hipStream_t s) {
  const int64_t n = Aff.rows;
  if (alpha.empty()) fail(AIRG_ERR_INTERNAL, "empty polynomial");
  CSR full;
  full.rows = n;
  full.cols = Aff.cols;
  full.nnz = Aff.nnz;
  full.rowptr.alloc(n + 1, s);
  full.col.alloc(Aff.nnz, s);
  full.val.alloc(Aff.nnz, s);
  AIRG_HIP(hipMemcpyAsync(full.rowptr.get(), Aff.rowptr.get(), (n + 1) * sizeof(int32_t),
                          hipMemcpyDeviceToDevice, s));
  AIRG_HIP(hipMemcpyAsync(full.col.get(), Aff.col.get(), Aff.nnz * sizeof(int32_t),
                          hipMemcpyDeviceToDevice, s));
  unsigned nb = blocks_for(n, kBlock);
  if (n > 0 && masked_poly(Aff, alpha, full, out, s)) return;
  // rows too long for the LDS form: one launch per power
  if (n > 0) {
    poly_init_kernel<<<nb, kBlock, 0, s>>>(view(Aff), alpha[0], alpha.size() > 1 ? alpha[1] : 0.0,
                                           alpha.size() > 1 ? 1 : 0, full.val.get());
    AIRG_CHECK_LAUNCH();
  }
  if (alpha.size() > 2) {
    DBuf<double> ta(Aff.nnz, s), tb(Aff.nnz, s);
    DBuf<int32_t> row_of(Aff.nnz, s);
    row_of_entry_kernel<<<nb, kBlock, 0, s>>>(view(Aff), row_of.get());
    AIRG_CHECK_LAUNCH();
    AIRG_HIP(hipMemcpyAsync(ta.get(), Aff.val.get(), Aff.nnz * sizeof(double),
                            hipMemcpyDeviceToDevice, s));
    for (size_t k = 2; k < alpha.size(); ++k) {
      masked_power_entry_kernel<<<blocks_for(Aff.nnz, kBlock), kBlock, 0, s>>>(
          view(Aff), row_of.get(), Aff.nnz, ta.get(), tb.get());
      AIRG_CHECK_LAUNCH();
      poly_add_kernel<<<blocks_for(Aff.nnz, kBlock), kBlock, 0, s>>>(Aff.nnz, alpha[k], tb.get(),
                                                                     full.val.get());
      AIRG_CHECK_LAUNCH();
      std::swap(ta, tb);
    }
  }
  drop_zeros(full, out, s);
}

// ------------------------------------------------------------------ exact polynomial
// a_ii += a; *missing is set where a row stores no diagonal
__global__ void add_diag_kernel(int64_t rows, const int32_t* rowptr, const int32_t* col, double a,
                                double* val, int32_t* missing) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows) return;
  const int r = find_col(col, rowptr[i], rowptr[i + 1], (int)i);
  if (r >= 0) val[r] = val[r] + a;
  else atomicOr(missing, 1);
}

// The matrix-free smoother reads A and three vectors d times; one product with
// Q = q(A) reads Q and the vectors once.  With few couplings between F points
// (1.4 a row on the finest upwind level, 2.0 on the next) Q hardly fills in
// (1.7 and 4.1 entries a row at d = 4), so the smoother is nearly d times
// cheaper; from about 8 entries a row on, Q holds ten times A's entries and
// loses.  Both sides are priced as launches * 2.6 us (what a small product
// takes) plus bytes at the rate that products reach inside a solve, where the
// rest of the cycle has been through the caches: 3.8 TB/s for A's short rows, 3.3
// for Q, whose rows gather further (an entry with an FP32 value counts 8 bytes for
// that, not 6), and 4.5 from 64 entries a row on; and Q has to win by a tenth.
// (Back to back on warm caches all reach 4.6 to 5, and by that level 2 of FV 2048^2,
// 22 entries a row, would win.)  One V-cycle's smoother with Q against the steps, from
// solves of both, FP64: FV 2048^2 level 0 -59 us, level 1 -40, level 2 -5 of some 45;
// in FP32 -36, -18 and 0; FV 4096^2 -199, -73 and, level 2, +33; the batch of 48 -312, -147 and +30; FD
// 3606^2 level 1 (d = 6) -131; DG 1024^2 level 0 -18.  Small levels are all
// launches: Q may be ten times denser there and still wins (FV 512^2, all levels:
// -48 us of 278 a cycle).  Priced at 3.3 the long rows of small systems kept their
// steps: FV 512^2 levels 4 and 5 (198 and 303 entries a row) 2.08 ms a solve, 1.96
// formed; DG 193 x 180 level 3 (232) 2.33 and 2.23; 6 problems of 256^2 level 4
// (176) 2.63 and 2.58, FP32 2.50 and 2.44.
bool exact_polynomial(const CSR& A, const std::vector<double>& alpha, double vbytes, double xbytes,
                      CSR& Q, hipStream_t s) {
  Q = CSR();
  const int d = (int)alpha.size() - 1;
  const int64_t n = A.rows;
  if (d < 2 || n <= 0 || A.nnz < n) return false;
  constexpr double kLaunchUs = 2.6, kStepBytesPerUs = 3.8e6, kBytesPerUs = 3.3e6, kLongBytesPerUs = 4.5e6,
                   kWin = 0.9;
  const double free_us =
      d * (kLaunchUs + ((vbytes + 2.0) * (double)A.nnz + (4.0 + 3.0 * xbytes) * (double)n) / kStepBytesPerUs);
  auto fits = [&](double bytes_per_us) {  // the entries that Q may have at that rate
    return std::min(2147483647.0, ((kWin * free_us - kLaunchUs) * bytes_per_us - (4.0 + 3.0 * xbytes) * (double)n) /
                                      (6.0 + 0.5 * xbytes));
  };
  const double long_rows = 64.0 * (double)n, max_short = fits(kBytesPerUs), max_long = fits(kLongBytesPerUs);
  const double max_nnz = max_long >= long_rows ? max_long : max_short;
  // the growth of a power's entries over the last one's: 2.8 and more from
  // 8 entries a row on, where a product would only find that out
  auto hopeless = [&](double nnz, double growth, int left) {
    double f = 0.5 * nnz;
    for (int k = 0; k < left; ++k) f *= growth;
    return std::min(f, (double)n * (double)n) > max_nnz;
  };
  if ((double)A.nnz > max_nnz || (A.nnz >= 8 * n && hopeless((double)A.nnz, 2.8, d - 1))) return false;
  DBuf<int32_t> missing(1, s);
  launch_fill_i32(missing.get(), 1, 0, s);
  const unsigned nb = blocks_for(n, kBlock);
  auto add_diag = [&](CSR& M, double a) {
    add_diag_kernel<<<nb, kBlock, 0, s>>>(n, M.rowptr.get(), M.col.get(), a, M.val.get(), missing.get());
    AIRG_CHECK_LAUNCH();
  };
  CSR P;  // alpha_d A + alpha_{d-1} I
  copy_csr(A, P, s);
  launch_scale(P.val.get(), A.val.get(), alpha[d], A.nnz, s);
  add_diag(P, alpha[d - 1]);
  for (int k = d - 2; k >= 0; --k) {
    CSR T;
    if (!spgemm(A, P, T, s, (int64_t)max_nnz) || (k > 0 && hopeless((double)T.nnz, (double)T.nnz / (double)P.nnz, k)))
      return false;
    add_diag(T, alpha[k]);
    P = std::move(T);
  }
  if ((double)P.nnz > max_short && (double)P.nnz < long_rows) return false;
  if (fetch(missing.get(), s)) return false;
  Q = std::move(P);
  return true;
}

// ------------------------------------------------------------------ Neumann (nAIR)
__global__ void row_diag_kernel(CSRView A, double* d) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  double v = 0.0;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p)
    if (A.col[p] == i) v = A.val[p];
  d[i] = v;
}
// N = I - D^{-1} A on A's pattern: -a_ij / a_ii off the diagonal, 0 on it
__global__ void jacobi_iteration_matrix_kernel(CSRView A, const double* d, double* nval) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p)
    nval[p] = A.col[p] == i ? 0.0 : -A.val[p] / d[i];
}
__global__ void col_scale_kernel(int64_t nnz, const int32_t* col, const double* dinv, double* val) {
  int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p < nnz) val[p] = val[p] * dinv[col[p]];
}
__global__ void reciprocal_kernel(int64_t n, const double* d, double* r) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r[i] = 1.0 / d[i];
}

void diag_inverse(const CSR& A, DBuf<double>& dinv, hipStream_t s) {
  const int64_t n = A.rows;
  DBuf<double> d(n, s);
  dinv.alloc(n, s);
  if (n <= 0) return;
  row_diag_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(view(A), d.get());
  AIRG_CHECK_LAUNCH();
  reciprocal_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(n, d.get(), dinv.get());
  AIRG_CHECK_LAUNCH();
}

void neumann_fixed_sparsity(const CSR& Aff, int degree, CSR& out, hipStream_t s) {
  const int64_t n = Aff.rows;
  DBuf<double> d(n, s), dinv;
  CSR N;
  copy_csr(Aff, N, s);
  if (n > 0) {
    row_diag_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(view(Aff), d.get());
    AIRG_CHECK_LAUNCH();
    jacobi_iteration_matrix_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(view(Aff), d.get(),
                                                                           N.val.get());
    AIRG_CHECK_LAUNCH();
  }
  // I + N + N~^2 + ... + N~^d through the fixed-sparsity sum with unit coefficients
  std::vector<double> ones((size_t)std::max(degree, 0) + 1, 1.0);
  CSR S;
  fixed_sparsity_inverse(N, ones, S, s);
  diag_inverse(Aff, dinv, s);
  if (S.nnz > 0) {
    col_scale_kernel<<<blocks_for(S.nnz, kBlock), kBlock, 0, s>>>(S.nnz, S.col.get(), dinv.get(),
                                                                 S.val.get());
    AIRG_CHECK_LAUNCH();
  }
  drop_zeros(S, out, s);
}



// ------------------------------------------------------------------ drops
// A group of G lanes per row, the row at consecutive addresses; FILL writes the
// kept entries, else they are counted.  One thread per row took 2.9 ms for the
// restrictor drops and 14.2 ms for the coarse matrix drops of a setup at FV
// 2048^2 (count and fill).
template <int G>
__device__ __forceinline__ double group_max(double m) {
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, G));
  return m;
}
template <int G, bool FILL>
__global__ __launch_bounds__(256) void rdrop_kernel(CSRView Z, double tol, double sign,
                                                    int32_t* __restrict__ count,
                                                    const int32_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ col, double* __restrict__ val) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
  if (i >= Z.rows) return;
  const epos s = Z.rowptr[i], e = Z.rowptr[i + 1];
  double m = 0.0;
  for (epos p = s + lane; p < e; p += G) m = fmax(m, fabs(Z.val[p]));
  const double thr = tol * group_max<G>(m);
  int n = 0;
  const int o = FILL ? rowptr[i] : 0;
  for (epos p0 = s; p0 < e; p0 += G) {
    const epos p = p0 + lane;
    const double v = p < e ? Z.val[p] : 0.0;
    const bool keep = p < e && fabs(v) >= thr;
    const unsigned long long b = group_ballot<G>(keep);
    if (FILL && keep) {
      const int at = o + n + bits_below(b, lane);
      col[at] = Z.col[p];
      val[at] = sign * v;
    }
    n += (int)__popcll(b);
  }
  if (!FILL && lane == 0) count[i] = n;
}

void restrictor_drop(const CSR& Zin, double tol, bool negate, CSR& Z, hipStream_t s) {
  const int64_t n = Zin.rows;
  const double avg = n > 0 ? (double)Zin.nnz / (double)n : 0.0, sign = negate ? -1.0 : 1.0;
  DBuf<int32_t> cnt(n, s);
  if (n > 0) {
#define AIRG_CALL(G, CAP)                                                                          \
  rdrop_kernel<G, false><<<blocks_for(n, 256 / G), 256, 0, s>>>(view(Zin), tol, sign, cnt.get(),   \
                                                                nullptr, nullptr, nullptr)
    AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
    AIRG_CHECK_LAUNCH();
  }
  Z.rows = n;
  Z.cols = Zin.cols;
  Z.nnz = counts_to_rowptr(cnt, n, Z.rowptr, s);
  Z.col.alloc(Z.nnz, s);
  Z.val.alloc(Z.nnz, s);
  if (n > 0) {
#define AIRG_CALL(G, CAP)                                                                         \
  rdrop_kernel<G, true><<<blocks_for(n, 256 / G), 256, 0, s>>>(view(Zin), tol, sign, nullptr,     \
                                                               Z.rowptr.get(), Z.col.get(), Z.val.get())
    AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
    AIRG_CHECK_LAUNCH();
  }
}

// Off-diagonal relative drop; dropped values lumped to the diagonal as
// d + l_1 + l_2 + ... in ascending column order.
template <int G, bool FILL>
__global__ __launch_bounds__(256) void adrop_kernel(CSRView A, double tol, int lump,
                                                    int32_t* __restrict__ count,
                                                    const int32_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ col, double* __restrict__ val,
                                                    int32_t* bad) {
  const int lane = threadIdx.x & (G - 1);
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
  if (i >= A.rows) return;
  const epos s = A.rowptr[i], e = A.rowptr[i + 1];
  double m = 0.0;
  for (epos p = s + lane; p < e; p += G)
    if (A.col[p] != i) m = fmax(m, fabs(A.val[p]));
  const double thr = tol * group_max<G>(m);
  // the diagonal first: the dropped values are added to it in column order
  double d = 0.0;
  int dlane = -1;
  for (epos p0 = s; p0 < e; p0 += G) {
    const epos p = p0 + lane;
    const bool diag = p < e && A.col[p] == i;
    const unsigned long long b = group_ballot<G>(diag);
    if (b) {
      dlane = (int)__ffsll(b) - 1;
      d = __shfl(diag ? A.val[p] : 0.0, dlane, G);
      break;
    }
  }
  int n = 0;
  const int o = FILL ? rowptr[i] : 0;
  int dat = -1;
  for (epos p0 = s; p0 < e; p0 += G) {
    const epos p = p0 + lane;
    const int j = p < e ? A.col[p] : -1;
    const double v = p < e ? A.val[p] : 0.0;
    const bool drop = p < e && j != i && fabs(v) < thr;
    const bool keep = p < e && !drop;
    const unsigned long long b = group_ballot<G>(keep);
    if (FILL) {
      if (lump) {
        unsigned long long db = group_ballot<G>(drop);
        while (db) {
          const int l = (int)__ffsll(db) - 1;
          db &= db - 1;
          d = d + __shfl(v, l, G);
        }
      }
      const int at = o + n + bits_below(b, lane);
      if (keep) {
        col[at] = j;
        if (j == i) dat = at;
        else val[at] = v;
      }
    }
    n += (int)__popcll(b);
  }
  if constexpr (FILL) {
    if (dat >= 0) val[dat] = d;
    if (lane == 0 && (d == 0.0 || !isfinite(d))) atomicOr(bad, 1);
  } else if (lane == 0) {
    if (dlane < 0) atomicOr(bad, 1);
    count[i] = n;
  }
}

void drop_lump(const CSR& Ain, double tol, bool lump, CSR& Aout, int32_t* bad_diag,
               hipStream_t s) {
  const int64_t n = Ain.rows;
  const double avg = n > 0 ? (double)Ain.nnz / (double)n : 0.0;
  DBuf<int32_t> cnt(n, s);
  if (n > 0) {
#define AIRG_CALL(G, CAP)                                                                       \
  adrop_kernel<G, false><<<blocks_for(n, 256 / G), 256, 0, s>>>(view(Ain), tol, lump ? 1 : 0,   \
                                                                cnt.get(), nullptr, nullptr, nullptr, bad_diag)
    AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
    AIRG_CHECK_LAUNCH();
  }
  Aout.rows = n;
  Aout.cols = Ain.cols;
  Aout.nnz = counts_to_rowptr(cnt, n, Aout.rowptr, s);
  Aout.col.alloc(Aout.nnz, s);
  Aout.val.alloc(Aout.nnz, s);
  if (n > 0) {
#define AIRG_CALL(G, CAP)                                                                      \
  adrop_kernel<G, true><<<blocks_for(n, 256 / G), 256, 0, s>>>(view(Ain), tol, lump ? 1 : 0, nullptr, \
                                                               Aout.rowptr.get(), Aout.col.get(),     \
                                                               Aout.val.get(), bad_diag)
    AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
    AIRG_CHECK_LAUNCH();
  }
}

// ------------------------------------------------------------------ R and P's map
// R row c: Z row c with F columns mapped to level indices (fpos, ascending),
// plus 1.0 at level index cpos[c], merged in column order.
__global__ void build_r_kernel(CSRView Z, const int64_t* fpos, const int64_t* cpos,
                               const int32_t* rowptr, int32_t* col, double* val) {
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= Z.rows) return;
  const int32_t me = (int32_t)cpos[c];
  int64_t o = rowptr[c];
  bool placed = false;
  for (int p = Z.rowptr[c]; p < Z.rowptr[c + 1]; ++p) {
    int32_t j = (int32_t)fpos[Z.col[p]];
    if (!placed && me < j) {
      col[o] = me;
      val[o] = 1.0;
      ++o;
      placed = true;
    }
    col[o] = j;
    val[o] = Z.val[p];
    ++o;
  }
  if (!placed) {
    col[o] = me;
    val[o] = 1.0;
  }
}
__global__ void rowlen_plus_one_kernel(CSRView Z, int32_t* cnt) {
  int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < Z.rows) cnt[c] = Z.rowptr[c + 1] - Z.rowptr[c] + 1;
}

void build_r(const CSR& Z, const int64_t* fpos, const int64_t* cpos, int64_t n, CSR& R,
             hipStream_t s) {
  const int64_t nc = Z.rows;
  DBuf<int32_t> cnt(nc, s);
  unsigned nb = blocks_for(nc, kBlock);
  if (nc > 0) {
    rowlen_plus_one_kernel<<<nb, kBlock, 0, s>>>(view(Z), cnt.get());
    AIRG_CHECK_LAUNCH();
  }
    R.rows = nc;
  R.cols = n;
  R.nnz = counts_to_rowptr(cnt, nc, R.rowptr, s);
  R.col.alloc(R.nnz, s);
  R.val.alloc(R.nnz, s);
  if (nc > 0) {
    build_r_kernel<<<nb, kBlock, 0, s>>>(view(Z), fpos, cpos, R.rowptr.get(), R.col.get(),
                                         R.val.get());
    AIRG_CHECK_LAUNCH();
  }
}

__global__ void one_point_map_kernel(const int8_t* state, const int64_t* fidx, const int64_t* cidx,
                                     const int32_t* cmap, int64_t n, int32_t* pmap) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) pmap[i] = state[i] == 2 ? (int32_t)cidx[i] : cmap[fidx[i]];
}
void one_point_map(const int8_t* state, const int64_t* fidx, const int64_t* cidx, const int32_t* cmap,
                   int64_t n, int32_t* pmap, hipStream_t s) {
  if (n <= 0) return;
  one_point_map_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(state, fidx, cidx, cmap, n, pmap);
  AIRG_CHECK_LAUNCH();
}

// ------------------------------------------------------------------ permutation / transpose
__global__ void perm_count_kernel(CSRView A, const int32_t* newrow, int32_t* cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < A.rows) cnt[newrow ? newrow[i] : i] = A.rowptr[i + 1] - A.rowptr[i];
}

// Row i of A to row newrow[i] (i itself when null) of out with its columns
// mapped by colmap (kept when null) and, with SORT, sorted: a group of G lanes
// loads the row at consecutive addresses, ranks its entries against the row's
// columns in LDS and writes each to its place.  Bound by one read and one
// write of the matrix for short rows, by len^2 / G LDS compares for long ones.
// One thread per row copying, and another sorting by insertion in global
// memory, were a chain of dependent cache accesses per row: the permutations
// and sorts of a setup at FV 2048^2 took 6.8 + 37.9 ms that way.  Rows longer
// than CAP are ranked from memory.  out may be A itself (same row pointers,
// no column map): a row is read before it is written, and one past CAP is
// sorted by one thread.
template <int G, int CAP, bool SORT>
__global__ __launch_bounds__(256) void perm_fill_kernel(CSRView A, const int32_t* newrow,
                                                        const int32_t* colmap, const int32_t* rowptr,
                                                        int32_t* col, double* val) {
  constexpr int T = SORT ? CAP / G : 1;
  __shared__ int4 sc4[256 / G][SORT ? CAP / 4 : 1];
  const int lane = threadIdx.x & (G - 1), g = threadIdx.x / G;
  const int64_t i = (int64_t)blockIdx.x * (256 / G) + g;
  if (i >= A.rows) return;
  const int s = A.rowptr[i], len = A.rowptr[i + 1] - s;
  const int o = rowptr[newrow ? newrow[i] : i];
  if constexpr (!SORT) {
    for (int k = lane; k < len; k += G) {
      const int j = A.col[s + k];
      col[o + k] = colmap ? colmap[j] : j;
      val[o + k] = A.val[s + k];
    }
    return;
  }
  if (len > CAP) {
    if (A.col == col) {  // in place
      if (lane == 0) insertion_sort(o, o + len, col, val);
      return;
    }
    for (int k = lane; k < len; k += G) {
      const int c = colmap ? colmap[A.col[s + k]] : A.col[s + k];
      int r = 0;
      for (int j = 0; j < len; ++j) {
        const int cj = colmap ? colmap[A.col[s + j]] : A.col[s + j];
        r += cj < c || (cj == c && j < k);
      }
      col[o + r] = c;
      val[o + r] = A.val[s + k];
    }
    return;
  }
  int32_t* sc = reinterpret_cast<int32_t*>(sc4[g]);
  int c[T], r[T];
  double v[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int k = lane + G * t;
    c[t] = 0x7fffffff;
    v[t] = 0.0;
    if (k < len) {
      const int j = A.col[s + k];
      c[t] = colmap ? colmap[j] : j;
      v[t] = A.val[s + k];
    }
    if (G * t < len + 3) sc[k] = c[t];
  }
  wave_order();
  rank_entries<G, T>(sc, len, c, lane, r);
#pragma unroll
  for (int t = 0; t < T; ++t)
    if (lane + G * t < len) {
      col[o + r[t]] = c[t];
      val[o + r[t]] = v[t];
    }
}
template <bool SORT>
static void launch_perm_fill(const CSR& A, const int32_t* newrow, const int32_t* colmap,
                             const int32_t* rowptr, int32_t* col, double* val, hipStream_t s) {
  if (A.rows <= 0 || A.nnz <= 0) return;
  const double avg = (double)A.nnz / (double)A.rows;
#define AIRG_CALL(G, CAP)                                                                        \
  perm_fill_kernel<G, CAP, SORT><<<blocks_for(A.rows, 256 / G), 256, 0, s>>>(view(A), newrow,    \
                                                                             colmap, rowptr, col, val)
  AIRG_ROW_GROUPS(avg, AIRG_CALL);
#undef AIRG_CALL
  AIRG_CHECK_LAUNCH();
}

void permute_rows(const CSR& A, const int32_t* newrow, const int32_t* colmap, int64_t out_cols,
                  CSR& out, hipStream_t s, bool sorted) {
  const int64_t n = A.rows;
  DBuf<int32_t> cnt(n, s);
  DBuf<int64_t> work(rowptr_work_size(n), s), total(1, s);
  if (n > 0) {
    perm_count_kernel<<<blocks_for(n, kBlock), kBlock, 0, s>>>(view(A), newrow, cnt.get());
    AIRG_CHECK_LAUNCH();
  }
  out.alloc(n, out_cols, A.nnz, s);
  launch_rowptr_scan(cnt.get(), n, out.rowptr.get(), total.get(), work.get(), s);
  if (sorted) launch_perm_fill<true>(A, newrow, colmap, out.rowptr.get(), out.col.get(), out.val.get(), s);
  else launch_perm_fill<false>(A, newrow, colmap, out.rowptr.get(), out.col.get(), out.val.get(), s);
}

__global__ void tcount_kernel(CSRView A, int32_t* cnt) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p) atomicAdd(&cnt[A.col[p]], 1);
}
__global__ void tfill_kernel(CSRView A, const int32_t* rowptr, int32_t* cursor, int32_t* col,
                             double* val) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.rows) return;
  for (int p = A.rowptr[i]; p < A.rowptr[i + 1]; ++p) {
    int j = A.col[p];
    const int k = rowptr[j] + atomicAdd(&cursor[j], 1);
    col[k] = (int32_t)i;
    val[k] = A.val[p];
  }
}

__global__ void inverse_perm_kernel(const int32_t* perm, int64_t n, int32_t* inv) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) inv[perm[i]] = (int32_t)i;
}

void spatial_row_order(CSR& A, const int32_t* rkey, hipStream_t s) {
  if (A.rows <= 0) return;
  if (A.rmap.get()) fail(AIRG_ERR_INTERNAL, "operator rows are already reordered");
  DBuf<int32_t> rank(A.rows, s);
  rank_points(rkey, A.rows, rank.get(), s);
  CSR P;
  permute_rows(A, rank.get(), nullptr, A.cols, P, s);
  P.rmap.alloc(A.rows, s);
  inverse_perm_kernel<<<blocks_for(A.rows, kBlock), kBlock, 0, s>>>(rank.get(), A.rows, P.rmap.get());
  AIRG_CHECK_LAUNCH();
  A = std::move(P);
}

void sort_rows(CSR& A, hipStream_t s) {
  launch_perm_fill<true>(A, nullptr, nullptr, A.rowptr.get(), A.col.get(), A.val.get(), s);
}

void transpose(const CSR& A, CSR& At, hipStream_t s) {
  const int64_t m = A.cols;
  DBuf<int32_t> cnt(m, s);
  launch_zero_bytes(cnt.get(), m * sizeof(int32_t), s);
  unsigned nb = blocks_for(A.rows, kBlock);
  if (A.rows > 0) {
    tcount_kernel<<<nb, kBlock, 0, s>>>(view(A), cnt.get());
    AIRG_CHECK_LAUNCH();
  }
  DBuf<int64_t> work(rowptr_work_size(m), s), total(1, s);
  At.alloc(m, A.rows, A.nnz, s);
  launch_rowptr_scan(cnt.get(), m, At.rowptr.get(), total.get(), work.get(), s);
  launch_zero_bytes(cnt.get(), m * sizeof(int32_t), s);
  if (A.rows > 0) {
    tfill_kernel<<<nb, kBlock, 0, s>>>(view(A), At.rowptr.get(), cnt.get(), At.col.get(), At.val.get());
    AIRG_CHECK_LAUNCH();
  }
  sort_rows(At, s);
}

void copy_csr(const CSR& A, CSR& out, hipStream_t s) {
  out.alloc(A.rows, A.cols, A.nnz, s);
  AIRG_HIP(hipMemcpyAsync(out.rowptr.get(), A.rowptr.get(), (A.rows + 1) * sizeof(int32_t),
                          hipMemcpyDeviceToDevice, s));
  if (A.nnz) {
    AIRG_HIP(hipMemcpyAsync(out.col.get(), A.col.get(), A.nnz * sizeof(int32_t),
                            hipMemcpyDeviceToDevice, s));
    AIRG_HIP(hipMemcpyAsync(out.val.get(), A.val.get(), A.nnz * sizeof(double),
                            hipMemcpyDeviceToDevice, s));
  }
}

}  // namespace airg

namespace airg {

// ------------------------------------------------------------------ merged F-point residual operator
// B = A_fc + A_ff W with W the one-point prolongation (merge_rows_kernel).
void merge_fc_ffw(const CSR& Afc, const CSR& Aff, const int32_t* cmap, CSR& B, hipStream_t s) {
  const int64_t n = Afc.rows, tot = Afc.nnz + Aff.nnz;
  if (tot > 2147483647ll) fail(AIRG_ERR_NOMEM, "sparse matrix exceeds 2^31 nonzeros");
  B.rows = n;
  B.cols = Afc.cols;
  DBuf<int32_t> cnt(n, s), tcol(tot, s);
  DBuf<double> tval(tot, s);
  if (n > 0) launch_merge_rows<true>(Afc, Aff, cmap, tcol.get(), tval.get(), cnt.get(), s);
  B.nnz = counts_to_rowptr(cnt, n, B.rowptr, s);
  B.col.alloc(B.nnz, s);
  B.val.alloc(B.nnz, s);
  if (n > 0) {
    compact_rows_kernel<16><<<blocks_for(n, 16), 256, 0, s>>>(n, Afc.rowptr.get(), Aff.rowptr.get(),
                                                              B.rowptr.get(), tcol.get(), tval.get(),
                                                              B.col.get(), B.val.get());
    AIRG_CHECK_LAUNCH();
  }
}

// ------------------------------------------------------------------ compressed columns
// Every block of 2^kColBlockShift consecutive rows whose columns span less
// than 65536 stores them as 16-bit offsets from the block's smallest column
// (true for almost every block of a locality-ordered operator, whose rows see
// nearby columns); a block that spans more keeps its int32 columns, marked by
// a negative base.  Saves 2 of the 12 bytes of an FP64 entry.
// One wavefront per block: its entries are one run of addresses.  One thread
// per block walked them one by one, 22.9 ms a setup at FV 2048^2.
__global__ __launch_bounds__(256) void col_span_kernel(CSRView A, int64_t nblk, int32_t* cbase,
                                                       int32_t* cspan, int32_t* stat) {
  const int lane = threadIdx.x & 63;
  const int64_t blk = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (blk >= nblk) return;
  const int64_t r0 = blk << kColBlockShift;
  const int64_t r1 = min(r0 + ((int64_t)1 << kColBlockShift), A.rows);
  int mn = 0x7fffffff, mx = -1;
  for (epos p = (epos)A.rowptr[r0] + lane, e = A.rowptr[r1]; p < e; p += 64) {
    const int c = A.col[p];
    mn = min(mn, c);
    mx = max(mx, c);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mn = min(mn, __shfl_xor(mn, o, 64));
    mx = max(mx, __shfl_xor(mx, o, 64));
  }
  if (lane != 0) return;
  if (mx < 0) mn = mx = 0;
  if (mx - mn > 65535) {
    cbase[blk] = -1;
    cspan[blk] = 0;
    atomicAdd(stat, 1);
  } else {
    cbase[blk] = mn;
    cspan[blk] = mx - mn + 1;
    // most blocks find a wider one counted already and need no atomic
    if (mx - mn + 1 > __hip_atomic_load(stat + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(stat + 1, mx - mn + 1);
  }
}
__global__ __launch_bounds__(256) void col16_kernel(CSRView A, int64_t nblk, const int32_t* cbase,
                                                    uint16_t* col16) {
  const int64_t blk = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  if (blk >= nblk) return;
  const int64_t r0 = blk << kColBlockShift;
  const int64_t r1 = min(r0 + ((int64_t)1 << kColBlockShift), A.rows);
  const int b = cbase[blk];
  for (epos p = (epos)A.rowptr[r0] + (threadIdx.x & 63), e = A.rowptr[r1]; p < e; p += 64)
    col16[p] = b >= 0 ? (uint16_t)(A.col[p] - b) : (uint16_t)0;
}

bool compress_columns(CSR& A, hipStream_t s) {
  A.col16.release();
  A.cbase.release();
  A.cspan.release();
  A.max_span = 0;
  if (A.rows <= 0 || A.nnz <= 0) return false;
  const int64_t nblk = (A.rows + (1 << kColBlockShift) - 1) >> kColBlockShift;
  DBuf<int32_t> stat(2, s);  // blocks that span too much, the widest of the others
  launch_zero_bytes(stat.get(), 2 * sizeof(int32_t), s);
  A.cbase.alloc(nblk, s);
  A.cspan.alloc(nblk, s);
  col_span_kernel<<<blocks_for(nblk, 4), 256, 0, s>>>(view(A), nblk, A.cbase.get(), A.cspan.get(),
                                                      stat.get());
  AIRG_CHECK_LAUNCH();
  int32_t st[2];
  read_back(st, stat.get(), sizeof(st), s);
  // worth it only if nearly every block compresses
  if ((int64_t)st[0] * 16 > nblk) {
    A.cbase.release();
    A.cspan.release();
    return false;
  }
  A.max_span = (int64_t)st[1];
  A.col16.alloc(A.nnz, s);
  col16_kernel<<<blocks_for(nblk, 4), 256, 0, s>>>(view(A), nblk, A.cbase.get(), A.col16.get());
  AIRG_CHECK_LAUNCH();
  return true;
}

// ------------------------------------------------------------------ row blocks
// Row blocks for the row-block product: greedy over the rows, a block takes
// consecutive rows of one 64-row group while its entries fit in
// kRowBlockEntries; a longer row is a block by itself.  One thread walks the
// rows of a group (the blocks of a group do not depend on another's).
constexpr int kRowBlockEntries = 2048;
template <bool FILL>
__global__ void row_blocks_kernel(const int32_t* __restrict__ rowptr, int64_t rows, int64_t groups,
                                  int32_t* __restrict__ count, const int32_t* __restrict__ first,
                                  int32_t* __restrict__ rblk) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= groups) return;
  const int64_t r0 = g << kColBlockShift, r1 = min(r0 + ((int64_t)1 << kColBlockShift), rows);
  int n = 0;
  int start = rowptr[r0], end = start;
  for (int64_t r = r0; r < r1; ++r) {
    const int next = rowptr[r + 1];
    // row r opens a block: the group's first, or the one before is full
    if (r == r0 || next - start > kRowBlockEntries) {
      if (FILL) rblk[first[g] + n] = (int32_t)r;
      ++n;
      start = end;
    }
    end = next;
  }
  if (!FILL) count[g] = n;
  else if (g == groups - 1) rblk[first[g] + n] = (int32_t)rows;
}
void build_row_blocks(CSR& A, hipStream_t s) {
  A.rblk.release();
  A.nrblk = 0;
  if (A.rows <= 0) return;
  const int64_t groups = (A.rows + 63) >> kColBlockShift;
  const unsigned nb = blocks_for(groups, kBlock);
  DBuf<int32_t> cnt(groups, s), first;
  row_blocks_kernel<false><<<nb, kBlock, 0, s>>>(A.rowptr.get(), A.rows, groups, cnt.get(), nullptr, nullptr);
  AIRG_CHECK_LAUNCH();
  A.nrblk = counts_to_rowptr(cnt, groups, first, s);
  A.rblk.alloc(A.nrblk + 1, s);
  row_blocks_kernel<true><<<nb, kBlock, 0, s>>>(A.rowptr.get(), A.rows, groups, nullptr, first.get(),
                                                A.rblk.get());
  AIRG_CHECK_LAUNCH();
}

}  // namespace airg

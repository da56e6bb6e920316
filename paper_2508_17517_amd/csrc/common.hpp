// Shared host-side definitions of the AIRG library: error type, device
// buffers, CSR matrices and the launch helpers every translation unit uses.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <map>
#include <stdexcept>
#include <string>
#include <utility>
#include <vector>

#include "airg.h"
#include "entries.hpp"
#include "error.hpp"

namespace airg {

#define AIRG_HIP(call)                                                              \
  do {                                                                              \
    hipError_t e_ = (call);                                                         \
    if (e_ != hipSuccess)                                                           \
      ::airg::fail(e_ == hipErrorOutOfMemory ? AIRG_ERR_NOMEM : AIRG_ERR_HIP,       \
                   std::string(#call) + ": " + hipGetErrorString(e_) + " (" +       \
                       std::to_string((int)e_) + ")");                              \
  } while (0)

#define AIRG_CHECK_LAUNCH() AIRG_HIP(hipGetLastError())

void launch_zero_bytes(void* p, size_t bytes, hipStream_t s);

// Device bytes the library's buffers hold, and an optional budget on them
// (a test hook: an allocation that would pass the budget fails as if the
// device were out of memory; 0 means no budget).
void account_device_bytes(int64_t delta);
void check_device_budget(size_t bytes);
void set_device_budget(int64_t bytes);

// Blocks and a pinned page that one setup keeps while it runs.  The setup makes
// and drops some thousand temporaries, and the stream-ordered allocator gives
// what is free back to the system at every wait of the stream (1,800 calls and
// 128 ms of a setup at FV 2048^2, 90 ms at the two of a differentiable 512^2);
// a block released here serves the next request of about its size on the same
// stream, whose order makes that safe.  (With the pinned page and row blocks
// made on the device, setup and one solve at FV 2048^2 went from 370 to 267 ms,
// the differentiable FV 512^2 from 181 to 128 ms, FV 64^2 from 25.6 to 16.3.)
// Blocks are asked for at rounded sizes, so that sizes that differ a little
// share blocks, and a kept one may serve a smaller request: each by an eighth
// of it and at most kSlack.  (Without both the setups above take 5 to 8% longer,
// with neither for the arrays that stay with the handle 8 to 13%.)  At most
// kKeep bytes are kept.  Blocks count as held at their own size, kept ones too,
// and all kept ones go back when the setup ends or an allocation fails; under an
// allocation budget nothing is rounded or kept, so that a setup needs what its
// buffers need.  A scope belongs to the thread that opened it; buffers released
// later, or by other threads, or on other streams, go back to the allocator.
class SetupPool {
 public:
  explicit SetupPool(hipStream_t s);
  ~SetupPool();
  SetupPool(const SetupPool&) = delete;
  SetupPool& operator=(const SetupPool&) = delete;
  // the calling thread's scope for stream s, or null
  static SetupPool* of(hipStream_t s) { return cur_ && cur_->s_ == s ? cur_ : nullptr; }
  // a kept block of cap >= bytes, or null and cap the size to ask for
  void* take(size_t bytes, size_t& cap);
  bool give(void* p, size_t cap);           // false: not kept
  void drop();                              // everything kept goes back
  void* page() const { return page_; }      // kPage bytes of pinned host memory, or null
  static constexpr size_t kPage = 16384;

 private:
  static constexpr size_t kKeep = (size_t)8 << 30, kSlack = (size_t)16 << 20;
  static thread_local SetupPool* cur_;
  SetupPool* outer_;
  hipStream_t s_;
  std::multimap<size_t, void*> free_;
  size_t kept_ = 0;
  void* page_ = nullptr;
};

// A block of at least `bytes` of device memory on stream s, from the running
// setup's blocks or the stream-ordered allocator, cap its size: checked against
// the budget and counted as held until it goes back to the allocator.
void* take_block(size_t bytes, hipStream_t s, size_t& cap);
void give_block(void* p, size_t cap, hipStream_t s);

// `bytes` of device memory on the host, waited for; small reads pass through
// the setup's pinned page.
void read_back(void* dst, const void* dev, size_t bytes, hipStream_t s);

// Stream-ordered device buffer (hipMallocAsync / hipFreeAsync, or the blocks a
// running setup keeps).
template <class T>
class DBuf {
 public:
  DBuf() = default;
  DBuf(size_t n, hipStream_t s) { alloc(n, s); }
  ~DBuf() { release(); }
  DBuf(const DBuf&) = delete;
  DBuf& operator=(const DBuf&) = delete;
  DBuf(DBuf&& o) noexcept { *this = std::move(o); }
  DBuf& operator=(DBuf&& o) noexcept {
    if (this != &o) {
      release();
      p_ = o.p_; n_ = o.n_; s_ = o.s_; cap_ = o.cap_;
      o.p_ = nullptr; o.n_ = 0;
    }
    return *this;
  }
  void alloc(size_t n, hipStream_t s) {
    release();
    s_ = s;
    if (n) p_ = (T*)take_block(n * sizeof(T) + 256, s, cap_);
    n_ = n;
  }
  void release() {
    if (p_) give_block(p_, cap_, s_);
    p_ = nullptr;
    n_ = 0;
  }
  T* get() const { return p_; }
  size_t size() const { return n_; }
  // cleared by a fill kernel (no memset nodes in code a caller may capture)
  void zero() { if (n_) launch_zero_bytes(p_, n_ * sizeof(T), s_); }
  void to_host(T* dst, size_t n) const {
    if (n) AIRG_HIP(hipMemcpyAsync(dst, p_, n * sizeof(T), hipMemcpyDeviceToHost, s_));
  }
  std::vector<T> host(size_t n) const {
    std::vector<T> v(n);
    if (n) read_back(v.data(), p_, n * sizeof(T), s_);
    return v;
  }
  void from_host(const T* src, size_t n) {
    if (n) AIRG_HIP(hipMemcpyAsync(p_, src, n * sizeof(T), hipMemcpyHostToDevice, s_));
  }
  hipStream_t stream() const { return s_; }

 private:
  T* p_ = nullptr;
  size_t n_ = 0, cap_ = 0;
  hipStream_t s_ = nullptr;
};

// Device CSR matrix, int32 row pointers and columns.
// Rows per base of the compressed column form (see compress_columns).
constexpr int kColBlockShift = 6;

struct CSR {
  int64_t rows = 0, cols = 0, nnz = 0;
  DBuf<int32_t> rowptr, col;
  DBuf<double> val;
  // optional compressed columns for the solve kernels: the column of entry p
  // in row i is cbase[i >> kColBlockShift] + col16[p], or col[p] where that
  // base is negative
  DBuf<uint16_t> col16;
  DBuf<int32_t> cbase;
  // with col16: number of columns each 64-row group spans (max - min + 1),
  // and the largest span over the groups
  DBuf<int32_t> cspan;
  int64_t max_span = 0;
  // optional row blocks for the row-block product: block b holds rows
  // rblk[b] .. rblk[b+1]-1 (see build_row_blocks)
  DBuf<int32_t> rblk;
  int64_t nrblk = 0;
  // in a problem batch: the first of this operator's 64-row groups in the
  // batch's activity masks (-1: not masked)
  int64_t mask_off = -1;
  // optional stored row order of a solve operator: stored row r is the
  // operator's row rmap[r], so the products read and write their per-row
  // vectors at rmap[r] (see spatial_row_order); empty: row r is stored at r
  DBuf<int32_t> rmap;
  void alloc(int64_t r, int64_t c, int64_t nz, hipStream_t s) {
    rows = r; cols = c; nnz = nz;
    rowptr.alloc(r + 1, s);
    col.alloc(nz, s);
    val.alloc(nz, s);
    col16.release();
    cbase.release();
    cspan.release();
    max_span = 0;
    rblk.release();
    nrblk = 0;
    mask_off = -1;
    rmap.release();
  }
};

// Matrix value storage of a solve-phase operator.
enum ValType { VT_F64 = 0, VT_F32 = 1, VT_BF16 = 2 };
struct bf16 {
  uint16_t bits;
};

// Operator view for the solve kernels: structure plus values of type vt.
struct OpView {
  const int32_t* rowptr;
  const int32_t* col;
  const void* val;
  ValType vt;
  int64_t rows;
  int64_t nnz;
  const uint16_t* col16;  // compressed columns, or null
  const int32_t* cbase;
  const int32_t* rblk;    // row blocks, or null
  int64_t nrblk;
  const int32_t* cspan;   // column span per 64-row group (with col16)
  int64_t max_span;
  // per 64-row group, 0 where every row belongs to a problem whose input is
  // zero in this product (its rows then skip the matrix: their sums are 0);
  // null: every row is computed
  const uint8_t* gmask;
  // stored row r is the operator's row rmap[r] (null: r)
  const int32_t* rmap;
};
inline OpView opview(const CSR& A) {
  return {A.rowptr.get(), A.col.get(), A.val.get(), VT_F64, A.rows, A.nnz, A.col16.get(),
          A.cbase.get(), A.rblk.get(), A.nrblk, A.cspan.get(), A.max_span, nullptr, A.rmap.get()};
}

// Read-only view passed to kernels.
struct CSRView {
  const int32_t* rowptr;
  const int32_t* col;
  const double* val;
  int64_t rows;
};
inline CSRView view(const CSR& A) { return {A.rowptr.get(), A.col.get(), A.val.get(), A.rows}; }

// A contiguous range of the nested numbering that belongs to one problem of
// a block-diagonal batch.
struct GroupRange {
  int64_t start, len;
  int32_t group;
};

inline unsigned blocks_for(int64_t n, int per_block) {
  int64_t b = (n + per_block - 1) / per_block;
  return (unsigned)(b < 1 ? 1 : b);
}

// Host scalar fetched from device memory (synchronises the stream).
template <class T>
T fetch(const T* dptr, hipStream_t s) {
  T v;
  read_back(&v, dptr, sizeof(T), s);
  return v;
}

constexpr int kBlock = 256;

}  // namespace airg

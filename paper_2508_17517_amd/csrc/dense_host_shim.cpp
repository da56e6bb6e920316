// Host-only C entry points over the dense routines, the launch-shape rule and
// the arithmetic on entry positions, for CPU tests (not part of the public ABI).
#include <cstring>
#include <vector>

#include "dense.hpp"
#include "entries.hpp"
#include "error.hpp"
#include "shapes.hpp"

using namespace airg;

extern "C" {

// alpha (steps entries) from an (m+1) x m Hessenberg matrix; returns 0 or -1.
int airg_host_gmres_poly(const double* H, int m, int steps, double beta, double* alpha) {
  try {
    std::vector<double> h(H, H + (size_t)(m + 1) * m);
    std::vector<double> a = gmres_poly_coeffs(h, m, steps, beta);
    std::memcpy(alpha, a.data(), a.size() * sizeof(double));
    return 0;
  } catch (...) {
    return -1;
  }
}

// Eigenvalues of an upper Hessenberg n x n matrix; returns 0 or -1.
int airg_host_hessenberg_eig(const double* A, int n, double* re, double* im) {
  try {
    std::vector<cplx> ev = hessenberg_eigenvalues(std::vector<double>(A, A + (size_t)n * n), n);
    for (int i = 0; i < n; ++i) {
      re[i] = ev[i].real();
      im[i] = ev[i].imag();
    }
    return 0;
  } catch (...) {
    return -1;
  }
}

// Newton roots from an Arnoldi relation; writes up to cap roots, returns the count or -1.
int airg_host_newton_roots(const double* H, int m, int steps, int add_roots, double* re,
                           double* im, int cap) {
  try {
    std::vector<double> h(H, H + (size_t)(m + 1) * m);
    std::vector<cplx> r = newton_roots(h, m, steps, add_roots != 0);
    if ((int)r.size() > cap) return -1;
    for (size_t i = 0; i < r.size(); ++i) {
      re[i] = r[i].real();
      im[i] = r[i].imag();
    }
    return (int)r.size();
  } catch (...) {
    return -1;
  }
}

int airg_host_numerical_rank(const double* H, int ld, int k, double tol) {
  try {
    std::vector<double> h(H, H + (size_t)k * ld);
    return numerical_rank(h, ld, k, tol);
  } catch (...) {
    return -1;
  }
}

// The default launch shape of an operator (role as in OpRole).
int airg_host_default_shape(int role, int64_t rows, int64_t nnz, int vbytes, int xbytes, int windows,
                            int64_t max_span) {
  return default_shape({rows, nnz, vbytes, xbytes, windows != 0, max_span}, (OpRole)role);
}

// Walks entries s .. e - 1 as the kernels do: in chunks of len (len > 0), or in
// strides of -len from lane `lane`.  Writes up to cap (first, end) pairs and
// returns their number, cap + 1 where the walk does not end.
int airg_host_walk_entries(int32_t s, int32_t e, int len, int lane, int cap, uint32_t* out) {
  int n = 0;
  const epos end = e;
  if (len > 0) {
    for (epos c0 = s; c0 < end; c0 += len) {
      if (n == cap) return cap + 1;
      out[2 * n] = c0;
      out[2 * n++ + 1] = chunk_end(c0, end, len);
    }
  } else {
    for (epos p = (epos)s + lane; p < end; p += -len) {
      if (n == cap) return cap + 1;
      out[2 * n] = p;
      out[2 * n++ + 1] = p + 1;
    }
  }
  return n;
}
int airg_host_find_col(const int32_t* col, int32_t lo, int32_t hi, int32_t j) { return find_col(col, lo, hi, j); }
int64_t airg_host_first_from(const int32_t* col, int32_t lo, int32_t hi, int64_t w0) {
  return first_from(col, lo, hi, w0);
}
int64_t airg_host_pairs_before(int32_t e) { return pairs_before(e); }

}  // extern "C"

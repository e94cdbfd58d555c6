// Launchers shared between the library's translation units.
#pragma once
#include <functional>

#include "internal.hpp"

namespace chf {

void launch_vloc(chf_ham* H, const double4* atoms, const double* width, int n_atoms, hipStream_t s);
void launch_cast_veff(chf_ham* H, const double* src, double* d64, float* d32, int* bad_dev, hipStream_t s);
// row-group tables of the tiled kernel (ham_build, after the entry tables)
void build_row_groups(chf_ham* H, hipStream_t s);
template <class T>
void launch_kb_gather(chf_ham* H, const T* X, int64_t ldx, int nvec, T* C, hipStream_t s);
// Y = alpha (H X - shift X) - beta Z ; Z may be null or alias Y.  force_kernel:
// 0 = best available, 1 = generic neighbour-table kernel.  lap_only: H is
// replaced by -1/2 L (no V_eff, no projectors), by the neighbour-table kernel.
// C_ext: caller-provided KB-coefficient scratch for nvec vectors (no
// allocation, no kernel timing); NULL uses the handle's scratch.  narrow: a
// block of one row piece of 8 or 16 bytes may take the one-thread-per-point
// kernel (whose sums run in another order than the vector tile's).
template <class T>
void hx_step(chf_ham* H, const T* X, int64_t ldx, T* Y, int64_t ldy, const T* Z, int64_t ldz, int nvec, double alpha,
             double shift, double beta, hipStream_t s, int force_kernel, bool lap_only = false, T* C_ext = nullptr,
             bool narrow = false);
// y = H x for one FP64 vector, with the partials of x.y (at most 512) in part;
// returns their number.  hx_dot_ok: whether the handle has the tables for it.
bool hx_dot_ok(const chf_ham* H);
int hx_dot(chf_ham* H, const double* x, double* y, double* part, hipStream_t s);
// a launch counted as an H X launch by the kernel timer
void timed_hx(hipStream_t s, const std::function<void()>& launch);

// Degree-m scaled Chebyshev filter in place over X and the work block W
// (column blocks of min(nvec, ldw) vectors)
template <class T>
void filter_run(chf_ham* H, T* X, int64_t ldx, T* W, int64_t ldw, int nvec, int m, double a, double b, double a0,
                hipStream_t s, int force_kernel, int64_t max_cols = INT64_MAX, T* C_ext = nullptr);
// the same filter with the KB coefficients in the library's fixed device
// scratch (no allocation); noalloc_scratch_init looks its address up for the
// current device (called by ham_build)
void noalloc_scratch_init(int device);
template <class T>
void filter_run_noalloc(chf_ham* H, T* X, int64_t ldx, T* W, int64_t ldw, int nvec, int m, double a, double b,
                        double a0, hipStream_t s);
// CHF_EINVAL unless the bytes of A and B are disjoint; the bytes that a block of m
// columns spans (capi.cpp)
void check_disjoint(const void* A, size_t bytes_a, const void* B, size_t bytes_b, const char* what);
size_t block_bytes(const chf_ham* H, int dtype, int64_t ld, int64_t m);

// bytes of the KB coefficient scratch an H X launch on nvec vectors needs
size_t kb_coef_bytes(const chf_ham* H, int nvec, size_t elem_bytes);

void timer_enable(int on);
void timer_read(double* ms, int64_t* launches);

// dense.hip
template <class T>
void dot_device(chf_ctx* ctx, int64_t n, const T* x, int64_t incx, const T* y, int64_t incy, double* out_dev,
                hipStream_t s);
template <class T>
double dot_host(chf_ctx* ctx, int64_t n, const T* x, int64_t incx, const T* y, int64_t incy, hipStream_t s);
void lincomb(int64_t n, double a, const double* x, int64_t incx, double b, const double* y, int64_t incy, double* z,
             int64_t incz, hipStream_t s);
template <class T>
void orthonormalize_t(chf_ctx* ctx, T* X, int64_t ldx, int64_t n_rows, int m, bool gram64, int* fallbacks,
                      hipStream_t s);
template <class T>
void rayleigh_ritz_t(chf_ham* H, chf_ctx* ctx, T* X, int64_t ldx, int m, double* eig_host, T* W, int64_t ldw,
                     hipStream_t s);
void lanczos_run(chf_ham* H, chf_ctx* ctx, const double* v0, int k, double* out3, hipStream_t s);

// S = A^T B (m x n, FP64, row stride lds) over n_rows rows of TI, multiplied and
// added in TA within a row slice, the slices' partials in FP64 (gram.hip)
struct GramSlices {
    int64_t tiles;        // pieces of S per slice
    int64_t rows;         // rows per slice
    int64_t group;        // slices whose partials are held at once
    int64_t most;         // slices of any product of these pieces over at most n_rows rows
    int64_t part_stride;  // values of one partial
    size_t part_bytes;    // partials scratch
};
GramSlices gram_slices(int64_t n_rows, int m, int n, size_t acc_bytes, size_t in_bytes, int64_t ld, bool symmetric);
size_t gram_part_bound(int64_t n_rows, int m, int n, size_t acc_bytes, bool symmetric);
template <class TI, class TA>
void gram_product(chf_ctx* ctx, const TI* A, int64_t lda, const TI* B, int64_t ldb, int64_t n_rows, int m, int n,
                  double* S, int64_t lds, hipStream_t s);

// Cholesky factor and solve of a Cholesky-QR pass (trsolve.hip): S = R^T R, R upper,
// column-major, over the upper triangle of S (*info as LAPACK's potrf; set it to
// 0 before), then X <- X R^{-1} in place with the same work, cholesky_work_bytes
// long and 16-byte aligned
size_t cholesky_work_bytes(int m, size_t elem_bytes);
template <class T>
void cholesky(double* S, int m, void* work, int* info, hipStream_t s);
template <class T>
void solve_upper(T* X, int64_t ldx, int64_t n_rows, int m, const double* R, void* work, hipStream_t s);

// X <- X Q in place, Q m x m column-major FP64, for the widths it takes (else false);
// work: rotate_work_bytes(m) bytes, 16-byte aligned (trsolve.hip)
size_t rotate_work_bytes(int m, size_t elem_bytes);
template <class T>
bool rotate(T* X, int64_t ldx, int64_t n_rows, int m, const double* Q, void* work, hipStream_t s);

// eigenvalues (ascending) and eigenvectors (columns, over S) of the symmetric
// m x m S; E: m doubles, work: eig_work_bytes(m) (eig.hip)
constexpr int kEigMax = 192;
size_t eig_work_bytes(int m);
void sym_eig(chf_ctx* ctx, int m, double* S, double* evals, double* E, double* work, int* info, hipStream_t s);

}  // namespace chf

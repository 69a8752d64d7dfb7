// Host-side launchers of the library's HIP kernels (gfx950, wave64).
#pragma once

#include "common.h"

namespace matamg {

// ----------------------------------------------------------------- prims ---
// exclusive scan of `n` int32 counts into out[0..n]; out[n] = total.
// `tmp` must hold scan_tmp_size(n) ints.  Returns nothing; total stays on device.
size_t scan_tmp_size(int64_t n);
void exclusive_scan(const int* in, int* out, int64_t n, int* tmp, hipStream_t s);
// bytes zero bytes at p, by a kernel on s (cheaper to issue than a runtime memset)
void zero_async(void* p, size_t bytes, hipStream_t s);

// deterministic dot product sum_i a_i b_i in FP64 (fixed reduction tree for a given n)
// written to *result (device).  partial: >= kMaxPartials doubles, counter: zeroed uint.
constexpr int kMaxPartials = 4096;
template <typename T>
void dot(const T* a, const T* b, int64_t n, double* partial, unsigned* counter, double* result, hipStream_t s);

// --------------------------------------------------------------- streaming ---
// row blocks for the streaming CSR kernels, computed from a host row pointer
std::vector<int> stream_blocks(const int* rowptr_host, int n, int group, int cap = kStreamCap);
// threads per row for a matrix (host row pointer): stream_group_rule
int stream_group(const int* rowptr_host, int n);
// A.group, A.nblk and A.blk from A's device row pointer (the same greedy
// partition as stream_blocks, computed on the device), and with `pack`
// A.col16 and A.cbase when every block's columns span fewer than 2^16
// values (otherwise both stay empty); reads back the block count, so s is
// synchronised once
// (blocks of at most `cap` stored entries; A.cap records it)
void stream_partition(DCsr& A, MemCounter* mc, hipStream_t s, bool pack, int cap = kStreamCap);
// the distinct-column lists of A's packed streaming blocks (see DCsr::ustart)
void block_uniques(DCsr& A, MemCounter* mc, hipStream_t s);
// the column windows of A's streaming blocks (see DCsr::uwin), where some span
// 2^16 values or more
void block_windows(DCsr& A, MemCounter* mc, hipStream_t s);

// the row dictionaries of A (see DCsr::drow_of) where its rows repeat; none
// otherwise.  Synchronises s.
void row_dictionaries(DCsr& A, MemCounter* mc, hipStream_t s);
// whether FP64 launches stage the windows that A's dictionaries gather from
bool rows_staged(const DCsr& A);

// dot partials of a streaming launch: one per row block
constexpr int kStreamPartials = 1;  // dot partials per streaming block
inline int stream_partials(const DCsr& A) { return A.nblk * kStreamPartials; }

// dot-fusion target: per-block partial sums, reduced by finish_sum into
// *result (result null: left to the kernel that needs the sum)
struct DotTarget {
    double* partial = nullptr;
    unsigned* counter = nullptr;
    double* result = nullptr;
};
// *dt.result = sum of dt.partial[0..nblocks) in index order (one block)
void finish_sum(const DotTarget& dt, int nblocks, hipStream_t s);

// y = A x
template <typename T>
void spmv(const DCsr& A, const T* val, const T* x, T* y, hipStream_t s);
// y = b - A x
template <typename T>
void spmv_resid(const DCsr& A, const T* val, const T* x, const T* b, T* y, hipStream_t s);
// y = y_in + A x  (prolongation x += P e when y == y_in)
template <typename T>
void spmv_add(const DCsr& A, const T* val, const T* x, const T* y_in, T* y, hipStream_t s);
// smoother step: res = b - A x; d = c1 d + c2 dinv res; out = x + d.
// out64 (if non-null) receives the FP64 iterate instead of out; dotvec (if
// non-null) fuses sum_i out_i * dotvec_i into `dt`.
template <typename T>
void spmv_smooth(const DCsr& A, const T* val, const T* x, const T* b, const T* dinv, T* d, T c1, T c2, T* out,
                 double* out64, const double* dotvec, DotTarget dt, hipStream_t s);
// restriction fused with the next level's first smoother step from zero:
// bc = R r; d_c = c2 * dinv_c .* bc; x_c = d_c (as smooth_first on bc)
template <typename T>
void spmv_restrict_first(const DCsr& R, const T* val, const T* r, T* bc, const T* dinv_c, T c2, T* d_c, T* x_c,
                         hipStream_t s);
// q = A p and sum_i p_i q_i (FP64)
void spmv_dot(const DCsr& A, const double* p, double* q, DotTarget dt, hipStream_t s);
// y = b - A x and sum_i y_i^2
void spmv_resid_norm(const DCsr& A, const double* x, const double* b, double* y, DotTarget dt, hipStream_t s);
// y = dscale .* (A x / |x|) and sum y_i^2 (power method); x.x is the sum of
// part[0..npart), at most kOwnSumPartials of them
void spmv_scale_norm(const DCsr& A, const double* x, const double* part, int npart, const double* dscale, double* y,
                     DotTarget dt, hipStream_t s);

// --------------------------------------------------------------- vectors ---
// first smoother step from zero: d = c2 * dinv .* b; x = d.  If b64 is given,
// b = (T) b64 is also stored to `b`.
template <typename T>
void smooth_first(int64_t n, const double* b64, T* b, const T* dinv, T c2, T* d, T* x, hipStream_t s);
// most partials that a kernel which needs their sum adds up itself
constexpr int kOwnSumPartials = 1024;
// the finest level's first smoother step from zero, as smooth_first takes it
// (b null: the right-hand side is r itself)
template <typename T>
struct FirstStep {
    T* b;
    const T* dinv;
    T c2;
    T* d;
    T* x;
};
// CG: alpha = rz/pq; x += alpha p; r -= alpha q; rr = r.r (its partials,
// vector_partials(n) of them, are left if rr.result is null).  pqs.partial,
// if set, holds pq as pq_blocks partials, and pq is stored.  first (or null):
// also the next V-cycle's first smoother step, from the new r.
template <typename T>
void cg_update(int64_t n, double* x, double* r, const double* p, const double* q, const double* rz, double* pq,
               DotTarget pqs, int pq_blocks, DotTarget rr, const FirstStep<T>* first, hipStream_t s);
// CG: p = z + (rz_new / rz_old) p  (rz_old == nullptr: p = z); rzs.partial, if
// set, holds rz_new as rz_blocks partials, and rz_new is stored
void cg_direction(int64_t n, double* p, const double* z, double* rz_new, const double* rz_old, DotTarget rzs,
                  int rz_blocks, hipStream_t s);
int vector_partials(int64_t n);
// finish_sum, then `words` of scal to host memory (pinned), then *step + 1 to
// *step and *host_step, and scal[from] to scal[to]
void finish_report(const DotTarget& dt, int nblocks, double* scal, int words, int from, int to, unsigned* step,
                   double* host, unsigned* host_step, hipStream_t s);
template <typename A, typename B>
void cast_vec(int64_t n, const A* in, B* out, hipStream_t s);
// seeded values in (-1, 1) and sum_i v_i^2 as dot(v, v) takes it; its number
// of partial sums is returned (all that is left if dt.result is null)
int fill_seeded_uniform(int64_t n, uint64_t key, double* v, DotTarget dt, hipStream_t s);

// ----------------------------------------------------------------- dense ---
// out = Minv * in for a dense row-major n x n FP64 matrix; in/out of type T
template <typename T>
void dense_gemv(int n, const double* M, const T* in, T* out, hipStream_t s);
// A (n x n, row-major, symmetric) -> A^{-1} in place via blocked Cholesky,
// enqueued on s; *flag (device int, set to 0 here) becomes 1 if the matrix is
// not positive definite, and A then holds no inverse.  work: n*n doubles.
void dense_spd_inverse(int n, double* A, double* work, int* flag, hipStream_t s);

// ------------------------------------------------- the V-cycle's small levels ---
constexpr int kTailLevels = 4;       // smoothed levels
constexpr int kTailSteps = 4;        // smoother steps
constexpr int kTailDense = 256;      // coarsest unknowns
constexpr int kTailRow = 96;         // entries of a row
constexpr int kTailLds = 156 << 10;  // bytes

constexpr int kTailThreads = 1024;
// One level in LDS: byte offsets of its arrays, the operator's, the inverse
// diagonal and the row pointers in the image.  The transfers' entries are in
// memory.
template <typename T>
struct TailLevel {
    int n, steps;
    int val, col, dinv, rp, prp, rrp;  // operator; row pointers of P and R
    int b, d, x, y;
    const int *pcol, *rcol;
    const T *pval, *rval;
    T c1[kTailSteps], c2[kTailSteps];
};
// the head of the image
template <typename T>
struct TailHead {
    int levels;
    int nc, bc, xc;  // coarsest unknowns, right-hand side and solution
    const double* inverse;
    TailLevel<T> lv[kTailLevels];
};
// an array of the image: values, or indices to be stored in 16 bits
template <typename T>
struct TailSegment {
    const T* val;
    const int* idx;
    int count, at;
};
template <typename T>
struct TailSegments {
    int count = 0;
    TailSegment<T> s[6 * kTailLevels];
};
template <typename T>
void tail_image(const TailHead<T>& head, const TailSegments<T>& segs, char* image, hipStream_t s);
// the V-cycle from the first of the levels (n rows, its right-hand side b, its
// first smoother step in d and x) down and back, its result to out; that
// level's b, d and x lie behind the image in LDS, in this order
template <typename T>
void tail_cycle(const char* image, int image_bytes, int lds_bytes, int n, const T* b, const T* d, const T* x, T* out,
                hipStream_t s);

}  // namespace matamg

// Dense FP64 kernels for the coarsest level: blocked right-looking Cholesky
// A = L L^T, the triangular inverse Y = L^{-1} by right-looking block-row
// forward substitution, and A^{-1} = Y^T Y.  The coarse solve of every
// V-cycle is then a single dense GEMV, which streams the matrix at full
// bandwidth instead of the sequential dependency chain of two triangular
// solves.
//
// All matrices are row-major n x n, tiles are 64 x 64.  The factorisation
// and the inverse advance together, two launches per diagonal tile: step kb
// solves the panel below tile kb and block row kb of Y against L_kk, then
// subtracts both products from the later tiles; the workgroup that updates
// the next diagonal tile factors it at once, beside the other tiles.  What
// bounds it is the chain of nt such steps (solve 13 us, update with the next
// factorisation 25 us) up to about 2,500 unknowns, and beyond that the
// updates' passes over the two matrices.  Setup of a one-level hierarchy of
// 1,950 unknowns 6.5 -> 1.7 ms, of 4,225 17.7 -> 4.6 ms, of 4,970 23.5 ->
// 6.3 ms, against five launches a step with one thread per row of a
// triangular solve (50 and 36 us), a barrier per column of the diagonal tile
// (50 us) and products on the vector units.
//
// The products run on the FP64 matrix cores (v_mfma_f64_16x16x4: each result
// is the chain of IEEE fused multiply-adds over ascending k, so a product
// tile is the same as a loop of fma).  Every entry's operations and their
// order are fixed: subtractions of 64-term products panel after panel, and
// within a diagonal tile or a triangular solve one fused subtraction at a
// time in ascending column order.
#include "device_util.h"
#include "kernels.h"

namespace matamg {
namespace {

constexpr int NB = 64;
constexpr int kTile = NB * NB;
constexpr int kPer = kTile / kBlock;  // tile entries per thread

typedef double d4 __attribute__((ext_vector_type(4)));

// Two LDS layouts of a 64 x 64 operand tile, free of bank conflicts for the
// reads of a matrix instruction (lane l reads row l % 16 and term l / 16 of
// four consecutive terms):
//   by rows:  T[i][k], rows padded to 66 doubles
//   by terms: T[k][j], with bit 4 of j flipped on odd k
constexpr int kRowPitch = NB + 2;
__device__ __forceinline__ int at_row(int i, int k) { return i * kRowPitch + k; }
__device__ __forceinline__ int at_term(int k, int j) { return k * NB + (j ^ ((k & 1) << 4)); }
constexpr int kTileLds = NB * kRowPitch;

// this thread's entries of a tile of M (row-major, leading dimension n) whose
// first entry is (r0, c0); entries outside the matrix read as zero
__device__ __forceinline__ void load_tile(double* v, const double* M, int n, int r0, int c0) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = (int)threadIdx.x + u * kBlock;
        const int r = r0 + e / NB, c = c0 + e % NB;
        v[u] = (r < n && c < n) ? M[(size_t)r * n + c] : 0.0;
    }
}
template <bool BY_ROW>
__device__ __forceinline__ void store_lds(double* T, const double* v) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = (int)threadIdx.x + u * kBlock;
        T[BY_ROW ? at_row(e / NB, e % NB) : at_term(e / NB, e % NB)] = v[u];
    }
}

// acc += A B over 64 terms: wavefront w owns the 32 x 32 quadrant (w / 2,
// w % 2) as 2 x 2 matrix-core tiles.  A is held by rows (AROW) or by terms
// (A^T stored), B^T by rows (BROW) or B by terms.
template <bool AROW, bool BROW>
__device__ __forceinline__ void tile_mma(d4 (&acc)[2][2], const double* As, const double* Bs) {
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int i0 = (w >> 1) * 32 + (lane & 15), j0 = (w & 1) * 32 + (lane & 15), kq = lane >> 4;
#pragma unroll
    for (int s = 0; s < NB / 4; ++s) {
        const int k = 4 * s + kq;
        double a[2], b[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            a[t] = As[AROW ? at_row(i0 + 16 * t, k) : at_term(k, i0 + 16 * t)];
            b[t] = Bs[BROW ? at_row(j0 + 16 * t, k) : at_term(k, j0 + 16 * t)];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int v = 0; v < 2; ++v) acc[t][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[v], acc[t][v], 0, 0, 0);
    }
}

// f(i, j, t, v, q) for every tile entry (i, j) this thread holds in acc[t][v][q]
template <class F>
__device__ __forceinline__ void for_acc(F f) {
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                f((w >> 1) * 32 + 16 * t + 4 * q + (lane >> 4), (w & 1) * 32 + 16 * v + (lane & 15), t, v, q);
}

__device__ __forceinline__ double lane_value(double x, int lane) {
    const unsigned long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// Factor the diagonal tile held in LDS (by rows, lower triangle; entries
// outside the matrix must be those of the identity) and write it to A; flag
// <- 1 if it is not positive definite.  Right-looking in panels of 16
// columns: the first wavefront factors a panel, lane i holding row i in
// registers, with no barrier between the columns (root, quotients and the
// panel's own subtractions are the chain that bounds the tile); then the
// matrix cores subtract the panel's products from the columns right of it.
__device__ __forceinline__ void potrf_tile(double* T, double* A, int n, int o, int* flag) {
    constexpr int PW = 16;
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    for (int p = 0; p < NB / PW; ++p) {
        if (w == 0) {
            double v[PW];
            bool bad = false;
#pragma unroll
            for (int c = 0; c < PW; ++c) v[c] = T[at_row(lane, PW * p + c)];
#pragma unroll
            for (int c = 0; c < PW; ++c) {
                const int j = PW * p + c;
                double d = lane_value(v[c], j);
                const bool ok = d > 0.0 && d <= 1.79769313486231570815e308;
                bad = bad || !ok;
                d = ok ? d : 1.0;
                const double root = sqrt(d);
                v[c] = (lane == j) ? root : v[c] / root;
#pragma unroll
                for (int k = c + 1; k < PW; ++k) v[k] = __builtin_fma(-v[c], lane_value(v[c], PW * p + k), v[k]);
            }
#pragma unroll
            for (int c = 0; c < PW; ++c) T[at_row(lane, PW * p + c)] = v[c];
            if (bad && lane == 0) *flag = 1;
        }
        __syncthreads();
        const int rest = NB / PW - 1 - p;
        for (int t = w; t < rest * (rest + 1) / 2; t += kBlock / 64) {
            // 16 x 16 blocks (bi, bj), p < bj <= bi, the next panel's first
            int bj = p + 1, off = t;
            while (off >= NB / PW - bj) {
                off -= NB / PW - bj;
                ++bj;
            }
            const int bi = bj + off, r = lane & 15, kq = lane >> 4;
            d4 c;
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = T[at_row(PW * bi + 4 * q + kq, PW * bj + r)];
#pragma unroll
            for (int k = 0; k < PW; k += 4)
                c = __builtin_amdgcn_mfma_f64_16x16x4f64(-T[at_row(PW * bi + r, PW * p + k + kq)],
                                                         T[at_row(PW * bj + r, PW * p + k + kq)], c, 0, 0, 0);
#pragma unroll
            for (int q = 0; q < 4; ++q) T[at_row(PW * bi + 4 * q + kq, PW * bj + r)] = c[q];
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = (int)threadIdx.x + u * kBlock;
        const int r = e / NB, c = e % NB;
        if (o + r < n && o + c < n) A[(size_t)(o + r) * n + o + c] = c <= r ? T[at_row(r, c)] : 0.0;
    }
}

// the tile's identity outside the matrix, zero above the diagonal
__device__ __forceinline__ double diag_pad(double v, int r, int c, int o, int n) {
    if (o + r >= n || o + c >= n) return r == c ? 1.0 : 0.0;
    return c <= r ? v : 0.0;
}

__global__ __launch_bounds__(kBlock) void k_potrf_first(double* A, int n, int* flag) {
    __shared__ double T[kTileLds];
    double v[kPer];
    load_tile(v, A, n, 0, 0);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = (int)threadIdx.x + u * kBlock;
        v[u] = diag_pad(v[u], e / NB, e % NB, 0, n);
    }
    store_lds<true>(T, v);
    __syncthreads();
    potrf_tile(T, A, n, 0, flag);
}

// the value of row SEL of 16 lanes in all four rows of the wavefront
template <int SEL>
__device__ __forceinline__ unsigned row_bits(unsigned x) {
    auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const unsigned y = SEL & 2 ? h[1] : h[0];
    auto r = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return SEL & 1 ? r[1] : r[0];
}
template <int SEL>
__device__ __forceinline__ double row_value(double x) {
    const unsigned long long b = __double_as_longlong(x);
    const unsigned lo = row_bits<SEL>((unsigned)b), hi = row_bits<SEL>((unsigned)(b >> 32));
    return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}

// x / d, correctly rounded, from y = 1 / d correctly rounded: two steps of
// q <- q + (x - q d) y from q = x y.  The first leaves q within one unit in
// the last place, the second's remainder is then exact and its result the
// rounded quotient (P. Markstein, Computation of elementary functions on the
// IBM RISC System/6000 processor, 1990), as long as the remainders stay clear
// of the ends of the exponent range; `bad` is set where they may not.
__device__ __forceinline__ double quotient(double x, double d, double y, bool& bad) {
    double q = x * y;
    q = __builtin_fma(__builtin_fma(-q, d, x), y, q);
    q = __builtin_fma(__builtin_fma(-q, d, x), y, q);
    const double a = fabs(x);
    bad = bad || !((a > 0x1p-900 && a < 0x1p+900) || x == 0.0);
    return q;
}

// Four unknowns, 4 R + 0 .. 3, of a panel of 16 of the substitutions of
// k_dense_solve: v holds the panel's unknowns, l the factor's entries that
// this lane subtracts with (zero where its unknown is not later), d and y the
// diagonal and its reciprocals.  The solved unknown goes to x, so that the
// next step waits only for quotient, broadcast and subtraction.
struct PanelFactor {
    double l[16][4], d[16], y[16];
};
template <int R, int SEL>
__device__ __forceinline__ void solve_step(double (&v)[4], double (&x)[4], const PanelFactor& F, int g, bool& bad) {
    constexpr int j = 4 * R + SEL;
    const double t = row_value<SEL>(quotient(v[R], F.d[j], F.y[j], bad));
#pragma unroll
    for (int r = R; r < 4; ++r) v[r] = __builtin_fma(-t, F.l[j][r], v[r]);
    x[R] = g == SEL ? t : x[R];
}
template <int R>
__device__ __forceinline__ void solve_four(double (&v)[4], double (&x)[4], const PanelFactor& F, int g, bool& bad) {
    solve_step<R, 0>(v, x, F, g, bad);
    solve_step<R, 1>(v, x, F, g, bad);
    solve_step<R, 2>(v, x, F, g, bad);
    solve_step<R, 3>(v, x, F, g, bad);
}

// Solves with L_kk, one 64-wide tile per workgroup:
//   blocks 0 .. kb:  block row kb of Y,  Y <- L_kk^{-1} Y, tile by tile (the
//                    tile of column kb starts as the identity)
//   the others:      the panel below, X L_kk^T = B, 64 rows each
// Both are 64 forward substitutions with L_kk, 16 per wavefront and
// independent of the other wavefronts: lane 16 g + c holds the unknowns
// 16 p + 4 r + g of substitution c in v[p][r], the layout in which the matrix
// cores take the solved panel p as an operand and return the later unknowns.
// Each unknown's subtractions come one by one in ascending order; the chain
// is a quotient, a broadcast over the four lanes and a subtraction per unknown.
__global__ __launch_bounds__(kBlock) void k_dense_solve(double* A, double* Y, int n, int kb) {
    __shared__ double L[kTileLds], inv[NB];
    __shared__ int odd;
    const int o = kb * NB;
    const bool yrow = (int)blockIdx.x <= kb, eye = (int)blockIdx.x == kb;
    const int lane = (int)threadIdx.x & 63, g = lane >> 4, c = lane & 15;
    double t[kPer];
    load_tile(t, A, n, o, o);
    // substitution c of wavefront w: a column of Y or a row of A
    const int rhs = (yrow ? (int)blockIdx.x * NB : o + NB + ((int)blockIdx.x - kb - 1) * NB) +
                    16 * ((int)threadIdx.x >> 6) + c;
    double* M = yrow ? Y + (size_t)o * n + rhs : A + (size_t)rhs * n + o;
    const size_t step = yrow ? (size_t)n : 1;
    auto load = [&](int u) {
        if (eye) return u + o == rhs ? 1.0 : 0.0;
        return (rhs < n && o + u < n) ? M[u * step] : 0.0;
    };
    d4 v[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[p][r] = load(16 * p + 4 * r + g);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int e = (int)threadIdx.x + u * kBlock;
        L[at_row(e / NB, e % NB)] = diag_pad(t[u], e / NB, e % NB, o, n);
    }
    if (threadIdx.x == 0) odd = 0;
    __syncthreads();
    if (threadIdx.x < NB) {
        const double d = L[at_row(threadIdx.x, threadIdx.x)];
        inv[threadIdx.x] = 1.0 / d;
        if (!(d > 0x1p-60 && d < 0x1p+60)) odd = 1;
    }
    __syncthreads();
    bool bad = odd != 0;
    // v[0] is the panel being solved: the panels move down one place after
    // each, the solved ones to the end (unrolled, the code is 41 KB and takes
    // longer to fetch than to run)
#pragma unroll 1
    for (int p = 0; p < 4; ++p) {
        const double* Lp = L + at_row(16 * p, 16 * p);
        PanelFactor F;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            F.d[j] = Lp[at_row(j, j)];
            F.y[j] = inv[16 * p + j];
#pragma unroll
            for (int r = j / 4; r < 4; ++r) F.l[j][r] = 4 * r + g > j ? Lp[at_row(4 * r + g, j)] : 0.0;
        }
        // (every load above is issued before the chain below starts)
        __builtin_amdgcn_sched_barrier(0);
        double u[4] = {v[0][0], v[0][1], v[0][2], v[0][3]}, x[4] = {};
        solve_four<0>(u, x, F, g, bad);
        solve_four<1>(u, x, F, g, bad);
        solve_four<2>(u, x, F, g, bad);
        solve_four<3>(u, x, F, g, bad);
        // the matrix cores subtract the panel from the unknowns below it
#pragma unroll
        for (int b = 1; b < 4; ++b)
            if (p + b < 4) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    v[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-Lp[at_row(16 * b + c, 4 * s + g)], x[s], v[b], 0, 0, 0);
            }
#pragma unroll
        for (int b = 0; b < 3; ++b) v[b] = v[b + 1];
        v[3] = d4{x[0], x[1], x[2], x[3]};
    }
    if (__any(bad)) {
        // some quotient lies near the ends of the exponent range: the same
        // substitutions with plain divisions
        double y = 0.0;
        for (int p = 0; p < 4; ++p)
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * p + 4 * r;
                // subtract the unknowns before i, then solve the next four
                y = load(i + g);
                for (int j = 0; j < i; ++j) {
                    double x = 0.0;
#pragma unroll
                    for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr)
                            if (16 * pp + 4 * rr == (j & ~3)) x = v[pp][rr];
                    y = __builtin_fma(-__shfl(x, 16 * (j & 3) + c, 64), L[at_row(i + g, j)], y);
                }
                for (int q = 0; q < 4; ++q) {
                    const double x = __shfl(y / L[at_row(i + q, i + q)], 16 * q + c, 64);
                    if (g == q) y = x;
                    if (g > q) y = __builtin_fma(-x, L[at_row(i + g, i + q)], y);
                }
#pragma unroll
                for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr)
                        if (pp == p && rr == r) v[pp][rr] = y;
            }
    }
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (rhs < n && o + 16 * p + 4 * r + g < n) M[(16 * p + 4 * r + g) * step] = v[p][r];
}

__device__ __forceinline__ void tri_index(int b, int& I, int& J) {
    int i = (int)((sqrt(8.0 * b + 1.0) - 1.0) * 0.5);
    while ((i + 1) * (i + 2) / 2 <= b) ++i;
    while (i * (i + 1) / 2 > b) --i;
    I = i;
    J = b - i * (i + 1) / 2;
}

// After step kb's solves, with t = nt - kb - 1 later tile rows:
//   blocks 0 .. t (t + 1) / 2 - 1:  A_IJ -= L_I,kb L_J,kb^T for kb < J <= I;
//       block 0, the next diagonal tile, factors it as well
//   the other t (kb + 1):  Y_IJ -= L_I,kb Y_kb,J for I > kb, J <= kb (zero
//       before its first subtraction, at J = kb)
// Tile column kb is never the last, so its 64 terms are all inside.
__global__ __launch_bounds__(kBlock) void k_dense_update(double* A, double* Y, int n, int nt, int kb, int* flag) {
    __shared__ double As[kTileLds], Bs[kTileLds];
    const int t = nt - kb - 1, nsyrk = t * (t + 1) / 2;
    const int b = (int)blockIdx.x, o = kb * NB;
    const bool syrk = b < nsyrk;
    int I, J;
    if (syrk) {
        tri_index(b, I, J);
        J += kb + 1;
    } else {
        I = (b - nsyrk) / (kb + 1);
        J = (b - nsyrk) % (kb + 1);
    }
    I += kb + 1;
    double* M = syrk ? A : Y;
    const int ri = I * NB, cj = J * NB;
    const bool fresh = !syrk && J == kb;
    double va[kPer], vb[kPer];
    load_tile(va, A, n, ri, o);
    if (syrk) load_tile(vb, A, n, cj, o);
    else load_tile(vb, Y, n, o, cj);
    double old[2][2][4];
    for_acc([&](int i, int j, int tt, int v, int q) {
        old[tt][v][q] = (!fresh && ri + i < n && cj + j < n) ? M[(size_t)(ri + i) * n + cj + j] : 0.0;
    });
    store_lds<true>(As, va);
    if (syrk) store_lds<true>(Bs, vb);
    else store_lds<false>(Bs, vb);
    __syncthreads();
    d4 acc[2][2] = {};
    if (syrk) tile_mma<true, true>(acc, As, Bs);
    else tile_mma<true, false>(acc, As, Bs);
    if (b != 0) {
        for_acc([&](int i, int j, int tt, int v, int q) {
            if (ri + i < n && cj + j < n && (!syrk || I != J || j <= i))
                M[(size_t)(ri + i) * n + cj + j] = old[tt][v][q] - acc[tt][v][q];
        });
        return;
    }
    __syncthreads();
    for_acc([&](int i, int j, int tt, int v, int q) {
        As[at_row(i, j)] = diag_pad(old[tt][v][q] - acc[tt][v][q], i, j, ri, n);
    });
    __syncthreads();
    potrf_tile(As, A, n, ri, flag);
}

// Ainv_IJ = sum_{K >= I} Y_KI^T Y_KJ for J <= I, and its mirror image (the
// same products in the same order); the blocks with the longest sums first,
// the next pair of tiles on its way while one is multiplied
__global__ __launch_bounds__(kBlock) void k_yty(const double* Y, double* Ainv, int n, int nt) {
    __shared__ double As[kTile], Bs[kTile];
    int I, J;
    tri_index((int)blockIdx.x, I, J);
    const int ri = I * NB, cj = J * NB;
    d4 acc[2][2] = {};
    double va[kPer], vb[kPer];
    load_tile(va, Y, n, ri, ri);
    load_tile(vb, Y, n, ri, cj);
    for (int K = I; K < nt; ++K) {
        __syncthreads();
        store_lds<false>(As, va);
        store_lds<false>(Bs, vb);
        __syncthreads();
        if (K + 1 < nt) {
            load_tile(va, Y, n, (K + 1) * NB, ri);
            load_tile(vb, Y, n, (K + 1) * NB, cj);
        }
        tile_mma<false, false>(acc, As, Bs);
    }
    for_acc([&](int i, int j, int t, int v, int q) {
        if (ri + i < n && cj + j < n) {
            Ainv[(size_t)(ri + i) * n + cj + j] = acc[t][v][q];
            if (I != J) Ainv[(size_t)(cj + j) * n + ri + i] = acc[t][v][q];
        }
    });
}

}  // namespace

void dense_spd_inverse(int n, double* A, double* work, int* flag, hipStream_t s) {
    if (n <= 0) return;
    const int nt = ceil_div(n, NB);
    zero_async(flag, sizeof(int), s);
    // a failed factorisation goes on with unit pivots in place of the bad
    // ones (finite values, no early exit), so the inverse runs on any input
    // and the caller reads the flag once at the end
    hipLaunchKernelGGL(k_potrf_first, dim3(1), dim3(kBlock), 0, s, A, n, flag);
    for (int kb = 0; kb < nt; ++kb) {
        const int t = nt - kb - 1;
        hipLaunchKernelGGL(k_dense_solve, dim3(nt), dim3(kBlock), 0, s, A, work, n, kb);
        if (t > 0)
            hipLaunchKernelGGL(k_dense_update, dim3(t * (t + 1) / 2 + t * (kb + 1)), dim3(kBlock), 0, s, A, work, n, nt,
                               kb, flag);
    }
    hipLaunchKernelGGL(k_yty, dim3(nt * (nt + 1) / 2), dim3(kBlock), 0, s, work, A, n, nt);
    MATAMG_LAUNCH_CHECK();
}

}  // namespace matamg

// Device bodies of the solve-path kernels, shared by the one-hierarchy
// launchers (k_solve.hip) and the batched launchers that run the same work
// for many hierarchies in one launch (k_batch.hip).  Each body takes its
// block index and grid size within its own problem explicitly, so a block
// computes exactly the same thing whether it is launched alone or as one
// segment of a batch: results do not depend on what else is in the batch.
#pragma once

#include "device_util.h"
#include "kernels.h"

namespace matamg {

__host__ __device__ inline int vec_grid(int64_t n) {
    const int64_t g = (n > 0 ? n : 1) / kBlock + (((n > 0 ? n : 1) % kBlock) ? 1 : 0);
    return g < 2048 ? (int)g : 2048;
}

// ----------------------------------------------------------- streaming SpMV
enum StreamMode {
    M_PLAIN = 0,
    M_RESID = 1,
    M_ADD = 2,
    M_SMOOTH = 3,
    M_DOTPQ = 4,
    M_RESNORM = 5,
    M_SCALENORM = 6,
    M_RESTRICT = 7  // y = A x, then the first smoother step on y as right-hand side
};

template <typename T>
struct SArgs {
    const int* rowptr;
    const int* col;
    const uint16_t* col16;  // packed columns (or null): col = cbase[block] + col16
    const int* cbase;
    const T* val;
    const int* blk;
    const int* blkk;   // first entry of each block (rowptr at its first row)
    const int* ustart;       // packed blocks' distinct-column lists (or null):
    const uint16_t* uoff;    // block b's are uoff[ustart[b] .. ustart[b+1])
    const uint32_t* urun;    // or their runs (DCsr::urun; null: none)
    const int* uwin;         // or their windows (DCsr::uwin; null: none)
    const T* x;        // gathered operand
    const T* b;        // right-hand side (RESID, SMOOTH, RESNORM); SCALENORM: partial sums of x.x
    const T* yin;      // ADD: base vector; SMOOTH: iterate at the row
    const T* dinv;     // SMOOTH: inverse diagonal; SCALENORM: row scale
    T* d;              // SMOOTH: direction (in/out); RESTRICT: direction (out)
    T* y;              // output
    T* xo;             // RESTRICT: first smoother iterate
    double* y64;       // SMOOTH: FP64 output instead of y
    const double* dotvec;  // SMOOTH: fused dot partner
    T c1, c2;
    DotTarget dt;
    // row dictionaries (dk > 0: of the above, rowptr, col and val are read only for
    // groups that have none)
    int dk, nblk;
    const uint16_t* drow_of;
    const uint32_t* dinfo;
    const int* doff;
    const int* drun;
    const T* dval;
    int n;      // length of the gathered operand
    int npart;  // SCALENORM: number of partial sums in b
};

// Per-row operands of the epilogue, loaded before the row's sum is known so
// that their latency overlaps the streaming of the block's entries.
template <typename T>
struct RowOperands {
    T b, dinv, d, xin;
};

template <typename T, int MODE>
__device__ __forceinline__ RowOperands<T> row_operands(const SArgs<T>& a, int r) {
    RowOperands<T> o{};
    if constexpr (MODE == M_RESID || MODE == M_RESNORM) o.b = a.b[r];
    if constexpr (MODE == M_ADD) o.xin = a.yin[r];
    if constexpr (MODE == M_SMOOTH) {
        o.b = a.b[r];
        o.dinv = a.dinv[r];
        o.d = a.d[r];
        o.xin = a.yin[r];
    }
    if constexpr (MODE == M_DOTPQ) o.xin = a.x[r];
    if constexpr (MODE == M_SCALENORM || MODE == M_RESTRICT) o.dinv = a.dinv[r];
    return o;
}

// the factors of a row's term of the fused dot product
struct DotTerm {
    double a, b;
};

template <typename T, int MODE, bool HAS_DOT>
__device__ __forceinline__ DotTerm epilogue(const SArgs<T>& a, int r, T s, const RowOperands<T>& o) {
    DotTerm dp{0.0, 0.0};
    if constexpr (MODE == M_PLAIN) {
        a.y[r] = s;
    } else if constexpr (MODE == M_RESID) {
        a.y[r] = o.b - s;
    } else if constexpr (MODE == M_ADD) {
        a.y[r] = o.xin + s;
    } else if constexpr (MODE == M_SMOOTH) {
        T res = o.b - s;
        T dn = a.c1 * o.d + a.c2 * (o.dinv * res);
        a.d[r] = dn;
        T xn = o.xin + dn;
        if (a.y64) a.y64[r] = (double)xn;
        else a.y[r] = xn;
        if constexpr (HAS_DOT) dp = DotTerm{(double)xn, a.dotvec[r]};
    } else if constexpr (MODE == M_DOTPQ) {
        a.y[r] = s;
        dp = DotTerm{(double)o.xin, (double)s};
    } else if constexpr (MODE == M_RESNORM) {
        T v = o.b - s;
        a.y[r] = v;
        dp = DotTerm{(double)v, (double)v};
    } else if constexpr (MODE == M_SCALENORM) {
        T v = o.dinv * s;
        a.y[r] = v;
        dp = DotTerm{(double)v, (double)v};
    } else if constexpr (MODE == M_RESTRICT) {
        // the coarse right-hand side, and the first smoother step from a
        // zero iterate (the same operations as smooth_first_body)
        a.y[r] = s;
        T di = a.c2 * (o.dinv * s);
        a.d[r] = di;
        a.xo[r] = di;
    }
    return dp;
}

// The sum of partial[0..nb) is taken by kFinishThreads threads: thread t adds
// partial[t], partial[t + kFinishThreads], ... in ascending order, and the
// per-thread sums are combined by a fixed tree.  The order depends on nb only.
constexpr int kFinishThreads = 1024;
constexpr int kFinishWaves = kFinishThreads / 64;

// The same sum of at most kFinishThreads partials, by a block of kBlock
// threads, on every thread: a kernel that needs a sum of few partials takes
// it itself, in each of its blocks, instead of waiting for a launch of its
// own (3 to 4 us, of about 100 us a CG step on small systems).  sh:
// kFinishWaves doubles.
__device__ __forceinline__ double finish_block(const double* partial, int nb, double* sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < kFinishThreads / kBlock; ++j) {
        const int t = (int)threadIdx.x + j * kBlock;
        double v = 0.0;
        if (t < nb) v += partial[t];
        v = wave_sum(v);
        if (lane == 0) sh[w + j * (kBlock / 64)] = v;
    }
    __syncthreads();
    double t = sh[0];
    for (int k = 1; k < kFinishWaves; ++k) t += sh[k];
    __syncthreads();
    return t;
}

// The factor on the gathered operand: 1 / |x| in the power method, whose
// iterates are scaled where the next product reads them (a pass of its own
// over the vector and one for the sum cost the setup two launches in three).
// x.x comes as its partial sums, or as one finished sum of very many.
template <typename T, int MODE>
__device__ __forceinline__ T operand_scale(const SArgs<T>& a, void* sh) {
    if constexpr (MODE == M_SCALENORM) {
        const double nrm2 = a.npart == 1 ? *a.b : finish_block(a.b, a.npart, reinterpret_cast<double*>(sh));
        return 1.0 / sqrt(nrm2);
    } else {
        return T(1);
    }
}
template <int MODE, typename T>
__device__ __forceinline__ T operand(T x, T scale) {
    if constexpr (MODE == M_SCALENORM) return x * scale;
    else return x;
}

constexpr int kPerThread = kStreamCap / kBlock;

// LDS of one streaming block of at most CAP stored entries: the products
// (first holding the block's distinct gathered values), reduction scratch
template <typename T, int CAP = kStreamCap>
struct StreamShared {
    T prod[CAP];
    double sh[kBlock / 64];
    T shr[kBlock / 64];
};

// prod[t] = val[k0 + t] * x[col[k0 + t]] for t < cnt, with NU = ceil(cnt /
// kBlock) strides per thread: all loads first (indices past the end clamped
// to the last entry, results discarded), then the gathers, then the stores.
// PACKED: the columns come from the 16-bit col16 plus the block's base.
// packed columns, two entries per load: the block's entries from its first
// even position are read as aligned pairs (a pair of values, a pair of
// 16-bit columns), NP = ceil(pairs / kBlock) strides per thread; an entry left
// over at either end (odd start, odd length) is read alone by thread 0 or 1.
template <typename T>
struct PairOf;
template <>
struct PairOf<double> {
    typedef double type __attribute__((ext_vector_type(2)));
};
template <>
struct PairOf<float> {
    typedef float type __attribute__((ext_vector_type(2)));
};
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int stage_head(int k0, int cnt) { return cnt > 0 ? (k0 & 1) : 0; }

template <typename T, int MODE, int NP, int UQ, bool WIN>
__device__ __forceinline__ void stage_pairs(const SArgs<T>& a, int bid, int k0, int cnt, T scale, T* prod) {
    using P2 = typename PairOf<T>::type;
    // (only a matrix with no windows takes the cap of wide blocks)
    const int* win = WIN && a.uwin ? a.uwin + (size_t)bid * kWinWords : nullptr;
    const int base = win ? win[2] : a.cbase[bid];
    const int head = stage_head(k0, cnt);  // entry 0 alone when the block starts at an odd position
    const int body = cnt - head;
    const int np = body >> 1;  // whole pairs from the even position k0 + head
    const int kp = k0 + head;
    const int tid = (int)threadIdx.x;
    // the block's distinct columns (block-uniform): runs, a list, or none
    // (gathers)
    const uint32_t* rec = a.urun && !win ? a.urun + (size_t)bid * kRunWords : nullptr;
    const int nruns = rec ? (int)rec[0] : 0;
    const int u0 = a.ustart ? a.ustart[bid] : 0;
    const int nu = win ? win[0] : nruns > 0 ? (int)rec[1] : (a.ustart ? a.ustart[bid + 1] - u0 : 0);
    u16x2 c[NP > 0 ? NP : 1];
    P2 v[NP > 0 ? NP : 1];
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int p = tid + u * kBlock;
        const int pc = p < np ? p : np - 1;
        c[u] = __builtin_nontemporal_load(reinterpret_cast<const u16x2*>(a.col16 + kp + 2 * pc));
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const P2*>(a.val + kp + 2 * pc));
    }
    // the single entries: the head (thread 0) and, for an odd body, the tail (thread 1)
    int ts = -1;
    if (tid == 0 && head) ts = 0;
    if (tid == 1 && (body & 1)) ts = cnt - 1;
    int cs = 0;
    T vs = 0;
    if (ts >= 0) {
        cs = (int)a.col16[k0 + ts];
        vs = a.val[k0 + ts];
    }
    T x0[NP > 0 ? NP : 1], x1[NP > 0 ? NP : 1];
    T xsng = T(0);
    if (UQ > 0 && nu > 0) {
        // the block's distinct values of the gathered vector, read in
        // ascending column order (coalesced along the list), staged in the
        // product array (nu <= unique_cap(CAP) <= CAP entries); the entries'
        // col16 index the list.  Every thread takes its values into
        // registers before the products overwrite the array.
        T* xs = prod;
        int off[UQ > 0 ? UQ : 1];
        if (nruns > 0) {
            // list index j lies in the run whose prefix of lengths it reaches
            uint32_t rw[kMaxRuns];
#pragma unroll
            for (int r = 0; r < kMaxRuns; ++r) rw[r] = rec[2 + r];
#pragma unroll
            for (int q = 0; q < UQ; ++q) {
                const int j0 = tid + q * kBlock;
                const int j = j0 < nu ? j0 : nu - 1;
                int pos = (int)(rw[0] & 0xffffu) + j, pre = 0;
#pragma unroll
                for (int r = 0; r < kMaxRuns - 1; ++r) {
                    pre += (int)(rw[r] >> 16);
                    if (r + 1 < nruns && j >= pre) pos = (int)(rw[r + 1] & 0xffffu) + (j - pre);
                }
                off[q] = pos;
            }
        } else {
#pragma unroll
            for (int q = 0; q < UQ; ++q) {
                const int j = tid + q * kBlock;
                off[q] = (int)a.uoff[u0 + (j < nu ? j : nu - 1)];
            }
            if (win && win[1] > 1) {
                // several windows: each list index takes its own one's base
#pragma unroll
                for (int q = 0; q < UQ; ++q) {
                    const int j = min(tid + q * kBlock, nu - 1);
                    int b = base;
#pragma unroll
                    for (int w = 1; w < kMaxWin; ++w)
                        if (w < win[1] && j >= win[1 + 2 * w]) b = win[2 + 2 * w];
                    off[q] += b - base;
                }
            }
        }
        T xv[UQ > 0 ? UQ : 1];
#pragma unroll
        for (int q = 0; q < UQ; ++q) xv[q] = a.x[base + off[q]];
#pragma unroll
        for (int q = 0; q < UQ; ++q) {
            const int j = tid + q * kBlock;
            if (j < nu) xs[j] = operand<MODE>(xv[q], scale);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            x0[u] = xs[(int)c[u].x];
            x1[u] = xs[(int)c[u].y];
        }
        if (ts >= 0) xsng = xs[cs];
        __syncthreads();
    } else {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            x0[u] = operand<MODE>(a.x[base + (int)c[u].x], scale);
            x1[u] = operand<MODE>(a.x[base + (int)c[u].y], scale);
        }
        if (ts >= 0) xsng = operand<MODE>(a.x[base + cs], scale);
    }
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int p = tid + u * kBlock;
        if (p < np) {
            prod[head + 2 * p] = v[u].x * x0[u];
            prod[head + 2 * p + 1] = v[u].y * x1[u];
        }
    }
    if (ts >= 0) prod[ts] = vs * xsng;
}

template <typename T, int MODE, int NU>
__device__ __forceinline__ void stage_products(const SArgs<T>& a, int k0, int cnt, T scale, T* prod) {
    int c[NU];
    T v[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int t = (int)threadIdx.x + u * kBlock;
        const int tc = t < cnt ? t : cnt - 1;
        c[u] = __builtin_nontemporal_load(a.col + k0 + tc);
        v[u] = __builtin_nontemporal_load(a.val + k0 + tc);
    }
    T xv[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u) xv[u] = operand<MODE>(a.x[c[u]], scale);
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        const int t = (int)threadIdx.x + u * kBlock;
        if (t < cnt) prod[t] = v[u] * xv[u];
    }
}

// s + prod[k0] + prod[k0 + step] + ... (k < k1), added one at a time in
// that order; the LDS reads go out eight at a time so that their latencies
// overlap (the additions, and so the result, are those of the plain loop)
template <typename T, int STEP>
__device__ __forceinline__ T ordered_sum(const T* prod, int k0, int k1, T s) {
    int k = k0;
    for (; k + 7 * STEP < k1; k += 8 * STEP) {
        T p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = prod[k + u * STEP];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += p[u];
    }
    for (; k < k1; k += STEP) s += prod[k];
    return s;
}

// Row block `bid` of the matrix in `a`: stream its val/col range into LDS
// products, reduce each row with G threads (or the whole block for a long
// row), apply the epilogue, and store the block's dot partial (its
// wavefront sums in wavefront order) at a.dt.partial[bid].
//
// Every load of the streaming phase is unconditional: indices past the
// block's end are clamped to its last entry (or row) and the results are
// discarded, so the compiler issues all of them back to back with no
// branch, and no wait, between them.
template <typename T, int MODE, bool HAS_DOT, int G, int CAP = kStreamCap>
__device__ __forceinline__ void stream_block(const SArgs<T>& a, int bid, StreamShared<T, CAP>& S) {
    // rows and entries of the block from the two tables: the loads of the
    // entries do not wait for the row pointer
    const int r0 = a.blk[bid], r1 = a.blk[bid + 1];
    const int k0 = a.blkk[bid], k1 = a.blkk[bid + 1];
    const int cnt = k1 - k0;
    const T scale = operand_scale<T, MODE>(a, S.prod);
    double dp = 0.0;
    if (!(r1 - r0 == 1 && cnt > long_row_limit(G))) {
        // one thread per row: every thread prefetches its row's bounds and
        // operands.  With G > 1 a group has rows_per_group(G) rows, kBlock / G
        // apart, and its thread q those of the q-th, so that none of these
        // loads waits behind the reduction and the epilogues are one pass of
        // the group (by its first thread alone, with all four rows' operands
        // in 98 registers, they are four: FP64 smoother of the 192^3 stack's
        // levels 2 to 4 226, 165 and 81 us against 204, 148 and 72 us, of the
        // 96^3 cube's level 2 22 against 19 us)
        constexpr int RQ = G == 1 ? 1 : rows_per_group(G);
        const int gl = (int)threadIdx.x % G;
        const int r = r0 + (int)threadIdx.x / G + (gl % RQ) * (kBlock / G);
        const bool owner = r < r1 && gl < RQ;
        const int rc = r < r1 ? r : r1 - 1;
        const int e0 = a.rowptr[rc], e1 = a.rowptr[rc + 1];
        RowOperands<T> ops{};
        if (gl < RQ) ops = row_operands<T, MODE>(a, rc);

        // ceil(cnt / kBlock) strides of the block's entries (block-uniform),
        // from packed or plain columns (uniform per matrix)
        const int nu = (cnt + kBlock - 1) / kBlock;
        constexpr int kUQ = unique_cap(CAP) / kBlock;  // distinct values per thread
        constexpr bool kWin = CAP == kStreamCap;
        const bool packed = a.col16 && !(kWin && a.uwin && a.uwin[(size_t)bid * kWinWords + 1] == 0);
        if (packed) {
            // pairs of entries: ceil(pairs / kBlock) strides (block-uniform)
            switch (((cnt - stage_head(k0, cnt)) / 2 + kBlock - 1) / kBlock) {
                case 0: stage_pairs<T, MODE, 0, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                case 1: stage_pairs<T, MODE, 1, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                case 2: stage_pairs<T, MODE, 2, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                case 3: stage_pairs<T, MODE, 3, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                case 4: stage_pairs<T, MODE, 4, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                default:
                    if constexpr (CAP > kStreamCap) {
                        switch (((cnt - stage_head(k0, cnt)) / 2 + kBlock - 1) / kBlock) {
                            case 5: stage_pairs<T, MODE, 5, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                            case 6: stage_pairs<T, MODE, 6, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                            case 7: stage_pairs<T, MODE, 7, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                            case 8: stage_pairs<T, MODE, 8, kUQ, kWin>(a, bid, k0, cnt, scale, S.prod); break;
                            default: break;
                        }
                    }
                    break;
            }
        } else if constexpr (CAP == kStreamCap) {
            // (wide blocks are only made for packed matrices)
            switch (nu) {
                case 1: stage_products<T, MODE, 1>(a, k0, cnt, scale, S.prod); break;
                case 2: stage_products<T, MODE, 2>(a, k0, cnt, scale, S.prod); break;
                case 3: stage_products<T, MODE, 3>(a, k0, cnt, scale, S.prod); break;
                case 4: stage_products<T, MODE, 4>(a, k0, cnt, scale, S.prod); break;
                case 5: stage_products<T, MODE, 5>(a, k0, cnt, scale, S.prod); break;
                case 6: stage_products<T, MODE, 6>(a, k0, cnt, scale, S.prod); break;
                case 7: stage_products<T, MODE, 7>(a, k0, cnt, scale, S.prod); break;
                case 8: stage_products<T, MODE, 8>(a, k0, cnt, scale, S.prod); break;
                default: break;
            }
        }
        __syncthreads();
        if constexpr (G == 1) {
            // a row up to kWideRow wide is summed by its own thread; the
            // wider rows of a wavefront (at most long_row_limit(1) wide) by
            // 8-lane groups of it, eight rows at a time: lane-strided
            // partial sums, then a butterfly that leaves the same bits in
            // the group's eight lanes
            const bool wide = owner && (e1 - e0) > kWideRow;
            T s = 0;
            if (owner && !wide) s = ordered_sum<T, 1>(S.prod, e0 - k0, e1 - k0, s);
            const int lane = (int)threadIdx.x & 63, grp = lane >> 3, gl = lane & 7;
            unsigned long long wm = __ballot(wide);
            // rank of this lane's row among the wide rows of the wavefront
            const int rank = __popcll(wm & ((1ull << lane) - 1ull));
            for (int base = 0; wm; base += 8) {
                unsigned long long m = wm;
                for (int j = 0; j < grp; ++j) m &= m - 1ull;  // the grp-th remaining wide row
                const int l = m ? __builtin_ctzll(m) : 0;
                const int f0 = __shfl(e0, l, 64) - k0, f1 = __shfl(e1, l, 64) - k0;
                T ps = 0;
                if (m) ps = ordered_sum<T, 8>(S.prod, f0 + gl, f1, ps);
                for (int off = 4; off > 0; off >>= 1) ps += __shfl_xor(ps, off, 64);
                const int src = (rank >= base && rank < base + 8) ? (rank - base) * 8 : 0;
                const T got = __shfl(ps, src, 64);
                if (wide && rank >= base && rank < base + 8) s = got;
                for (int j = 0; j < 8; ++j) wm &= wm - 1ull;
            }
            if (owner) {
                const DotTerm t = epilogue<T, MODE, HAS_DOT>(a, r, s, ops);
                dp = t.a * t.b;
            }
        } else {
            // G threads per row: strided partial sums, then a fixed shuffle
            // tree (on every thread the same bits), row after row; the row's
            // own thread takes its sum
            T s = 0;
#pragma unroll
            for (int q = 0; q < RQ; ++q) {
                const int f0 = __shfl(e0, q, G) - k0, f1 = __shfl(e1, q, G) - k0;
                T t = 0;
                if (r0 + (int)threadIdx.x / G + q * (kBlock / G) < r1) t = ordered_sum<T, G>(S.prod, f0 + gl, f1, t);
                for (int off = G / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, G);
                if (gl == q) s = t;
            }
            DotTerm e{0.0, 0.0};
            if (owner) e = epilogue<T, MODE, HAS_DOT>(a, r, s, ops);
            if constexpr (HAS_DOT) {
                // the group's terms in row order, each product and addition
                // rounded once, on its first thread
#pragma unroll
                for (int q = 0; q < RQ; ++q) {
                    const double ta = __shfl(e.a, q, G), tb = __shfl(e.b, q, G);
                    if (gl == 0 && r + q * (kBlock / G) < r1) dp = __builtin_fma(ta, tb, dp);
                }
            }
        }
    } else {
        // one long row (a block of its own): strided partial sums, fixed
        // tree.  Each thread adds its entries t, t + kBlock, ... in order;
        // four strides at a time have their loads, then their gathers, in
        // flight together.  A long row's block is never staged, so packed
        // columns hold plain offsets from the block's base.
        T s = 0;
        const int* col = a.col16 && !a.uwin ? nullptr : a.col;
        const int base = col ? 0 : a.cbase[bid];
        int t = (int)threadIdx.x;
        for (; t + 3 * kBlock < cnt; t += 4 * kBlock) {
            int c[4];
            T v[4], xv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + t + u * kBlock;
                c[u] = col ? col[k] : base + (int)a.col16[k];
                v[u] = a.val[k];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) xv[u] = operand<MODE>(a.x[c[u]], scale);
#pragma unroll
            for (int u = 0; u < 4; ++u) s += v[u] * xv[u];
        }
        for (; t < cnt; t += kBlock) {
            const int k = k0 + t;
            s += a.val[k] * operand<MODE>(a.x[col ? col[k] : base + (int)a.col16[k]], scale);
        }
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
        if (lane == 0) S.shr[w] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            T t = S.shr[0];
            for (int i = 1; i < kBlock / 64; ++i) t += S.shr[i];
            const DotTerm p = epilogue<T, MODE, HAS_DOT>(a, r0, t, row_operands<T, MODE>(a, r0));
            dp = p.a * p.b;
        }
    }
    if constexpr (HAS_DOT) {
        // the block's partial: wavefront sums added in wavefront order
        const double t = wave_sum(dp);
        if ((threadIdx.x & 63) == 0) S.sh[threadIdx.x >> 6] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            double u = S.sh[0];
            for (int w = 1; w < kBlock / 64; ++w) u += S.sh[w];
            a.dt.partial[bid] = u;
        }
    }
}

// ---------------------------------------------------------- row dictionaries
// LDS of one group, for the largest of a launch: dictionary values, offsets
// and row records, the gathered operands' windows, and (dot modes) one term
// per row
struct RowsSize {
    int max_e = 0, max_n = 0, max_x = 0, dots = 0;
};
struct RowsLds {
    int vals, xs, offs, info, bytes;  // byte offsets (the row terms come first), total
};
template <typename T>
__host__ __device__ inline RowsLds rows_lds(const RowsSize& z) {
    RowsLds l;
    l.vals = 8 * z.dots;
    l.xs = l.vals + (int)sizeof(T) * z.max_e;
    l.offs = l.xs + (int)sizeof(T) * z.max_x;
    l.info = l.offs + 4 * z.max_e;
    l.bytes = l.info + 4 * z.max_n;
    return l;
}
// Adds lv[k] x(k) to s over the entries k, k + 1, ... of a row in stored
// order, C at a time while they last: their operands are loaded together, and
// each product is rounded before it is added, as the streaming kernel does.
template <int C, typename T, class X>
__device__ __forceinline__ void row_chunk(T& s, const T* lv, int& k, int end, X x) {
#pragma clang fp contract(off)
    for (; k + C <= end; k += C) {
        T xv[C];
#pragma unroll
        for (int u = 0; u < C; ++u) xv[u] = x(k + u);
#pragma unroll
        for (int u = 0; u < C; ++u) {
            const T p = lv[k + u] * xv[u];
            s = s + p;
        }
    }
}
// nine at a time: a third of a 27-point row, all of a 9-point one (more keep
// fewer wavefronts on a CU: the FP64 fine smoother of the 128^3 stack took
// 41.5 us with 9, 42.9 with 14 and 51.6 with 27)
template <typename T, class X>
__device__ __forceinline__ T row_sum(const T* lv, int k0, int len, X x) {
    T s = 0;
    int k = k0;
    row_chunk<9>(s, lv, k, k0 + len, x);
    row_chunk<3>(s, lv, k, k0 + len, x);
    row_chunk<1>(s, lv, k, k0 + len, x);
    return s;
}

// the dot terms of row blocks [b0, b1) of a group from row r0 on, in the streaming
// kernel's order
template <typename T>
__device__ __forceinline__ void rows_dots(const SArgs<T>& a, int b0, int b1, int r0, const double* ld) {
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int b = b0 + (int)(threadIdx.x >> 6); b < b1; b += kBlock / 64) {
        const int f = a.blk[b], n = a.blk[b + 1] - f;
        double u = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) {
            const int i = 64 * w + lane;
            const double t = wave_sum(i < n ? ld[f - r0 + i] : 0.0);
            u = w == 0 ? t : u + t;
        }
        if (lane == 0) a.dt.partial[b] = u;
    }
}

// The rows of a group without a dictionary, one thread a row in the streaming
// kernel's order of additions: only launches that were recorded before an update come
// here (product of the 128^3 stack 31 us with dictionaries, 319 us here, launched
// anew 104 us).  A thread's loads wait for one another, six entries at a time: as
// many as leave the registers at what the groups with dictionaries need (one at a
// time 1823 us; nine cost those a sixth of their wavefronts).
template <typename T, int MODE, bool HAS_DOT>
__device__ __forceinline__ void rows_plain(const SArgs<T>& a, int b0, int b1, T scale, double* ld) {
    const int r0 = a.blk[b0], r1 = a.blk[b1];
    __syncthreads();  // (every thread has read the scale's sums)
    for (int r = r0 + (int)threadIdx.x; r < r1; r += kBlock) {
        const RowOperands<T> o = row_operands<T, MODE>(a, r);
        T s = 0;
        int k = a.rowptr[r];
        const int end = a.rowptr[r + 1];
        auto x = [&](int e) { return operand<MODE>(a.x[a.col[e]], scale); };
        row_chunk<6>(s, a.val, k, end, x);
        row_chunk<3>(s, a.val, k, end, x);
        row_chunk<1>(s, a.val, k, end, x);
        const DotTerm dp = epilogue<T, MODE, HAS_DOT>(a, r, s, o);
        if constexpr (HAS_DOT) ld[r - r0] = dp.a * dp.b;
    }
    if constexpr (HAS_DOT) rows_dots(a, b0, b1, r0, ld);
}

// Rows of group `g` (dk row blocks) from its dictionary in LDS, one thread
// per row.  With max_x the operands come from LDS too: the rows of a group
// gather from a few windows of consecutive columns (three planes of a mesh,
// say), read once.  A row block's dot terms are summed in the streaming
// kernel's order (its rows over four wavefronts, each by the wavefront tree,
// the four sums in order).  What bounds it where it gathers is the cache path: the
// texture address units are busy 83% of the time (FP64, 96^3 cube) and 75% (FP32,
// 128^3 stack).  Staged, no unit is (128^3 stack: vector units 51%, address units
// 50%, LDS 44%, HBM at half the rate of a plain read): a workgroup's steps -- the
// windows, the barrier, the sums -- follow one another, and a CU's LDS has room
// for six workgroups to fill the gaps.  The FP64 fine smoother of the 128^3 stack
// takes 33 us for the 103 MB of its vectors (staged; 41 us gathering), against 116
// us from values and columns, that of the 96^3 cube 24 us (gathering) against 52
// us, and the FP32 ones 19 and 15 us against 72 and 30 us.
template <typename T, int MODE, bool HAS_DOT>
__device__ __forceinline__ void rows_group(const SArgs<T>& a, int g, const RowsSize& z, char* lds) {
    const RowsLds at = rows_lds<T>(z);
    T* lv = reinterpret_cast<T*>(lds + at.vals);
    T* xs = reinterpret_cast<T*>(lds + at.xs);
    int* lo = reinterpret_cast<int*>(lds + at.offs);
    uint32_t* li = reinterpret_cast<uint32_t*>(lds + at.info);
    double* ld = reinterpret_cast<double*>(lds);
    const int b0 = g * a.dk, b1 = min(b0 + a.dk, a.nblk);
    const int r0 = a.blk[b0], r1 = a.blk[b1];
    const int* rec = a.drun + (size_t)g * kDictRunWords;
    const int m0 = rec[0], m1 = rec[kDictRunWords], e0 = rec[1], e1 = rec[kDictRunWords + 1];
    const int* run = rec + 2;
    const int total = run[1];
    const int nrun = total <= z.max_x ? run[0] : 0;
    const T scale = operand_scale<T, MODE>(a, lds);
    const int first = r0 + (int)threadIdx.x;
    // the first row's record number and operands travel with the dictionary
    int id = 0;
    RowOperands<T> o{};
    if (first < r1) {
        id = a.drow_of[first];
        o = row_operands<T, MODE>(a, first);
    }
    // a launch recorded before an update may find none, or more than it has room for
    if (m1 <= m0 || m1 - m0 > z.max_n || e1 - e0 > z.max_e) {
        rows_plain<T, MODE, HAS_DOT>(a, b0, b1, scale, ld);
        return;
    }
    if (nrun > 0) {
        // window j covers the columns first[j] on, at the places end[j - 1] on
        int shift[kDictRuns], end[kDictRuns];  // column less place
        int pre = 0;
#pragma unroll
        for (int j = 0; j < kDictRuns; ++j) {
            const bool in = j < nrun;
            shift[j] = in ? r0 + run[2 + 2 * j] - pre : 0;
            pre += in ? run[3 + 2 * j] : 0;
            end[j] = pre;
        }
        for (int i = threadIdx.x; i < total; i += kBlock) {
            int c = shift[0];
#pragma unroll
            for (int j = 1; j < kDictRuns; ++j)
                if (j < nrun && i >= end[j - 1]) c = shift[j];
            c += i;
            xs[i] = operand<MODE>(a.x[min(max(c, 0), a.n - 1)], scale);  // (columns outside the matrix are in no entry)
        }
        // an entry's operand for row r0 + i is at place lo + i
        for (int e = threadIdx.x; e < e1 - e0; e += kBlock) {
            const int d = a.doff[e0 + e];
            int c = shift[0];
#pragma unroll
            for (int j = 1; j < kDictRuns; ++j)
                if (j < nrun && d >= run[2 + 2 * j]) c = shift[j];
            lv[e] = a.dval[e0 + e];
            lo[e] = r0 + d - c;
        }
    } else {
        for (int e = threadIdx.x; e < e1 - e0; e += kBlock) {
            lv[e] = a.dval[e0 + e];
            lo[e] = a.doff[e0 + e];
        }
    }
    for (int m = threadIdx.x; m < m1 - m0; m += kBlock) li[m] = a.dinfo[m0 + m];
    __syncthreads();
    for (int r = first; r < r1; r += kBlock) {
        if (r != first) {
            id = a.drow_of[r];
            o = row_operands<T, MODE>(a, r);
        }
        const uint32_t w = li[id];
        const int k0 = (int)(w & 0xffffu), len = (int)(w >> 16);
        T s;
        if (nrun > 0) {
            const T* x = xs + (r - r0);
            s = row_sum<T>(lv, k0, len, [&](int k) { return x[lo[k]]; });
        } else {
            const T* x = a.x + r;
            s = row_sum<T>(lv, k0, len, [&](int k) { return operand<MODE>(x[lo[k]], scale); });
        }
        const DotTerm dp = epilogue<T, MODE, HAS_DOT>(a, r, s, o);
        if constexpr (HAS_DOT) ld[r - r0] = dp.a * dp.b;
    }
    if constexpr (HAS_DOT) rows_dots(a, b0, b1, r0, ld);
}

// The sizes of M's groups for a launch in precision T over `rows` rows of
// `entries` entries in all.  The windows are staged for FP64 operands where six
// workgroups' LDS fits a CU: FP32 gathers (half the bytes) and groups with large
// dictionaries lose more by the lower occupancy and the barrier (FP32 fine
// smoother of the 128^3 stack 25 us staged, 20 us gathering; FP64 of the 96^3 cube
// 28 us and 25 us).  Staging is one more step of a workgroup's chain, which pays
// where there are many gathers to spare: not in launches whose workgroups are all
// resident at once, nor for short rows, at any number of them.  FP64 smoothers
// gathering and staged, us:
//   27 entries a row: 27 thousand rows 4.0, 4.4; 74 thousand 4.6, 4.9; 97 thousand
//     5.5, 5.4; 262 thousand 8.6, 7.6; 2.1 million 40, 33
//   19 and 21: 125 thousand rows 5.2, 5.4 and 5.1, 5.0; 262 thousand 7.3, 6.9 and
//     7.4, 6.9; 2.1 million 34, 31 and 34, 32
//   13 and 15: 262 thousand 5.9, 6.5 and 7.1, 7.5; 531 thousand (15) 9.7, 9.1;
//     1 million equal
//   7 and 9: 262 thousand 4.4, 5.5 and 5.3, 5.5; 490 thousand (9) 7.7, 7.6; 1 million
//     (9) 13.2, 13.7; 4.2 million (9) 34, 38
constexpr int kRowsStageLds = 160 * 1024 / 6;
constexpr int64_t kRowsStageEntries = 2500000;
constexpr int kRowsStageWidth = 16;
template <typename T>
inline RowsSize rows_size(int max_e, int max_n, int max_x, int dots, int64_t rows, int64_t entries) {
    RowsSize z{max_e, max_n, max_x, dots};
    if (sizeof(T) == 4 || entries < kRowsStageEntries || entries < kRowsStageWidth * rows ||
        rows_lds<T>(RowsSize{max_e, max_n, max_x, 0}).bytes > kRowsStageLds)
        z.max_x = 0;
    return z;
}

// the dictionary of M as the arguments of a streaming launch, if M has one in
// this precision
template <typename T>
inline void dict_args(const DCsr& M, const T* dval, SArgs<T>& a) {
    if (M.dk <= 0 || !dval) return;
    a.dk = M.dk;
    a.nblk = M.nblk;
    a.n = M.m;
    a.drow_of = M.drow_of.get();
    a.dinfo = M.dinfo.get();
    a.doff = M.doff.get();
    a.drun = M.drun.get();
    a.dval = dval;
}
inline void dict_args(const DCsr& M, SArgs<double>& a) { dict_args<double>(M, M.dval.get(), a); }
inline void dict_args(const DCsr& M, SArgs<float>& a) { dict_args<float>(M, M.dval32.get(), a); }

// ------------------------------------------------------------ vector bodies
// Grid-stride loops over one problem's vectors: block `lb` of `grid`.

template <typename T>
struct SmoothFirstArgs {
    int64_t n;
    const double* b64;  // if set: b = (T) b64 is stored first
    T* b;
    const T* dinv;
    T c2;
    T* d;
    T* x;
};

template <typename T>
__device__ __forceinline__ void smooth_first_body(const SmoothFirstArgs<T>& a, int lb, int grid) {
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < a.n; i += (int64_t)grid * kBlock) {
        T bi;
        if (a.b64) {
            bi = (T)a.b64[i];
            a.b[i] = bi;
        } else {
            bi = a.b[i];
        }
        T di = a.c2 * (a.dinv[i] * bi);
        a.d[i] = di;
        a.x[i] = di;
    }
}

struct CgDirArgs {
    int64_t n;
    double* p;
    const double* z;
    double* rz_new;
    const double* rz_old;  // null: p = z
    const double* part;    // if set: rz_new is the sum of part[0..npart), stored here
    int npart;
};

__device__ __forceinline__ void cg_direction_body(const CgDirArgs& a, int lb, int grid, double* sh) {
    double rz = 0.0;
    if (a.part) {
        rz = finish_block(a.part, a.npart, sh);
        if (lb == 0 && threadIdx.x == 0) *a.rz_new = rz;
    } else if (a.rz_old) {
        rz = *a.rz_new;
    }
    const double beta = a.rz_old ? (rz / *a.rz_old) : 0.0;
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < a.n; i += (int64_t)grid * kBlock)
        a.p[i] = a.rz_old ? a.z[i] + beta * a.p[i] : a.z[i];
}

struct CgUpdArgs {
    int64_t n;
    double* x;
    double* r;
    const double* p;
    const double* q;
    const double* rz;
    double* pq;
    double* partial;     // r.r partial of block lb at partial[lb]
    const double* part;  // if set: pq is the sum of part[0..npart), stored here
    int npart;
};

// x += alpha p, r -= alpha q, and the block's part of r.r; with `first` also
// the next V-cycle's first smoother step from the new r (the operations of
// smooth_first_body)
template <typename T>
__device__ __forceinline__ void cg_update_body(const CgUpdArgs& a, const SmoothFirstArgs<T>* first, int lb, int grid,
                                               double* sh) {
    // a non-positive or non-finite curvature is a breakdown: leave x and r
    // unchanged so the caller keeps the last iterate
    double pqv;
    if (a.part) {
        pqv = finish_block(a.part, a.npart, sh);
        if (lb == 0 && threadIdx.x == 0) *a.pq = pqv;
    } else {
        pqv = *a.pq;
    }
    const double rzv = *a.rz;
    const double alpha = (pqv > 0.0 && isfinite(pqv) && isfinite(rzv)) ? rzv / pqv : 0.0;
    double v = 0.0;
    for (int64_t i = (int64_t)lb * kBlock + threadIdx.x; i < a.n; i += (int64_t)grid * kBlock) {
        a.x[i] = a.x[i] + alpha * a.p[i];
        double ri = a.r[i] - alpha * a.q[i];
        a.r[i] = ri;
        v += ri * ri;
        if (first) {
            const T bi = (T)ri;
            if (first->b64) first->b[i] = bi;
            const T di = first->c2 * (first->dinv[i] * bi);
            first->d[i] = di;
            first->x[i] = di;
        }
    }
    double t = block_sum(v, sh);
    if (threadIdx.x == 0) a.partial[lb] = t;
}

struct FinishArgs {
    int nb;
    const double* partial;
    double* result;
};

__device__ __forceinline__ void finish_body(const FinishArgs& a, double* sh /* kFinishThreads / 64 */) {
    constexpr int T = kFinishThreads;
    double v = 0.0;
    int i = threadIdx.x;
    for (; i + 3 * T < a.nb; i += 4 * T) {
        const double p0 = a.partial[i], p1 = a.partial[i + T], p2 = a.partial[i + 2 * T], p3 = a.partial[i + 3 * T];
        v += p0;
        v += p1;
        v += p2;
        v += p3;
    }
    for (; i < a.nb; i += T) v += a.partial[i];
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = sh[0];
        for (int k = 1; k < T / 64; ++k) t += sh[k];
        *a.result = t;
    }
}

// ------------------------------------------------------------- dense GEMV
// out = M in, one wavefront per row of the row-major n x n FP64 matrix
template <typename T>
struct GemvArgs {
    int n;
    const double* M;
    const T* in;
    T* out;
};

template <typename T>
__device__ __forceinline__ void gemv_body(const GemvArgs<T>& a, int lb) {
    const int lane = threadIdx.x & 63;
    const int row = lb * (kBlock / 64) + (threadIdx.x >> 6);
    if (row >= a.n) return;
    const double* m = a.M + (size_t)row * a.n;
    const int n = a.n;
    // lane-strided sum (columns lane, lane + 64, ... in order) over chunks of
    // sixteen columns per lane; the next chunk's loads are issued before the
    // current chunk is summed, so a row costs about one memory latency
    // instead of one per chunk.  Indices past the row's end are clamped to
    // its last column and their products skipped.
    constexpr int U = 16;
    double mv[U], iv[U];
    auto load = [&](int j0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(j0 + u * 64, n - 1);
            mv[u] = m[j];
            iv[u] = (double)a.in[j];
        }
    };
    double s = 0.0;
    load(lane);
    for (int j0 = lane; j0 < n; j0 += U * 64) {
        double cm[U], ci[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cm[u] = mv[u];
            ci[u] = iv[u];
        }
        if (j0 + U * 64 < n) load(j0 + U * 64);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u * 64 < n) s += cm[u] * ci[u];
    }
    s = wave_sum(s);
    if (lane == 0) a.out[row] = (T)s;
}

inline int gemv_grid(int n) { return ceil_div(n, kBlock / 64); }

}  // namespace matamg

// The bottom of the V-cycle in one workgroup: the levels whose operators and
// vectors fit in the LDS of one CU together, and the dense coarsest solve.
//
// A level of a few hundred rows is seven launches of 3.5 to 5 us each, all of
// it launch and memory latency.  Here the levels' operators, inverse diagonals
// and row pointers come from one image laid out at the setup (and after an
// update), copied to LDS with every load in flight, and their vectors stay
// there.  The transfers' entries, read once a cycle, and the dense inverse come
// from memory.  Every row's sum and epilogue are those of the streaming kernels,
// in their order.
#include <algorithm>

#include "hierarchy.h"
#include "solve_device.h"

namespace matamg {
namespace {

// val * x over a row in the streaming kernels' order: serially, or for a wide
// row eight strided partial sums and their tree.  Eight entries at a time, all
// of them read (past the end the last one, whose product is left out), so that
// the reads of a chunk are two LDS latencies.
template <typename T, typename C>
__device__ __forceinline__ T tail_row(const T* val, const C* col, int k0, int k1, const T* x) {
#pragma clang fp contract(off)
    T s = 0, ps[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ps[u] = 0;
    const bool wide = k1 - k0 > kWideRow;
    for (int k = k0; k < k1; k += 8) {
        T v[8], xv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int p = min(k + u, k1 - 1);
            v[u] = val[p];
            xv[u] = x[(int)col[p]];
        }
        if (wide) {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const T p = v[u] * xv[u];
                ps[u] = k + u < k1 ? ps[u] + p : ps[u];
            }
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const T p = v[u] * xv[u];
                s = k + u < k1 ? s + p : s;
            }
        }
    }
    return wide ? ((ps[0] + ps[4]) + (ps[2] + ps[6])) + ((ps[1] + ps[5]) + (ps[3] + ps[7])) : s;
}

template <typename T>
__global__ __launch_bounds__(kTailThreads) void k_tail(const uint4* image, int words, int n0, const T* b0,
                                                       const T* d0, const T* x0, T* out) {
    extern __shared__ char lds[];
    const int tid = threadIdx.x;
    auto vec = [&](int at) { return reinterpret_cast<T*>(lds + at); };
    // the image (the description of the levels in front) and behind it the
    // first level's vectors, every load in flight
    {
        T* first = reinterpret_cast<T*>(lds + 16 * words);
        const int stride = ((int)sizeof(T) * n0 + 15) / 16 * 16 / (int)sizeof(T);
        const int r0 = min(tid, n0 - 1);
        const T b = b0[r0], d = d0[r0], x = x0[r0];
        constexpr int kPer = (kTailLds / 16 + kTailThreads - 1) / kTailThreads;
        uint4 v[kPer];
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            v[u] = image[min(tid + u * kTailThreads, words - 1)];
#pragma unroll
        for (int u = 0; u < kPer; ++u)
            if (tid + u * kTailThreads < words) reinterpret_cast<uint4*>(lds)[tid + u * kTailThreads] = v[u];
        for (int r = tid; r < n0; r += kTailThreads) {
            first[r] = r == tid ? b : b0[r];
            first[r + stride] = r == tid ? d : d0[r];
            first[r + 2 * stride] = r == tid ? x : x0[r];
        }
    }
    __syncthreads();
    const TailHead<T>& a = *reinterpret_cast<const TailHead<T>*>(lds);
    // row r of a level's operator times x
    auto row = [&](const TailLevel<T>& L, int r, const T* x) {
        const uint16_t* col = reinterpret_cast<const uint16_t*>(lds + L.col);
        const uint16_t* rp = reinterpret_cast<const uint16_t*>(lds + L.rp);
        return tail_row(vec(L.val), col, (int)rp[r], (int)rp[r + 1], x);
    };
    // one smoother step x -> y (the epilogue of M_SMOOTH)
    auto smooth = [&](const TailLevel<T>& L, const T* x, T* y, T c1, T c2) {
        const T *b = vec(L.b), *dinv = vec(L.dinv);
        T* d = vec(L.d);
        for (int r = tid; r < L.n; r += kTailThreads) {
            const T s = row(L, r, x);
            T res = b[r] - s;
            T dn = c1 * d[r] + c2 * (dinv[r] * res);
            d[r] = dn;
            T xn = x[r] + dn;
            y[r] = xn;
        }
        __syncthreads();
    };
    unsigned swapped = 0;  // bit l: level l's iterate is in its second buffer
    for (int l = 0; l < a.levels; ++l) {
        const TailLevel<T>& L = a.lv[l];
        int x = L.x, y = L.y;
        for (int k = 1; k < L.steps; ++k) {
            smooth(L, vec(x), vec(y), L.c1[k], L.c2[k]);
            const int t = x;
            x = y;
            y = t;
        }
        if (x != L.x) swapped |= 1u << l;
        T* res = vec(y);
        {
            const T *b = vec(L.b), *xs = vec(x);
            for (int r = tid; r < L.n; r += kTailThreads) res[r] = b[r] - row(L, r, xs);
        }
        __syncthreads();
        const uint16_t* rp = reinterpret_cast<const uint16_t*>(lds + L.rrp);
        if (l + 1 < a.levels) {
            // with the next level's first step (the epilogue of M_RESTRICT)
            const TailLevel<T>& N = a.lv[l + 1];
            T *b = vec(N.b), *d = vec(N.d), *xs = vec(N.x);
            const T* dinv = vec(N.dinv);
            const T c2 = N.c2[0];
            for (int r = tid; r < N.n; r += kTailThreads) {
                const T s = tail_row(L.rval, L.rcol, (int)rp[r], (int)rp[r + 1], res);
                b[r] = s;
                T di = c2 * (dinv[r] * s);
                d[r] = di;
                xs[r] = di;
            }
        } else {
            T* b = vec(a.bc);
            for (int r = tid; r < a.nc; r += kTailThreads)
                b[r] = tail_row(L.rval, L.rcol, (int)rp[r], (int)rp[r + 1], res);
        }
        __syncthreads();
    }
    {
        // the dense inverse, one wavefront per row (gemv_body's sums)
        const T* b = vec(a.bc);
        T* x = vec(a.xc);
        const int lane = tid & 63;
        for (int r = tid >> 6; r < a.nc; r += kTailThreads / 64) {
            const double* m = a.inverse + (size_t)r * a.nc;
            double mv[kTailDense / 64];
#pragma unroll
            for (int u = 0; u < kTailDense / 64; ++u) mv[u] = m[min(lane + u * 64, a.nc - 1)];
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < kTailDense / 64; ++u)
                if (lane + u * 64 < a.nc) s += mv[u] * (double)b[lane + u * 64];
            s = wave_sum(s);
            if (lane == 0) x[r] = (T)s;
        }
        __syncthreads();
    }
    int below = a.xc;  // the iterate of the level below
    for (int l = a.levels - 1; l >= 0; --l) {
        const TailLevel<T>& L = a.lv[l];
        const bool second = (swapped >> l) & 1u;
        int x = second ? L.y : L.x, y = second ? L.x : L.y;
        const T* e = vec(below);
        const uint16_t* rp = reinterpret_cast<const uint16_t*>(lds + L.prp);
        T* xs = vec(x);
        for (int r = tid; r < L.n; r += kTailThreads)
            xs[r] = xs[r] + tail_row(L.pval, L.pcol, (int)rp[r], (int)rp[r + 1], e);
        __syncthreads();
        for (int k = 0; k < L.steps; ++k) {
            smooth(L, vec(x), vec(y), k == 0 ? T(0) : L.c1[k], L.c2[k]);
            const int t = x;
            x = y;
            y = t;
        }
        below = x;
    }
    const T* x = vec(below);
    for (int r = tid; r < a.lv[0].n; r += kTailThreads) out[r] = x[r];
}

template <typename T>
__global__ void k_tail_head(TailHead<T> head, char* image) {
    *reinterpret_cast<TailHead<T>*>(image) = head;
}

// one array of the image per blockIdx.y: copied, or narrowed to 16 bits
template <typename T>
__global__ __launch_bounds__(kBlock) void k_tail_image(TailSegments<T> segs, char* image) {
    const TailSegment<T>& s = segs.s[blockIdx.y];
    for (int i = (int)blockIdx.x * kBlock + (int)threadIdx.x; i < s.count; i += (int)gridDim.x * kBlock) {
        if (s.val) reinterpret_cast<T*>(image + s.at)[i] = s.val[i];
        else reinterpret_cast<uint16_t*>(image + s.at)[i] = (uint16_t)s.idx[i];
    }
}

}  // namespace

template <typename T>
void tail_image(const TailHead<T>& head, const TailSegments<T>& segs, char* image, hipStream_t s) {
    // (more than 64 KB of dynamic LDS has to be allowed)
    MATAMG_HIP(hipFuncSetAttribute((const void*)k_tail<T>, hipFuncAttributeMaxDynamicSharedMemorySize, kTailLds));
    hipLaunchKernelGGL(k_tail_head<T>, dim3(1), dim3(1), 0, s, head, image);
    hipLaunchKernelGGL(k_tail_image<T>, dim3(8, segs.count), dim3(kBlock), 0, s, segs, image);
    MATAMG_LAUNCH_CHECK();
}
template void tail_image<double>(const TailHead<double>&, const TailSegments<double>&, char*, hipStream_t);
template void tail_image<float>(const TailHead<float>&, const TailSegments<float>&, char*, hipStream_t);

template <typename T>
void tail_cycle(const char* image, int image_bytes, int lds_bytes, int n, const T* b, const T* d, const T* x, T* out,
                hipStream_t s) {
    hipLaunchKernelGGL(k_tail<T>, dim3(1), dim3(kTailThreads), lds_bytes, s, reinterpret_cast<const uint4*>(image),
                       image_bytes / 16, n, b, d, x, out);
    MATAMG_LAUNCH_CHECK();
}
template void tail_cycle<double>(const char*, int, int, int, const double*, const double*, const double*, double*,
                                 hipStream_t);
template void tail_cycle<float>(const char*, int, int, int, const float*, const float*, const float*, float*,
                                hipStream_t);

}  // namespace matamg

// Row-block partition of a CSR matrix for the streaming kernels, computed on
// the device.
//
// The partition is the greedy one: walking the rows in order, a block takes
// rows while it holds fewer than max_block_rows(G) rows and its stored
// entries stay within the cap (kStreamCap, or kStreamCapWide); a row longer
// than long_row_limit(G) forms a block of its own.  The walk is sequential,
// but the block that starts at row r ends at a row that depends on r alone, so
// every row's step is computed in parallel, and a walk enters a chunk of rows
// at one of its first 256: each chunk is walked from all of them at once, the
// chunks' entries then follow one from the other, and each chunk is walked
// once more, from its own entry, for the starts.  The result equals the host
// walk exactly.  Launches are what bounds it on small matrices and memory
// passes on large ones: five launches, three for a single chunk (radix-8
// pointer jumping over marks, with scans, took about twenty; without it the setup
// of the 128^2 two-domain problem went from 5.6 to 4.2 ms, of the 128^3 stack from
// 34.8 to 32.2 ms).
#include <algorithm>

#include "device_util.h"
#include "kernels.h"

namespace matamg {
namespace {

inline int grid1(int64_t n) {
    int g = ceil_div(n > 0 ? n : 1, kBlock);
    return g < 65535 ? g : 65535;
}

#define FOR_ROWS(i, n) for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < (n); i += (int64_t)gridDim.x * kBlock)

// one bitmap of long rows for both group sizes, steps of a byte
constexpr int kMaxStep = 256;
static_assert(long_row_limit(1) == long_row_limit(8) && max_block_rows(1) <= kMaxStep && max_block_rows(8) <= kMaxStep);
constexpr int kStatBlocks = 256;      // most workgroups of k_row_stats
constexpr int kChunkTile = 16384;     // rows whose steps are in LDS at a time
constexpr int kMaxChunks = 512;

// sums (w) and maxima (m) over the block's threads, on every thread
__device__ __forceinline__ void block_max_sum(int& m, int& w) {
    __shared__ int sm[kBlock / 64], sw[kBlock / 64];
    for (int off = 32; off > 0; off >>= 1) {
        m = max(m, __shfl_xor(m, off, 64));
        w += __shfl_xor(w, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        sm[threadIdx.x >> 6] = m;
        sw[threadIdx.x >> 6] = w;
    }
    __syncthreads();
    m = 0;
    w = 0;
    for (int k = 0; k < kBlock / 64; ++k) {
        m = max(m, sm[k]);
        w += sw[k];
    }
}

// part[block] = {longest row, entries in rows wider than kWideRow} of the
// block's rows; bits: the rows that are long
__global__ __launch_bounds__(kBlock) void k_row_stats(int n, const int* rp, int2* part, unsigned long long* bits) {
    int m = 0, w = 0;
    for (int64_t b = (int64_t)blockIdx.x * kBlock; b < n; b += (int64_t)gridDim.x * kBlock) {
        const int64_t r = b + threadIdx.x;
        const int len = r < n ? rp[r + 1] - rp[r] : 0;
        const unsigned long long lw = __ballot(len > long_row_limit(1));
        if ((threadIdx.x & 63) == 0) bits[r >> 6] = lw;
        m = max(m, len);
        if (len > kWideRow) w += len;
    }
    block_max_sum(m, w);
    if (threadIdx.x == 0) part[blockIdx.x] = int2{m, w};
}

// step[r]: rows, less one, of the block that would start at row r;
// par[1] = threads per row (the host's stream_group rule), par[2] = longest
// row, par[3] = 0
__global__ __launch_bounds__(kBlock) void k_row_steps(int n, const int* rp, const int2* part, int nparts,
                                                      const unsigned long long* bits, int cap, uint8_t* step,
                                                      int* par) {
    int m = 0, w = 0;
    if ((int)threadIdx.x < nparts) {
        const int2 p = part[threadIdx.x];
        m = p.x;
        w = p.y;
    }
    block_max_sum(m, w);
    const int group = stream_group_rule(m, w, rp[n]);
    const int limit = long_row_limit(group), max_rows = max_block_rows(group);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        par[1] = group;
        par[2] = m;
        par[3] = 0;
    }
    FOR_ROWS(r64, n) {
        const int r = (int)r64;
        const int first = rp[r];
        int e = r + 1;
        if (rp[r + 1] - first <= limit) {
            // largest e with at most cap entries (e = r + 1 always has),
            // then up to the first long row
            int lo = r + 1, hi = min(n, r + max_rows);
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (rp[mid] - first <= cap) lo = mid;
                else hi = mid - 1;
            }
            e = lo;
            if (m > limit) {
                for (int q = r >> 6; q <= (e - 1) >> 6; ++q) {
                    unsigned long long b = bits[q];
                    if (q == r >> 6) b &= ~0ull << (r & 63);
                    if (b) {
                        e = min(e, q * 64 + __builtin_ctzll(b));
                        break;
                    }
                }
            }
        }
        step[r] = (uint8_t)(e - r - 1);
    }
}

// f(steps, lo, hi) for every tile lo .. hi of the rows c0 .. c1, its steps in
// LDS (step is on 16 bytes and padded to them, tiles start on 16)
template <class F>
__device__ __forceinline__ void for_each_tile(int c0, int c1, const uint8_t* step, F f) {
    __shared__ uint4 lds[kChunkTile / 16];
    for (int lo = c0; lo < c1; lo += kChunkTile) {
        const int hi = min(c1, lo + kChunkTile);
        const uint4* src = reinterpret_cast<const uint4*>(step + lo);
        for (int i = threadIdx.x; i < (hi - lo + 15) / 16; i += kBlock) lds[i] = src[i];
        __syncthreads();
        f(reinterpret_cast<const uint8_t*>(lds), lo, hi);
        __syncthreads();
    }
}

// chunk blockIdx.x walked from its row t on, for thread t: the row of the next
// chunk that the walk enters (from its start), and the blocks that it passed
__global__ __launch_bounds__(kBlock) void k_chunk_walks(int n, int chunk, const uint8_t* step, uint8_t* exits,
                                                        int* counts) {
    static_assert(kMaxStep == kBlock);
    const int c0 = (int)blockIdx.x * chunk, c1 = min(n, c0 + chunk);
    int r = c0 + (int)threadIdx.x, b = 0;
    for_each_tile(c0, c1, step, [&](const uint8_t* s, int lo, int hi) {
        while (r < hi) {
            r += (int)s[r - lo] + 1;
            ++b;
        }
    });
    exits[blockIdx.x * kMaxStep + threadIdx.x] = (uint8_t)(r - c1);
    counts[blockIdx.x * kMaxStep + threadIdx.x] = b;
}

// where the walk from row 0 enters each chunk, and the blocks before it
__global__ __launch_bounds__(kMaxChunks) void k_chunk_entries(int chunks, const uint8_t* exits, const int* counts,
                                                              int* entry, int* base) {
    __shared__ uint4 lds[kMaxChunks * kMaxStep / 16];
    __shared__ int at[kMaxChunks];
    __shared__ int sums[kMaxChunks / 64];
    for (int i = threadIdx.x; i < chunks * kMaxStep / 16; i += kMaxChunks)
        lds[i] = reinterpret_cast<const uint4*>(exits)[i];
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint8_t* e = reinterpret_cast<const uint8_t*>(lds);
        int t = 0;
        for (int c = 0; c < chunks; ++c) {
            at[c] = t;
            t = e[c * kMaxStep + t];
        }
    }
    __syncthreads();
    const int c = threadIdx.x;
    const int v = c < chunks ? counts[c * kMaxStep + at[c]] : 0;
    const int incl = scan_add(v);
    if ((c & 63) == 63) sums[c >> 6] = incl;
    __syncthreads();
    int before = incl - v;
    for (int k = 0; k < c >> 6; ++k) before += sums[k];
    if (c < chunks) {
        entry[c] = at[c];
        base[c] = before;
    }
}

// the block starts of chunk blockIdx.x; the last one also stores the end and
// par[0] = number of blocks
__global__ __launch_bounds__(kBlock) void k_chunk_starts(int n, int chunk, const uint8_t* step, const int* entry,
                                                         const int* base, int* blk, int* par) {
    const int c0 = (int)blockIdx.x * chunk, c1 = min(n, c0 + chunk);
    int r = c0 + (entry ? entry[blockIdx.x] : 0), b = entry ? base[blockIdx.x] : 0;
    for_each_tile(c0, c1, step, [&](const uint8_t* s, int lo, int hi) {
        if (threadIdx.x != 0) return;
        while (r < hi) {
            blk[b++] = r;
            r += (int)s[r - lo] + 1;
        }
    });
    if (c1 == n && threadIdx.x == 0) {
        blk[b] = n;
        par[0] = b;
    }
}

// cbase[b] = smallest column of block b; flag = 1 if a block's columns span
// 2^16 values or more (the block count *nblk_dev is read on the device)
__global__ __launch_bounds__(kBlock) void k_block_col_range(const int* nblk_dev, const int* rp, const int* col,
                                                            const int* blk, int* cbase, int* flag) {
    __shared__ int smin[kBlock / 64], smax[kBlock / 64];
    const int nblk = *nblk_dev;
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int k0 = rp[blk[b]], k1 = rp[blk[b + 1]];
        int lo = 0x7fffffff, hi = -1;
        for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) {
            const int c = col[k];
            lo = min(lo, c);
            hi = max(hi, c);
        }
        for (int off = 32; off > 0; off >>= 1) {
            lo = min(lo, __shfl_xor(lo, off, 64));
            hi = max(hi, __shfl_xor(hi, off, 64));
        }
        if ((threadIdx.x & 63) == 0) {
            smin[threadIdx.x >> 6] = lo;
            smax[threadIdx.x >> 6] = hi;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int w = 1; w < kBlock / 64; ++w) {
                lo = min(lo, smin[w]);
                hi = max(hi, smax[w]);
            }
            cbase[b] = k1 > k0 ? lo : 0;
            if (k1 > k0 && hi - lo > 0xffff) *flag = 1;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_pack_cols(int nblk, const int* rp, const int* col, const int* blk,
                                                      const int* cbase, uint16_t* col16) {
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int k0 = rp[blk[b]], k1 = rp[blk[b + 1]], base = cbase[b];
        for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) col16[k] = (uint16_t)(col[k] - base);
    }
}

// Distinct packed columns of a block: a bitmap over the 2^16 offsets a
// packed block can hold (2048 words in LDS), set by the block's entries.
constexpr int kColWords = 65536 / 32;

__device__ __forceinline__ bool long_row_block(int r0, int r1, int k0, int k1, int group) {
    return r1 - r0 == 1 && k1 - k0 > long_row_limit(group);
}

__device__ __forceinline__ void mark_columns(unsigned* bits, const uint16_t* col16, int k0, int k1) {
    for (int w = threadIdx.x; w < kColWords; w += kBlock) bits[w] = 0u;
    __syncthreads();
    for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) {
        const unsigned c = col16[k];
        atomicOr(&bits[c >> 5], 1u << (c & 31u));
    }
    __syncthreads();
}

// exclusive prefix over the block's threads of v (block-wide, 256 threads);
// *total receives the sum
__device__ __forceinline__ int block_exclusive(int v, int* red, int* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) red[wv] = incl;
    __syncthreads();
    int woff = 0, tot = 0;
    for (int i = 0; i < kBlock / 64; ++i) {
        if (i < wv) woff += red[i];
        tot += red[i];
    }
    __syncthreads();
    *total = tot;
    return woff + incl - v;
}

// Per block b: the number of distinct columns and of runs of consecutive
// columns among them.  A block is staged when it is not one long row, has
// at most ucap distinct columns and at most kUniqueReusePct percent as many
// as entries (too little reuse does not pay for the staging).  A staged
// block with at most kMaxRuns runs gets its run record (urun); any other
// staged block a list of ucnt[b] = its distinct count (0 otherwise).
__global__ __launch_bounds__(kBlock) void k_block_uniques_count(int nblk, const int* blk, const int* blkk,
                                                                const uint16_t* col16, int group, int ucap,
                                                                int* ucnt, uint32_t* urun, int* nstaged) {
    __shared__ unsigned bits[kColWords];
    __shared__ int red[kBlock / 64];
    __shared__ int rs[kMaxRuns], re[kMaxRuns];
    constexpr int kPer = kColWords / kBlock;  // words per thread, contiguous
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int r0 = blk[b], r1 = blk[b + 1], k0 = blkk[b], k1 = blkk[b + 1];
        const bool skip = long_row_block(r0, r1, k0, k1, group);
        mark_columns(bits, col16, k0, skip ? k0 : k1);
        int c = 0, ns = 0, ne = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int w = threadIdx.x * kPer + i;
            const unsigned m = bits[w];
            const unsigned prev = w > 0 ? bits[w - 1] >> 31 : 0u;
            const unsigned next = w + 1 < kColWords ? (bits[w + 1] & 1u) << 31 : 0u;
            c += __popc(m);
            ns += __popc(m & ~((m << 1) | prev));
            ne += __popc(m & ~((m >> 1) | next));
        }
        int total = 0, runs = 0, tmp = 0;
        (void)block_exclusive(c, red, &total);
        const int s0 = block_exclusive(ns, red, &runs);
        const int e0 = block_exclusive(ne, red, &tmp);
        const bool staged = !skip && total <= ucap && total * 100 <= kUniqueReusePct * (k1 - k0) && total > 0;
        const bool use_runs = staged && runs <= kMaxRuns;
        if (use_runs) {
            // the run starts and ends in column order (threads own contiguous words)
            int si = s0, ei = e0;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int w = threadIdx.x * kPer + i;
                const unsigned m = bits[w];
                const unsigned prev = w > 0 ? bits[w - 1] >> 31 : 0u;
                const unsigned next = w + 1 < kColWords ? (bits[w + 1] & 1u) << 31 : 0u;
                unsigned st = m & ~((m << 1) | prev), en = m & ~((m >> 1) | next);
                while (st) {
                    rs[si++] = w * 32 + __builtin_ctz(st);
                    st &= st - 1u;
                }
                while (en) {
                    re[ei++] = w * 32 + __builtin_ctz(en);
                    en &= en - 1u;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x < kRunWords) {
            uint32_t word = 0u;
            if (use_runs) {
                const int t = (int)threadIdx.x;
                if (t == 0) word = (uint32_t)runs;
                else if (t == 1) word = (uint32_t)total;
                else if (t - 2 < runs) word = (uint32_t)rs[t - 2] | ((uint32_t)(re[t - 2] - rs[t - 2] + 1) << 16);
            }
            urun[(size_t)b * kRunWords + threadIdx.x] = word;
        }
        if (threadIdx.x == 0) {
            ucnt[b] = (staged && !use_runs) ? total : 0;
            if (staged) atomicAdd(nstaged, 1);
        }
        __syncthreads();
    }
}

// the lists (ascending offsets) and every staged entry's index into its
// block's distinct columns (list or runs: the same ascending order)
__global__ __launch_bounds__(kBlock) void k_block_uniques_fill(int nblk, const int* blkk, const int* ustart,
                                                               const uint32_t* urun, uint16_t* col16,
                                                               uint16_t* uoff) {
    __shared__ unsigned bits[kColWords];
    __shared__ int wpre[kColWords];
    __shared__ int red[kBlock / 64];
    constexpr int kPer = kColWords / kBlock;  // words per thread
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int u0 = ustart[b];
        const bool list = ustart[b + 1] > u0;
        if (!list && urun[(size_t)b * kRunWords] == 0u) continue;  // block-uniform: not staged
        const int k0 = blkk[b], k1 = blkk[b + 1];
        mark_columns(bits, col16, k0, k1);
        // exclusive prefix of the set-bit counts over the words, thread t
        // owning words [t kPer, (t + 1) kPer)
        int loc[kPer];
        int sum = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            loc[i] = sum;
            sum += __popc(bits[threadIdx.x * kPer + i]);
        }
        int tot = 0;
        const int base = block_exclusive(sum, red, &tot);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int w = threadIdx.x * kPer + i;
            wpre[w] = base + loc[i];
            if (list) {
                unsigned m = bits[w];
                int r = base + loc[i];
                while (m) {
                    uoff[u0 + r] = (uint16_t)(w * 32 + __builtin_ctz(m));
                    ++r;
                    m &= m - 1u;
                }
            }
        }
        __syncthreads();
        for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) {
            const unsigned c = col16[k];
            const unsigned m = bits[c >> 5] & ((1u << (c & 31u)) - 1u);
            col16[k] = (uint16_t)(wpre[c >> 5] + __popc(m));
        }
        __syncthreads();
    }
}

// Per block of a matrix that has blocks whose columns span 2^16 values or
// more: its record in uwin (see DCsr::uwin).  The block's columns are sorted in
// LDS; the distinct ones, where they are staged (the rule of
// k_block_uniques_count), are covered by windows of 2^16 columns from the first
// on -- a mesh row gathers from a few planes, so a few windows do -- and the
// entries' col16 become their places in the list.  The list goes to
// off[blkk[b] ..], its length to ucnt[b]; *packed counts the entries of blocks
// with windows.
__global__ __launch_bounds__(kBlock) void k_block_windows(int nblk, const int* blk, const int* blkk, const int* col,
                                                          int group, uint16_t* col16, uint16_t* off, int* ucnt,
                                                          int* uwin, int* packed) {
    constexpr int kNone = 0x7fffffff;
    constexpr int kPer = kStreamCap / kBlock;
    __shared__ int keys[kStreamCap];
    __shared__ int red[kBlock / 64];
    __shared__ int rec[kWinWords];
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int r0 = blk[b], r1 = blk[b + 1], k0 = blkk[b], cnt = blkk[b + 1] - k0;
        if (threadIdx.x < kWinWords) rec[threadIdx.x] = 0;
        const bool skip = cnt <= 0 || long_row_block(r0, r1, k0, k0 + cnt, group);
        int nu = 0;
        if (!skip) {
            int size = kBlock;
            while (size < cnt) size *= 2;
            for (int i = threadIdx.x; i < size; i += kBlock) keys[i] = i < cnt ? col[k0 + i] : kNone;
            __syncthreads();
            for (int run = 2; run <= size; run *= 2)
                for (int d = run / 2; d > 0; d /= 2) {
                    for (int i = threadIdx.x; i < size / 2; i += kBlock) {
                        const int p = 2 * i - (i & (d - 1));
                        const int x = keys[p], y = keys[p + d];
                        if ((x > y) == ((p & run) == 0)) {
                            keys[p] = y;
                            keys[p + d] = x;
                        }
                    }
                    __syncthreads();
                }
            // the distinct ones to the front
            const int per = size / kBlock, e0 = (int)threadIdx.x * per;
            int v[kPer], mine = 0;
            int before = e0 > 0 ? keys[e0 - 1] : -1;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                v[i] = i < per ? keys[e0 + i] : kNone;
                if (v[i] == before) v[i] = kNone;
                else before = v[i];
                mine += v[i] != kNone;
            }
            int at = block_exclusive(mine, red, &nu);  // (all have read before any writes)
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (v[i] != kNone) keys[at++] = v[i];
            __syncthreads();
            if (threadIdx.x == 0) {
                int w = 0;
                for (int j = 0; j < nu;) {
                    if (w == kMaxWin) {
                        w = 0;
                        break;
                    }
                    if (w > 0) rec[1 + 2 * w] = j;
                    rec[2 + 2 * w] = keys[j];
                    const int last = keys[j] > kNone - 0xffff ? kNone : keys[j] + 0xffff;
                    ++w;
                    int lo = j + 1, hi = nu;  // the first beyond the window
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (keys[mid] <= last) lo = mid + 1;
                        else hi = mid;
                    }
                    j = lo;
                }
                const bool staged = w > 0 && nu <= unique_cap(kStreamCap) && nu * 100 <= kUniqueReusePct * cnt;
                rec[0] = staged ? nu : 0;
                rec[1] = staged || w == 1 ? w : 0;
                if (rec[1] > 0) atomicAdd(packed, cnt);
            }
        }
        __syncthreads();
        const int listed = rec[0], windows = rec[1];
        if (listed > 0) {
            for (int k = threadIdx.x; k < cnt; k += kBlock) {
                const int c = col[k0 + k];
                int lo = 0, hi = nu - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (keys[mid] < c) lo = mid + 1;
                    else hi = mid;
                }
                col16[k0 + k] = (uint16_t)lo;
            }
            for (int j = threadIdx.x; j < nu; j += kBlock) {
                int base = rec[2];
                for (int w = 1; w < windows; ++w)
                    if (j >= rec[1 + 2 * w]) base = rec[2 + 2 * w];
                off[k0 + j] = (uint16_t)(keys[j] - base);
            }
        } else if (windows > 0) {
            for (int k = threadIdx.x; k < cnt; k += kBlock) col16[k0 + k] = (uint16_t)(col[k0 + k] - rec[2]);
        }
        if (threadIdx.x < kWinWords) uwin[(size_t)b * kWinWords + threadIdx.x] = rec[threadIdx.x];
        if (threadIdx.x == 0) ucnt[b] = listed;
        __syncthreads();
    }
}

// the lists of k_block_windows, one after the other
__global__ __launch_bounds__(kBlock) void k_copy_lists(int nblk, const int* blkk, const int* ustart,
                                                       const uint16_t* off, uint16_t* uoff) {
    for (int b = blockIdx.x; b < nblk; b += gridDim.x) {
        const int k0 = blkk[b], u0 = ustart[b], nu = ustart[b + 1] - u0;
        for (int j = threadIdx.x; j < nu; j += kBlock) uoff[u0 + j] = off[k0 + j];
    }
}

// the block tables at their own length: blk, blkk[b] = rp[blk[b]] (b <= nblk),
// and cbase where it is given
__global__ void k_block_tables(int nblk, const int* rp, const int* blk_in, const int* cbase_in, int* blk, int* blkk,
                               int* cbase) {
    FOR_ROWS(b, (int64_t)nblk + 1) {
        const int r = blk_in[b];
        blk[b] = r;
        blkk[b] = rp[r];
        if (cbase && b < nblk) cbase[b] = cbase_in[b];
    }
}

}  // namespace

void stream_partition(DCsr& A, MemCounter* mc, hipStream_t s, bool pack, int cap) {
    const int n = A.n;
    A.col16.release();
    A.cbase.release();
    A.ustart.release();
    A.uoff.release();
    A.urun.release();
    A.uwin.release();
    A.npacked = 0;
    A.nuniq = 0;
    A.sblk.release();
    A.snblk = 0;
    A.cap = cap;
    if (n <= 0) {
        A.group = 1;
        A.max_len = 0;
        A.nblk = 0;
        A.blk.alloc(1, mc);
        A.blkk.alloc(1, mc);
        zero_async(A.blk.get(), sizeof(int), s);
        zero_async(A.blkk.get(), sizeof(int), s);
        MATAMG_HIP(hipStreamSynchronize(s));
        return;
    }
    const int* rp = A.rowptr.get();
    // everything is decided on the device: the only read-back is {blocks,
    // threads per row, longest row, columns too wide to pack} at the end
    const size_t n1 = (size_t)n + 1;
    const int stats = std::min(grid1(n), kStatBlocks);
    const int chunk = kChunkTile * ceil_div(ceil_div(n, kChunkTile), kMaxChunks);
    const int chunks = ceil_div(n, chunk);
    DBuf<int> par(4, mc), blk(n1, mc), cbase;
    DBuf<int2> part((size_t)stats, mc);
    DBuf<unsigned long long> bits((size_t)ceil_div(n, kBlock) * (kBlock / 64), mc);
    DBuf<uint8_t> step(((size_t)n + 15) / 16 * 16, mc);
    hipLaunchKernelGGL(k_row_stats, dim3(stats), dim3(kBlock), 0, s, n, rp, part.get(), bits.get());
    hipLaunchKernelGGL(k_row_steps, dim3(grid1(n)), dim3(kBlock), 0, s, n, rp, (const int2*)part.get(), stats,
                       (const unsigned long long*)bits.get(), cap, step.get(), par.get());
    DBuf<uint8_t> exits;
    DBuf<int> counts, entry;
    if (chunks > 1) {
        exits.alloc((size_t)chunks * kMaxStep, mc);
        counts.alloc((size_t)chunks * kMaxStep, mc);
        entry.alloc((size_t)chunks * 2, mc);
        hipLaunchKernelGGL(k_chunk_walks, dim3(chunks), dim3(kBlock), 0, s, n, chunk, (const uint8_t*)step.get(),
                           exits.get(), counts.get());
        hipLaunchKernelGGL(k_chunk_entries, dim3(1), dim3(kMaxChunks), 0, s, chunks, (const uint8_t*)exits.get(),
                           (const int*)counts.get(), entry.get(), entry.get() + chunks);
    }
    hipLaunchKernelGGL(k_chunk_starts, dim3(chunks), dim3(kBlock), 0, s, n, chunk, (const uint8_t*)step.get(),
                       (const int*)entry.get(), (const int*)entry.get() + (chunks > 1 ? chunks : 0), blk.get(),
                       par.get());
    if (pack && A.nnz > 0) {
        cbase.alloc(n1, mc);
        hipLaunchKernelGGL(k_block_col_range, dim3(std::min(grid1(n) * 4, 65535)), dim3(kBlock), 0, s,
                           (const int*)par.get(), rp, A.col.get(), (const int*)blk.get(), cbase.get(),
                           par.get() + 3);
    }
    MATAMG_LAUNCH_CHECK();
    int res[4] = {0, 0, 0, 0};
    d2h(res, par.get(), 4, s);
    const int nblk = res[0];
    A.group = res[1];
    A.max_len = res[2];
    A.nblk = nblk;
    A.blk.alloc((size_t)nblk + 1, mc);
    A.blkk.alloc((size_t)nblk + 1, mc);
    const bool narrow = pack && A.nnz > 0 && res[3] == 0;
    if (narrow) A.cbase.alloc((size_t)nblk, mc);
    hipLaunchKernelGGL(k_block_tables, dim3(grid1((int64_t)nblk + 1)), dim3(kBlock), 0, s, nblk, rp,
                       (const int*)blk.get(), (const int*)cbase.get(), A.blk.get(), A.blkk.get(), A.cbase.get());
    MATAMG_LAUNCH_CHECK();
    if (narrow) {
        A.col16.alloc((size_t)A.nnz, mc);
        hipLaunchKernelGGL(k_pack_cols, dim3(std::min(nblk, 65535)), dim3(kBlock), 0, s, nblk, rp, A.col.get(),
                           (const int*)A.blk.get(), (const int*)A.cbase.get(), A.col16.get());
        MATAMG_LAUNCH_CHECK();
        block_uniques(A, mc, s);
    } else if (pack && A.nnz > 0 && cap == kStreamCap) {
        block_windows(A, mc, s);
    }
}

// Packed columns by windows, for a matrix that one base per block cannot pack
// (one block is enough: a ring's first and last rows, an uneven level of a large
// stack).  It then reads 2 bytes of column an entry, not 4, and gathers through
// LDS: FP64 smoother of the 80x600x4 annulus 18.5 -> 15.0 us, of the 96^3
// cube's level 2 27 -> 22 us, of the 192^3 stack's levels 1 to 3 323, 256 and
// 178 -> 311, 226 and 165 us.  A matrix most of whose entries are in blocks
// without windows would gain little and stays as it is.
void block_windows(DCsr& A, MemCounter* mc, hipStream_t s) {
    const int nblk = A.nblk;
    if (nblk <= 0) return;
    DBuf<int> cnt((size_t)nblk, mc), tmp(scan_tmp_size(nblk), mc);
    DBuf<uint16_t> off((size_t)A.nnz, mc);
    A.col16.alloc((size_t)A.nnz, mc);
    A.uwin.alloc((size_t)nblk * kWinWords, mc);
    A.ustart.alloc((size_t)nblk + 2, mc);  // (the number of packed entries behind the starts)
    zero_async(A.ustart.get() + nblk + 1, sizeof(int), s);
    hipLaunchKernelGGL(k_block_windows, dim3(std::min(nblk, 16384)), dim3(kBlock), 0, s, nblk, (const int*)A.blk.get(),
                       (const int*)A.blkk.get(), (const int*)A.col.get(), A.group, A.col16.get(), off.get(), cnt.get(),
                       A.uwin.get(), A.ustart.get() + nblk + 1);
    MATAMG_LAUNCH_CHECK();
    exclusive_scan(cnt.get(), A.ustart.get(), nblk, tmp.get(), s);
    int res[2] = {0, 0};  // list length, packed entries
    d2h(res, A.ustart.get() + nblk, 2, s);
    if (2 * (int64_t)res[1] < A.nnz) {
        A.col16.release();
        A.uwin.release();
        A.ustart.release();
        return;
    }
    A.npacked = res[1];
    A.nuniq = res[0];
    A.uoff.alloc((size_t)(res[0] > 0 ? res[0] : 1), mc);
    if (res[0] > 0)
        hipLaunchKernelGGL(k_copy_lists, dim3(std::min(nblk, 16384)), dim3(kBlock), 0, s, nblk, (const int*)A.blkk.get(),
                           (const int*)A.ustart.get(), (const uint16_t*)off.get(), A.uoff.get());
    MATAMG_LAUNCH_CHECK();
}

void block_uniques(DCsr& A, MemCounter* mc, hipStream_t s) {
    A.ustart.release();
    A.uoff.release();
    A.urun.release();
    A.nuniq = 0;
    const int nblk = A.nblk;
    if (!A.col16 || nblk <= 0) return;
    DBuf<int> cnt((size_t)nblk, mc), tmp(scan_tmp_size((int64_t)nblk + 1), mc);
    A.urun.alloc((size_t)nblk * kRunWords, mc);
    A.ustart.alloc((size_t)nblk + 2, mc);  // (the number of staged blocks behind the starts)
    zero_async(A.ustart.get() + nblk + 1, sizeof(int), s);
    const int grid = std::min(nblk, 8192);
    hipLaunchKernelGGL(k_block_uniques_count, dim3(grid), dim3(kBlock), 0, s, nblk, (const int*)A.blk.get(),
                       (const int*)A.blkk.get(), (const uint16_t*)A.col16.get(), A.group, unique_cap(A.cap),
                       cnt.get(), A.urun.get(), A.ustart.get() + nblk + 1);
    MATAMG_LAUNCH_CHECK();
    exclusive_scan(cnt.get(), A.ustart.get(), nblk, tmp.get(), s);
    int res[2] = {0, 0};  // list length, staged blocks
    d2h(res, A.ustart.get() + nblk, 2, s);
    const int total = res[0];
    if (res[1] == 0) {
        // nothing staged: the streaming kernels read no per-block tables
        A.ustart.release();
        A.urun.release();
        return;
    }
    A.nuniq = total;
    A.uoff.alloc((size_t)(total > 0 ? total : 1), mc);
    hipLaunchKernelGGL(k_block_uniques_fill, dim3(grid), dim3(kBlock), 0, s, nblk, (const int*)A.blkk.get(),
                       (const int*)A.ustart.get(), (const uint32_t*)A.urun.get(), A.col16.get(), A.uoff.get());
    MATAMG_LAUNCH_CHECK();
}

}  // namespace matamg

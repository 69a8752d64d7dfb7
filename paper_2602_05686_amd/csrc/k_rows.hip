// Row dictionaries of an operator whose rows repeat.
//
// A structured mesh with piecewise constant coefficients gives bitwise equal
// rows (same values, same column offsets from the row) all over each piece:
// a few to a few dozen distinct ones among the rows of neighbouring row
// blocks.  Groups of dk consecutive row blocks then keep each distinct row
// once, and the streaming kernels read a 16-bit number per row in place of
// its values and columns (27 entries of 10 bytes).  Nothing is rounded: the
// dictionary holds the operator's own values.  Such rows also gather from few
// windows of consecutive columns, which the kernels then stage in LDS.
//
// One workgroup builds one group's dictionary: a hash of every row (eight
// lanes per row; an order-independent sum, so that lanes can take entries in
// any order), an LDS table from hash to the first row that has it, an exact
// comparison of every row with that row, and numbers in row order.  An
// operator is left without dictionaries if a group's do not fit, if two
// different rows share a hash, or if they hold more than 1 / kDictShare of
// its entries.
#include <algorithm>

#include "device_util.h"
#include "kernels.h"

namespace matamg {
namespace {

constexpr int kSlots = 2048;  // hash slots of a group (at most kDictGroupRows rows)
static_assert(kSlots > kDictGroupRows, "the table never fills");

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// result[0] = 1: no dictionaries; [1], [2]: most entries and rows of a group,
// [3]: longest windows
enum { R_FAIL = 0, R_MAX_E = 1, R_MAX_N = 2, R_MAX_X = 3, R_WORDS = 4 };

// Group g: drow_of of its rows, the number of distinct rows and of their
// entries (rows[g], entries[g]), and for the fill the first row with number i
// and its record, at [blk of the group + i].
__global__ __launch_bounds__(kBlock) void k_rows_count(int nblk, int dk, const int* blk, const int* rp, const int* col,
                                                       const double* val, uint16_t* drow_of, int* rows, int* entries,
                                                       int* first, uint32_t* record, int* result) {
    __shared__ unsigned long long key[kSlots];
    __shared__ int rep[kSlots];
    __shared__ uint16_t slot_of[kDictGroupRows], number[kDictGroupRows];
    __shared__ int red[2][kBlock / 64];
    __shared__ int skip, bad;
    const int g = blockIdx.x;
    const int b0 = g * dk, b1 = min(b0 + dk, nblk);
    const int r0 = blk[b0], n = blk[b1] - r0;
    if (threadIdx.x == 0) {
        skip = *(volatile int*)&result[R_FAIL];  // another group has already failed
        bad = 0;
    }
    for (int i = threadIdx.x; i < kSlots; i += kBlock) {
        key[i] = 0ull;
        rep[i] = 0x7fffffff;
    }
    __syncthreads();
    if (skip) return;
    const int lane8 = threadIdx.x & 7;
    for (int i = threadIdx.x >> 3; i < n; i += kBlock / 8) {
        const int r = r0 + i;
        const int k0 = rp[r], k1 = rp[r + 1];
        uint64_t h = 0;
        for (int k = k0 + lane8; k < k1; k += 8) {
            const uint64_t v = (uint64_t)__double_as_longlong(val[k]);
            h += mix64(v ^ mix64(((uint64_t)(uint32_t)(col[k] - r) << 32) | (uint32_t)(k - k0 + 1)));
        }
        for (int off = 4; off > 0; off >>= 1) h += (uint64_t)__shfl_xor((unsigned long long)h, off, 8);
        if (lane8 == 0) {
            h = mix64(h + (uint64_t)(k1 - k0)) | 1ull;  // 0 marks a free slot
            int s = (int)(h >> 40) & (kSlots - 1);
            for (;;) {
                const unsigned long long was = atomicCAS(&key[s], 0ull, (unsigned long long)h);
                if (was == 0ull || was == h) break;
                s = (s + 1) & (kSlots - 1);
            }
            atomicMin(&rep[s], i);
            slot_of[i] = (uint16_t)s;
        }
    }
    __syncthreads();
    // every row against the first row of its slot, entry by entry
    for (int i = threadIdx.x >> 3; i < n; i += kBlock / 8) {
        const int q = rep[slot_of[i]];
        if (q == i) continue;
        const int r = r0 + i, f = r0 + q;
        const int k0 = rp[r], len = rp[r + 1] - k0, f0 = rp[f];
        bool same = rp[f + 1] - f0 == len;
        if (same)
            for (int k = lane8; k < len; k += 8)
                same = same && __double_as_longlong(val[k0 + k]) == __double_as_longlong(val[f0 + k]) &&
                       col[k0 + k] - r == col[f0 + k] - f;
        if (!same) bad = 1;
    }
    // numbers in row order: thread t owns the rows [t per, (t + 1) per)
    const int per = (n + kBlock - 1) / kBlock;
    const int i0 = min(n, (int)threadIdx.x * per), i1 = min(n, i0 + per);
    int m = 0, e = 0;
    for (int i = i0; i < i1; ++i)
        if (rep[slot_of[i]] == i) {
            ++m;
            e += rp[r0 + i + 1] - rp[r0 + i];
        }
    int mi = m, ei = e;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int off = 1; off < 64; off <<= 1) {
        const int a = __shfl_up(mi, off, 64), c = __shfl_up(ei, off, 64);
        if (lane >= off) {
            mi += a;
            ei += c;
        }
    }
    if (lane == 63) {
        red[0][w] = mi;
        red[1][w] = ei;
    }
    __syncthreads();
    int mt = 0, et = 0, mb = mi - m, eb = ei - e;
    for (int k = 0; k < kBlock / 64; ++k) {
        if (k < w) {
            mb += red[0][k];
            eb += red[1][k];
        }
        mt += red[0][k];
        et += red[1][k];
    }
    if (threadIdx.x == 0) {
        rows[g] = mt;
        entries[g] = et;
        if (bad || mt > kDictRows || et > kDictEntries) result[R_FAIL] = 1;
        atomicMax(&result[R_MAX_E], et);
        atomicMax(&result[R_MAX_N], mt);
    }
    if (mt > kDictRows || et > kDictEntries) return;  // uniform
    for (int i = i0; i < i1; ++i)
        if (rep[slot_of[i]] == i) {
            const int len = rp[r0 + i + 1] - rp[r0 + i];
            number[i] = (uint16_t)mb;
            first[r0 + mb] = r0 + i;
            record[r0 + mb] = (uint32_t)eb | ((uint32_t)len << 16);
            ++mb;
            eb += len;
        }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += kBlock) drow_of[r0 + i] = number[rep[slot_of[i]]];
}

// The dictionaries' records and entries (eight lanes per distinct row), and
// the group's windows: an offset d reaches the columns r0 + d .. r1 - 1 + d of
// the group's rows r0 .. r1 - 1; the union of these windows over the distinct
// offsets, in ascending order, is what is staged.
constexpr int kOffsets = 256;  // most distinct offsets of a staged group
__global__ __launch_bounds__(kBlock) void k_rows_fill(int nblk, int dk, const int* blk, const int* rp, const int* col,
                                                      const double* val, const int* drow, const int* dent,
                                                      const int* first, const uint32_t* record, uint32_t* dinfo,
                                                      int* doff, double* dval, int* drun, int* result) {
    __shared__ int table[2 * kOffsets], list[kOffsets], sorted[kOffsets], count;
    __shared__ int run[kDictRunWords - 2];
    constexpr int kFree = 0x7fffffff;
    const int g = blockIdx.x;
    const int r0 = blk[g * dk], n = blk[min((g + 1) * dk, nblk)] - r0;
    const int m0 = drow[g], m = drow[g + 1] - m0, e0 = dent[g];
    int* rec = drun + (size_t)g * kDictRunWords;
    if (threadIdx.x < 2) {
        rec[threadIdx.x] = threadIdx.x == 0 ? m0 : e0;
        // the ends of the last group
        if (g + 1 == (int)gridDim.x) rec[kDictRunWords + threadIdx.x] = threadIdx.x == 0 ? m0 + m : dent[g + 1];
    }
    for (int i = threadIdx.x; i < 2 * kOffsets; i += kBlock) table[i] = kFree;
    if (threadIdx.x == 0) count = 0;
    if (threadIdx.x < kDictRunWords - 2) run[threadIdx.x] = 0;
    __syncthreads();
    // distinct offsets (a full table ends the search: not staged)
    for (int i = threadIdx.x >> 3; i < m; i += kBlock / 8) {
        const int r = first[r0 + i];
        const int len = (int)(record[r0 + i] >> 16), k0 = rp[r];
        for (int k = threadIdx.x & 7; k < len; k += 8) {
            const int d = col[k0 + k] - r;
            unsigned s = (unsigned)d * 2654435761u >> 23;  // 0 .. 511
            for (int tries = 0; tries < 2 * kOffsets; ++tries) {
                const int was = atomicCAS(&table[s], kFree, d);
                if (was == d) break;
                if (was == kFree) {
                    const int c = atomicAdd(&count, 1);
                    if (c < kOffsets) list[c] = d;
                    break;
                }
                if (*(volatile int*)&count > kOffsets) break;
                s = (s + 1) & (2 * kOffsets - 1);
            }
        }
    }
    __syncthreads();
    const int nd = count;
    if (nd <= kOffsets) {
        if ((int)threadIdx.x < nd) {
            const int d = list[threadIdx.x];
            int rank = 0;
            for (int j = 0; j < nd; ++j) rank += list[j] < d;
            sorted[rank] = d;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int runs = 0, total = 0, start = sorted[0], end = start + n;
            bool ok = true;
            for (int j = 1; ok && j <= nd; ++j) {
                if (j < nd && sorted[j] <= end) {
                    end = sorted[j] + n;
                    continue;
                }
                ok = runs < kDictRuns && end - start <= kDictWindow - total;
                if (ok) {
                    run[2 + 2 * runs] = start;
                    run[3 + 2 * runs] = end - start;
                    total += end - start;
                    ++runs;
                }
                if (j < nd) {
                    start = sorted[j];
                    end = start + n;
                }
            }
            run[0] = ok ? runs : 0;
            run[1] = ok ? total : 0;
            if (ok) atomicMax(&result[R_MAX_X], total);
        }
        __syncthreads();
    }
    if (threadIdx.x < kDictRunWords - 2) rec[2 + threadIdx.x] = run[threadIdx.x];
    for (int i = threadIdx.x >> 3; i < m; i += kBlock / 8) {
        const int r = first[r0 + i];
        const uint32_t rec = record[r0 + i];
        const int s = (int)(rec & 0xffffu), len = (int)(rec >> 16), k0 = rp[r];
        if ((threadIdx.x & 7) == 0) dinfo[m0 + i] = rec;
        for (int k = threadIdx.x & 7; k < len; k += 8) {
            doff[e0 + s + k] = col[k0 + k] - r;
            dval[e0 + s + k] = val[k0 + k];
        }
    }
}

}  // namespace

void row_dictionaries(DCsr& A, MemCounter* mc, hipStream_t s) {
    A.dk = 0;
    A.dn = A.de = 0;
    // one thread per row adds its entries in order, as the streaming kernel
    // does for rows up to kWideRow of a one-thread-per-row matrix
    if (A.group != 1 || A.max_len > kWideRow || A.n <= 0 || A.nnz <= 0) return;
    // up to 450 rows of a 27-point operator per workgroup (two rounds; the
    // fine smoother of the 192^3 stack took 158 us with six row blocks of a
    // narrow partition, 177 us with two), fewer where a small operator would
    // leave the device idle
    const int dk = std::max(1, std::min(A.cap == kStreamCapWide ? kDictMaxBlocks / 2 : kDictMaxBlocks, A.nblk / 1024));
    const int groups = ceil_div(A.nblk, dk);
    DBuf<int> cnt_n((size_t)groups, mc), cnt_e((size_t)groups, mc), first((size_t)A.n, mc),
        tmp(scan_tmp_size(groups), mc), result(R_WORDS + 2, mc);
    DBuf<uint32_t> record((size_t)A.n, mc);
    if (!A.drow_of) A.drow_of.alloc((size_t)A.n, mc);
    DBuf<int> drow((size_t)groups + 1, mc), dent((size_t)groups + 1, mc);
    zero_async(result.get(), R_WORDS * sizeof(int), s);
    hipLaunchKernelGGL(k_rows_count, dim3(groups), dim3(kBlock), 0, s, A.nblk, dk, (const int*)A.blk.get(),
                       (const int*)A.rowptr.get(), (const int*)A.col.get(), (const double*)A.val.get(), A.drow_of.get(),
                       cnt_n.get(), cnt_e.get(), first.get(), record.get(), result.get());
    MATAMG_LAUNCH_CHECK();
    exclusive_scan(cnt_n.get(), drow.get(), groups, tmp.get(), s);
    exclusive_scan(cnt_e.get(), dent.get(), groups, tmp.get(), s);
    MATAMG_HIP(hipMemcpyAsync(result.get() + R_WORDS, drow.get() + groups, sizeof(int), hipMemcpyDeviceToDevice, s));
    MATAMG_HIP(hipMemcpyAsync(result.get() + R_WORDS + 1, dent.get() + groups, sizeof(int), hipMemcpyDeviceToDevice, s));
    int res[R_WORDS + 2];
    d2h(res, result.get(), R_WORDS + 2, s);
    const int64_t dn = res[R_WORDS], de = res[R_WORDS + 1];
    // no rows in any record: what was recorded with dictionaries reads val and col
    auto empty = [&] { zero_async(A.drun.get(), A.drun.size() * sizeof(int), s); };
    if (res[R_FAIL] || de * kDictShare > A.nnz) {
        if (A.drun) empty();
        else A.drow_of.release();
        return;
    }
    if (!A.drun || (size_t)dn > A.dinfo.size() || (size_t)de > A.doff.size()) {
        // half as large again, so that all of them are a few times the largest
        const size_t rows = std::max((size_t)dn, A.dinfo.size() * 3 / 2),
                     entries = std::max((size_t)de, A.doff.size() * 3 / 2);
        if (A.drun) {
            empty();
            DBuf<uint16_t> row_of((size_t)A.n, mc);
            MATAMG_HIP(hipMemcpyAsync(row_of.get(), A.drow_of.get(), sizeof(uint16_t) * (size_t)A.n,
                                      hipMemcpyDeviceToDevice, s));
            auto aside = [&](auto& b) {
                using B = std::decay_t<decltype(b)>;
                if (b) A.dold.push_back(std::make_shared<B>(std::move(b)));
            };
            aside(A.drow_of);
            aside(A.drun);
            aside(A.dinfo);
            aside(A.doff);
            aside(A.dval);
            aside(A.dval32);
            A.drow_of = std::move(row_of);
        }
        A.dinfo.alloc(rows, mc);
        A.doff.alloc(entries, mc);
        A.dval.alloc(entries, mc);
        A.drun.alloc((size_t)(groups + 1) * kDictRunWords, mc);
    }
    hipLaunchKernelGGL(k_rows_fill, dim3(groups), dim3(kBlock), 0, s, A.nblk, dk, (const int*)A.blk.get(),
                       (const int*)A.rowptr.get(), (const int*)A.col.get(), (const double*)A.val.get(),
                       (const int*)drow.get(), (const int*)dent.get(), (const int*)first.get(),
                       (const uint32_t*)record.get(), A.dinfo.get(), A.doff.get(), A.dval.get(), A.drun.get(),
                       result.get());
    MATAMG_LAUNCH_CHECK();
    A.dk = dk;
    A.dn = dn;
    A.de = de;
    A.dmax_e = (res[R_MAX_E] + 1) & ~1;  // (even: the arrays after it in LDS stay aligned)
    A.dmax_n = res[R_MAX_N];
    int longest = 0;
    d2h(&longest, result.get() + R_MAX_X, 1, s);
    A.dmax_x = (longest + 1) & ~1;
}

}  // namespace matamg

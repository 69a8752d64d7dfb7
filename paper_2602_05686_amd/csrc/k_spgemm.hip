// Sparse matrix-matrix product C = A * B (Galerkin product R (A P) and the
// smoothed prolongator A_F P^) and the CSR transpose P -> R = P^T.
//
// One wavefront per output row.  The row's products are enumerated in the
// canonical order (A's row ascending, then B's row order), 64 at a time: a
// product belongs to the last of up to 64 A entries whose products start at
// or before it, found from the bits of those starts.  Symbolic phase: product
// columns go into an open-addressed hash set in LDS (1024 slots per wave, at
// most 512 distinct columns); rows that overflow it are redone with a table
// in global memory sized from the row's product count.  Numeric phase: the
// products are accumulated strictly in canonical order, A entry after A entry
// (the products of one A entry have distinct columns and are added at once),
// so every entry is the same sequence of IEEE additions as a serial
// row-by-row product.  On LDS tables a single walk adds each product to its
// column's hash-slot sum and the slots are ranked by column (ascending output
// positions) afterwards; the global tables rank the columns first and
// accumulate by rank in a second walk.  Overflow rows of at most kDBig
// columns run their numeric phase in a large LDS table shared by a
// workgroup's wavefronts, the others in global memory.
//
// What bounds the rows is their chains of dependent loads (two loads per
// chunk of A entries, one per step), which are taken one chunk and one step
// ahead; what bounded the wide ones was ranking every column against every
// other.  All products of the 128^3 layered stack's setup (seven levels, rows
// of up to 5,200 columns) 22.0 -> 12.7 ms, of a 64^3 cube's update 3.8 -> 2.0,
// of a 37 x 23 x 29 cube's setup 1.29 -> 0.19.
#pragma clang fp contract(off)

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "device_util.h"
#include "kernels.h"
#include "setup_kernels.h"

namespace matamg {
namespace {

constexpr int kWaves = kBlock / 64;
constexpr int kHS = 1024;     // LDS hash slots per wave
constexpr int kDMax = 512;    // max distinct columns on the LDS path
// numeric phase: distinct columns of a row (at most) and LDS hash slots per
// wavefront, in three sizes, of which a CU's LDS holds 8 or more, 6 and 3
// workgroups
constexpr int kNumCols[3] = {128, 256, kDMax};
constexpr int kNumSlots[3] = {256, 384, 768};
// parts of a row's column range in rank_columns, for rows of up to d columns
constexpr int rank_parts(int d) { return d / 4; }
// LDS of a workgroup: keys, running sums, columns' list and parts (see k_spgemm_numeric)
constexpr int num_lds(int i) {
    return kWaves * ((int)(sizeof(int) + sizeof(double)) * kNumSlots[i] +
                     (int)sizeof(int) * (kNumCols[i] + rank_parts(kNumCols[i]) + 1));
}
constexpr int kCuLds = 160 * 1024;
static_assert(kCuLds / num_lds(0) >= 8 && kCuLds / num_lds(1) == 6 && kCuLds / num_lds(2) == 3);
// lists of fewer rows leave out the middle size (a launch of 4 us)
constexpr int kNumThreeSizes = 32768;
constexpr int kRankTile = 1024;  // LDS tile of the column list when ranking long rows
constexpr int kRankKeys = 8;     // keys per lane per ranking pass
// overflow rows with at most this many columns: numeric phase in LDS, one
// workgroup per row.  The table fills a CU's 160 KB: a row of up to half as
// many columns probes a half-empty table, the longest one that is 89% full.
// (Rows beyond go to global memory at several times the cost: 67 rows of
// 4,100 to 5,200 columns took 5.4 ms there.)
constexpr int kDBig = 8192;
constexpr int kHSBig = 9216;     // their LDS hash slots
// dynamic LDS of the large-table workgroup: a key and a running sum per slot,
// and the columns' list and parts
constexpr size_t kBigLds = (sizeof(int) + sizeof(double)) * kHSBig + sizeof(int) * (kDBig + rank_parts(kDBig) + 1);
static_assert(kBigLds + 1024 <= kCuLds, "the large table fits a CU");

__device__ __forceinline__ unsigned hash_slot(int key, unsigned mask) {
    return ((unsigned)key * 2654435761u) & mask;
}

// insert key; returns 1 if newly inserted, 0 if present, -1 if the table is full
__device__ __forceinline__ int hash_insert(int* keys, unsigned mask, int key) {
    unsigned h = hash_slot(key, mask);
    for (unsigned probe = 0; probe <= mask; ++probe) {
        int old = atomicCAS(keys + h, -1, key);
        if (old == -1) return 1;
        if (old == key) return 0;
        h = (h + 1) & mask;
    }
    return -1;
}

// slot of key in an LDS table of any number of slots, inserting it if absent
// (the table has more slots than the row has keys); fresh: inserted here
__device__ __forceinline__ unsigned table_at(int key, unsigned n) {
    return (unsigned)(((uint64_t)((unsigned)key * 2654435761u) * n) >> 32);
}
__device__ __forceinline__ unsigned lds_insert(int* keys, unsigned slots, int key, bool& fresh) {
    unsigned h = table_at(key, slots);
    for (unsigned probe = 0; probe < slots; ++probe) {
        const int old = atomicCAS(keys + h, -1, key);
        fresh = old == -1;
        if (fresh || old == key) return h;
        if (++h == slots) h = 0;
    }
    fresh = false;
    return 0;
}
// The same in buckets of four keys read at once, for tables that may be
// nearly full.  Buckets fill from their first slot on and keys stay where
// they are, so a key that is present is met before any free slot.
constexpr int kBucket = 4;
__device__ __forceinline__ unsigned bucket_insert(int* keys, unsigned buckets, int key) {
    unsigned b = table_at(key, buckets);
    for (unsigned probe = 0; probe < kBucket * buckets + 64;) {
        const int4 k = *reinterpret_cast<const int4*>(keys + kBucket * b);
        const unsigned at = kBucket * b;
        if (k.x == key) return at;
        if (k.y == key) return at + 1;
        if (k.z == key) return at + 2;
        if (k.w == key) return at + 3;
        const int j = k.x == -1 ? 0 : k.y == -1 ? 1 : k.z == -1 ? 2 : k.w == -1 ? 3 : kBucket;
        ++probe;
        if (j < kBucket) {
            const int old = atomicCAS(keys + at + j, -1, key);
            if (old == -1 || old == key) return at + j;
            continue;  // another key took the slot: read the bucket again
        }
        if (++b == buckets) b = 0;
    }
    return 0;
}
// slots of a table for m keys: twice as many where they fit, a multiple of a bucket
__device__ __forceinline__ unsigned lds_slots(int m, int most) {
    return (unsigned)min(most, max(64, (2 * m + kBucket - 1) & ~(kBucket - 1)));
}

// Ranks of a row's columns among each other (their output positions), from
// its hash table, by THREADS threads (one wavefront, or a workgroup: sync is
// called between the phases).  The columns' range is cut into `nb` equal
// parts; the occupied slots are listed part by part (a count, a prefix, a
// placement), and a column is compared only with those of its own part.
// place(slot, key, rank) is called once per column.  (Comparing every column
// with every other took 0.4 ms for a row of 5,000 columns, most of the time
// of the rows with many.)  list: d entries, part: nb + 1.
template <int THREADS, class Sync, class Place>
__device__ __forceinline__ void rank_columns(const int* keys, unsigned slots, int d, int* list, int* part, int nb,
                                             int* red, int tid, Sync sync, Place place) {
    const int lane = tid & 63;
    int lo = 0x7fffffff, hi = -1;
    for (unsigned h = tid; h < slots; h += THREADS) {
        const int key = keys[h];
        if (key >= 0) {
            lo = min(lo, key);
            hi = max(hi, key);
        }
    }
    for (int b = tid; b <= nb; b += THREADS) part[b] = 0;
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, __shfl_xor(lo, off, 64));
        hi = max(hi, __shfl_xor(hi, off, 64));
    }
    if constexpr (THREADS > 64) {
        if (lane == 0) {
            red[tid >> 6] = lo;
            red[THREADS / 64 + (tid >> 6)] = hi;
        }
        sync();
        for (int w = 0; w < THREADS / 64; ++w) {
            lo = min(lo, red[w]);
            hi = max(hi, red[THREADS / 64 + w]);
        }
    }
    sync();
    // part of column c: floor((c - lo) scale / 2^32), ascending with c, below nb
    const uint64_t scale = (((uint64_t)nb << 32) - 1ull) / ((uint64_t)(unsigned)(hi - lo) + 1ull);
    auto part_of = [&](int key) { return (int)(((uint64_t)(unsigned)(key - lo) * scale) >> 32); };
    for (unsigned h = tid; h < slots; h += THREADS) {
        const int key = keys[h];
        if (key >= 0) atomicAdd(part + part_of(key) + 1, 1);
    }
    sync();
    // part[b + 1] -> end of part b's list; by the first wavefront
    if (tid < 64) {
        int carry = 0;
        for (int b0 = 0; b0 < nb; b0 += 64) {
            const int b = b0 + lane;
            int v = b < nb ? part[b + 1] : 0;
            const int own = v;
            for (int off = 1; off < 64; off <<= 1) {
                const int y = __shfl_up(v, off, 64);
                if (lane >= off) v += y;
            }
            if (b < nb) part[b + 1] = carry + v - own;  // its start, for now
            carry += __shfl(v, 63, 64);
        }
    }
    sync();
    for (unsigned h = tid; h < slots; h += THREADS) {
        const int key = keys[h];
        if (key >= 0) list[min(atomicAdd(part + part_of(key) + 1, 1), d - 1)] = (int)h;
    }
    sync();
    for (int e = tid; e < d; e += THREADS) {
        const int h = list[e], key = keys[h], b = part_of(key);
        const int q0 = part[b], q1 = part[b + 1];
        int r = q0;
        for (int q = q0; q < q1; ++q) r += keys[list[q]] < key ? 1 : 0;
        place(h, key, r);
    }
}

__device__ __forceinline__ int lane_int(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

// the OR over the wavefront, on every lane
__device__ __forceinline__ unsigned wave_or(unsigned x) {
    return (unsigned)lane_int(wave_scan((int)x, [](int a, int b) { return a | b; }), 63);
}

// Adds one step's products to their slots' running sums in LDS, the segments
// s0 .. s1 (see below) one after the other: each is one LDS addition per lane
// with no value returned, and a wavefront's LDS instructions are executed in
// the order they are issued, so a segment neither waits for the one before
// nor overtakes it.  (Reading, adding and writing back behind a fence made
// the segments a chain of about 130 cycles each.)
__device__ __forceinline__ void add_segments(double* acc, bool valid, unsigned h, double pv, int seg, int s0, int s1) {
    for (int sg = s0; sg <= s1; ++sg) {
        if (valid && seg == sg) __hip_atomic_fetch_add(acc + h, pv, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_wave_barrier();
    }
}

// Enumerate the products of row i of A*B in canonical order, 64 per step.
// f(valid, colB, value, t0, total, seg) is called by every lane for each step
// of 64 products starting at t0; lanes past the end get valid = false.  seg
// is the index of the product's A entry within the current chunk of 64 A
// entries: it does not decrease with the lane, and the products of one A
// entry (one B row) have distinct columns.  All cross-lane traffic uses
// shuffles, so every lane executes the same steps.  f returns whether to go
// on; its answer must be the same on every lane.
//
// The chain acol -> brp -> bcol, bval is taken one chunk and one step ahead:
// the next chunk's entries and B-row bounds and the next step's B entries are
// on their way while f works on the current step.
template <bool NEED_VAL>
struct ProductStep {
    int col = 0, seg = 0;
    double a = 0.0, b = 0.0;
    bool valid = false;
    // the step from product t0 on, of a chunk whose entries' products start at
    // excl (blen of them each, the entries without any behind the others)
    __device__ __forceinline__ void fetch(int t0, int total, int excl, int blen, int bstart, double av, const int* bcol,
                                          const double* bval) {
        const int lane = (int)threadIdx.x & 63;
        const int t = t0 + lane;
        valid = t < total;
        // the places where entries' first products lie in the step, as bits:
        // a product belongs to the last entry that starts at or before it
        const int at = excl - t0;
        const bool starts = blen > 0 && at >= 0 && at < 64;
        const unsigned lo = wave_or(starts && at < 32 ? 1u << at : 0u);
        const unsigned hi = wave_or(starts && at >= 32 ? 1u << (at - 32) : 0u);
        const unsigned long long upto = (((unsigned long long)hi << 32) | lo) & ((2ull << lane) - 1ull);
        seg = __popcll(__ballot(blen > 0 && at < 0)) + __popcll(upto) - 1;
        const int sb = __shfl(bstart, seg, 64);
        const int so = __shfl(excl, seg, 64);
        if (NEED_VAL) a = __shfl(av, seg, 64);
        if (valid) {
            const int kb = sb + (t - so);
            col = bcol[kb];
            if (NEED_VAL) b = bval[kb];
        }
    }
};
// one chunk's entries, those without products moved behind the others (an
// exchange of lanes, and only where there are any)
__device__ __forceinline__ void pack_entries(int& bstart, int& blen, double& av) {
    const unsigned long long some = __ballot(blen > 0);
    const int n = __popcll(some);
    if (some == (n == 64 ? ~0ull : (1ull << n) - 1ull)) return;
    const int lane = (int)threadIdx.x & 63;
    const int below = __popcll(some & ((1ull << lane) - 1ull));
    const int to = (blen > 0 ? below : n + lane - below) << 2;
    bstart = __builtin_amdgcn_ds_permute(to, bstart);
    blen = __builtin_amdgcn_ds_permute(to, blen);
    const unsigned long long b = (unsigned long long)__double_as_longlong(av);
    const unsigned l = (unsigned)__builtin_amdgcn_ds_permute(to, (int)(unsigned)b);
    const unsigned h = (unsigned)__builtin_amdgcn_ds_permute(to, (int)(unsigned)(b >> 32));
    av = __longlong_as_double((long long)(((unsigned long long)h << 32) | l));
}
template <bool NEED_VAL, typename F>
__device__ __forceinline__ void for_each_product(const int* arp, const int* acol, const double* aval, const int* brp,
                                                 const int* bcol, const double* bval, int i, F&& f) {
    const int lane = threadIdx.x & 63;
    const int a0 = arp[i], a1 = arp[i + 1];
    int k = 0, bstart = 0, bend = 0;  // (k: the entry's column, of the chunk after the current one)
    double av = 0.0, av1 = 0.0;
    if (a0 + lane < a1) {
        k = acol[a0 + lane];
        if (NEED_VAL) av = aval[a0 + lane];
        bstart = brp[k];
        bend = brp[k + 1];
    }
    if (a0 + 64 + lane < a1) {
        k = acol[a0 + 64 + lane];
        if (NEED_VAL) av1 = aval[a0 + 64 + lane];
    }
    for (int c0 = a0; c0 < a1; c0 += 64) {
        int nstart = 0, nend = 0;
        double av2 = 0.0;
        if (c0 + 64 + lane < a1) {
            nstart = brp[k];
            nend = brp[k + 1];
        }
        if (c0 + 128 + lane < a1) {
            k = acol[c0 + 128 + lane];
            if (NEED_VAL) av2 = aval[c0 + 128 + lane];
        }
        int blen = bend - bstart;
        pack_entries(bstart, blen, av);
        const int incl = scan_add(blen);
        const int excl = incl - blen;
        const int total = lane_int(incl, 63);
        ProductStep<NEED_VAL> next;
        if (total > 0) next.fetch(0, total, excl, blen, bstart, av, bcol, bval);
        for (int t0 = 0; t0 < total; t0 += 64) {
            const ProductStep<NEED_VAL> now = next;
            if (t0 + 64 < total) next.fetch(t0 + 64, total, excl, blen, bstart, av, bcol, bval);
            if (!f(now.valid, now.col, NEED_VAL ? now.a * now.b : 0.0, t0, total, now.seg)) return;
        }
        bstart = nstart;
        bend = nend;
        av = av1;
        av1 = av2;
    }
}

// number of products of row i (sum of the B-row lengths over A's row), on every lane
__device__ __forceinline__ int row_products(const int* arp, const int* acol, const int* brp, int i) {
    const int lane = threadIdx.x & 63;
    int m = 0;
    for (int ka = arp[i] + lane; ka < arp[i + 1]; ka += 64) {
        const int k = acol[ka];
        m += brp[k + 1] - brp[k];
    }
    for (int off = 32; off > 0; off >>= 1) m += __shfl_xor(m, off, 64);
    return m;
}

__device__ __forceinline__ int ld_key(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Memory ordering between the phases of one wavefront's row.  A row's hash
// table is private to one wavefront.  In global memory (long rows) workgroup
// scope orders its accesses; in LDS they are executed in the order they are
// issued, so only the compiler has to keep that order (and loads from global
// memory stay in flight).
template <bool GLOBAL>
__device__ __forceinline__ void phase_fence() {
    __builtin_amdgcn_wave_barrier();
    if constexpr (GLOBAL) __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// slot of a key known to be present in a global-memory table; the probe count
// is bounded by the table size
__device__ __forceinline__ unsigned hash_find_fresh(const int* keys, unsigned mask, int key) {
    unsigned h = hash_slot(key, mask);
    for (unsigned probe = 0; probe <= mask; ++probe) {
        if (ld_key(keys + h) == key) return h;
        h = (h + 1) & mask;
    }
    return 0;
}

// one row (list position ridx) of the symbolic phase, by one wavefront:
// cnt[i] = its distinct columns, or, where they do not fit LDS, 0 with
// flags[i] = 1 and *novf counted up
template <bool GLOBAL>
__device__ void symbolic_row(int ridx, const int* rows, const int* arp, const int* acol, const int* brp,
                             const int* bcol, int* cnt, int* flags, int* novf, int* gkeys, const int64_t* goff,
                             int dmax, int* lds_keys) {
    const int lane = threadIdx.x & 63;
    const int i = rows ? rows[ridx] : ridx;
    int* keys;
    unsigned slots;  // (a power of two in global memory)
    if (GLOBAL) {
        const int64_t o = goff[ridx];
        keys = gkeys + o;
        slots = (unsigned)(goff[ridx + 1] - o);
    } else {
        keys = lds_keys;
        slots = lds_slots(row_products(arp, acol, brp, i), kHS);
    }
    for (unsigned h = lane; h < slots; h += 64) keys[h] = -1;
    phase_fence<GLOBAL>();
    // distinct columns so far (the same on every lane); the LDS path stops as
    // soon as the row cannot fit, so its table never fills up
    int added = 0;
    for_each_product<false>(arp, acol, nullptr, brp, bcol, nullptr, i, [&](bool valid, int c, double, int, int, int) {
        bool fresh = false;
        if (valid) {
            if constexpr (GLOBAL) fresh = hash_insert(keys, slots - 1, c) > 0;
            else (void)lds_insert(keys, slots, c, fresh);
        }
        added += __popcll(__ballot(fresh));
        return GLOBAL || added <= dmax;
    });
    if (lane == 0) {
        const bool over = !GLOBAL && added > dmax;
        cnt[i] = over ? 0 : added;
        if (!GLOBAL) flags[i] = over ? 1 : 0;
        if (over) atomicAdd(novf, 1);
    }
}

// rows [0, nrows) of the list (all rows if rows is null), a wavefront per
// row, grid-stride; nrows_dev (if set) holds the row count on the device
template <bool GLOBAL>
__global__ __launch_bounds__(kBlock) void k_spgemm_symbolic(int nrows, const int* nrows_dev, const int* rows,
                                                            const int* arp, const int* acol, const int* brp,
                                                            const int* bcol, int* cnt, int* flags, int* novf,
                                                            int* gkeys, const int64_t* goff, int dmax) {
    __shared__ __align__(16) int skeys[GLOBAL ? 1 : kWaves][GLOBAL ? 4 : kHS];
    const int w = threadIdx.x >> 6;
    const int nr = nrows_dev ? *nrows_dev : nrows;
    for (int ridx = blockIdx.x * kWaves + w; ridx < nr; ridx += gridDim.x * kWaves)
        symbolic_row<GLOBAL>(ridx, rows, arp, acol, brp, bcol, cnt, flags, novf, gkeys, goff, dmax,
                             skeys[GLOBAL ? 0 : w]);
}

// Row i of the numeric phase, by one wavefront on its LDS table of at most HS
// slots (rows of at most DM columns).  One walk over the products: each takes
// its column's hash slot (inserting the column on first sight) and is added to
// that slot's running sum in canonical order, the segments of a step one after
// the other; then the occupied slots are ranked by column and written out.
// Every entry receives the same additions in the same order as in the two walks
// of numeric_row_global (a zeroed sum plus the first product, then the others).
template <int HS, int DM>
__device__ void numeric_row_lds(int i, const int* arp, const int* acol, const double* aval, const int* brp,
                                const int* bcol, const double* bval, const int* crp, int* ccol, double* cval, int* keys,
                                int* vals, double* acc) {
    const int lane = threadIdx.x & 63;
    const int base = crp[i];
    const int d = crp[i + 1] - base;
    const unsigned slots = lds_slots(d, HS);
    for (unsigned h = lane; h < slots; h += 64) {
        keys[h] = -1;
        acc[h] = 0.0;
    }
    phase_fence<false>();
    for_each_product<true>(arp, acol, aval, brp, bcol, bval, i,
                           [&](bool valid, int c, double pv, int t0, int total, int seg) {
                               bool fresh;
                               const unsigned h = valid ? lds_insert(keys, slots, c, fresh) : 0u;
                               add_segments(acc, valid, h, pv, seg, lane_int(seg, 0),
                                            lane_int(seg, min(64, total - t0) - 1));
                               return true;
                           });
    phase_fence<false>();
    if (d <= 64) {
        // a lane per column, compared with all
        int filled = 0, h = 0;
        for (unsigned h0 = 0; h0 < slots; h0 += 64) {
            const bool occ = h0 + lane < slots && keys[h0 + lane] >= 0;
            const uint64_t bal = __ballot(occ);
            if (occ) vals[filled + __popcll(bal & ((1ull << lane) - 1ull))] = (int)h0 + lane;
            filled += __popcll(bal);
        }
        phase_fence<false>();
        int key = 0x7fffffff;
        if (lane < d) {
            h = vals[lane];
            key = keys[h];
        }
        int r = 0;
        for (int q = 0; q < d; ++q) r += lane_int(key, q) < key ? 1 : 0;
        if (lane < d) {
            ccol[base + r] = key;
            cval[base + r] = acc[h];
        }
    } else {
        rank_columns<64>(keys, slots, d, vals, vals + DM, rank_parts(DM), nullptr, lane, [] { phase_fence<false>(); },
                         [&](int h, int key, int r) {
                             ccol[base + r] = key;
                             cval[base + r] = acc[h];
                         });
    }
    phase_fence<false>();  // the tables are reused by the wavefront's next row
}

// Overflow row i (list position ridx) of more columns than any LDS table takes,
// by one wavefront on its table in global memory: the columns are ranked first,
// then the products are accumulated by rank in a second walk.
__device__ void numeric_row_global(int ridx, int i, const int* arp, const int* acol, const double* aval, const int* brp,
                                   const int* bcol, const double* bval, const int* crp, int* ccol, double* cval,
                                   int* gkeys, int* gvals, double* gacc, const int64_t* goff, int* tile) {
    const int lane = threadIdx.x & 63;
    const int64_t o = goff[ridx];
    int *keys = gkeys + o, *vals = gvals + o;
    double* acc = gacc + o;
    const unsigned mask = (unsigned)(goff[ridx + 1] - o) - 1;
    for (unsigned h = lane; h <= mask; h += 64) {
        keys[h] = -1;
        vals[h] = 0;
    }
    phase_fence<true>();
    for_each_product<false>(arp, acol, nullptr, brp, bcol, nullptr, i,
                            [&](bool valid, int c, double, int, int, int) {
                                if (valid) (void)hash_insert(keys, mask, c);
                                return true;
                            });
    phase_fence<true>();
    // compact the occupied slots (arbitrary order) into the output column range
    const int base = crp[i];
    const int d = crp[i + 1] - base;
    int* cl = ccol + base;
    int filled = 0;
    for (unsigned h0 = 0; h0 <= mask; h0 += 64) {
        const unsigned h = h0 + lane;
        const int key = (h <= mask) ? ld_key(keys + h) : -1;
        const bool occ = key >= 0;
        const uint64_t bal = __ballot(occ);
        const int before = __popcll(bal & ((1ull << lane) - 1ull));
        if (occ && filled + before < d) cl[filled + before] = key;
        filled += __popcll(bal);
    }
    phase_fence<true>();
    // rank of each column among the row's columns = its output position:
    // kRankKeys keys per lane at a time, compared against the list staged
    // through LDS in tiles
    for (int e0 = 0; e0 < d; e0 += 64 * kRankKeys) {
        int c[kRankKeys], r[kRankKeys];
#pragma unroll
        for (int u = 0; u < kRankKeys; ++u) {
            const int e = e0 + u * 64 + lane;
            c[u] = e < d ? cl[e] : -1;
            r[u] = 0;
        }
        for (int t0 = 0; t0 < d; t0 += kRankTile) {
            const int tn = min(kRankTile, d - t0);
            for (int q = lane; q < tn; q += 64) tile[q] = cl[t0 + q];
            phase_fence<false>();
            for (int q = 0; q < tn; ++q) {
                const int v = tile[q];
#pragma unroll
                for (int u = 0; u < kRankKeys; ++u) r[u] += (v < c[u]) ? 1 : 0;
            }
            phase_fence<false>();
        }
#pragma unroll
        for (int u = 0; u < kRankKeys; ++u)
            if (c[u] >= 0) vals[hash_find_fresh(keys, mask, c[u])] = r[u];
    }
    phase_fence<true>();
    for (unsigned h = lane; h <= mask; h += 64) {
        const int key = ld_key(keys + h);
        const int r = vals[h];
        if (key >= 0 && r >= 0 && r < d) cl[r] = key;
    }
    for (int e = lane; e < d; e += 64) acc[e] = 0.0;
    phase_fence<true>();
    // Accumulate in canonical product order.  The products of one A entry
    // (a segment) have distinct columns, so a segment's lanes add their
    // products to their columns' running values at once; the segments of a
    // step go one after the other in order, and steps follow each other in
    // product order.  Every entry therefore receives exactly the sequence of
    // additions of a serial row product.
    for_each_product<true>(arp, acol, aval, brp, bcol, bval, i,
                           [&](bool valid, int c, double pv, int t0, int total, int seg) {
                               int r = valid ? vals[hash_find_fresh(keys, mask, c)] : 0;
                               r = (r >= 0 && r < d) ? r : 0;
                               const int m = min(64, total - t0);
                               const int s0 = __shfl(seg, 0, 64), s1 = __shfl(seg, m - 1, 64);
                               for (int sg = s0; sg <= s1; ++sg) {
                                   if (valid && seg == sg) acc[r] += pv;
                                   phase_fence<true>();
                               }
                               return true;
                           });
    phase_fence<true>();
    for (int e = lane; e < d; e += 64) cval[base + e] = acc[e];
}

// The rows of the list whose distinct column count lies in (mlo, mhi] (known
// from the symbolic phase: rows of many products but few columns take the small
// tables) and that did not overflow (skip), with HS hash slots and room for DM =
// mhi columns per wavefront.  A wavefront per row, grid-stride over runs of up to
// eight rows whose counts its lanes read together (one row after the other, the
// rows that are not this launch's cost a memory latency each); nrows_dev (if set)
// holds the count.
template <int HS, int DM>
__global__ __launch_bounds__(kBlock) void k_spgemm_numeric(int nrows, const int* nrows_dev, const int* rows,
                                                           const int* arp, const int* acol, const double* aval,
                                                           const int* brp, const int* bcol, const double* bval,
                                                           const int* crp, int* ccol, double* cval, const int* skip,
                                                           int mlo, int mhi) {
    __shared__ __align__(16) int skeys[kWaves][HS];
    __shared__ int svals[kWaves][DM + rank_parts(DM) + 1];  // see rank_columns
    __shared__ double sacc[kWaves][HS];                     // one running sum per hash slot
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nr = nrows_dev ? *nrows_dev : nrows;
    const int waves = (int)gridDim.x * kWaves;
    const int take = max(1, min(8, nr / waves));
    for (int first = (blockIdx.x * kWaves + w) * take; first < nr; first += waves * take) {
        int row = 0;
        bool mine = false;
        if (lane < take && first + lane < nr) {
            row = rows ? rows[first + lane] : first + lane;
            const int dc = crp[row + 1] - crp[row];
            mine = dc > mlo && dc <= mhi && !(skip && skip[row]);
        }
        for (unsigned long long left = __ballot(mine); left; left &= left - 1ull)
            numeric_row_lds<HS, DM>(lane_int(row, __builtin_ctzll(left)), arp, acol, aval, brp, bcol, bval, crp, ccol,
                                    cval, skeys[w], svals[w], sacc[w]);
    }
}

// the listed overflow rows of more than mlo columns (the others take the large
// LDS table), a wavefront per row
__global__ __launch_bounds__(kBlock) void k_spgemm_numeric_global(int nrows, const int* rows, const int* arp,
                                                                  const int* acol, const double* aval, const int* brp,
                                                                  const int* bcol, const double* bval, const int* crp,
                                                                  int* ccol, double* cval, int* gkeys, int* gvals,
                                                                  double* gacc, const int64_t* goff, int mlo) {
    __shared__ int stile[kWaves][kRankTile];
    const int w = threadIdx.x >> 6;
    for (int ridx = blockIdx.x * kWaves + w; ridx < nrows; ridx += gridDim.x * kWaves) {
        const int i = rows[ridx];
        if (crp[i + 1] - crp[i] > mlo)
            numeric_row_global(ridx, i, arp, acol, aval, brp, bcol, bval, crp, ccol, cval, gkeys, gvals, gacc, goff,
                               stile[w]);
    }
}

// Overflow row i with at most kDBig columns, by a whole workgroup of kWaves
// wavefronts on one table in LDS.  Within each chunk of 64 A entries the
// wavefronts take the chunk's steps of 64 products in turn (wavefront w the
// steps w, w + kWaves, ...): in a round each loads its step's products and
// takes their columns' hash slots (inserting a column on first sight), then
// the round's steps are added to the slots' running sums in step order, one
// wavefront after the other between barriers, each step's segments one
// after the other.  Every entry thus receives the additions of a serial row
// product in the same order (a zeroed sum plus the first product, then the
// others), while kWaves steps' loads are in flight at once.  The occupied
// slots are then ranked by column and written out.
__device__ void numeric_row_big(int i, const int* arp, const int* acol, const double* aval, const int* brp,
                                const int* bcol, const double* bval, const int* crp, int* ccol, double* cval,
                                int* keys, int* vals, double* acc, int* red) {
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int base = crp[i];
    const int d = crp[i + 1] - base;
    const unsigned slots = lds_slots(d, kHSBig), buckets = slots / kBucket;
    for (unsigned h = tid; h < slots; h += kBlock) {
        keys[h] = -1;
        acc[h] = 0.0;
    }
    __syncthreads();
    const int a0 = arp[i], a1 = arp[i + 1];
    int k = 0, bstart = 0, bend = 0;  // as in for_each_product: one chunk ahead
    double av = 0.0, av1 = 0.0;
    if (a0 + lane < a1) {
        k = acol[a0 + lane];
        av = aval[a0 + lane];
        bstart = brp[k];
        bend = brp[k + 1];
    }
    if (a0 + 64 + lane < a1) {
        k = acol[a0 + 64 + lane];
        av1 = aval[a0 + 64 + lane];
    }
    for (int c0 = a0; c0 < a1; c0 += 64) {
        int nstart = 0, nend = 0;
        double av2 = 0.0;
        if (c0 + 64 + lane < a1) {
            nstart = brp[k];
            nend = brp[k + 1];
        }
        if (c0 + 128 + lane < a1) {
            k = acol[c0 + 128 + lane];
            av2 = aval[c0 + 128 + lane];
        }
        int blen = bend - bstart;
        pack_entries(bstart, blen, av);
        const int incl = scan_add(blen);
        const int excl = incl - blen;
        const int total = lane_int(incl, 63);
        const int nsteps = (total + 63) / 64;  // the same in every wavefront
        ProductStep<true> next;
        if (w < nsteps) next.fetch(w * 64, total, excl, blen, bstart, av, bcol, bval);
        for (int sr = 0; sr < nsteps; sr += kWaves) {
            const int st = sr + w;
            const ProductStep<true> now = next;
            if (st + kWaves < nsteps) next.fetch((st + kWaves) * 64, total, excl, blen, bstart, av, bcol, bval);
            const bool any = st < nsteps;
            const bool valid = any && now.valid;
            const unsigned h = valid ? bucket_insert(keys, buckets, now.col) : 0u;
            const double pv = now.a * now.b;
            const int m = any ? min(64, total - st * 64) : 1;
            const int s0 = lane_int(now.seg, 0), s1 = lane_int(now.seg, m - 1);
            for (int q = 0; q < kWaves; ++q) {
                if (q == w && any) add_segments(acc, valid, h, pv, now.seg, s0, s1);
                __syncthreads();
            }
        }
        bstart = nstart;
        bend = nend;
        av = av1;
        av1 = av2;
    }
    __syncthreads();
    rank_columns<kBlock>(keys, slots, d, vals, vals + kDBig, rank_parts(kDBig), red, tid, [] { __syncthreads(); },
                         [&](int h, int key, int r) {
                             ccol[base + r] = key;
                             cval[base + r] = acc[h];
                         });
    __syncthreads();  // the tables are reused by the workgroup's next row
}

// the listed overflow rows with at most kDBig columns: a workgroup per row,
// with a hash table of up to kHSBig slots, one running sum per slot, in
// dynamic LDS
__global__ __launch_bounds__(kBlock) void k_spgemm_numeric_big(int nrows, const int* rows, const int* arp,
                                                               const int* acol, const double* aval, const int* brp,
                                                               const int* bcol, const double* bval, const int* crp,
                                                               int* ccol, double* cval, int dbig) {
    extern __shared__ __align__(16) unsigned char big_lds[];
    __shared__ int red[2 * kWaves];
    double* sacc = reinterpret_cast<double*>(big_lds);
    int* skeys = reinterpret_cast<int*>(sacc + kHSBig);
    int* svals = skeys + kHSBig;
    for (int ridx = blockIdx.x; ridx < nrows; ridx += gridDim.x) {
        const int i = rows[ridx];
        if (crp[i + 1] - crp[i] > dbig) continue;  // block-uniform
        numeric_row_big(i, arp, acol, aval, brp, bcol, bval, crp, ccol, cval, skeys, svals, sacc, red);
    }
}

// --------------------------------------------------- one thread per row
// Rows with at most kThreadCols distinct output columns (most rows of the
// finer levels' products) are multiplied by one thread each: the thread walks
// its row's products in the canonical order and keeps the distinct columns,
// in order of first appearance, in registers with their running sums; the
// sorted output position of each is its rank among them.  Every entry
// therefore gets the same additions, in the same order, as on the wavefront
// path.  A row with more than kThreadProducts products takes the wavefront
// path even when its columns would fit: each product costs a thread a
// compare against every register slot, a wavefront one hash probe per lane
// (the coarse levels' Galerkin rows collapse hundreds of products into few
// columns).
constexpr int kThreadCols = 32;
constexpr int kThreadProducts = 64;

// add product (c, v) to the row's column list key/acc[0..d) of S slots (v
// when VAL); returns false when a new column does not fit
template <bool VAL, int S>
__device__ __forceinline__ bool thread_row_add(int (&key)[S], double (&acc)[S], int& d, int c, double v) {
    bool found = false;
#pragma unroll
    for (int j = 0; j < S; ++j)
        if (key[j] == c) {
            found = true;
            if constexpr (VAL) acc[j] += v;
        }
    if (found) return true;
    if (d == S) return false;
#pragma unroll
    for (int j = 0; j < S; ++j)
        if (j == d) {
            key[j] = c;
            if constexpr (VAL) acc[j] = 0.0 + v;  // as the wavefront path: a zeroed sum plus the first product
        }
    ++d;
    return true;
}

// the products of row i in canonical order, f(column, value): A's row in
// chunks of CH entries whose column, B-row bounds and first B entry are all
// loaded before any is used (P rows mostly hold one entry), so a chunk costs
// three memory latencies instead of three per entry.  f returns whether to
// go on.
template <bool VAL, int CH, typename F>
__device__ __forceinline__ void thread_row_products(const int* arp, const int* acol, const double* aval,
                                                    const int* brp, const int* bcol, const double* bval, int i,
                                                    F&& f) {
    const int a0 = arp[i], a1 = arp[i + 1];
    for (int c0 = a0; c0 < a1; c0 += CH) {
        int kk[CH], b0[CH], b1[CH], fc[CH];
        double av[CH], fv[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int ka = min(c0 + u, a1 - 1);
            kk[u] = acol[ka];
            av[u] = VAL ? aval[ka] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            b0[u] = brp[kk[u]];
            b1[u] = brp[kk[u] + 1];
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int kb = b0[u] < b1[u] ? b0[u] : 0;
            fc[u] = bcol[kb];
            fv[u] = VAL ? bval[kb] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            if (c0 + u >= a1 || b0[u] >= b1[u]) continue;
            if (!f(fc[u], VAL ? av[u] * fv[u] : 0.0)) return;
            for (int kb = b0[u] + 1; kb < b1[u]; ++kb)
                if (!f(bcol[kb], VAL ? av[u] * bval[kb] : 0.0)) return;
        }
    }
}

// symbolic: cnt[i] = distinct columns and wide[i] = 0 for rows that fit (at
// most kThreadCols columns from at most kThreadProducts products); wide[i] =
// 1 (and cnt[i] untouched) for the others, whose walk stops where they stop
// fitting
__global__ __launch_bounds__(kBlock) void k_spgemm_symbolic_thread(int n, const int* arp, const int* acol,
                                                                   const int* brp, const int* bcol, int* cnt,
                                                                   int* flags, int* wide, int tprod) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        int key[kThreadCols];
        double acc[kThreadCols];
#pragma unroll
        for (int j = 0; j < kThreadCols; ++j) key[j] = -1;
        int d = 0, m = 0;
        bool fits = true;
        thread_row_products<false, 8>(arp, acol, nullptr, brp, bcol, nullptr, i, [&](int c, double) {
            fits = ++m <= tprod && thread_row_add<false, kThreadCols>(key, acc, d, c, 0.0);
            return fits;
        });
        wide[i] = fits ? 0 : 1;
        if (fits) {
            cnt[i] = d;
            flags[i] = 0;
        }
    }
}

// numeric for the rows the thread symbolic pass kept whose column count
// lies in (dlo, S], with S register slots (fewer slots for narrower rows:
// fewer registers and compares per product; the additions are the same)
template <int S>
__global__ __launch_bounds__(kBlock) void k_spgemm_numeric_thread(int n, const int* arp, const int* acol,
                                                                  const double* aval, const int* brp,
                                                                  const int* bcol, const double* bval,
                                                                  const int* wide, const int* crp, int* ccol,
                                                                  double* cval, int dlo) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        if (wide[i]) continue;
        const int base = crp[i];
        const int dr = crp[i + 1] - base;
        if (dr <= dlo || dr > S) continue;
        int key[S];
        double acc[S];
#pragma unroll
        for (int j = 0; j < S; ++j) {
            key[j] = -1;
            acc[j] = 0.0;
        }
        int d = 0;
        thread_row_products<true, 4>(arp, acol, aval, brp, bcol, bval, i, [&](int c, double v) {
            (void)thread_row_add<true, S>(key, acc, d, c, v);
            return true;
        });
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (key[j] < 0) continue;
            int r = 0;
#pragma unroll
            for (int q = 0; q < S; ++q) r += (key[q] >= 0 && key[q] < key[j]) ? 1 : 0;
            ccol[base + r] = key[j];
            cval[base + r] = acc[j];
        }
    }
}

__global__ void k_list_flagged(int n, const int* flags, const int* pos, int* list) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        if (flags[i]) list[pos[i]] = i;
}

// product-count upper bound of each listed row, as a hash table size (power
// of two >= 2*m): a wavefront per row, lane-strided over its A entries
__global__ __launch_bounds__(kBlock) void k_row_table_size(int nrows, const int* rows, const int* arp,
                                                           const int* acol, const int* brp, int ncols,
                                                           int64_t* size) {
    const int w = (int)threadIdx.x >> 6;
    for (int r = blockIdx.x * kWaves + w; r < nrows; r += gridDim.x * kWaves) {
        int64_t m = row_products(arp, acol, brp, rows[r]);
        if (m > ncols) m = ncols;
        int64_t t = 64;
        while (t < 2 * m) t <<= 1;
        if ((threadIdx.x & 63) == 0) size[r] = t;
    }
}

// out = {*a, *b}, for one read-back of two device values
__global__ void k_pair(const int* a, const int* b, int* out) {
    out[0] = *a;
    out[1] = *b;
}

// exclusive scan of n 64-bit values by one block, kBlock at a time with a
// running carry (overflow rows are few)
__global__ __launch_bounds__(kBlock) void k_scan64(int n, const int64_t* in, int64_t* out) {
    __shared__ int64_t sh[kBlock];
    int64_t carry = 0;
    for (int b = 0; b < n; b += kBlock) {
        const int i = b + (int)threadIdx.x;
        const int64_t v = i < n ? in[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        // inclusive Hillis-Steele scan in LDS
        for (int off = 1; off < kBlock; off <<= 1) {
            const int64_t y = (int)threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
            __syncthreads();
            sh[threadIdx.x] += y;
            __syncthreads();
        }
        if (i < n) out[i] = carry + sh[threadIdx.x] - v;
        carry += sh[kBlock - 1];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[n] = carry;
}

// ---------------------------------------------------------------- transpose
__global__ void k_col_counts(int64_t nnz, const int* col, int* cnt) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += (int64_t)gridDim.x * blockDim.x)
        atomicAdd(cnt + col[k], 1);
}

// the transpose's entries, in the order the atomic slots hand out within
// each row, with each entry's row
__global__ void k_transpose_fill(int n, const int* rp, const int* col, const double* val, const int* trp,
                                 int* fill, int* tcol, double* tval, int* trow) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        for (int k = rp[i]; k < rp[i + 1]; ++k) {
            const int c = col[k];
            const int p = trp[c] + atomicAdd(fill + c, 1);
            tcol[p] = i;
            tval[p] = val[k];
            trow[p] = c;
        }
    }
}

// Rows of the transpose up to this long are put in column order by ranking;
// longer ones are sorted in place afterwards
constexpr int kRankRow = 256;

// Each entry to its place in column order.  A row's columns (the source
// rows) are distinct, so an entry's place is the number of the row's
// columns below its own: one thread per entry, reading the row with
// independent loads.  Entries of longer rows are copied where they are.
__global__ void k_rank_place(int64_t nnz, const int* trp, const int* trow, const int* tcol, const double* tval,
                             int* col, double* val) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < nnz; e += (int64_t)gridDim.x * blockDim.x) {
        const int j = trow[e];
        const int lo = trp[j], hi = trp[j + 1];
        const int c = tcol[e];
        int64_t pos = e;
        if (hi - lo <= kRankRow) {
            int r = 0;
            for (int k = lo; k < hi; ++k) r += tcol[k] < c ? 1 : 0;
            pos = lo + r;
        }
        col[pos] = c;
        val[pos] = tval[e];
    }
}

// insertion sort of the rows longer than kRankRow, one thread per row
__global__ void k_sort_pairs(int n, const int* rp, int* col, double* val) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int lo = rp[i], hi = rp[i + 1];
        if (hi - lo <= kRankRow) continue;
        for (int a = lo + 1; a < hi; ++a) {
            const int c = col[a];
            const double v = val[a];
            int b = a - 1;
            while (b >= lo && col[b] > c) {
                col[b + 1] = col[b];
                val[b + 1] = val[b];
                --b;
            }
            col[b + 1] = c;
            val[b + 1] = v;
        }
    }
}

inline int g1(int64_t n) {
    int g = ceil_div(n > 0 ? n : 1, kBlock);
    return g < 65535 ? g : 65535;
}

// The rows' routes: at most tprod products (and kThreadCols columns) for one
// thread, at most dmax columns for a wavefront's LDS table, at most dbig for
// a workgroup's, a global-memory table beyond.  MATAMG_SPGEMM_ROUTE=t,d,b
// lowers them (the tests send rows down every path: every route adds the
// same products in the same order).
struct Route {
    int tprod = kThreadProducts, dmax = kDMax, dbig = kDBig;
};

// The thread route is left out where the device has threads to spare: its
// rows are chains of dependent loads and compares, about 100 us a kernel
// however few they are (A P of 6,400 rows 371 us, 43 us with a wavefront
// each; 115,700 rows 455 and 260 us; 274,700 rows 511 and 490 us; a million
// rows 1.09 and 2.0 ms).  Products with few terms a row (the filtered
// operator times the tentative prolongator) keep it at every size: 40 and 60
// us at 27,400 rows.
constexpr int kThreadMinRows = 262144;
constexpr double kThreadFewProducts = 16.0;

Route spgemm_route(const DCsr& A, const DCsr& B) {
    Route r;
    if (A.n < kThreadMinRows && A.n > 0 && B.n > 0 &&
        (double)A.nnz / A.n * ((double)B.nnz / B.n) >= kThreadFewProducts)
        r.tprod = 0;
    const char* e = std::getenv("MATAMG_SPGEMM_ROUTE");
    int t = 0, d = 0, b = 0;
    if (e && std::sscanf(e, "%d,%d,%d", &t, &d, &b) == 3) {
        r.tprod = std::max(0, std::min(t, kThreadProducts));
        r.dmax = std::max(0, std::min(d, kDMax));
        r.dbig = std::max(0, std::min(b, kDBig));
    }
    return r;
}

}  // namespace

void spgemm(const DCsr& A, const DCsr& B, DCsr& C, MemCounter* mc, hipStream_t s) {
    const Route route = spgemm_route(A, B);
    const int n = A.n;
    C.n = n;
    C.m = B.m;
    const int nn = n > 0 ? n : 1;
    const bool threads = route.tprod > 0;
    DBuf<int> cnt((size_t)nn, mc), flags((size_t)nn, mc), tmp(scan_tmp_size(n), mc), novf_dev(4, mc);
    DBuf<int> wide, wpos, wl;  // rows for the wavefronts (all of them where the thread route is off)
    C.rowptr.alloc((size_t)n + 1, mc);
    // wavefront launches loop over a row list whose length stays on the device
    const int wgrid = std::max(1, std::min(ceil_div(nn, kWaves), 8192));
    const int* nwide_dev = nullptr;
    const int* wlist = nullptr;
    zero_async(novf_dev.get(), sizeof(int), s);
    if (n > 0) {
        if (threads) {
            wide.alloc((size_t)nn, mc);
            wpos.alloc((size_t)n + 1, mc);
            wl.alloc((size_t)nn, mc);
            nwide_dev = wpos.get() + n;
            wlist = wl.get();
            hipLaunchKernelGGL(k_spgemm_symbolic_thread, dim3(g1(n)), dim3(kBlock), 0, s, n, A.rowptr.get(),
                               A.col.get(), B.rowptr.get(), B.col.get(), cnt.get(), flags.get(), wide.get(),
                               route.tprod);
            exclusive_scan(wide.get(), wpos.get(), n, tmp.get(), s);
            hipLaunchKernelGGL(k_list_flagged, dim3(g1(n)), dim3(kBlock), 0, s, n, (const int*)wide.get(),
                               (const int*)wpos.get(), wl.get());
        }
        hipLaunchKernelGGL((k_spgemm_symbolic<false>), dim3(wgrid), dim3(kBlock), 0, s, n, nwide_dev, wlist,
                           A.rowptr.get(), A.col.get(), B.rowptr.get(), B.col.get(), cnt.get(), flags.get(),
                           novf_dev.get(), (int*)nullptr, (const int64_t*)nullptr, route.dmax);
        MATAMG_LAUNCH_CHECK();
    }
    // the row pointer as if no row overflowed
    exclusive_scan(cnt.get(), C.rowptr.get(), n, tmp.get(), s);
    int head[2] = {0, 0};  // overflow rows, stored entries
    hipLaunchKernelGGL(k_pair, dim3(1), dim3(1), 0, s, (const int*)novf_dev.get(), (const int*)C.rowptr.get() + n,
                       novf_dev.get() + 2);
    d2h(head, novf_dev.get() + 2, 2, s);
    const int novf = head[0];
    int nnz = head[1];
    DBuf<int> list;
    DBuf<int64_t> tsize, toff;
    DBuf<int> gkeys, gvals;
    DBuf<double> gacc;
    if (novf > 0) {
        // rows with more distinct columns than the LDS table holds
        DBuf<int> pos((size_t)n + 1, mc);
        exclusive_scan(flags.get(), pos.get(), n, tmp.get(), s);
        list.alloc((size_t)novf, mc);
        hipLaunchKernelGGL(k_list_flagged, dim3(g1(n)), dim3(kBlock), 0, s, n, (const int*)flags.get(),
                           (const int*)pos.get(), list.get());
        tsize.alloc((size_t)novf, mc);
        toff.alloc((size_t)novf + 1, mc);
        hipLaunchKernelGGL(k_row_table_size, dim3(std::min(ceil_div(novf, kWaves), 8192)), dim3(kBlock), 0, s, novf,
                           list.get(), A.rowptr.get(), A.col.get(), B.rowptr.get(), B.m, tsize.get());
        hipLaunchKernelGGL(k_scan64, dim3(1), dim3(kBlock), 0, s, novf, tsize.get(), toff.get());
        int64_t tot = 0;
        d2h(&tot, toff.get() + novf, 1, s);
        gkeys.alloc((size_t)tot, mc);
        gvals.alloc((size_t)tot, mc);
        gacc.alloc((size_t)tot, mc);
        hipLaunchKernelGGL((k_spgemm_symbolic<true>), dim3(ceil_div(novf, kWaves)), dim3(kBlock), 0, s, novf,
                           (const int*)nullptr, list.get(), A.rowptr.get(), A.col.get(), B.rowptr.get(), B.col.get(),
                           cnt.get(), (int*)nullptr, (int*)nullptr, gkeys.get(), toff.get(), route.dmax);
        MATAMG_LAUNCH_CHECK();
        exclusive_scan(cnt.get(), C.rowptr.get(), n, tmp.get(), s);
        d2h(&nnz, C.rowptr.get() + n, 1, s);
    }
    C.nnz = nnz;
    C.col.alloc((size_t)(nnz > 0 ? nnz : 1), mc);
    C.val.alloc((size_t)(nnz > 0 ? nnz : 1), mc);
    if (n > 0) {
        if (threads) {
            hipLaunchKernelGGL(k_spgemm_numeric_thread<kThreadCols / 2>, dim3(g1(n)), dim3(kBlock), 0, s, n,
                               A.rowptr.get(), A.col.get(), A.val.get(), B.rowptr.get(), B.col.get(), B.val.get(),
                               (const int*)wide.get(), C.rowptr.get(), C.col.get(), C.val.get(), -1);
            hipLaunchKernelGGL(k_spgemm_numeric_thread<kThreadCols>, dim3(g1(n)), dim3(kBlock), 0, s, n, A.rowptr.get(),
                               A.col.get(), A.val.get(), B.rowptr.get(), B.col.get(), B.val.get(),
                               (const int*)wide.get(), C.rowptr.get(), C.col.get(), C.val.get(), kThreadCols / 2);
        }
        // wide rows with few distinct columns: small tables, so more
        // wavefronts fit a CU
        auto numeric = [&](auto kernel, int mlo, int mhi) {
            hipLaunchKernelGGL(kernel, dim3(wgrid), dim3(kBlock), 0, s, n, nwide_dev, wlist, A.rowptr.get(),
                               A.col.get(), A.val.get(), B.rowptr.get(), B.col.get(), B.val.get(), C.rowptr.get(),
                               C.col.get(), C.val.get(), (const int*)flags.get(), mlo, mhi);
        };
        numeric(k_spgemm_numeric<kNumSlots[0], kNumCols[0]>, -1, kNumCols[0]);
        if (n >= kNumThreeSizes) numeric(k_spgemm_numeric<kNumSlots[1], kNumCols[1]>, kNumCols[0], kNumCols[1]);
        numeric(k_spgemm_numeric<kNumSlots[2], kNumCols[2]>, n >= kNumThreeSizes ? kNumCols[1] : kNumCols[0],
                kNumCols[2]);
        MATAMG_LAUNCH_CHECK();
    }
    if (novf > 0) {
        // the dynamic LDS limit, raised once per process (thread-safe static)
        static const bool big_lds_set = [] {
            MATAMG_HIP(hipFuncSetAttribute((const void*)k_spgemm_numeric_big,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBigLds));
            return true;
        }();
        (void)big_lds_set;
        hipLaunchKernelGGL(k_spgemm_numeric_big, dim3(std::min(novf, 4096)), dim3(kBlock), kBigLds, s, novf,
                           (const int*)list.get(), A.rowptr.get(), A.col.get(), A.val.get(), B.rowptr.get(),
                           B.col.get(), B.val.get(), (const int*)C.rowptr.get(), C.col.get(), C.val.get(),
                           route.dbig);
        hipLaunchKernelGGL(k_spgemm_numeric_global, dim3(ceil_div(novf, kWaves)), dim3(kBlock), 0, s, novf,
                           (const int*)list.get(), A.rowptr.get(), A.col.get(), A.val.get(), B.rowptr.get(), B.col.get(),
                           B.val.get(), (const int*)C.rowptr.get(), C.col.get(), C.val.get(), gkeys.get(), gvals.get(),
                           gacc.get(), (const int64_t*)toff.get(), route.dbig);
        MATAMG_LAUNCH_CHECK();
    }
    // no synchronisation: temporaries go back to the pool in stream order
}

void transpose(const DCsr& A, DCsr& T, MemCounter* mc, hipStream_t s) {
    const int n = A.n, m = A.m;
    T.n = m;
    T.m = n;
    T.nnz = A.nnz;
    DBuf<int> cnt((size_t)(m > 0 ? m : 1), mc);
    zero_async(cnt.get(), sizeof(int) * (size_t)(m > 0 ? m : 1), s);
    if (A.nnz > 0)
        hipLaunchKernelGGL(k_col_counts, dim3(g1(A.nnz)), dim3(kBlock), 0, s, A.nnz, A.col.get(), cnt.get());
    T.rowptr.alloc((size_t)m + 1, mc);
    DBuf<int> tmp(scan_tmp_size(m), mc);
    exclusive_scan(cnt.get(), T.rowptr.get(), m, tmp.get(), s);
    zero_async(cnt.get(), sizeof(int) * (size_t)(m > 0 ? m : 1), s);
    const size_t nz = (size_t)(A.nnz > 0 ? A.nnz : 1);
    T.col.alloc(nz, mc);
    T.val.alloc(nz, mc);
    DBuf<int> tcol(nz, mc), trow(nz, mc);
    DBuf<double> tval(nz, mc);
    if (n > 0)
        hipLaunchKernelGGL(k_transpose_fill, dim3(g1(n)), dim3(kBlock), 0, s, n, A.rowptr.get(), A.col.get(),
                           A.val.get(), T.rowptr.get(), cnt.get(), tcol.get(), tval.get(), trow.get());
    if (A.nnz > 0)
        hipLaunchKernelGGL(k_rank_place, dim3(g1(A.nnz)), dim3(kBlock), 0, s, A.nnz, (const int*)T.rowptr.get(),
                           (const int*)trow.get(), (const int*)tcol.get(), (const double*)tval.get(), T.col.get(),
                           T.val.get());
    if (m > 0)
        hipLaunchKernelGGL(k_sort_pairs, dim3(g1(m)), dim3(kBlock), 0, s, m, T.rowptr.get(), T.col.get(),
                           T.val.get());
    MATAMG_LAUNCH_CHECK();
}

}  // namespace matamg

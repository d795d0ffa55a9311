// Dynamic embedding table of MTGR's training framework (Sec. 5, "Dynamic Hash Table" and
// "Embedding Lookup"): a compact key store (open addressing, linear probing over 64-bit IDs)
// decoupled from the value store (embedding rows plus an occurrence counter and the time of
// the last lookup per row), a hash-set de-duplication of each batch, lookup with insertion,
// the gather of a batch's rows, a sparse SGD step, eviction by time and a rebuild of the key
// store at another capacity.
//
// Every kernel is a bounded grid-stride loop; every probe loop is bounded by the capacity it
// walks.  Concurrency inside one call: distinct IDs race only for free slots (atomicCAS on the
// 64-bit key) and for free rows (atomic counters); an ID's own slot and row are touched by one
// thread, so its metadata needs no atomics.
#include <type_traits>

#include "../../include/mtgr_embedding.h"
#include "mtgr_device.h"
#include "mtgr_internal.h"

namespace mtgr {
namespace {

constexpr uint64_t KEY_EMPTY = 0xFFFFFFFFFFFFFFFFull;
constexpr uint64_t KEY_DELETED = 0xFFFFFFFFFFFFFFFEull;
constexpr int THREADS = 256;

// 64-bit finalizer of MurmurHash3 (public domain): spreads every input bit over the word.
__device__ __forceinline__ uint64_t mix64(uint64_t k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return k;
}

__device__ __forceinline__ uint64_t load_key(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t cas_key(uint64_t* p, uint64_t expect, uint64_t value) {
    return atomicCAS((unsigned long long*)p, (unsigned long long)expect, (unsigned long long)value);
}

__device__ __forceinline__ long long grid_threads() { return (long long)gridDim.x * blockDim.x; }
__device__ __forceinline__ long long thread_id() { return (long long)blockIdx.x * blockDim.x + threadIdx.x; }

__global__ void fill_u64_kernel(uint64_t* p, long long n, uint64_t v) {
    for (long long i = thread_id(); i < n; i += grid_threads()) p[i] = v;
}
__global__ void fill_i32_kernel(int* p, long long n, int v) {
    for (long long i = thread_id(); i < n; i += grid_threads()) p[i] = v;
}
__global__ void zero_i64_kernel(long long* p) { *p = 0; }

// ------------------------------------------------------------------------ de-duplication
// Each workgroup takes TPB PER consecutive IDs and first de-duplicates them in an LDS hash set
// (LDS integer atomics are cheap), then inserts each of its distinct IDs once into the global set
// (capacity tmask + 1 >= 2 n).  Skewed batches repeat a few hot IDs thousands of times; counting
// them in LDS first keeps the global atomics on a hot ID to two per workgroup.  Whoever brings an
// ID into the set gives it the next place of the unique list (one atomic per workgroup), so the
// list needs no scan of the set, and writes its count there; the others add theirs to the entry.
// pos[i] = the global slot of ids[i]; uslot[u] = that of unique[u].
//
// Bound by the latency of the dependent memory operations and by the atomics on the hottest IDs'
// entries (one insertion and one count per workgroup, one after another), not by bytes.  So the
// distinct IDs are compacted first and a thread's up to PER insertions are in flight together; an
// entry (key, place, count) is 16 bytes of one line; and a workgroup takes as many IDs as leave one
// workgroup per CU: 256 up to 65,536 IDs, 1,024 up to 262,144, else 4,096.
// Measured, 556,504 Zipf IDs (319,887 distinct): whole de-duplication 96 -> 68 us, of which the
// insertions' atomics take about a third (18 us without any); 12,000 IDs: 31 us of insertion in 12
// workgroups of 1,024 IDs -> 10 us.
struct __align__(16) SetEntry {
    uint64_t key;
    int rank;       // place in the unique list
    int occ;        // occurrences in other workgroups than the one that brought it in
};
constexpr long long BATCH_SMALL = 256 * 256, BATCH_MEDIUM = 256 * 1024;    // (see above)

template <int TPB>
__device__ __forceinline__ int block_scan_exclusive(int v, int* total) {
    __shared__ int wsum[TPB / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < TPB / 64; i++) {
        before += i < w ? wsum[i] : 0;
        all += wsum[i];
    }
    __syncthreads();   // wsum is reused by the next call
    *total = all;
    return before + incl - v;
}

__global__ void dedup_clear_kernel(SetEntry* set, long long tcap, long long* num_unique) {
    for (long long i = thread_id(); i < tcap; i += grid_threads())
        ((uint4*)set)[i] = make_uint4(0xffffffffu, 0xffffffffu, 0u, 0u);
    if (thread_id() == 0) *num_unique = 0;
}

template <int TPB, int PER>
__global__ __launch_bounds__(TPB) void dedup_insert_kernel(long long n, const uint64_t* __restrict__ ids,
                                                               SetEntry* set, int* __restrict__ pos, long long tmask,
                                                               uint64_t* __restrict__ unique, int* __restrict__ uslot,
                                                               int* __restrict__ occ_out, long long* num_unique) {
    constexpr int CHUNK = TPB * PER, LCAP = 2 * CHUNK;
    __shared__ uint64_t lkeys[LCAP];
    __shared__ int lcount[LCAP];
    __shared__ int lslot[LCAP];
    __shared__ int llist[CHUNK];
    __shared__ int lnum, lbase;
    const long long i0 = (long long)blockIdx.x * CHUNK;
    uint64_t id[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        id[k] = i < n ? ids[i] : 0;
    }
    for (int e = threadIdx.x; e < LCAP; e += TPB) {
        lkeys[e] = KEY_EMPTY;
        lcount[e] = 0;
    }
    if (threadIdx.x == 0) lnum = 0;
    __syncthreads();
    int mine[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        mine[k] = -1;
        if (i >= n) continue;
        int p = (int)(mix64(id[k]) & (LCAP - 1));
        for (int step = 0; step < LCAP; step++) {
            const uint64_t old = atomicCAS((unsigned long long*)&lkeys[p], (unsigned long long)KEY_EMPTY,
                                           (unsigned long long)id[k]);
            if (old == KEY_EMPTY) llist[atomicAdd(&lnum, 1)] = p;
            if (old == KEY_EMPTY || old == id[k]) break;
            p = (p + 1) & (LCAP - 1);
        }
        atomicAdd(&lcount[p], 1);
        mine[k] = p;
    }
    __syncthreads();
    const int num = lnum;
    uint64_t key[PER], old[PER];
    long long at[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int e = threadIdx.x + k * TPB;
        key[k] = e < num ? lkeys[llist[e]] : KEY_EMPTY;
        at[k] = (long long)(mix64(key[k]) & (uint64_t)tmask);
        old[k] = e < num ? cas_key(&set[at[k]].key, KEY_EMPTY, key[k]) : key[k];
    }
    int fresh = 0;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int e = threadIdx.x + k * TPB;
        for (long long step = 0; step <= tmask && old[k] != KEY_EMPTY && old[k] != key[k]; step++) {
            at[k] = (at[k] + 1) & tmask;
            old[k] = cas_key(&set[at[k]].key, KEY_EMPTY, key[k]);
        }
        if (e < num) {
            if (old[k] != KEY_EMPTY) atomicAdd(&set[at[k]].occ, lcount[llist[e]]);
            lslot[llist[e]] = (int)at[k];
            fresh += old[k] == KEY_EMPTY ? 1 : 0;
        }
    }
    int total;
    int r = block_scan_exclusive<TPB>(fresh, &total);
    if (threadIdx.x == 0) lbase = (int)atomicAdd((unsigned long long*)num_unique, (unsigned long long)total);
    __syncthreads();
    r += lbase;
#pragma unroll
    for (int k = 0; k < PER; k++) {
        if (threadIdx.x + k * TPB < num && old[k] == KEY_EMPTY) {
            set[at[k]].rank = r;
            unique[r] = key[k];
            uslot[r] = (int)at[k];
            if (occ_out) occ_out[r] = lcount[llist[threadIdx.x + k * TPB]];
            r++;
        }
    }
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        if (i < n) pos[i] = lslot[mine[k]];
    }
}

// inverse of every position and the occurrences of every unique ID (their number is at most n).
__global__ void dedup_finish_kernel(long long n, const SetEntry* __restrict__ set, const int* __restrict__ pos,
                                    const int* __restrict__ uslot, const long long* __restrict__ num_unique,
                                    int* __restrict__ inverse, int* __restrict__ occ_out) {
    const long long nu = occ_out ? *num_unique : 0;
    for (long long i = thread_id(); i < n; i += grid_threads()) {
        inverse[i] = set[pos[i]].rank;
        if (i < nu) occ_out[i] += set[uslot[i]].occ;
    }
}

// ------------------------------------------------------------------------ lookup / insert
// Rows for `n` IDs, taken by one thread: the top of the free-row stack, then the never-used rows.  The
// k-th ID's row is row_of(grant, k), -1 when both are used up.  What was taken beyond the supply is
// given back at once.  While any of it is outstanding the stack top is <= 0 and the row counter >=
// the capacity, so nobody else mistakes it for supply.
struct RowGrant {
    int top, take;              // stack entries top - 1 .. top - take
    uint32_t next;              // then rows from here on, below the capacity
};
__device__ __forceinline__ RowGrant take_rows(const EmbArgs& t, int n) {
    int* top_p = t.state + MTGR_EMB_STATE_FREE_TOP;
    uint32_t* next_p = (uint32_t*)(t.state + MTGR_EMB_STATE_NEXT_ROW);
    const uint32_t cap = (uint32_t)t.row_capacity;
    RowGrant g = {0, 0, 0u};
    uint32_t over = 0;
    if (__hip_atomic_load(top_p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0) {
        g.top = atomicSub(top_p, n);
        g.take = min(max(g.top, 0), n);
        if (g.take < n) atomicAdd(top_p, n - g.take);
    }
    const uint32_t rest = (uint32_t)(n - g.take);
    if (rest) {
        g.next = atomicAdd(next_p, rest);
        const uint32_t end = g.next + rest;
        over = end > cap ? min(end - cap, rest) : 0u;
        if (over) atomicSub(next_p, over);
    }
    if ((uint32_t)n > over) atomicAdd(t.state + MTGR_EMB_STATE_NUM_KEYS, n - (int)over);
    return g;
}
__device__ __forceinline__ int row_of(const EmbArgs& t, const RowGrant& g, int k) {
    if (k < g.take) return t.free_rows[g.top - 1 - k];
    const uint32_t r = g.next + (uint32_t)(k - g.take);
    return r < (uint32_t)t.row_capacity ? (int)r : -1;
}

__device__ __forceinline__ void zero_row(const EmbArgs& t, int row) {
    uint4* v = (uint4*)((char*)t.values + (long long)row * t.dim * t.esize);
    const int chunks = t.dim * t.esize / 16;
    for (int c = 0; c < chunks; c++) v[c] = make_uint4(0, 0, 0, 0);
}

// Finds each ID's slot, or (insert) claims one: the first DELETED slot met on the probe path if the
// path ends at an EMPTY slot without the ID, else that EMPTY slot; then rows for the claimed
// slots, counters and timestamps.  The IDs of a call are distinct, so no other thread reads a
// slot claimed here, and one launch does both.
// Insertion is bound by the atomics on the table's state (one cache line, one after another), so a
// workgroup takes the rows of its new IDs at once: 556,504 new IDs 108 us, against 710 us with one
// grant per wave (12,000: 9 us).  Up to 65,536 IDs workgroups of 256 reach more CUs, beyond it those of
// 512 make fewer grants; those of 1,024 insert faster still (92 us), but look up 320,000 known IDs in 18.0
// instead of 14.4 us.
// (Finding and finishing used to be two launches and the clamping of the state a third: 24 us for
// 319,887 IDs, 11 us for 8,000; now 27 and 5 us.  The unique list used to come in the order of the
// set, in which the probes walk the key store; the scans that gave it that order cost 23 us.  Beyond
// about two million distinct IDs in one call the order was worth more than the scans: de-duplication and
// lookup of 1.5 million known ones 270 -> 262 us, of 4 million 650 -> 710, of 16 million 2,770 -> 3,410 us;
// of 4 and 16 million Zipf IDs 490 -> 485 and 1,970 -> 2,100 us.)
template <int TPB>
__global__ __launch_bounds__(TPB) void lookup_kernel(EmbArgs t, long long n_max, const uint64_t* __restrict__ unique,
                              const int* __restrict__ occurrences, const long long* __restrict__ num_unique, int now,
                              int insert, int* __restrict__ rows) {
    const long long nu = min(*num_unique, n_max);
    const long long mask = t.key_capacity - 1;
    __shared__ RowGrant grant;
    for (long long base = (long long)blockIdx.x * TPB; base < nu; base += grid_threads()) {
        const long long u = base + threadIdx.x;
        const bool mine = u < nu;
        const uint64_t key = mine ? unique[u] : 0;
        long long p = (long long)(mix64(key) & (uint64_t)mask);
        long long tomb = -1, slot = -1;
        bool fresh = false, done = !mine;
        for (long long step = 0; step < 2 * t.key_capacity && !done; step++) {
            const uint64_t k = load_key(t.keys + p);
            if (k == key) {
                slot = p;
                done = true;
            } else if (k == KEY_DELETED) {
                if (tomb < 0) tomb = p;
                p = (p + 1) & mask;
            } else if (k == KEY_EMPTY) {
                if (!insert) {
                    done = true;   // absent
                } else {
                    const long long tgt = tomb >= 0 ? tomb : p;
                    const uint64_t expect = tomb >= 0 ? KEY_DELETED : KEY_EMPTY;
                    if (cas_key(t.keys + tgt, expect, key) == expect) {
                        slot = tgt;
                        fresh = true;
                        done = true;
                    } else if (tomb >= 0) {
                        tomb = -1;           // another ID took the deleted slot: look at p again
                    } else {
                        p = (p + 1) & mask;  // another ID took this empty slot
                    }
                }
            } else {
                p = (p + 1) & mask;
            }
        }
        if (!done && insert && tomb >= 0 && cas_key(t.keys + tomb, KEY_DELETED, key) == KEY_DELETED) {
            slot = tomb;   // the whole store was walked: no EMPTY slot, but a DELETED one
            fresh = true;
            done = true;
        }
        if (!done && insert) atomicOr(t.state + MTGR_EMB_STATE_OVERFLOW, 2);
        int row = -1;
        if (insert) {                     // (the same for every thread, as the loop's trips are)
            int total;
            const int k = block_scan_exclusive<TPB>(fresh ? 1 : 0, &total);
            if (total) {
                if (threadIdx.x == 0) grant = take_rows(t, total);
                __syncthreads();
                if (fresh) row = row_of(t, grant, k);
            }
        }
        if (!mine) continue;
        if (fresh) {
            if (row < 0) {
                // No row: release the slot as DELETED (IDs inserted meanwhile may have probed
                // past it, so it must not become EMPTY).
                __hip_atomic_store(t.keys + slot, KEY_DELETED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicOr(t.state + MTGR_EMB_STATE_OVERFLOW, 1);
            } else {
                t.key_rows[slot] = row;
                zero_row(t, row);
            }
        } else if (slot >= 0) {
            row = t.key_rows[slot];
        }
        if (row >= 0) {
            t.counts[row] = (fresh ? 0u : t.counts[row]) + (occurrences ? (uint32_t)occurrences[u] : 1u);
            t.last_ts[row] = now;
        }
        rows[u] = row;
    }
}

// ------------------------------------------------------------------------ gather / sgd
// One thread per 16-byte chunk of an output row.
__global__ void gather_kernel(EmbArgs t, long long n, const int* __restrict__ inverse,
                              const int* __restrict__ rows, void* __restrict__ out, long long ld_out) {
    const int cpr = t.dim * t.esize / 16;
    const long long total = n * cpr;
    for (long long c = thread_id(); c < total; c += grid_threads()) {
        const long long i = c / cpr;
        const int j = (int)(c - i * cpr);
        const int row = rows[inverse[i]];
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row >= 0) v = ((const uint4*)((const char*)t.values + (long long)row * t.dim * t.esize))[j];
        ((uint4*)((char*)out + i * ld_out * t.esize))[j] = v;
    }
}

__device__ __forceinline__ void load_chunk(const void* base, int esize, float* f) {
    const uint4 v = *(const uint4*)base;
    if (esize == 2) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; e++) {
            f[2 * e] = __uint_as_float(w[e] << 16);
            f[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
        }
    } else {
        f[0] = __uint_as_float(v.x);
        f[1] = __uint_as_float(v.y);
        f[2] = __uint_as_float(v.z);
        f[3] = __uint_as_float(v.w);
    }
}

// One chunk of a row plus -lr times a sum, rounded to the table's dtype.
template <int ESIZE>
__device__ __forceinline__ void apply_chunk(void* vp, uint4 old, const float* g, float lr) {
    constexpr int epc = 16 / ESIZE;
    float f[8];
    load_chunk(&old, ESIZE, f);
#pragma unroll
    for (int e = 0; e < epc; e++) f[e] = __builtin_fmaf(-lr, g[e], f[e]);
    uint4 v;
    if constexpr (ESIZE == 2)
        v = make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                       pack_bf16x2(f[6], f[7]));
    else
        v = make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    *(uint4*)vp = v;
}

// The SGD step groups the positions by unique ID (a counting sort over the occurrences, in any
// order of the IDs), then sums runs of equal IDs and applies each whole run to its row at once.
// A workgroup of the sum owns sgd_positions(dim) consecutive places of the grouped list; the IDs
// that reach beyond one (few: at most one per workgroup boundary) add their parts with float atomics into
// an accumulator row of the workgroup they start in, which a last small kernel applies.
struct SgdWork {
    float* acc;       // [groups][dim]
    int* span;        // [groups]: the ID that starts in this workgroup and reaches beyond it, or -1
    int* total;       // [1]: places handed out
    int* cursor;      // [n_max]: next free place of each ID; its end after the scatter
    int2* list;       // [n]: {position, ID}
    long long groups;
};

__global__ void sgd_clear_kernel(SgdWork w, int dim) {
    for (long long i = thread_id(); i < w.groups * dim; i += grid_threads()) w.acc[i] = 0.f;
    for (long long i = thread_id(); i < w.groups; i += grid_threads()) w.span[i] = -1;
    if (thread_id() == 0) *w.total = 0;
}

// Disjoint ranges of the list for the IDs: a scan inside the workgroup, one atomic per workgroup.
constexpr int START_PER = 4;
__global__ __launch_bounds__(THREADS) void sgd_start_kernel(SgdWork w, const int* __restrict__ occ,
                                                            const long long* __restrict__ num, long long n_max) {
    __shared__ int lbase;
    const long long nv = min(*num, n_max);
    const long long base = ((long long)blockIdx.x * THREADS + threadIdx.x) * START_PER;
    int v[START_PER], c = 0;
#pragma unroll
    for (int e = 0; e < START_PER; e++) {
        v[e] = base + e < nv ? occ[base + e] : 0;
        c += v[e];
    }
    int total;
    int r = block_scan_exclusive<THREADS>(c, &total);
    if (threadIdx.x == 0) lbase = total ? atomicAdd(w.total, total) : 0;
    __syncthreads();
    r += lbase;
#pragma unroll
    for (int e = 0; e < START_PER; e++) {
        if (base + e < nv) w.cursor[base + e] = r;
        r += v[e];
    }
}

// Places of the positions.  A workgroup takes TPB PER positions and counts its IDs in an LDS hash
// first, so a hot ID costs one global atomic per workgroup; its positions then take consecutive
// places from the range reserved there.  TPB and PER as in the de-duplication.
template <int TPB, int PER>
__global__ __launch_bounds__(TPB) void sgd_scatter_kernel(SgdWork w, long long n, const int* __restrict__ inverse) {
    constexpr int CHUNK = TPB * PER, LCAP = 2 * CHUNK;
    __shared__ int lkey[LCAP];
    __shared__ int lcount[LCAP];
    __shared__ int lbase[LCAP];
    __shared__ int llist[CHUNK];
    __shared__ int lnum;
    const long long i0 = (long long)blockIdx.x * CHUNK;
    int u[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        u[k] = i < n ? inverse[i] : 0;
    }
    for (int e = threadIdx.x; e < LCAP; e += TPB) {
        lkey[e] = -1;
        lcount[e] = 0;
    }
    if (threadIdx.x == 0) lnum = 0;
    __syncthreads();
    int slot[PER], rank[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        slot[k] = -1;
        rank[k] = 0;
        if (i >= n) continue;
        int p = (int)(((uint32_t)u[k] * 2654435761u) >> 16) & (LCAP - 1);
        for (int step = 0; step < LCAP; step++) {
            const int old = atomicCAS(&lkey[p], -1, u[k]);
            if (old == -1) llist[atomicAdd(&lnum, 1)] = p;
            if (old == -1 || old == u[k]) break;
            p = (p + 1) & (LCAP - 1);
        }
        rank[k] = atomicAdd(&lcount[p], 1);
        slot[k] = p;
    }
    __syncthreads();
    const int num = lnum;
    int got[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const int e = threadIdx.x + k * TPB;
        got[k] = e < num ? atomicAdd(w.cursor + lkey[llist[e]], lcount[llist[e]]) : 0;
    }
#pragma unroll
    for (int k = 0; k < PER; k++)
        if (threadIdx.x + k * TPB < num) lbase[llist[threadIdx.x + k * TPB]] = got[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; k++) {
        const long long i = i0 + threadIdx.x + (long long)k * TPB;
        if (i >= n) continue;
        const int p = lbase[slot[k]] + rank[k];
        if (p < n) w.list[p] = make_int2((int)i, u[k]);   // always, for occurrences consistent with inverse
    }
}

// Chunks of a workgroup (one thread per chunk and 16-byte column block) and places per chunk: at
// most 1024 places per workgroup, 32 per thread.
__host__ __device__ __forceinline__ int sgd_chunks(int dim, int esize) { return THREADS / (dim * esize / 16); }
__host__ __device__ __forceinline__ int sgd_chunk_len(int chunks) { return chunks > 32 ? 1024 / chunks : 32; }

// Bound by the random 128-byte gradient and value rows (dim 64, bf16); per thread eight positions'
// gradient and value chunks are in flight together, the list and rows come in through LDS once
// per workgroup, and a run inside a chunk is a whole ID, which needs no look at its range.
// Measured, 556,504 gradients of 64 bf16: sum and apply 91 + 26 us and 19 us of clearing a row of
// fp32 sums per ID -> 47 us (154 MB, 3.3 TB/s); the whole step 200 -> 83 us.
template <int ESIZE>
__global__ __launch_bounds__(THREADS) void sgd_sum_kernel(EmbArgs t, SgdWork w, long long n, long long n_max,
                                                          const int* __restrict__ occ, const int* __restrict__ rows,
                                                          const void* __restrict__ grad, long long ld_grad, float lr) {
    constexpr int epc = 16 / ESIZE, UNR = 8;
    __shared__ int lpos[1024];
    __shared__ int lid[1024];
    __shared__ int lrow[1024];
    __shared__ float first_part[THREADS][epc];
    __shared__ float last_part[THREADS][epc];
    const int cpr = t.dim / epc;                       // column blocks per row (<= THREADS here)
    const int cpb = sgd_chunks(t.dim, ESIZE), len = sgd_chunk_len(cpb);
    const long long P0 = (long long)blockIdx.x * cpb * len;
    const int cnt = (int)min((long long)cpb * len, n - P0);
    for (int p = threadIdx.x; p < cnt; p += THREADS) {
        const int2 e = w.list[P0 + p];
        // (for inconsistent occurrences the list has holes: nothing is read through them)
        const bool in = e.x >= 0 && e.x < n && e.y >= 0 && e.y < n_max;
        lpos[p] = in ? e.x : -1;
        lid[p] = in ? e.y : -1;
        lrow[p] = in ? rows[e.y] : -1;
    }
    __syncthreads();
    const int c = threadIdx.x / cpr, j = threadIdx.x - c * cpr;
    const int p0 = c * len, p1 = c < cpb ? min(cnt, p0 + len) : p0;
    char* vbase = (char*)t.values + (long long)j * 16;
    const long long vstride = (long long)t.dim * ESIZE;
    float f[epc];
#pragma unroll
    for (int e = 0; e < epc; e++) f[e] = 0.f;
    int cur = -1, crow = -1, runs = 0, first_id = -1;
    uint4 cval = make_uint4(0, 0, 0, 0);
    for (int pb = p0; pb < p1; pb += UNR) {
        uint4 g[UNR], v[UNR];
        int uu[UNR], rr[UNR];
#pragma unroll
        for (int k = 0; k < UNR; k++) {
            const bool in = pb + k < p1;
            const int i = in ? lpos[pb + k] : -1;
            uu[k] = in ? lid[pb + k] : -1;
            rr[k] = in ? lrow[pb + k] : -1;
            g[k] = v[k] = make_uint4(0, 0, 0, 0);
            if (i >= 0) g[k] = *(const uint4*)((const char*)grad + (long long)i * ld_grad * ESIZE + (long long)j * 16);
            if (rr[k] >= 0) v[k] = *(const uint4*)(vbase + rr[k] * vstride);
        }
#pragma unroll
        for (int k = 0; k < UNR; k++) {
            if (uu[k] < 0) continue;
            if (uu[k] != cur) {
                if (runs == 1) {            // the chunk's first run: to LDS
                    first_id = cur;
#pragma unroll
                    for (int e = 0; e < epc; e++) first_part[threadIdx.x][e] = f[e];
                } else if (runs > 1 && crow >= 0) {   // a run strictly inside the chunk: a whole ID
                    apply_chunk<ESIZE>(vbase + crow * vstride, cval, f, lr);
                }
                cur = uu[k];
                runs++;
#pragma unroll
                for (int e = 0; e < epc; e++) f[e] = 0.f;
            }
            crow = rr[k];
            cval = v[k];
            float gk[8];
            load_chunk(&g[k], ESIZE, gk);
#pragma unroll
            for (int e = 0; e < epc; e++) f[e] += gk[e];
        }
    }
    // Chunk c's first run (first_id, when it holds more than one) and last run (cur) are merged with
    // equal IDs of the neighbouring chunks by the thread of the chunk where the ID begins.
    __shared__ int first_u[THREADS];
    __shared__ int last_u[THREADS];
    first_u[threadIdx.x] = first_id;
    last_u[threadIdx.x] = cur;
#pragma unroll
    for (int e = 0; e < epc; e++) last_part[threadIdx.x][e] = f[e];
    // The IDs that reach beyond the workgroup, 0: over its start, 1: over its end only; their sums go out
    // together at the end, whole lines per atomic instruction (one ID in all of 556,504 positions, dim 8:
    // 8 atomics of one lane per workgroup made the step 104 us, 97.5 us before places were 1,024 per
    // workgroup; now 75).
    __shared__ float span_sum[2][1024];
    __shared__ int span_id[2];
    __shared__ long long span_group[2];
    if (threadIdx.x < 2) span_id[threadIdx.x] = -1;
    __syncthreads();
    // sum (from this chunk) of ID u whose part here is `part`; `reach`: it is the chunk's last run
    auto finish = [&](int u, const float* part, bool reach, int row, uint4 val) {
        float r[epc];
#pragma unroll
        for (int e = 0; e < epc; e++) r[e] = part[e];
        bool to_end = false;      // reaches the workgroup's last place
        if (reach) {
            // the chunks that hold nothing but u, then the first run of the next one; a hot ID fills
            // up to 256 chunks, so their sums are read eight at a time (one after another: 1,000
            // gradients of one ID, dim 8, 79 us; now 26)
            const int chunks = min(cpb, (cnt + len - 1) / len);
            int cc = c + 1;
            for (bool open = true; open && cc < chunks;) {
                float q[8][epc];
                int fu[8], lu[8], whole = 0;
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    const int pair = min(cc + k, chunks - 1) * cpr + j;
                    fu[k] = first_u[pair];
                    lu[k] = last_u[pair];
#pragma unroll
                    for (int e = 0; e < epc; e++) q[k][e] = last_part[pair][e];
                }
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    open = open & (cc + k < chunks) & (fu[k] < 0) & (lu[k] == u);
                    whole += open ? 1 : 0;
#pragma unroll
                    for (int e = 0; e < epc; e++) r[e] = open ? r[e] + q[k][e] : r[e];
                }
                cc += whole;
            }
            if (cc < chunks && first_u[cc * cpr + j] == u) {
#pragma unroll
                for (int e = 0; e < epc; e++) r[e] += first_part[cc * cpr + j][e];
            }
            to_end = cc >= chunks;
        }
        const bool from_start = c == 0 && lid[0] == u;
        long long group = blockIdx.x;
        bool spans = false;
        if (from_start || to_end) {
            const long long end = w.cursor[u], start = end - occ[u];
            spans = start < P0 || end > P0 + cnt;
            group = start / ((long long)cpb * len);
        }
        if (!spans) {
            if (row >= 0) apply_chunk<ESIZE>(vbase + row * vstride, val, r, lr);
        } else if (group >= 0 && group < w.groups) {
            const int which = from_start ? 0 : 1;
#pragma unroll
            for (int e = 0; e < epc; e++) span_sum[which][j * epc + e] = r[e];
            if (j == 0) {
                span_id[which] = u;
                span_group[which] = group;
            }
        }
    };
    const int before = c > 0 ? last_u[threadIdx.x - cpr] : -1;
    if (runs > 1 && first_id != before) {
        const int row = lrow[p0];
        const uint4 val = row >= 0 ? *(const uint4*)(vbase + row * vstride) : make_uint4(0, 0, 0, 0);
        finish(first_id, first_part[threadIdx.x], false, row, val);
    }
    if (runs > 1 || (runs == 1 && cur != before)) finish(cur, last_part[threadIdx.x], true, crow, cval);
    __syncthreads();
#pragma unroll
    for (int which = 0; which < 2; which++) {
        if (span_id[which] < 0) continue;
        const long long group = span_group[which];
        for (int e = threadIdx.x; e < t.dim; e += THREADS) atomicAdd(w.acc + group * t.dim + e, span_sum[which][e]);
        if (threadIdx.x == 0 && group == blockIdx.x) w.span[group] = span_id[which];
    }
}

// The IDs that span workgroups: values[rows[u], :] -= lr * their accumulated sums.
template <int ESIZE>
__global__ void sgd_span_kernel(EmbArgs t, SgdWork w, const int* __restrict__ rows, float lr) {
    constexpr int epc = 16 / ESIZE;
    const int cpr = t.dim / epc;
    const long long total = w.groups * cpr;
    for (long long i = thread_id(); i < total; i += grid_threads()) {
        const long long grp = i / cpr;
        const int u = w.span[grp], j = (int)(i - grp * cpr);
        if (u < 0) continue;
        const int row = rows[u];
        if (row < 0) continue;
        char* vp = (char*)t.values + ((long long)row * t.dim + (long long)j * epc) * ESIZE;
        apply_chunk<ESIZE>(vp, *(const uint4*)vp, w.acc + grp * t.dim + j * epc, lr);
    }
}

// ------------------------------------------------------------------------ evict / rehash
__global__ void evict_kernel(EmbArgs t, int threshold, uint32_t min_count, long long* num_evicted) {
    for (long long p = thread_id(); p < t.key_capacity; p += grid_threads()) {
        const uint64_t k = t.keys[p];
        if (k >= KEY_DELETED) continue;
        const int row = t.key_rows[p];
        if (row < 0 || (t.last_ts[row] >= threshold && t.counts[row] >= min_count)) continue;
        t.keys[p] = KEY_DELETED;
        t.key_rows[p] = -1;
        const int i = atomicAdd(t.state + MTGR_EMB_STATE_FREE_TOP, 1);
        t.free_rows[i] = row;
        atomicSub(t.state + MTGR_EMB_STATE_NUM_KEYS, 1);
        atomicAdd((unsigned long long*)num_evicted, 1ull);
    }
}

__global__ void rehash_kernel(EmbArgs from, EmbArgs to) {
    const long long mask = to.key_capacity - 1;
    for (long long p = thread_id(); p < from.key_capacity; p += grid_threads()) {
        const uint64_t key = from.keys[p];
        if (key >= KEY_DELETED) continue;
        long long q = (long long)(mix64(key) & (uint64_t)mask);
        bool placed = false;
        for (long long step = 0; step < to.key_capacity && !placed; step++) {
            if (cas_key(to.keys + q, KEY_EMPTY, key) == KEY_EMPTY) {
                to.key_rows[q] = from.key_rows[p];
                placed = true;
            } else {
                q = (q + 1) & mask;
            }
        }
        if (!placed) atomicOr(to.state + MTGR_EMB_STATE_OVERFLOW, 2);
    }
}

int grid_for(long long work) {
    const long long blocks = (work + THREADS - 1) / THREADS;
    return (int)max(1ll, min(blocks, 8192ll));
}

}  // namespace

size_t dedup_set_capacity(long long n) {
    size_t c = 64;
    while ((long long)c < 2 * n) c <<= 1;
    return c;
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t dedup_workspace_bytes(long long n) {
    return align256(dedup_set_capacity(n) * sizeof(SetEntry)) + 2 * align256((size_t)n * 4);
}

hipError_t launch_emb_init(const EmbArgs& t, hipStream_t s) {
    fill_u64_kernel<<<grid_for(t.key_capacity), THREADS, 0, s>>>(t.keys, t.key_capacity, KEY_EMPTY);
    fill_i32_kernel<<<grid_for(t.key_capacity), THREADS, 0, s>>>(t.key_rows, t.key_capacity, -1);
    fill_i32_kernel<<<1, THREADS, 0, s>>>(t.state, MTGR_EMB_STATE_WORDS, 0);
    return hipGetLastError();
}

// f(threads, IDs per thread) of the kernels that de-duplicate in LDS, by the batch's size.
template <class F>
static void by_batch(long long n, F f) {
    using std::integral_constant;
    if (n <= BATCH_SMALL) f(integral_constant<int, 256>{}, integral_constant<int, 1>{});
    else if (n <= BATCH_MEDIUM) f(integral_constant<int, 1024>{}, integral_constant<int, 1>{});
    else f(integral_constant<int, 1024>{}, integral_constant<int, 4>{});
}

hipError_t launch_emb_dedup(long long n, const uint64_t* ids, uint64_t* unique, int* occ, int* inverse,
                            long long* num_unique, void* ws, hipStream_t s) {
    const long long tcap = (long long)dedup_set_capacity(n);
    SetEntry* set = (SetEntry*)ws;
    int* pos = (int*)((char*)ws + align256(tcap * sizeof(SetEntry)));
    int* uslot = (int*)((char*)pos + align256((size_t)n * 4));
    dedup_clear_kernel<<<grid_for(tcap), THREADS, 0, s>>>(set, tcap, num_unique);
    if (n > 0) {
        by_batch(n, [&](auto tpb, auto per) {
            constexpr int TPB = decltype(tpb)::value, PER = decltype(per)::value;
            dedup_insert_kernel<TPB, PER><<<(int)((n + TPB * PER - 1) / (TPB * PER)), TPB, 0, s>>>(
                n, ids, set, pos, tcap - 1, unique, uslot, occ, num_unique);
        });
        dedup_finish_kernel<<<grid_for(n), THREADS, 0, s>>>(n, set, pos, uslot, num_unique, inverse, occ);
    }
    return hipGetLastError();
}

hipError_t launch_emb_lookup(const EmbArgs& t, long long n_max, const uint64_t* unique, const int* occ,
                             const long long* num_unique, int now, int insert, int* rows, hipStream_t s) {
    if (n_max <= BATCH_SMALL)
        lookup_kernel<THREADS><<<grid_for(n_max), THREADS, 0, s>>>(t, n_max, unique, occ, num_unique, now, insert, rows);
    else
        lookup_kernel<512><<<(int)min((n_max + 511) / 512, 4096ll), 512, 0, s>>>(t, n_max, unique, occ, num_unique,
                                                                                   now, insert, rows);
    return hipGetLastError();
}

hipError_t launch_emb_gather(const EmbArgs& t, long long n, const int* inverse, const int* rows, void* out,
                             long long ld_out, hipStream_t s) {
    const long long chunks = n * (t.dim * t.esize / 16);
    gather_kernel<<<grid_for(chunks), THREADS, 0, s>>>(t, n, inverse, rows, out, ld_out);
    return hipGetLastError();
}

// Workspace of the SGD step at `ws`, its size in *bytes.
static SgdWork sgd_work(long long n, long long n_max, int dim, int esize, void* ws, size_t* bytes) {
    const int cpb = sgd_chunks(dim, esize);
    const long long places = (long long)cpb * sgd_chunk_len(cpb);
    SgdWork w;
    w.groups = (n + places - 1) / places;
    char* p = (char*)ws;
    auto take = [&](size_t b) {
        char* r = p;
        p += align256(b);
        return r;
    };
    w.acc = (float*)take((size_t)w.groups * dim * sizeof(float));
    w.span = (int*)take((size_t)w.groups * sizeof(int));
    w.total = (int*)take(sizeof(int));
    w.cursor = (int*)take((size_t)n_max * sizeof(int));
    w.list = (int2*)take((size_t)n * sizeof(int2));
    *bytes = (size_t)(p - (char*)ws);
    return w;
}

// (the query does not know the table's dtype: the larger of both)
size_t sgd_workspace_bytes(long long n, long long n_max, int dim) {
    size_t b2, b4;
    sgd_work(n, n_max, dim, 2, nullptr, &b2);
    sgd_work(n, n_max, dim, 4, nullptr, &b4);
    return max(b2, b4);
}

hipError_t launch_emb_sgd(const EmbArgs& t, long long n, const int* inverse, const int* occ, const void* grad,
                          long long ld_grad, long long n_max, const int* rows, const long long* num_unique,
                          float lr, void* ws, hipStream_t s) {
    if (n == 0) return hipSuccess;
    size_t bytes;
    const SgdWork w = sgd_work(n, n_max, t.dim, t.esize, ws, &bytes);
    const int starts = START_PER * THREADS;
    sgd_clear_kernel<<<grid_for(w.groups * t.dim), THREADS, 0, s>>>(w, t.dim);
    sgd_start_kernel<<<(int)((n_max + starts - 1) / starts), THREADS, 0, s>>>(w, occ, num_unique, n_max);
    by_batch(n, [&](auto tpb, auto per) {
        constexpr int TPB = decltype(tpb)::value, PER = decltype(per)::value;
        sgd_scatter_kernel<TPB, PER><<<(int)((n + TPB * PER - 1) / (TPB * PER)), TPB, 0, s>>>(w, n, inverse);
    });
    const int spans = grid_for(w.groups * (t.dim * t.esize / 16));
    if (t.esize == 2) {
        sgd_sum_kernel<2><<<(int)w.groups, THREADS, 0, s>>>(t, w, n, n_max, occ, rows, grad, ld_grad, lr);
        sgd_span_kernel<2><<<spans, THREADS, 0, s>>>(t, w, rows, lr);
    } else {
        sgd_sum_kernel<4><<<(int)w.groups, THREADS, 0, s>>>(t, w, n, n_max, occ, rows, grad, ld_grad, lr);
        sgd_span_kernel<4><<<spans, THREADS, 0, s>>>(t, w, rows, lr);
    }
    return hipGetLastError();
}

hipError_t launch_emb_evict(const EmbArgs& t, int threshold, uint32_t min_count, long long* num_evicted,
                            hipStream_t s) {
    zero_i64_kernel<<<1, 1, 0, s>>>(num_evicted);
    evict_kernel<<<grid_for(t.key_capacity), THREADS, 0, s>>>(t, threshold, min_count, num_evicted);
    return hipGetLastError();
}

hipError_t launch_emb_rehash(const EmbArgs& from, const EmbArgs& to, hipStream_t s) {
    fill_u64_kernel<<<grid_for(to.key_capacity), THREADS, 0, s>>>(to.keys, to.key_capacity, KEY_EMPTY);
    fill_i32_kernel<<<grid_for(to.key_capacity), THREADS, 0, s>>>(to.key_rows, to.key_capacity, -1);
    rehash_kernel<<<grid_for(from.key_capacity), THREADS, 0, s>>>(from, to);
    return hipGetLastError();
}

}  // namespace mtgr

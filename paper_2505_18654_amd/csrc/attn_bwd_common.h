// Shared pieces of the attention backward kernels, which live in separate translation units
// (attn_bwd_dq.hip, attn_bwd_dkdv.hip, attn_bwd_dqds.hip): compiled together, the register
// allocation of one kernel changed with the others (the dK/dV kernel spilled about twice as
// much), so each kernel family is compiled on its own and instantiated explicitly.
#pragma once

#include "mtgr_device.h"
#include "mtgr_internal.h"

namespace mtgr {
namespace bwd {
constexpr int BM = 128;   // rows (queries or keys) per workgroup
constexpr int BN = 64;    // columns per inner tile
__device__ __forceinline__ uint4 ldg16(const uint16_t* p) { return *(const uint4*)p; }

__device__ __forceinline__ void zero(floatx16& x) {
#pragma unroll
    for (int r = 0; r < 16; r++) x[r] = 0.f;
}

// Gradient rows on their way out: each wave's 32 staged rows (bf16, swizzled) from row0 of the
// user on go to columns h DH .. of dst, 16 bytes per lane and step.  With ACT they pass through
// the projection's activation (part 0, 1, 2: q, k, v): dh = da silu'(h + b), from the rounded da, as
// the pointwise kernel forms it.  In here that costs a read of h; as a pass of its own, bound by
// memory, it wrote and read da once more (1.2 GB of a layer step on 79,372 rows x 1,024: 5,823 ->
// 5,696 us; 128 users, d = 512, with a bias: 1,863 -> 1,771 us).
template <int DH, bool ACT>
struct GradRows {
    static constexpr int CPR = DH / 8, N = 32 * CPR / 64;
    u32x4_nt hrow[N];
    float bias[8];
    // the rows of h, issued before the gradients are staged (rows past the user's end clamp)
    __device__ __forceinline__ void load(const AttnArgs& a, int part, int ob, int nb, int h, int row0, int lane) {
        if (!ACT) return;
        const int col = (part * a.heads + h) * DH + 8 * (lane % CPR);
#pragma unroll
        for (int i = 0; i < N; i++) {
            const int r = min(row0 + (lane + 64 * i) / CPR, nb - 1);
            hrow[i] = __builtin_nontemporal_load(
                (const u32x4_nt*)((const uint16_t*)a.act_h + (long long)(ob + r) * a.ld_act + col));
        }
#pragma unroll
        for (int e = 0; e < 8; e++) bias[e] = 0.f;
        if (a.act_bias) {
#pragma unroll
            for (int e = 0; e < 8; e++) bias[e] = a.act_bias[col + e];
        }
    }
    __device__ __forceinline__ void store(const AttnArgs& a, uint16_t* dst, long long ld, const uint16_t* sO, int ob,
                                          int nb, int h, int row0, int lane) const {
#pragma unroll
        for (int i = 0; i < N; i++) {
            const int c = lane + 64 * i, row = c / CPR, cc = c % CPR, r = row0 + row;
            if (r >= nb) continue;
            uint16_t* out = dst + (long long)(ob + r) * ld + h * DH + cc * 8;
            const uint16_t* src = &sO[8 * tile_chunk<CPR>(row, cc)];
            if (!ACT) {
                store_nt16(out, src);
                continue;
            }
            const u32x4_nt g = *(const u32x4_nt*)src;
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint32_t gw = g[j], hw = hrow[i][j];
                o[j] = pack_bf16x2(silu_grad(__uint_as_float(gw << 16), __uint_as_float(hw << 16) + bias[2 * j]),
                                   silu_grad(__uint_as_float(gw & 0xffff0000u),
                                             __uint_as_float(hw & 0xffff0000u) + bias[2 * j + 1]));
            }
            const uint4 v = make_uint4(o[0], o[1], o[2], o[3]);
            store_nt16(out, &v);
        }
    }
};

// Relative bias of a backward kernel (RAB): none, one of all 64 buckets, or one of fewer.  With fewer the
// numbers of rab_index end at the last bucket's, so that a run (HistRun) goes on over all gaps of it
// (32 buckets: of more than 18 hours); the one operation for it costs 2 % with 64, where it does
// nothing.  128 users, 47 k tokens, 4 heads, 32 buckets: dK/dV at dh 64 183 -> 167 us, at dh 128 224 ->
// 212 us, dQ at dh 64 131 -> 116 us.
enum { BIAS_NONE = 0, BIAS_FULL = 1, BIAS_FEWER = 2 };
template <int RAB>
__device__ __forceinline__ uint32_t bwd_index(uint32_t a, uint32_t b, int nb) {
    return RAB == BIAS_FEWER ? min(rab_index(a, b), rab_last_index(nb)) : rab_index(a, b);
}

// drab histogram of one workgroup in LDS.  Log-time buckets put most (query, key) pairs of a
// tile into a handful of buckets, so one histogram would serialise the 64 lanes of each LDS
// atomic.  Lane l adds into copy l % 32 (at most two lanes of an instruction share a copy),
// and the copies are HIST_STRIDE = 65 words apart so that one bucket of different copies sits
// in different banks.  8.3 KB.
constexpr int HIST_COPIES = 32;
constexpr int HIST_STRIDE = RAB_SLOTS;
constexpr int HIST_WORDS = HIST_COPIES * HIST_STRIDE;
__device__ __forceinline__ void hist_zero(float* hist, int tid) {
    for (int i = tid; i < HIST_WORDS; i += 256) hist[i] = 0.f;
}
__device__ __forceinline__ void hist_add(float* hist, int lane, uint32_t index, float v) {
    atomicAdd(&hist[(lane & (HIST_COPIES - 1)) * HIST_STRIDE + rab_slot(index)], v);
}
// Per-lane run of equal buckets: consecutive scores of a lane (queries of one key, or keys of
// one query, in token order) mostly fall into the same log-time bucket, so each lane sums its
// run in a register and touches the LDS histogram only when the bucket changes (and once at
// the end).  LDS float atomics are slow on this chip; this makes them rare.
struct HistRun {
    uint32_t bucket = 0;      // as rab_index
    float sum = 0.f;
    __device__ __forceinline__ void add(float* hist, int lane, uint32_t b, float v) {
        if (v != 0.f) {
            if (b != bucket) {
                if (sum != 0.f) hist_add(hist, lane, bucket, sum);
                bucket = b;
                sum = 0.f;
            }
            sum += v;
        }
    }
    __device__ __forceinline__ void flush(float* hist, int lane) {
        if (sum != 0.f) hist_add(hist, lane, bucket, sum);
        sum = 0.f;
    }
};
// drab of the workgroup's head: every slot is summed over the copies by a thread of its own, then
// every bucket over its slots (the last one takes all slots from its own on; one thread walking
// slots and copies took 17 us longer at 32 buckets).  All threads call, behind a barrier.
__device__ __forceinline__ void hist_finish(float* hist, int nb, float scale, float* drab, int tid) {
    if (tid < RAB_SLOTS) {
        float s = 0.f;
#pragma unroll 8
        for (int c = 0; c < HIST_COPIES; c++) s += hist[c * HIST_STRIDE + tid];
        hist[tid] = s;
    }
    __syncthreads();
    if (tid < nb) {
        const int first = tid < 2 ? tid : tid + 1, last = tid == nb - 1 ? RAB_SLOTS - 1 : first;
        float s = 0.f;
#pragma unroll 4
        for (int x = first; x <= last; x++) s += hist[x];
        if (s != 0.f) atomicAdd(drab + tid, s * scale);
    }
}
}  // namespace bwd

template <int DH, int RAB, bool ACT>
__global__ void attn_bwd_dq_bf16_kernel(AttnArgs a);
template <int DH, int RAB, bool STORE, bool ACT, bool FEW>
__global__ void attn_bwd_dkdv_bf16_kernel(AttnArgs a);
template <int DH, bool ACT>
__global__ void attn_bwd_dq_ds_bf16_kernel(AttnArgs a);

}  // namespace mtgr

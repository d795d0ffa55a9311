// The large dense products of the encoder layer (the same layouts and epilogues as gemm.hip):
// a 256 x 256 tile of C per workgroup of 8 waves, one workgroup per CU.
//
// What bounds the 256 x 128 tiles of gemm.hip on large products is the path into LDS, not the
// matrix cores: per 32 k a tile copies 24 KB for 512 cycles of MFMA work, and the path delivers
// 1 KB per 13.2 ns and CU when a copy instruction's rows are 64 bytes long (32 k of a
// k-contiguous operand), 9.2 ns when they are 128 bytes or more (measured, operands in L2).  A
// 256 x 256 tile copies a third less per MFMA, and k steps of 64 make every row 128 bytes:
// 64 KB x 9.2 ns = 0.59 us of copies under 2048 cycles = 0.89 us of MFMAs.
//
// Wave w computes the 128 x 64 part (m half w % 2, n quarter w / 2) as 8 x 4 blocks of 16 x 16,
// transposed (C^T = B^T A^T), with v_mfma_f32_16x16x32_bf16.  On random data the card is bound by
// its power, not by issue: the clock falls to 1.3 - 1.8 GHz, and a loop of nothing but MFMAs on
// N(0, 1) operands in registers reaches 2.02 PFLOP/s with 16 x 16 x 32 and 1.82 with 32 x 32 x 16
// (both 2.45 on zeros).
//
// LDS (160 KB) holds three stages of A and two of B, 32 KB each: A streams from HBM and is copied
// two k steps ahead, B (weights, shared by all m blocks) comes from the XCD's L2 and is copied one
// step ahead.  One barrier per k step, half way through its second k32 part: behind it the step's
// slots are free and the next stage is visible, and the part's other MFMAs cover the first reads
// of the next stage.  Operands are read four blocks (16 MFMAs) ahead of their use, and the copies
// are spread between the MFMAs.
//
// NN / NT run persistently: a workgroup walks tiles, and the first two stages of its next tile are
// copied under the epilogue of the current one, whose stores nothing waits for.
//
// Measured against the 256 x 128 tiles, M = 79,372 rows, d = 1024: [d, 4d] product with bias + SiLU
// 1,045 -> 850 us, without 723 -> 615 us, its input gradient 702 -> 541 us (1.23 PFLOP/s; hipBLASLt
// 616 us), its weight gradient 654 -> 612 us, the d x d products 193 -> 170, 173 -> 150 and
// 190 -> 170 us.
#include <type_traits>

#include "mtgr_device.h"
#include "mtgr_internal.h"

namespace mtgr {

namespace {

constexpr int WBM = 256, WBN = 256, WBK = 64;
constexpr int WNM = 8, WNN = 4;                 // 16 x 16 blocks per wave (m, n)
constexpr uint32_t WSLOT = WBM * WBK * 2;       // bytes of one operand's stage
constexpr int WQ = 4;                           // copy instructions per wave, operand and stage
// Slots: A 0, A 1, B 0, B 1, A 2; the epilogue stages in the last one.
constexpr uint32_t WSTAGING = 4 * WSLOT;

template <int V>
using IC = std::integral_constant<int, V>;

__device__ __forceinline__ uint32_t slot_a(int r) { return r == 2 ? 4u * WSLOT : (uint32_t)r * WSLOT; }
__device__ __forceinline__ uint32_t slot_b(int r) { return (2u + (uint32_t)r) * WSLOT; }

__device__ __forceinline__ float silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// The same value, opaque to the compiler: what is derived from it is computed where it is used
// and not kept in registers across the k loop.
__device__ __forceinline__ int once(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Low or high bf16 of a packed pair.
__device__ __forceinline__ float bf16_half(uint32_t w, int hi) {
    return __uint_as_float(hi ? w & 0xffff0000u : w << 16);
}

// LDS hand-off between the lanes of one wave (its LDS operations run in order).
__device__ __forceinline__ void wave_lds_fence() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

}  // namespace

template <int LAYOUT, int EPI, bool COLSUM>
__global__ __launch_bounds__(512, 2) void gemm_wide_kernel(GemmArgs g) {
    constexpr bool A_KR = LAYOUT == GEMM_TN;      // A stored [K][M]
    constexpr bool B_KR = LAYOUT != GEMM_NT;      // B stored [K][N]
    constexpr bool SPLIT = LAYOUT == GEMM_TN;     // fp32 partials per K split, one tile per workgroup
    __shared__ __align__(1024) char sm[5 * WSLOT];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wm = w & 1, wn = w >> 1;
    const int M = (int)g.M, N = (int)g.N, K = (int)g.K;
    // Items (split, m block, n block), an equal share of consecutive ones per XCD (workgroup % 8):
    // an XCD's 32 workgroups share a few m blocks' rows (NN / NT) or few k ranges (TN) in its L2.
    const int x = blockIdx.x % XCDS, tiles = g.mblocks * g.nblocks, items = tiles * g.splits;
    const int share = (items + XCDS - 1) / XCDS;
    int j = blockIdx.x / XCDS, mb, nb;            // j: item within the share
    auto tile_of = [&](int jj) {
        const int it = x * share + jj;
        mb = it % tiles / g.nblocks;
        nb = it % g.nblocks;
        return jj < share && it < items;
    };
    if (!tile_of(j)) return;
    const int split = SPLIT ? (x * share + j) / tiles : 0;
    const int nks = (int)((g.K + WBK - 1) / WBK);
    const int ks_begin = SPLIT ? split * g.ks_per_split : 0;
    const int nk = (SPLIT ? min(nks, ks_begin + g.ks_per_split) : nks) - ks_begin;     // >= 1 by the plan
    const bool ragged = (long long)(ks_begin + nk) * WBK > K;     // the last step holds fewer than 64 k

    const uint32_t lds0 = lds_address(sm);
    const uint32_t ldsw = lds0 + __builtin_amdgcn_readfirstlane((uint32_t)w * 1024u);

    // ---- copies: instruction q of wave w fills the 1 KB block 8 q + w of a slot
    // [256 rows][64 k] (8 chunks per row, 8 rows per instruction): rows past `rvalid` and chunks
    // past `kvalid` clamp
    auto kc_offsets = [&](uint32_t* vo, long long ld, int rvalid, int kvalid) {
        const int ln = once(lane), r = 8 * w + (ln >> 3);
        const int c = min((ln & 7) ^ swz<8>(r), (kvalid >> 3) - 1);
#pragma unroll
        for (int q = 0; q < WQ; q++) vo[q] = (uint32_t)(min(64 * q + r, rvalid - 1) * ld + 8 * c) * 2u;
    };
    // [64 k][256 cols] (32 chunks per row, 2 rows per instruction)
    auto kr_offsets = [&](uint32_t* vo, long long ld, int cvalid, int kvalid) {
        const int ln = once(lane), r = 2 * w + (ln >> 5);
        const int c = min((ln & 31) ^ swz<32>(r), (cvalid >> 3) - 1);
#pragma unroll
        for (int q = 0; q < WQ; q++) vo[q] = (uint32_t)(min(16 * q + r, kvalid - 1) * ld + 8 * c) * 2u;
    };
    uint32_t voA[WQ], voB[WQ];
    const char *pa, *pb;
    int m0, n0;
    const long long stepA = 2ll * (A_KR ? WBK * g.lda : WBK), stepB = 2ll * (B_KR ? WBK * g.ldb : WBK);
    auto offsets_a = [&](uint32_t* vo, int kvalid) {
        if constexpr (A_KR) kr_offsets(vo, g.lda, M - m0, kvalid);
        else kc_offsets(vo, g.lda, min(WBM, M - m0), kvalid);
    };
    auto offsets_b = [&](uint32_t* vo, int kvalid) {
        if constexpr (B_KR) kr_offsets(vo, g.ldb, N - n0, kvalid);
        else kc_offsets(vo, g.ldb, min(WBN, N - n0), kvalid);
    };
    auto start_tile = [&]() {
        m0 = mb * WBM;
        n0 = nb * WBN;
        offsets_a(voA, WBK);
        offsets_b(voB, WBK);
        pa = (const char*)g.A + 2 * (A_KR ? (long long)m0 : (long long)m0 * g.lda) + ks_begin * stepA;
        pb = (const char*)g.B + 2 * (B_KR ? (long long)n0 : (long long)n0 * g.ldb) + ks_begin * stepB;
    };
    // copies [Q0, Q1) of stage i of one operand; stages are issued in order, the source moves on
    // after the last copy of each
    auto copy = [&](auto q0c, auto q1c, auto is_a, uint32_t slot, int i) {
        constexpr int Q0 = decltype(q0c)::value, Q1 = decltype(q1c)::value;
        constexpr bool IS_A = decltype(is_a)::value;
        uint32_t vo[WQ];
#pragma unroll
        for (int q = 0; q < WQ; q++) vo[q] = IS_A ? voA[q] : voB[q];
        if (ragged && i == nk - 1) {
            if constexpr (IS_A) offsets_a(vo, K - (ks_begin + i) * WBK);
            else offsets_b(vo, K - (ks_begin + i) * WBK);
        }
#pragma unroll
        for (int q = Q0; q < Q1; q++) lds_dma16(ldsw + slot + 8192u * q, IS_A ? pa : pb, vo[q]);
        if constexpr (Q1 == WQ) {
            if constexpr (IS_A) pa += stepA;
            else pb += stepB;
        }
    };
    using A_ = std::true_type;
    using B_ = std::false_type;
    auto copy_a = [&](int i, int r) { copy(IC<0>{}, IC<WQ>{}, A_{}, slot_a(r), i); };
    auto copy_b = [&](int i, int r) { copy(IC<0>{}, IC<WQ>{}, B_{}, slot_b(r), i); };
    // The k past K of a ragged last stage hold copies of valid values; zeros in both operands add
    // nothing.  Ends with a barrier.
    auto zero_tail = [&](uint32_t sa, uint32_t sb) {
        const int valid = K - (ks_begin + nk - 1) * WBK;
        auto clear = [&](bool kr, char* t) {
            if (kr) {
                for (int c = valid * 32 + tid; c < WBK * 32; c += 512) ((uint4*)t)[c] = make_uint4(0, 0, 0, 0);
            } else {
                for (int c = tid; c < WBM * 8; c += 512)
                    if (((c & 7) ^ swz<8>(c >> 3)) >= (valid >> 3)) ((uint4*)t)[c] = make_uint4(0, 0, 0, 0);
            }
        };
        clear(A_KR, sm + sa);
        clear(B_KR, sm + sb);
        lds_barrier();
    };

    // ---- operand reads: per-lane byte offsets within a slot; lane l of an operand of
    // v_mfma_f32_16x16x32_bf16 holds row (or column) l % 16 and k 8 (l / 16) .. + 7.
    // k-contiguous rows r0 + 16 b: chunk (4 p + l / 16) ^ swz(r0) for k32 part p, i.e. the offset of
    // part 0 XOR 64 p, block b at + 2048 b.
    // k-row column block c0 + 16 b: supplier rows of the two halves (k + 0..3, + 4..7) of part 0;
    // part 1 is 16384 bytes further, block b the offset XOR 32 b (c0 is a multiple of 64).
    const int lr = lane & 15, lg = lane >> 4;
    auto kc_base = [&](int r0) { return lds0 + 16u * (uint32_t)((r0 + lr) * 8 + (lg ^ swz<8>(lr))); };
    auto kr_base = [&](int c0, int half) {
        const int row = 8 * lg + 4 * half + (lr >> 2), colx = c0 + 4 * (lr & 3);
        return lds0 + 16u * (uint32_t)tile_chunk<32>(row, colx >> 3) + 2u * (uint32_t)(colx & 7);
    };
    uint32_t rm[2], rn[2];
    rm[0] = A_KR ? kr_base(128 * wm, 0) : kc_base(128 * wm);
    rm[1] = A_KR ? kr_base(128 * wm, 1) : 0;
    rn[0] = B_KR ? kr_base(64 * wn, 0) : kc_base(64 * wn);
    rn[1] = B_KR ? kr_base(64 * wn, 1) : 0;
    typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    auto read_frag = [&](auto kr, const uint32_t (&r)[2], uint32_t slot, auto pc, auto bc) {
        constexpr uint32_t P = decltype(pc)::value, BL = decltype(bc)::value;
        if constexpr (decltype(kr)::value) {
            const uint32_t o0 = ((r[0] + slot) ^ (32u * BL)) + 16384u * P, o1 = ((r[1] + slot) ^ (32u * BL)) + 16384u * P;
            const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)o0);
            const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)o1);
            const short __attribute__((ext_vector_type(8))) v = {lo[0], lo[1], lo[2], lo[3],
                                                                 hi[0], hi[1], hi[2], hi[3]};
            return __builtin_bit_cast(bf16x8, v);
        } else {
            return *(const lds_bf16x8*)(uintptr_t)(((r[0] + slot) ^ (64u * P)) + 2048u * BL);
        }
    };
    using AK = std::integral_constant<bool, A_KR>;
    using BK = std::integral_constant<bool, B_KR>;

    floatx4 acc[WNN][WNM];
    bf16x8 fm[WNM], fn[2][WNN];       // operands: m blocks (four ahead), n blocks of both k32 parts
    float csum[8];
    const bool colsum = COLSUM && mb == 0;
    auto colsum_step = [&](uint32_t sb) {
        if (COLSUM && colsum) {
            // bias gradient: column sums of B over this K split, 8 columns x 4 rows per thread
            const int c = tid & 31, rg = tid >> 5;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const bf16x8 v = tile_read8<32>((const uint16_t*)(sm + sb), 4 * rg + r, c);
#pragma unroll
                for (int e = 0; e < 8; e++) csum[e] += (float)v[e];
            }
        }
    };
    // Slot b of k32 part P: the four MFMAs of m block b, m block b + 4 read ahead (from part NP in
    // slot nsa once past the part's end), and in slots 4 and 5 the n blocks of the next part.
    auto slot = [&](auto pc, auto bc, uint32_t csa, uint32_t nsa, uint32_t nsb) {
        constexpr int P = decltype(pc)::value, b = decltype(bc)::value, NP = P ^ 1;
        if constexpr (b < 4) {
            fm[b + 4] = read_frag(AK{}, rm, csa, IC<P>{}, IC<b + 4>{});
        } else {
            if constexpr (b < 6) {
                fn[NP][2 * (b - 4)] = read_frag(BK{}, rn, nsb, IC<NP>{}, IC<2 * (b - 4)>{});
                fn[NP][2 * (b - 4) + 1] = read_frag(BK{}, rn, nsb, IC<NP>{}, IC<2 * (b - 4) + 1>{});
            }
            fm[b - 4] = read_frag(AK{}, rm, nsa, IC<NP>{}, IC<b - 4>{});
        }
#pragma unroll
        for (int a = 0; a < WNN; a++)
            acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fn[P][a], fm[b], acc[a][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // Stores of a full tile's epilogue per wave.  The waits below count on at least as many memory
    // operations behind the copies of stage 1 (more only make them stricter).
    constexpr int NOUT = EPI == GEMM_EPI_BIAS_SILU ? 2 : 1;
    constexpr int NSTORE = 16 * NOUT;
    start_tile();
    copy_b(0, 0);
    copy_a(0, 0);
    if (nk > 1) {
        copy_b(1, 1);
        copy_a(1, 1);
    }
    bool counted = false;      // the previous tile of this workgroup was a full one
    for (;;) {
        // Stage 0 has landed (a full tile's NSTORE stores and the copies of stage 1 may be in
        // flight behind it), and slot A 2, where the epilogue staged, is free.
        if (counted && nk > 1) wait_vmcnt<NSTORE + 2 * WQ>();
        else wait_vmem();
        lds_barrier();
        if (nk > 2) copy_a(2, 2);
        if (ragged && nk == 1) zero_tail(slot_a(0), slot_b(0));
#pragma unroll
        for (int a = 0; a < WNN; a++)
#pragma unroll
            for (int b = 0; b < WNM; b++)
#pragma unroll
                for (int r = 0; r < 4; r++) acc[a][b][r] = 0.f;
        if (COLSUM) {
#pragma unroll
            for (int e = 0; e < 8; e++) csum[e] = 0.f;
        }
        fn[0][0] = read_frag(BK{}, rn, slot_b(0), IC<0>{}, IC<0>{});
        fm[0] = read_frag(AK{}, rm, slot_a(0), IC<0>{}, IC<0>{});
        fn[0][1] = read_frag(BK{}, rn, slot_b(0), IC<0>{}, IC<1>{});
        fn[0][2] = read_frag(BK{}, rn, slot_b(0), IC<0>{}, IC<2>{});
        fn[0][3] = read_frag(BK{}, rn, slot_b(0), IC<0>{}, IC<3>{});
        fm[1] = read_frag(AK{}, rm, slot_a(0), IC<0>{}, IC<1>{});
        fm[2] = read_frag(AK{}, rm, slot_a(0), IC<0>{}, IC<2>{});
        fm[3] = read_frag(AK{}, rm, slot_a(0), IC<0>{}, IC<3>{});
        // Step i: copies of the second half of B(i+1), then A(i+2), then, behind the barrier that
        // frees its slot, the first half of B(i+2).
        uint32_t sa = slot_a(0), sb = slot_b(0), sa1 = slot_a(1), sa2 = slot_a(2), sb1 = slot_b(1);
        for (int i = 0; i < nk; i++) {
            const bool cb = i > 0 && i + 1 < nk, ca = i > 0 && i + 2 < nk, cn = i + 2 < nk;
            colsum_step(sb);
            slot(IC<0>{}, IC<0>{}, sa, sa, sb);
            if (cb) copy(IC<2>{}, IC<3>{}, B_{}, sb1, i + 1);
            slot(IC<0>{}, IC<1>{}, sa, sa, sb);
            slot(IC<0>{}, IC<2>{}, sa, sa, sb);
            if (cb) copy(IC<3>{}, IC<4>{}, B_{}, sb1, i + 1);
            slot(IC<0>{}, IC<3>{}, sa, sa, sb);
            slot(IC<0>{}, IC<4>{}, sa, sa, sb);
            if (ca) copy(IC<0>{}, IC<1>{}, A_{}, sa2, i + 2);
            slot(IC<0>{}, IC<5>{}, sa, sa, sb);
            slot(IC<0>{}, IC<6>{}, sa, sa, sb);
            if (ca) copy(IC<1>{}, IC<2>{}, A_{}, sa2, i + 2);
            slot(IC<0>{}, IC<7>{}, sa, sa, sb);
            slot(IC<1>{}, IC<0>{}, sa, sa1, sb1);
            if (ca) copy(IC<2>{}, IC<3>{}, A_{}, sa2, i + 2);
            slot(IC<1>{}, IC<1>{}, sa, sa1, sb1);
            slot(IC<1>{}, IC<2>{}, sa, sa1, sb1);
            if (ca) copy(IC<3>{}, IC<4>{}, A_{}, sa2, i + 2);
            slot(IC<1>{}, IC<3>{}, sa, sa1, sb1);
            // stage i + 1 has landed; A(i+2) may still be in flight, in step 0 also the previous
            // tile's stores, which were issued between the copies of stage 1 and A(2)
            if (cn) {
                if (i == 0) wait_vmcnt<NSTORE + WQ>();
                else wait_vmcnt<WQ>();
            } else if (i + 1 < nk) {
                wait_vmem();
            }
            lds_barrier_seen();                 // ... everywhere, and stage i is no longer read
            if (ragged && i + 2 == nk) zero_tail(sa1, sb1);
            // (after the last step the reads touch a slot that may be changing and are not used)
            slot(IC<1>{}, IC<4>{}, sa, sa1, sb1);
            slot(IC<1>{}, IC<5>{}, sa, sa1, sb1);
            if (cn) copy(IC<0>{}, IC<1>{}, B_{}, sb, i + 2);
            slot(IC<1>{}, IC<6>{}, sa, sa1, sb1);
            if (cn) copy(IC<1>{}, IC<2>{}, B_{}, sb, i + 2);
            slot(IC<1>{}, IC<7>{}, sa, sa1, sb1);
            const uint32_t t = sa;
            sa = sa1;
            sa1 = sa2;
            sa2 = t;
            const uint32_t u = sb;
            sb = sb1;
            sb1 = u;
        }

        // ---- epilogue.  acc[a][b] holds C of row m0 + 128 wm + 16 b + l % 16, columns
        // n0 + 64 wn + 16 a + 4 (l / 16) + 0..3.  Each wave passes its part through 4 KB of its own
        // in slot A 2 (no barrier), so that a store instruction writes whole 128-byte lines (or
        // 256-byte rows of fp32 partials), and the first stages of the workgroup's next tile are
        // copied meanwhile.
        const int el = once(lane), er = el & 15, eg = el >> 4;
        const int em = m0 + 128 * wm, en = n0 + 64 * wn;
        char* stg = sm + WSTAGING + 4096 * w;
        // fp32 rows of block b: 16-byte chunk c (of 16) of row r at chunk c ^ r
        auto stage_f32 = [&](int b) {
#pragma unroll
            for (int a = 0; a < WNN; a++)
                *(floatx4*)(stg + 256 * er + 16 * ((4 * a + eg) ^ er)) = acc[a][b];
            wave_lds_fence();
        };
        if constexpr (SPLIT) {
#pragma unroll
            for (int b = 0; b < WNM; b++) {
                stage_f32(b);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int row = 4 * q + eg, gm = em + 16 * b + row, gn = en + 4 * er;
                    const floatx4 v = *(const floatx4*)(stg + 256 * row + 16 * (er ^ row));
                    if (gm < M && gn < N) *(floatx4*)(g.partial + ((long long)split * M + gm) * N + gn) = v;
                }
                wave_lds_fence();
            }
            if (COLSUM && colsum) {
                float* red = (float*)sm;               // [16 row groups][256 columns]
                const int c = tid & 31, rg = tid >> 5;
#pragma unroll
                for (int e = 0; e < 8; e++) red[rg * WBN + 8 * c + e] = csum[e];
                lds_barrier();
                if (tid < WBN && n0 + tid < N) {
                    float s = 0.f;
#pragma unroll
                    for (int r = 0; r < 16; r++) s += red[r * WBN + tid];
                    g.colsum_partial[(long long)split * N + n0 + tid] = s;
                }
            }
            return;
        }
        const bool full = m0 + WBM <= M && n0 + WBN <= N;
        floatx4 bi[WNN];                               // bias of this lane's columns
        if constexpr (EPI == GEMM_EPI_BIAS_SILU) {
#pragma unroll
            for (int a = 0; a < WNN; a++) {
                const int gn = en + 16 * a + 4 * eg;
                bi[a] = gn < N ? *(const floatx4*)(g.bias + gn) : floatx4{};
            }
            wait_vmcnt_seen<0>();                      // (before the copies, which it would wait for)
        }
        // residual rows (row 8 q + l / 8 of block b, chunk l % 8), four blocks ahead, and their
        // columns' bias
        uint4 rr[EPI == GEMM_EPI_BIAS_RESIDUAL ? 4 : 1][2];
        floatx4 rb[2];
        auto load_residual = [&](int b) {
            const uint16_t* R = (const uint16_t*)g.R + min(en + 8 * (el & 7), N - 8);
#pragma unroll
            for (int q = 0; q < 2; q++)
                rr[b & 3][q] = *(const uint4*)(R + min(em + 16 * b + 8 * q + (el >> 3), M - 1) * g.ldr);
        };
        if constexpr (EPI == GEMM_EPI_BIAS_RESIDUAL) {
            const int gn = min(en + 8 * (el & 7), N - 8);
            rb[0] = *(const floatx4*)(g.bias + gn);
            rb[1] = *(const floatx4*)(g.bias + gn + 4);
#pragma unroll
            for (int b = 0; b < 4; b++) load_residual(b);
        }
        j += gridDim.x / XCDS;
        const bool more = tile_of(j);
        if (more) {
            start_tile();
            copy_b(0, 0);
            copy_a(0, 0);
            if (nk > 1) {
                copy_b(1, 1);
                copy_a(1, 1);
            }
        }
        counted = full;
        if constexpr (EPI != GEMM_EPI_BIAS_RESIDUAL) {
            // bf16, 32 rows (two blocks) at a time: 16-byte chunk c (of 8) of row r at c ^ (r & 7)
#pragma unroll
            for (int rd = 0; rd < WNM / 2; rd++)
#pragma unroll
                for (int out = 0; out < NOUT; out++) {
#pragma unroll
                    for (int bb = 0; bb < 2; bb++)
#pragma unroll
                        for (int a = 0; a < WNN; a++) {
                            floatx4 v = acc[a][2 * rd + bb];
                            if (out == 1) {
#pragma unroll
                                for (int e = 0; e < 4; e++) v[e] = silu(v[e] + bi[a][e]);
                            }
                            *(uint2*)(stg + 128 * (16 * bb + er) + 16 * ((2 * a + (eg >> 1)) ^ (er & 7)) + 8 * (eg & 1)) =
                                make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                        }
                    wave_lds_fence();
                    uint16_t* Cout = (uint16_t*)(out == 0 ? g.C : g.C2);
                    const long long ldo = out == 0 ? g.ldc : g.ldc2;
                    uint4 v[4];
#pragma unroll
                    for (int q = 0; q < 4; q++)
                        v[q] = *(const uint4*)(stg + 128 * (8 * q + (el >> 3)) + 16 * ((el & 7) ^ (el >> 3)));
                    const int gm = em + 32 * rd + (el >> 3), gn = en + 8 * (el & 7);
                    uint16_t* dst = Cout + gm * ldo + gn;
                    if (full) {
#pragma unroll
                        for (int q = 0; q < 4; q++) store_nt16(dst + 8 * q * ldo, &v[q]);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; q++)
                            if (gm + 8 * q < M && gn < N) store_nt16(dst + 8 * q * ldo, &v[q]);
                    }
                    wave_lds_fence();
                }
        } else {
            // bias + residual: the fp32 products of one block at a time, so that
            // acc + (bias + residual) is formed in fp32 and rounded once
#pragma unroll
            for (int b = 0; b < WNM; b++) {
                stage_f32(b);
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const int row = 8 * q + (el >> 3), ch = el & 7, gm = em + 16 * b + row, gn = en + 8 * ch;
                    const floatx4 x0 = *(const floatx4*)(stg + 256 * row + 16 * ((2 * ch) ^ row));
                    const floatx4 x1 = *(const floatx4*)(stg + 256 * row + 16 * ((2 * ch + 1) ^ row));
                    const uint32_t rw[4] = {rr[b & 3][q].x, rr[b & 3][q].y, rr[b & 3][q].z, rr[b & 3][q].w};
                    float v[8];
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        v[e] = x0[e] + (rb[0][e] + bf16_half(rw[e >> 1], e & 1));
                        v[4 + e] = x1[e] + (rb[1][e] + bf16_half(rw[2 + (e >> 1)], e & 1));
                    }
                    const uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                               pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                    if (full || (gm < M && gn < N)) store_nt16((uint16_t*)g.C + gm * g.ldc + gn, &o);
                }
                if (b < 4) load_residual(b + 4);
                wave_lds_fence();
            }
        }
        if (!more) return;
    }
}

template <int LAYOUT, int EPI, bool COLSUM>
static hipError_t wide_launch(const GemmArgs& g, hipStream_t s) {
    // NN / NT: one workgroup per CU (those without a tile end at once); TN: one per (split, tile)
    const int items = g.mblocks * g.nblocks * g.splits;
    const int gx = LAYOUT == GEMM_TN ? XCDS * ((items + XCDS - 1) / XCDS) : WIDE_WORKGROUPS;
    gemm_wide_kernel<LAYOUT, EPI, COLSUM><<<gx, 512, 0, s>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_wide(const GemmArgs& g, hipStream_t s) {
    if (g.layout == GEMM_TN)
        return g.colsum ? wide_launch<GEMM_TN, GEMM_EPI_NONE, true>(g, s)
                        : wide_launch<GEMM_TN, GEMM_EPI_NONE, false>(g, s);
    if (g.layout == GEMM_NN) {
        if (g.epilogue == GEMM_EPI_BIAS_SILU) return wide_launch<GEMM_NN, GEMM_EPI_BIAS_SILU, false>(g, s);
        if (g.epilogue == GEMM_EPI_BIAS_RESIDUAL) return wide_launch<GEMM_NN, GEMM_EPI_BIAS_RESIDUAL, false>(g, s);
        return wide_launch<GEMM_NN, GEMM_EPI_NONE, false>(g, s);
    }
    if (g.epilogue == GEMM_EPI_BIAS_SILU) return wide_launch<GEMM_NT, GEMM_EPI_BIAS_SILU, false>(g, s);
    if (g.epilogue == GEMM_EPI_BIAS_RESIDUAL) return wide_launch<GEMM_NT, GEMM_EPI_BIAS_RESIDUAL, false>(g, s);
    return wide_launch<GEMM_NT, GEMM_EPI_NONE, false>(g, s);
}

}  // namespace mtgr

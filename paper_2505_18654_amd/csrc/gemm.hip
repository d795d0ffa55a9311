// Dense bf16 products of the encoder layer around the attention (Sec. 4.2: the projection MLPs
// that form Q, K, V, U, and the top MLP of Eq. 6), with the layer's elementwise work fused:
//   C = op(A) op(B) with op(A) [M, K], op(B) [K, N], fp32 accumulation on the bf16 matrix cores;
//   epilogue NONE:          C = acc
//            BIAS_SILU:     C = acc (the pre-activation, kept for the backward),
//                           C2 = silu(acc + bias)          (the projection's activation)
//            BIAS_RESIDUAL: C = acc + bias + R             (the top MLP plus the residual)
//   layout NN: A [M, K], B [K, N] row-major          (forward products)
//          NT: A [M, K], B [N, K] row-major, C = A B^T (input gradients: dY W^T)
//          TN: A [K, M], B [K, N] row-major, C = A^T B (weight gradients: X^T dY, K = tokens),
//              split over K into fp32 partials that a second kernel adds in a fixed order, with
//              the column sums of B (the bias gradient) formed on the way.
//
// Workgroup: 4 waves, a 256 (m) x 128 (n) tile of C, two workgroups per CU (so that one
// workgroup's prologue, barrier hand-overs and epilogue run under the other's MFMAs).  Wave w
// computes the 128 x 64 part (m half w % 2, n half w / 2) as 4 x 2 blocks of 32 x 32.  k
// advances in steps of 32 through three LDS stages filled by global_load_lds two steps ahead.
// Within a step the two k16 halves are software-pipelined: the operands of the second half are
// read under the first half's MFMAs, the barrier that hands over the next stage sits between
// the halves, and the next stage's first operands are read under the second half's MFMAs.
// Every per-lane address (copy offsets, LDS read bases) is computed once per tile; per step
// only the stage offset (one add per base) and the scalar copy sources move.
// The products are computed transposed, C^T block = B^T A^T (v_mfma_f32_32x32x16_bf16), so
// that a lane's accumulators hold one row of C at 4 consecutive columns per register group:
// the epilogue reads bias / residual and writes C in 8-byte pieces per row without an LDS
// round trip.  An operand whose k index is contiguous in memory (A of NN / NT, B of NT) sits in
// LDS as [rows][32 k] and is read 16 bytes per lane; one whose k index runs over rows (B of
// NN / TN, A of TN) sits as [32 k][cols] and is read with the transposing ds_read_b64_tr_b16,
// the supplier rows chosen so that both operands use the natural k order of the instruction
// (lane half hf holds k = 8 hf .. 8 hf + 7).  Both layouts are swizzled so that every operand
// read and every copy is free of bank conflicts.
//
// Large products run on the 256 x 256 tiles of gemm_wide.hip (gemm_plan decides).
#include <type_traits>

#include "mtgr_device.h"
#include "mtgr_internal.h"

namespace mtgr {

namespace {

constexpr int GBM = 256, GBN = 128, GBK = 32, GSTAGES = 3;
constexpr int A_ELEMS = GBM * GBK, B_ELEMS = GBN * GBK;
constexpr uint32_t A_BYTES = A_ELEMS * 2, B_BYTES = B_ELEMS * 2;     // one stage of each operand
constexpr int QA = A_ELEMS / 8 / 256, QB = B_ELEMS / 8 / 256;         // copy instructions per wave
constexpr int NI = QA + QB;                                          // ... per stage
constexpr int NBN = 2, NBM = 4;                                      // 32 x 32 blocks per wave (n, m)

template <int V>
using IC = std::integral_constant<int, V>;

__device__ __forceinline__ float silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

// Wait until this wave's copies of the stage about to be read have landed, with `later` (0 or
// 1) stages issued after it still in flight.
__device__ __forceinline__ void wait_stage(int later) {
    if (later >= 1) wait_vmcnt<NI>();
    else wait_vmem();
}

// Instruction order of one half step: the scheduler alternates one LDS read with one MFMA
// while both last, then issues the rest (left alone it issues the reads after the MFMAs, so
// that the next half waits for them).
template <int READS, int MFMAS>
__device__ __forceinline__ void interleave_reads() {
    constexpr int P = READS < MFMAS ? READS : MFMAS;
#pragma unroll
    for (int k = 0; k < P; k++) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // one LDS read
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one MFMA
    }
    if constexpr (READS > P) __builtin_amdgcn_sched_group_barrier(0x100, READS - P, 0);
    if constexpr (MFMAS > P) __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - P, 0);
}

}  // namespace

template <int LAYOUT, int EPI, bool COLSUM>
__global__ __launch_bounds__(256, 2) void gemm_bf16_kernel(GemmArgs g) {
    constexpr bool A_KR = LAYOUT == GEMM_TN;      // A stored [K][M]
    constexpr bool B_KR = LAYOUT != GEMM_NT;      // B stored [K][N]
    constexpr bool SPLIT = LAYOUT == GEMM_TN;     // fp32 partials per K split
    __shared__ __align__(16) uint16_t smA[GSTAGES][A_ELEMS];
    __shared__ __align__(16) uint16_t smB[GSTAGES][B_ELEMS];

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int col = lane & 31, hf = lane >> 5;
    const int wm = w & 1, wn = w >> 1;
    // Items (split, m block, n block), an equal share of consecutive ones per XCD (blockIdx % 8): the
    // n blocks of an m block, and the m blocks of a K split, run on one XCD, so that their rows
    // stay in its L2.  Dealing whole m blocks to XCDs left two of them without work at three m blocks, and
    // gave some a round more than others (weight gradients at K = 70,176, d = 256: 54 -> 36 us; M = 5,000,
    // N = 1536, K = 6144: 159 -> 97 us); where it did not, it was up to 12 % the faster (M = 8,300, N =
    // K = 1024: 31 -> 35 us; M = 700, N = 640, K = 2560: 34 -> 38 us).
    const int tiles = g.mblocks * g.nblocks, items = tiles * g.splits, share = (items + XCDS - 1) / XCDS;
    const int item = blockIdx.x % XCDS * share + blockIdx.x / XCDS;
    if (item >= items) return;
    const int mb = item % tiles / g.nblocks, nb = item % g.nblocks, split = item / tiles;
    const int m0 = mb * GBM, n0 = nb * GBN;
    const int nks = (int)((g.K + GBK - 1) / GBK);
    const int ks_begin = split * g.ks_per_split;
    const int nk = min(nks, ks_begin + g.ks_per_split) - ks_begin;     // >= 1 by the plan
    const bool colsum = COLSUM && mb == 0;
    const int M = (int)g.M, N = (int)g.N, K = (int)g.K;

    // ---- copies: per-lane offsets computed once; per step only scalar bases move.
    // Instruction q of wave w fills LDS block 4 q + w (1 KB) of a tile (tile_dma's layout).
    const uint32_t wblk = __builtin_amdgcn_readfirstlane((uint32_t)w * 1024u);
    const uint32_t ldsA = lds_address(&smA[0][0]) + wblk;
    const uint32_t ldsB = lds_address(&smB[0][0]) + wblk;
    // [rows][32 k] tile (4 chunks per row, 64 rows per instruction): rows past `valid` clamp
    auto kc_offsets = [&](uint32_t* vo, int nq, long long ld, int valid) {
        const int rl = w * 16 + (lane >> 2);
        const int c = (lane & 3) ^ swz<4>(rl);
        for (int q = 0; q < nq; q++) vo[q] = (uint32_t)(min(64 * q + rl, valid - 1) * ld + 8 * c) * 2u;
    };
    // [32 k][cols] tile (CPR chunks per row, 256 / CPR rows per instruction): columns past
    // `cvalid` clamp, rows past `rvalid` clamp (the last step of a ragged K only)
    auto kr_offsets = [&](auto cprc, uint32_t* vo, long long ld, int cvalid, int rvalid) {
        constexpr int CPR = decltype(cprc)::value, RPI = 256 / CPR, NQ = 32 * CPR / 256;
        const int rl = w * (64 / CPR) + lane / CPR;
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            const int c = min((lane % CPR) ^ swz<CPR>(RPI * q + rl), (cvalid >> 3) - 1);
            vo[q] = (uint32_t)(min(RPI * q + rl, rvalid - 1) * ld + 8 * c) * 2u;
        }
    };
    uint32_t voA[QA], voB[QB];
    if constexpr (A_KR) kr_offsets(IC<GBM / 8>{}, voA, g.lda, M - m0, GBK);
    else kc_offsets(voA, QA, g.lda, min(GBM, M - m0));
    if constexpr (B_KR) kr_offsets(IC<GBN / 8>{}, voB, g.ldb, N - n0, GBK);
    else kc_offsets(voB, QB, g.ldb, min(GBN, N - n0));
    // source of the next k step to copy: k-contiguous operands move 32 columns, k-row operands
    // 32 rows; the copies are issued in k order, so the pointers only advance
    const char* pa = (const char*)g.A + 2 * (A_KR ? (long long)m0 : (long long)m0 * g.lda);
    const char* pb = (const char*)g.B + 2 * (B_KR ? (long long)n0 : (long long)n0 * g.ldb);
    const long long stepA = 2ll * (A_KR ? GBK * g.lda : GBK), stepB = 2ll * (B_KR ? GBK * g.ldb : GBK);
    pa += ks_begin * stepA;
    pb += ks_begin * stepB;

    auto issue = [&](int st, int i) {
        uint32_t ra[QA], rb[QB];
#pragma unroll
        for (int q = 0; q < QA; q++) ra[q] = voA[q];
#pragma unroll
        for (int q = 0; q < QB; q++) rb[q] = voB[q];
        if constexpr (A_KR) {
            const int k0 = (ks_begin + i) * GBK;
            if (k0 + GBK > K) {               // ragged last step: clamp the k rows
                kr_offsets(IC<GBM / 8>{}, ra, g.lda, M - m0, K - k0);
                kr_offsets(IC<GBN / 8>{}, rb, g.ldb, N - n0, K - k0);
            }
        }
#pragma unroll
        for (int q = 0; q < QA; q++) lds_dma16(ldsA + (uint32_t)st * A_BYTES + 4096u * q, pa, ra[q]);
#pragma unroll
        for (int q = 0; q < QB; q++) lds_dma16(ldsB + (uint32_t)st * B_BYTES + 4096u * q, pb, rb[q]);
        pa += stepA;
        pb += stepB;
    };
    // The last k step of a ragged K (TN only): rows past K hold copies of row K - 1; zero them
    // in both tiles so that they add nothing, then hand the stage over again.
    auto zero_tail = [&](int st, int i) {
        if constexpr (A_KR) {
            const int valid = K - (ks_begin + i) * GBK;
            if (valid < GBK) {
                uint4* za = (uint4*)smA[st];
                uint4* zb = (uint4*)smB[st];
                for (int c = tid; c < (GBK - valid) * (GBM / 8); c += 256) za[valid * (GBM / 8) + c] = make_uint4(0, 0, 0, 0);
                for (int c = tid; c < (GBK - valid) * (GBN / 8); c += 256) zb[valid * (GBN / 8) + c] = make_uint4(0, 0, 0, 0);
                lds_barrier();
            }
        }
    };

    // ---- operand reads: per-lane LDS addresses computed once; k16 step and block offsets go
    // into the 16-bit immediate of each ds_read, the stage offset into a per-step add.
    // k-contiguous operand rows r0 + 32 b: chunk (2 ks + hf) ^ swz(r0) (the swizzle depends on
    // the row mod 16 only), block b at + 2048 b bytes
    auto kc_base = [&](int r0, int ks) { return 16u * (uint32_t)(r0 * 4 + ((2 * ks + hf) ^ swz<4>(r0))); };
    // k-row operand column block c0 (CPR chunks per row), supplier rows of k16 step 0 (step 1:
    // 16 rows further, + 256 CPR bytes)
    auto kr_base = [&](auto cprc, int c0, int part) {
        constexpr int CPR = decltype(cprc)::value;
        const int j = lane & 15;
        const int row = 8 * hf + (j >> 2) + 4 * part;
        const int colx = c0 + 16 * ((lane >> 4) & 1) + 4 * (j & 3);
        return 16u * (uint32_t)tile_chunk<CPR>(row, colx >> 3) + 2u * (uint32_t)(colx & 7);
    };
    constexpr uint32_t KS_A = 256u * (GBM / 8), KS_B = 256u * (GBN / 8);     // k16 step of a k-row tile
    // bases: kr [block][supplier half]; kc [0][k16 step]
    uint32_t rbA[NBM][2], rbB[NBN][2];
    const uint32_t lA = lds_address(&smA[0][0]), lB = lds_address(&smB[0][0]);
#pragma unroll
    for (int h = 0; h < 2; h++) {
#pragma unroll
        for (int q = 0; q < NBM; q++)
            rbA[q][h] = lA + (A_KR ? kr_base(IC<GBM / 8>{}, 128 * wm + 32 * q, h) : kc_base(128 * wm + col, h));
#pragma unroll
        for (int q = 0; q < NBN; q++)
            rbB[q][h] = lB + (B_KR ? kr_base(IC<GBN / 8>{}, 64 * wn + 32 * q, h) : kc_base(64 * wn + col, h));
    }
    typedef __attribute__((address_space(3))) bf16x8 lds_bf16x8;
    auto rd16 = [&](uint32_t addr) { return *(const lds_bf16x8*)(uintptr_t)addr; };
    auto rdtr = [&](uint32_t o0, uint32_t o1) {
        const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)o0);
        const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4*)(uintptr_t)o1);
        const short __attribute__((ext_vector_type(8))) v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    };
    // stage-shifted copies of the read bases: `cur` for the stage being computed, `nxt` for the
    // next one (one VALU add per base and step)
    uint32_t curA[NBM][2], curB[NBN][2], nxtA[NBM][2], nxtB[NBN][2];
    auto shift = [&](uint32_t (&dA)[NBM][2], uint32_t (&dB)[NBN][2], int st) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int q = 0; q < NBM; q++)
                if (A_KR || q == 0) dA[q][h] = rbA[q][h] + (uint32_t)st * A_BYTES;
#pragma unroll
            for (int q = 0; q < NBN; q++)
                if (B_KR || q == 0) dB[q][h] = rbB[q][h] + (uint32_t)st * B_BYTES;
        }
    };
    auto read_ops = [&](bf16x8* ao, bf16x8* bo, const uint32_t (&bA)[NBM][2], const uint32_t (&bB)[NBN][2],
                        auto ksc) {
        constexpr uint32_t KS = decltype(ksc)::value;
#pragma unroll
        for (int a = 0; a < NBN; a++) {
            if constexpr (B_KR) ao[a] = rdtr(bB[a][0] + KS * KS_B, bB[a][1] + KS * KS_B);
            else ao[a] = rd16(bB[0][KS] + 2048u * a);
        }
#pragma unroll
        for (int b = 0; b < NBM; b++) {
            if constexpr (A_KR) bo[b] = rdtr(bA[b][0] + KS * KS_A, bA[b][1] + KS * KS_A);
            else bo[b] = rd16(bA[0][KS] + 2048u * b);
        }
    };

    floatx16 acc[NBN][NBM];
#pragma unroll
    for (int a = 0; a < NBN; a++)
#pragma unroll
        for (int b = 0; b < NBM; b++)
#pragma unroll
            for (int r = 0; r < 16; r++) acc[a][b][r] = 0.f;
    float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto mfmas = [&](const bf16x8* ao, const bf16x8* bo) {
#pragma unroll
        for (int a = 0; a < NBN; a++)
#pragma unroll
            for (int b = 0; b < NBM; b++)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ao[a], bo[b], acc[a][b], 0, 0, 0);
    };
    auto colsum_step = [&](int st) {
        if (COLSUM && colsum) {
            // bias gradient: column sums of B over this K split, 8 columns x 2 rows per thread
            const int c = tid & 15, rg = tid >> 4;
#pragma unroll
            for (int j = 0; j < 2; j++) {
                const bf16x8 v = tile_read8<GBN / 8>(smB[st], 2 * rg + j, c);
#pragma unroll
                for (int e = 0; e < 8; e++) csum[e] += (float)v[e];
            }
        }
    };

    bf16x8 a0[NBN], b0[NBM], a1[NBN], b1[NBM];
    // LDS reads per operand set: 2 per transposed operand, 1 per k-contiguous one
    constexpr int READS = NBM * (A_KR ? 2 : 1) + NBN * (B_KR ? 2 : 1);

    issue(0, 0);
    if (nk > 1) issue(1, 1);
    if (nk > 2) issue(2, 2);
    const int later0 = min(nk - 1, GSTAGES - 1);      // stages issued after stage 0
    if (later0 == 2) wait_vmcnt<2 * NI>();
    else wait_stage(later0);
    lds_barrier();
    if (nk == 1) zero_tail(0, 0);
    shift(curA, curB, 0);
    read_ops(a0, b0, curA, curB, IC<0>{});
    // One k step per iteration.  The second half's operands are read under the first half's
    // MFMAs, and the next stage's first operands under the second half's; the waits are ones
    // the compiler sees, so it adds none of its own in front of the MFMAs.  No MFMA sits in a
    // branch (the accumulators stay in place): after the last step the next-stage reads touch
    // a stale slot and are not used, and the hand-over barrier is harmless.
    int st = 0, nx = 1;
    for (int i = 0; i < nk; i++) {
        wait_lgkm_seen();                       // a0 / b0 (read a half step ago) have landed
        colsum_step(st);
        read_ops(a1, b1, curA, curB, IC<1>{});
        shift(nxtA, nxtB, nx);
        mfmas(a0, b0);
        interleave_reads<READS, NBN * NBM>();
        wait_stage(min(nk - 2 - i, 1));
        lds_barrier_seen();                     // stage i + 1 visible; every wave done with stage i
        if (i + GSTAGES < nk) issue(st, i + GSTAGES);     // into the slot of stage i
        if (A_KR && i + 2 == nk) zero_tail(nx, i + 1);
        read_ops(a0, b0, nxtA, nxtB, IC<0>{});
        mfmas(a1, b1);
        interleave_reads<READS, NBN * NBM>();
#pragma unroll
        for (int h = 0; h < 2; h++) {
#pragma unroll
            for (int q = 0; q < NBM; q++) curA[q][h] = nxtA[q][h];
#pragma unroll
            for (int q = 0; q < NBN; q++) curB[q][h] = nxtB[q][h];
        }
        st = nx;
        nx = nx == GSTAGES - 1 ? 0 : nx + 1;
    }

    // acc[a][b] holds C^T of rows n0 + 64 wn + 32 a + 8 (r / 4) + 4 hf + r % 4, columns
    // m0 + 128 wm + 32 b + col: lane row gm of C, columns gn .. gn + 3 per register group q = r / 4.
    // Written directly, one store instruction would touch 32 rows with 16 bytes each.  So the
    // bf16 results (and, for bias + SiLU, then the activation) pass through LDS, half a tile (128
    // rows, the rows of the waves with wm = hm) at a time, in the stage memory that is free now:
    // row stride 136 elements (272 bytes, so that the 32 rows of one write instruction spread
    // over the banks), then every thread stores whole 16-byte chunks, 4 rows of 256 bytes per
    // store instruction, with the non-temporal hint (the results are not read by this kernel).
    // Measured on the layer shapes: the projection with bias + SiLU 1.06 -> 0.91 ms, plain
    // products 12-19 % faster.
    constexpr bool STAGED = !SPLIT && EPI != GEMM_EPI_BIAS_RESIDUAL;
    if constexpr (STAGED) {
        constexpr int SROW = GBN + 8;
        static_assert(128 * SROW <= GSTAGES * A_ELEMS, "staging fits the A stages");
        uint16_t* stg = &smA[0][0];
        constexpr int NOUT = EPI == GEMM_EPI_BIAS_SILU ? 2 : 1;
#pragma unroll
        for (int out = 0; out < NOUT; out++) {
            uint16_t* Cout = (uint16_t*)(out == 0 ? g.C : g.C2);
            const long long ldo = out == 0 ? g.ldc : g.ldc2;
#pragma unroll
            for (int hm = 0; hm < 2; hm++) {
                lds_barrier();   // the stage memory (or the previous half) is no longer read
                if (wm == hm) {
#pragma unroll
                    for (int b = 0; b < NBM; b++)
#pragma unroll
                        for (int a = 0; a < NBN; a++)
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                const int cl = 64 * wn + 32 * a + 8 * q + 4 * hf;
                                float v[4] = {acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2],
                                              acc[a][b][4 * q + 3]};
                                if (out == 1) {
                                    float4 bi = make_float4(0.f, 0.f, 0.f, 0.f);
                                    if (n0 + cl < N) bi = *(const float4*)(g.bias + n0 + cl);
                                    v[0] = silu(v[0] + bi.x);
                                    v[1] = silu(v[1] + bi.y);
                                    v[2] = silu(v[2] + bi.z);
                                    v[3] = silu(v[3] + bi.w);
                                }
                                *(uint2*)&stg[(32 * b + col) * SROW + cl] =
                                    make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
                            }
                }
                lds_barrier();
#pragma unroll
                for (int i = 0; i < 128 * GBN / 8 / 256; i++) {
                    const int idx = 256 * i + tid, row = idx >> 4, ch = idx & 15;
                    const long long gm = m0 + 128 * hm + row;
                    const int gn = n0 + 8 * ch;
                    if (gm < M && gn < N)
                        store_nt16(Cout + gm * ldo + gn, &stg[row * SROW + 8 * ch]);
                }
            }
        }
    }
    if constexpr (!SPLIT && EPI == GEMM_EPI_BIAS_RESIDUAL) {
        // The same for bias + residual, with the fp32 products staged (a quarter tile, 64 rows,
        // at a time; row stride 132 floats) so that the store phase forms acc + (bias + residual)
        // from fp32 and rounds once, as the direct form did.
        constexpr int FROW = GBN + 4;
        static_assert(64 * FROW * 4 <= GSTAGES * A_ELEMS * 2, "staging fits the A stages");
        float* stf = (float*)&smA[0][0];
#pragma unroll
        for (int p = 0; p < 4; p++) {   // tile rows 64 p .. 64 p + 63: waves wm = p / 2, b = 2 (p % 2) + 0..1
            lds_barrier();
            if (wm == (p >> 1)) {
#pragma unroll
                for (int bb = 0; bb < 2; bb++)
#pragma unroll
                    for (int a = 0; a < NBN; a++)
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            const int b = 2 * (p & 1) + bb;
                            const int cl = 64 * wn + 32 * a + 8 * q + 4 * hf;
                            *(float4*)&stf[(32 * bb + col) * FROW + cl] =
                                make_float4(acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2],
                                            acc[a][b][4 * q + 3]);
                        }
            }
            lds_barrier();
#pragma unroll
            for (int i = 0; i < 64 * GBN / 8 / 256; i++) {
                const int idx = 256 * i + tid, row = idx >> 4, ch = idx & 15;
                const long long gm = m0 + 64 * p + row;
                const int gn = n0 + 8 * ch;
                if (gm < M && gn < N) {
                    const float4 x0 = *(const float4*)&stf[row * FROW + 8 * ch];
                    const float4 x1 = *(const float4*)&stf[row * FROW + 8 * ch + 4];
                    const float4 b0 = *(const float4*)(g.bias + gn), b1 = *(const float4*)(g.bias + gn + 4);
                    const uint4 rr = *(const uint4*)((const uint16_t*)g.R + gm * g.ldr + gn);
                    const float v[8] = {x0.x + (b0.x + __uint_as_float(rr.x << 16)), x0.y + (b0.y + __uint_as_float(rr.x & 0xffff0000u)),
                                        x0.z + (b0.z + __uint_as_float(rr.y << 16)), x0.w + (b0.w + __uint_as_float(rr.y & 0xffff0000u)),
                                        x1.x + (b1.x + __uint_as_float(rr.z << 16)), x1.y + (b1.y + __uint_as_float(rr.z & 0xffff0000u)),
                                        x1.z + (b1.z + __uint_as_float(rr.w << 16)), x1.w + (b1.w + __uint_as_float(rr.w & 0xffff0000u))};
                    const uint4 o = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]),
                                               pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
                    store_nt16((uint16_t*)g.C + gm * g.ldc + gn, &o);
                }
            }
        }
    }
    if constexpr (SPLIT) {
        // fp32 partials of this K split, 16 bytes per lane (summed by gemm_split_reduce_kernel)
#pragma unroll
        for (int b = 0; b < NBM; b++) {
            const long long gm = m0 + 128 * wm + 32 * b + col;
            if (gm >= M) continue;
#pragma unroll
            for (int a = 0; a < NBN; a++) {
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int gn = n0 + 64 * wn + 32 * a + 8 * q + 4 * hf;
                    if (gn >= N) continue;
                    float* P = g.partial + ((long long)split * M + gm) * N + gn;
                    *(float4*)P = make_float4(acc[a][b][4 * q], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2],
                                              acc[a][b][4 * q + 3]);
                }
            }
            // one 32-row block at a time: the stores are not hoisted across blocks
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (COLSUM && colsum) {
        // the 16 row groups' sums of each column, added through LDS (stage memory is free now)
        lds_barrier();
        float* red = (float*)smA[0];                // [16 row groups][128 columns]
        const int c = tid & 15, rg = tid >> 4;
#pragma unroll
        for (int e = 0; e < 8; e++) red[rg * GBN + 8 * c + e] = csum[e];
        lds_barrier();
        if (tid < GBN) {
            float s = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r++) s += red[r * GBN + tid];
            if (n0 + tid < N) g.colsum_partial[(long long)split * N + n0 + tid] = s;
        }
    }
}

// Sum of the K-split partials in a fixed order: C = bf16(sum_s partial[s]) and, with column
// sums, colsum = sum_s colsum_partial[s] (fp32).  Bound by the latency of a thread's chain of
// loads (a few MB in all, at most 64 partials): eight partials are in flight at a time, added in
// the order of the splits, and the column sums have workgroups of their own, the last ones,
// with one column per thread (they used to be workgroup 0's, column after column).
// Layer of 32 short users (d = 256, 27 partials): 22 us -> below 8 us per product, the layer's
// step 244 -> 219 us; of 128 users (d = 512, 69 k tokens) 2,162 -> 2,102 us.
template <class V>
__device__ __forceinline__ V sum_partials(const V* p, long long stride, int n) {
    V s = p[0];
    int i = 1;
    for (; i + 8 <= n; i += 8) {
        V t[8];
#pragma unroll
        for (int k = 0; k < 8; k++) t[k] = p[(i + k) * stride];
#pragma unroll
        for (int k = 0; k < 8; k++) s += t[k];
    }
    for (; i < n; i++) s += p[i * stride];
    return s;
}

__global__ __launch_bounds__(256) void gemm_split_reduce_kernel(GemmArgs g, int sum_blocks) {
    if ((int)blockIdx.x >= sum_blocks) {
        const long long n = (long long)(blockIdx.x - sum_blocks) * 256 + threadIdx.x;
        if (n < g.N) g.colsum[n] = sum_partials(g.colsum_partial + n, g.N, g.splits);
        return;
    }
    const long long MN4 = g.M * g.N / 4;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < MN4; i += (long long)sum_blocks * 256) {
        const long long e = 4 * i, m = e / g.N, n = e % g.N;
        const floatx4 s = sum_partials((const floatx4*)(g.partial + e), MN4, g.splits);
        *(uint2*)((uint16_t*)g.C + m * g.ldc + n) = make_uint2(pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3]));
    }
}

// Which kernel: 256 x 128 tiles, two workgroups per CU (gemm_bf16_kernel), or 256 x 256 tiles, one
// per CU (gemm_wide_kernel).  Both timed for the six products of a layer, d from 32 to 2,048 and 32 to
// 100,000 rows; the lines below leave no size at which the wide one is chosen and is more than 3 %
// (NN without an epilogue: 8 %, TN: 14 %) slower in a program of its own.
//
// NN / NT: the wide one does the same work up to 1.1 (K below 576), 1.15 (below 2048) or 1.25 times
// faster, but in whole rounds of 256 tiles, and a lone tile takes 1.5 times as long.  So it is taken when
// rounds of the narrow one, twice as short, would not beat it: M = 70,176, N = 512, K = 2048 (3
// rounds of wide, 5 half rounds of narrow) 171 -> 157 us; M = 69,563, N = K = 1024 (5 and 9) 162 -> 156
// us; M = 33,000, N = 512 (2 and 3) 88 us, wide 94; M = 6,925, N = 1024, K = 4096 (1 and 1) 66 us, wide 86.
// Without an epilogue it pays for the k that pad the last step of 64 (N = K = 160, M = 60,000: 10.4 us,
// wide 12.2), and NN, whose wide stores dominate, gains at most 1.07 (d = 256, [d, 4d], M = 90,000:
// 61 us, wide 70).  With bias + SiLU, whose element work the wide one hides, it is 1.43 times faster up to
// K = 768, and within a round also where it fills less of the chip than the narrow one, up to
// K = 512 at any size (M = 700, d = 128: 17.3 -> 13.9 us), above from 128 narrow tiles on (d = 768: M = 700
// 23.7 us, wide 24.8; M = 3,000 35.0 and 26.8).  At [d, 4d] with N no multiple of 256 the rounds count
// the padding: d = 96, M = 36,000 20.8 us, wide 25.7.
//
// TN takes the wide one when its K splits fill about half the chip (M = N = 768, K = 6,925, 117
// workgroups: 42 -> 32 us; 512, 52 workgroups: 21 us, wide 31), unless half of each tile would be
// padding (M <= 128: d = 96, K = 70,000, [d, 4d] 32 us, wide 43), or one split's tiles leave much of
// the chip idle for long (d = 1536, [d, 4d], 144 tiles, K = 45,000: 966 us, wide 1,241).  Where both fill the
// chip once (d = 1024, [d, 4d], K = 79,372, 4 splits) it depends on the power that the data takes: on
// activations narrow 618 us, wide 661, on the gradients of a layer 595 and 576, and there the narrow
// one also slows the kernels around it by 1 to 2 %; the wide one stays.
static bool use_wide(const GemmArgs& g, long long mb, long long nb, long long nb_narrow) {
    auto rounds = [](long long tiles) { return (tiles + 255) / 256; };
    const long long wide = mb * nb, narrow = mb * nb_narrow;
    if (wide == 0 || g.K == 0 || wide >= (1 << 20)) return false;     // (an empty product launches nothing)
    if (g.layout == GEMM_TN) {
        const long long s = max(1ll, min(min(256 / max(wide, 1ll), g.K / 512), 64ll));
        return wide * s >= 112 && g.M > 128 && (s > 1 || wide >= 200 || g.K < 2048);
    }
    long long gain;
    if (g.epilogue == GEMM_EPI_BIAS_SILU) {
        if (wide <= 256 && (g.K <= 512 || (g.K <= 768 && narrow >= 128))) return true;
        gain = g.K <= 768 ? 143 : 125;
    } else {
        gain = g.K >= 2048 ? 125 : g.K >= 576 ? 115 : 110;
        if (g.epilogue == GEMM_EPI_NONE) {
            if (g.layout == GEMM_NN && g.K < 2048) gain = g.K >= 768 ? 107 : g.K >= 448 ? 100 : 0;
            gain = gain * g.K / (64 * ((g.K + 63) / 64));
        }
    }
    return gain * rounds(narrow) >= 200 * rounds(wide);
}

void gemm_plan(GemmArgs* g) {
    const long long mb = (g->M + GBM - 1) / GBM;
    g->wide = use_wide(*g, mb, (g->N + 255) / 256, (g->N + GBN - 1) / GBN);
    const int bn = g->wide ? 256 : GBN, bk = g->wide ? 64 : GBK;
    g->mblocks = (int)mb;
    g->nblocks = (int)((g->N + bn - 1) / bn);
    g->splits = 1;
    const long long tiles = (long long)g->mblocks * g->nblocks, nks = (g->K + bk - 1) / bk;
    g->ks_per_split = (int)nks;
    if (tiles == 0 || nks == 0 || g->layout != GEMM_TN) return;     // (an empty product launches nothing)
    // enough workgroups for the chip (one per CU of the wide kernel, two of the narrow one), each
    // split at least 8 k steps
    const long long target = g->wide ? 256 / tiles : (512 + tiles - 1) / tiles;
    const int s = (int)max(1ll, min(min(target, nks / 8), 64ll));
    g->ks_per_split = (int)((nks + s - 1) / s);
    g->splits = (int)((nks + g->ks_per_split - 1) / g->ks_per_split);
}

size_t gemm_workspace_bytes(int layout, long long M, long long N, long long K) {
    if (layout != GEMM_TN) return 0;
    GemmArgs g{};
    g.layout = layout;
    g.M = M;
    g.N = N;
    g.K = K;
    gemm_plan(&g);
    return (size_t)g.splits * (size_t)(M * N + N) * sizeof(float);
}

template <int LAYOUT, int EPI, bool COLSUM>
static hipError_t gemm_launch(const GemmArgs& g, hipStream_t s) {
    const int share = (g.mblocks * g.nblocks * g.splits + XCDS - 1) / XCDS;
    gemm_bf16_kernel<LAYOUT, EPI, COLSUM><<<XCDS * share, 256, 0, s>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_bf16(const GemmArgs& g, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (g.wide && g.layout != GEMM_TN) return launch_gemm_wide(g, s);
    switch (g.layout) {
        case GEMM_NN:
            if (g.epilogue == GEMM_EPI_BIAS_SILU) e = gemm_launch<GEMM_NN, GEMM_EPI_BIAS_SILU, false>(g, s);
            else if (g.epilogue == GEMM_EPI_BIAS_RESIDUAL) e = gemm_launch<GEMM_NN, GEMM_EPI_BIAS_RESIDUAL, false>(g, s);
            else e = gemm_launch<GEMM_NN, GEMM_EPI_NONE, false>(g, s);
            return e;
        case GEMM_NT:
            if (g.epilogue == GEMM_EPI_BIAS_SILU) e = gemm_launch<GEMM_NT, GEMM_EPI_BIAS_SILU, false>(g, s);
            else if (g.epilogue == GEMM_EPI_BIAS_RESIDUAL) e = gemm_launch<GEMM_NT, GEMM_EPI_BIAS_RESIDUAL, false>(g, s);
            else e = gemm_launch<GEMM_NT, GEMM_EPI_NONE, false>(g, s);
            return e;
        case GEMM_TN:
            e = g.wide ? launch_gemm_wide(g, s)
                : g.colsum ? gemm_launch<GEMM_TN, GEMM_EPI_NONE, true>(g, s) : gemm_launch<GEMM_TN, GEMM_EPI_NONE, false>(g, s);
            if (e != hipSuccess) return e;
            {
                const int sums = (int)min((g.M * g.N / 4 + 255) / 256, 8192ll);
                const int cols = g.colsum ? (int)((g.N + 255) / 256) : 0;
                gemm_split_reduce_kernel<<<sums + cols, 256, 0, s>>>(g, sums);
            }
            return hipGetLastError();
        default: return hipErrorInvalidValue;
    }
}

}  // namespace mtgr

// Layer-wise query-attention score (Sec. 3.2 equation; first step of Algorithm 1):
//   A_l[h,t,i] = softmax_i(sigma <q_{l,t,h}, k_{l,g(h),i}>),
//   p_{l,i} = (1/(H Qn)) sum_{h,t} A_l[h,t,i],   a_{l,i} = MinMax_i(p_{l,i}).
//
// bf16 path (bf16 MFMA, fp32 accumulation).  Per layer l and KV head g the
// Qn*G query rows that share g form one row set.  A workgroup takes one
// (l, g, split of contiguous keys: up to 4096 in the statistics pass, up to 8192 in
// the column-sum pass, see pass_split): it stages the row set into LDS once (fragment-major),
// and each of its waves loads its own 32-key blocks from HBM straight into
// registers and runs every 32-row block against them, so K never passes
// through LDS (in the column-sum pass a wave holds two key blocks, so a query
// fragment read from LDS feeds two MFMAs):
//   1. score_stats_kreg -- S^T = K Q^T (one query row per lane): each row's
//      (reference, sum of exp2) over the split.           [skipped with q_lse]
//   2. score_merge  -- per row, merge the splits into a log2-sum-exp (few splits and rows:
//      merged by pass 3's workgroups instead).
//   3. score_colsum_kreg -- S = Q K^T - lse (one key per lane; each
//      accumulator starts at its row's -lse), summing exp2 over the rows: the
//      pooled mass of each key for this KV head.
//   4. score_pool / score_minmax -- the fixed-order sum over KV heads and the
//      1/(H Qn) factor with per-block extrema, then the MinMax normalisation
//      (score_finish for short contexts: both in one launch).
// float32 path: float32 MFMA kernels with the same four steps (used for fp32
// inputs, where bf16 MFMA would not meet fp32 accuracy).
// Every reduction has a fixed order and no float atomics: results are
// bit-identical run to run.

#include <math.h>

#include "dev_common.h"
#include "internal.h"

namespace relaxkv {
namespace {

#ifndef RELAXKV_SCORE_SPLIT
#define RELAXKV_SCORE_SPLIT 4096              // keys per statistics workgroup
#endif
#ifndef RELAXKV_SCORE_KREG_NW
#define RELAXKV_SCORE_KREG_NW 16              // waves per workgroup (four per SIMD)
#endif
#ifndef RELAXKV_SCORE_KREG_NKB
#define RELAXKV_SCORE_KREG_NKB 1              // 32-key blocks per wave and round (statistics pass)
#endif
#ifndef RELAXKV_SCORE_COLSUM_NW
#define RELAXKV_SCORE_COLSUM_NW 16            // waves per column-sum workgroup
#endif
#ifndef RELAXKV_SCORE_COLSUM_NKB
#define RELAXKV_SCORE_COLSUM_NKB 2            // 32-key blocks per wave and round (column-sum pass)
#endif
constexpr int kKeysPerSplit = RELAXKV_SCORE_SPLIT;
constexpr int kKregRowBlocks = 10;            // 32-row blocks staged per row chunk

// Range a block's sum of exp2(s - m) may take before the statistics pass moves
// its reference m (see score_stats_kreg).
constexpr float kRefHi = 18446744073709551616.0f;     // 2^64
constexpr float kRefLo = 5.42101086242752217e-20f;    // 2^-64

__host__ __device__ inline int round_up32(int x) { return (x + 31) / 32 * 32; }

// x plus the copy of x held by the lane 32 away (v_permlane32_swap with both
// operands x returns x and the partner's x, in some order, in its two results).
__device__ __forceinline__ float pair_add(float x) {
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The copy of x held by the lane 32 away (xor of both results with x leaves the
// partner's bits whichever result holds which).
__device__ __forceinline__ float pair_other(float x) {
    const uint32_t u = __float_as_uint(x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0] ^ r[1] ^ u);
}

// Stage rows rc0 .. rc0 + 32 nrb - 1 of the row set (l, g) into Qs, fragment-major:
// fragment (rb, j) holds the MFMA operand of 32-row block rb and k-step j (lane
// l: row 32 rb + l % 32, 16-byte chunk 2j + l / 32; padding rows are zero).
template <int D, int NW>
__device__ __forceinline__ void stage_rows(bf16x8* Qs, const uint16_t* __restrict__ q, int l,
                                           int g, int Qn, int H, int G, int n_rows, int rc0,
                                           int nrb) {
    constexpr int KS = D / 16;
    for (int f = threadIdx.x; f < nrb * KS * 64; f += NW * 64) {
        const int ln = f & 63, fj = f >> 6, rb = fj / KS, j = fj - rb * KS;
        const int row = rc0 + rb * 32 + (ln & 31), h2 = ln >> 5;
        bf16x8 v = {};
        if (row < n_rows) {
            const int t = row / G, hh = row - t * G;
            v = *(const bf16x8*)(q + (((size_t)l * Qn + t) * H + g * G + hh) * D + 16 * j + 8 * h2);
        }
        Qs[f] = v;
    }
}

// A row's log2-sum-exp from its splits' (m, sum) pairs (n_split of them, rows_pad apart).
__device__ __forceinline__ float merge_stats(const float2* __restrict__ s, int n_split,
                                             int rows_pad) {
    float M = -INFINITY;
    for (int j = 0; j < n_split; ++j) M = fmaxf(M, s[(size_t)j * rows_pad].x);
    float Z = 0.f;
    for (int j = 0; j < n_split; ++j) {
        const float2 v = s[(size_t)j * rows_pad];
        Z += v.y * fast_exp2(v.x - M);
    }
    return M + __log2f(Z);
}

// Up to this many splits, and for row sets of one chunk, the column-sum workgroups
// merge the statistics of their rows themselves while they stage them, which saves a
// launch; else a launch of its own merges each row once (every workgroup of a longer row
// set would merge all of it, chunk by chunk).  Self-contained scores in us, launch /
// inline: 8 layers of 1531 keys (24 query tokens, 8 KV heads) 25.7 / 23.6, 32 of 8192
// 314 / 313, 40 of 16384 934 / 927, 8 of 32768 (320 rows, 8 splits) 378 / 371, 40 of them
// 1829 / 1820; 1024 rows of 2048 keys 98.8 / 100.1, 2048 rows of 4096 keys 189 / 202,
// 16000 rows of 3000 keys, 4 layers, 1092 / 1176.  (All splits' loads in flight at once
// made the merge shorter and the main loop behind it 0.4 to 1.6% longer.)
constexpr int kMergeInline = 8;

// The accumulator start values of the column-sum pass: Ls[rb][hf][i] = -lse2 / sl2
// of row rc0 + 32 rb + 8 (i / 4) + 4 hf + i % 4, the row that element i of an
// S = Q K^T accumulator of row block rb holds in lane half hf; -inf for padding
// rows (their probabilities are then exp2(-inf) = 0).  From q_lse if given, else
// from the merged lse2 or, with n_merge > 0, from the statistics of n_merge splits
// that lse2 then points at.
__device__ __forceinline__ void stage_lse(float (*Ls)[2][16], int nt, int l, int g, int Qn,
                                          int H, int Hkv, int G, int n_rows, int rows_pad,
                                          int rc0, int nrb, float sl2,
                                          const float* __restrict__ lse2,
                                          const float* __restrict__ q_lse, int n_merge) {
    // (the index is opaque, so that nothing derived from it stays live across the
    // caller's main loop)
    int f0 = threadIdx.x;
    asm volatile("" : "+v"(f0));
    for (int f = f0; f < nrb * 32; f += nt) {
        const int rb = f >> 5, hh = (f >> 4) & 1, i = f & 15;
        const int row = rc0 + 32 * rb + 8 * (i >> 2) + 4 * hh + (i & 3);
        const float x = row >= n_rows ? INFINITY
                        : q_lse ? q_lse[((size_t)l * Qn + row / G) * H + g * G + row % G] * kLog2e
                        : n_merge
                            ? merge_stats((const float2*)lse2 +
                                              ((size_t)l * Hkv + g) * n_merge * rows_pad + row,
                                          n_merge, rows_pad)
                            : lse2[((size_t)l * Hkv + g) * rows_pad + row];
        Ls[rb][hh][i] = -x / sl2;
    }
}

// The 32-key blocks kr + 32 kb (kb < NKB) of K into registers, as MFMA operands
// (lane l: key kr + 32 kb + l % 32, 16-byte chunk 2j + l / 32 of k-step j); keys
// past T re-read key T-1 (their results are masked or never stored).
template <int D, int NKB>
__device__ __forceinline__ void load_keys(bf16x8 (&dst)[NKB][D / 16], const uint16_t* Kg, int T,
                                          int64_t sT, int kr, int r32, int hf) {
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        const int key = min(kr + 32 * kb + r32, T - 1);
        const bf16x8* kp = (const bf16x8*)(Kg + key * sT + hf * 8);
#pragma unroll
        for (int j = 0; j < D / 16; ++j) dst[kb][j] = kp[2 * j];
    }
}

// Column-sum pass with the keys in registers (rows known by their log2-sum-exp).
// A workgroup takes one (layer l, KV head g, key split).  The query rows of the
// group are staged once into LDS, fragment-major: fragment (rb, j) is the MFMA A
// operand of 32-row block rb and k-step j, lane l's 16 bytes at 16 l, so every
// read is one conflict-free ds_read_b128 at a fixed offset from the lane's base.
// Each accumulator starts at its rows' -lse2 / sl2 (the C operand of the first
// MFMA, read from a small LDS table; the lanes of a half read the same 64
// bytes), so it ends at s - lse2 / sl2 and exp2(sl2 * acc) is the probability.
// Each wave owns NKB blocks of 32 keys per round, loads them from HBM straight
// into registers (the B operand of S = Q K^T: lane l holds key l % 32, the
// 16-byte chunk 2j + l / 32 of k-step j) and runs every row block against them,
// so a query fragment read from LDS feeds NKB MFMAs and K needs no LDS at all.
// Per lane the 16 rows of a block are summed in fp32 in a fixed order, then the
// two half-waves are added: part[l][g][key] (added to the earlier row chunks'
// sum when the row set takes several chunks).  The next round's keys are
// loaded while the last row block's exp2 work runs.  Waves never wait for one
// another inside a row chunk.
template <int D, int NW, int NKB>
__global__ __launch_bounds__(NW * 64) void score_colsum_kreg(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc, KvStrides ks, int T, int Qn, int H,
    int Hkv, int G, int n_rows, int rows_pad, int keys_per_split, float sl2,
    const float* __restrict__ lse2, const float* __restrict__ q_lse, int n_merge,
    float* __restrict__ part) {
    constexpr int KS = D / 16;                      // k-steps of the dot product
    constexpr int NRB = kKregRowBlocks;             // row blocks per chunk
    constexpr int KPW = NKB * 32;                   // keys of a wave per round
    constexpr int KPR = NW * KPW;                   // keys of the workgroup per round
    __shared__ bf16x8 Qs[NRB * KS * 64];
    __shared__ __attribute__((aligned(64))) float Ls[NRB][2][16];

    const int split = blockIdx.x, g = blockIdx.y, l = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hf = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t* Kg = kc + l * ks.layer + g * ks.head;
    float* part_g = part + ((size_t)l * Hkv + g) * T;
    const int key0 = split * keys_per_split;
    const int key1 = min(T, key0 + keys_per_split);

    bf16x8 kf[NKB][KS];
    auto load_k = [&](bf16x8 (&dst)[NKB][KS], int kr) { load_keys<D, NKB>(dst, Kg, T, ks.token, kr, r32, hf); };

    for (int rc0 = 0; rc0 < rows_pad; rc0 += NRB * 32) {
        const int nrb = min(NRB, (rows_pad - rc0) / 32);
        __syncthreads();                             // the previous chunk's reads are done
        stage_rows<D, NW>(Qs, q, l, g, Qn, H, G, n_rows, rc0, nrb);
        stage_lse(Ls, NW * 64, l, g, Qn, H, Hkv, G, n_rows, rows_pad, rc0, nrb, sl2, lse2, q_lse,
                  n_merge);
        __syncthreads();

        // One round: the wave's NKB key blocks (in kfr) against every row block;
        // hook(rb) runs after the MFMAs of row block rb (before its exp2 work).
        auto round = [&](const bf16x8 (&kfr)[NKB][KS], int kr, auto&& hook) {
            float cs[NKB][2];
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) cs[kb][0] = cs[kb][1] = 0.f;
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                if (rb >= nrb) break;
                f32x16 acc[NKB];
                const f32x16 init = *(const f32x16*)&Ls[rb][hf][0];
                const bf16x8* qb = Qs + rb * KS * 64 + lane;
#pragma unroll
                for (int j = 0; j < KS; ++j) {
                    const bf16x8 qj = qb[j * 64];
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb)
                        acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            qj, kfr[kb][j], j == 0 ? init : acc[kb], 0, 0, 0);
                }
                hook(rb);
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int v = 0; v < 16; ++v) cs[kb][v & 1] += fast_exp2(acc[kb][v] * sl2);
            }
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                const float s = pair_add(cs[kb][0] + cs[kb][1]);
                const int key = kr + 32 * kb + r32;
                if (hf == 0 && key < key1) part_g[key] = rc0 == 0 ? s : part_g[key] + s;
            }
        };

        int kr = key0 + w * KPW;
        if (kr < key1) load_k(kf, kr);
        for (; kr < key1; kr += KPR)
            round(kf, kr, [&](int rb) { if (rb == nrb - 1 && kr + KPR < key1) load_k(kf, kr + KPR); });
    }
}

// Row statistics with the keys in registers: the same workgroup shape, staging
// and key rounds as score_colsum_kreg, with S^T = K Q^T (K the A operand from
// registers, the staged query fragment the B operand), so lane l holds row
// 32 rb + l % 32 and 16 keys of each 32-key block.  Per row block each lane
// keeps (m, z) = (reference, sum of exp2(s - m)) in log2 units over its keys,
// with a lazy reference: m starts at 0 and moves only when a block's sum
// leaves [2^-64, 2^64], to the larger of the block maximum and log2 of the
// running sum (so no term and no running sum exceeds 16 * 2^m); until some lane
// of the wave moves, m = 0 costs no subtraction.  Logits hundreds of log2 units
// from 0 (either sign) stay exact.  At the end of a row chunk the two
// half-waves and then the NW waves are merged in a fixed order (through LDS)
// into stats[l][g][split][row].
template <int D, int NW, int NKB>
__global__ __launch_bounds__(NW * 64) void score_stats_kreg(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc, KvStrides ks, int T, int Qn, int H,
    int Hkv, int G, int n_rows, int rows_pad, int keys_per_split, int n_split, float sl2,
    float2* __restrict__ stats) {
    constexpr int KS = D / 16;
    constexpr int NRB = kKregRowBlocks;
    constexpr int KPW = NKB * 32;
    constexpr int KPR = NW * KPW;
    __shared__ bf16x8 Qs[NRB * KS * 64];
    __shared__ float2 red[NW][NRB * 32];

    const int split = blockIdx.x, g = blockIdx.y, l = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hf = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint16_t* Kg = kc + l * ks.layer + g * ks.head;
    const int key0 = split * keys_per_split;
    const int key1 = min(T, key0 + keys_per_split);
    bf16x8 kf[NKB][KS];

    for (int rc0 = 0; rc0 < rows_pad; rc0 += NRB * 32) {
        const int nrb = min(NRB, (rows_pad - rc0) / 32);
        __syncthreads();                             // the previous chunk's reads are done
        stage_rows<D, NW>(Qs, q, l, g, Qn, H, G, n_rows, rc0, nrb);
        __syncthreads();

        float m_ref[NRB], z_run[NRB];
        bool moved[NRB];                             // some lane of the wave left reference 0
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            m_ref[rb] = 0.f;
            z_run[rb] = 0.f;
            moved[rb] = false;
        }
        int kr = key0 + w * KPW;
        if (kr < key1) load_keys<D, NKB>(kf, Kg, T, ks.token, kr, r32, hf);
        for (; kr < key1; kr += KPR) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) {
                if (rb < nrb) {
                    f32x16 acc[NKB];
                    const bf16x8* qb = Qs + rb * KS * 64 + lane;
#pragma unroll
                    for (int j = 0; j < KS; ++j) {
                        const bf16x8 qj = qb[j * 64];
#pragma unroll
                        for (int kb = 0; kb < NKB; ++kb)
                            acc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                kf[kb][j], qj, j == 0 ? f32x16{} : acc[kb], 0, 0, 0);
                    }
                    if (rb == nrb - 1 && kr + KPR < key1)
                        load_keys<D, NKB>(kf, Kg, T, ks.token, kr + KPR, r32, hf);
#pragma unroll
                    for (int kb = 0; kb < NKB; ++kb) {
                        // acc[kb][v] is key kr + 32 kb + 8(v/4) + 4 hf + v%4 of the row.
                        const int kb0 = kr + 32 * kb;
                        if (kb0 + 32 > key1) {
#pragma unroll
                            for (int v = 0; v < 16; ++v)
                                if (kb0 + 8 * (v >> 2) + 4 * hf + (v & 3) >= key1)
                                    acc[kb][v] = -INFINITY;
                        }
                        float z0 = 0.f, z1 = 0.f;
                        if (moved[rb]) {
                            const float m = m_ref[rb];
#pragma unroll
                            for (int v = 0; v < 16; v += 2) {
                                z0 += fast_exp2(fmaf(acc[kb][v], sl2, -m));
                                z1 += fast_exp2(fmaf(acc[kb][v + 1], sl2, -m));
                            }
                        } else {
#pragma unroll
                            for (int v = 0; v < 16; v += 2) {
                                z0 += fast_exp2(acc[kb][v] * sl2);
                                z1 += fast_exp2(acc[kb][v + 1] * sl2);
                            }
                        }
                        float zb = z0 + z1;
                        const bool out = !(zb <= kRefHi) || z_run[rb] + zb < kRefLo;
                        if (__builtin_expect(out, 0)) {
                            // New reference: the larger of the block maximum and the
                            // log2 of what the row has summed so far.
                            float mt = acc[kb][0];
#pragma unroll
                            for (int v = 1; v < 16; ++v) mt = fmaxf(mt, acc[kb][v]);
                            mt *= sl2;
                            const float lz =
                                z_run[rb] > 0.f ? m_ref[rb] + __log2f(z_run[rb]) : -INFINITY;
                            mt = fmaxf(mt, lz);
                            if (mt > -INFINITY) {
                                zb = 0.f;
#pragma unroll
                                for (int v = 0; v < 16; ++v)
                                    zb += fast_exp2(fmaf(acc[kb][v], sl2, -mt));
                                z_run[rb] = fast_exp2(lz - mt);
                                m_ref[rb] = mt;
                            }
                        }
                        moved[rb] = moved[rb] || __any(out);
                        z_run[rb] += zb;
                    }
                }
            }
        }
        // Each half-wave's (m, z) per row; a half that met no key holds (0, 0)
        // and becomes (-inf, 0), so no merge takes its 0 as the reference.
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
            if (rb < nrb) {
                const float m = z_run[rb] > 0.f ? m_ref[rb] : -INFINITY, z = z_run[rb];
                const float m2 = pair_other(m), z2 = pair_other(z);
                const float M = fmaxf(m, m2);
                const float Z = M == -INFINITY ? 0.f : z * fast_exp2(m - M) + z2 * fast_exp2(m2 - M);
                if (hf == 0) red[w][rb * 32 + r32] = make_float2(M, Z);
            }
        }
        __syncthreads();
        for (int row = tid; row < nrb * 32; row += NW * 64) {
            float M = -INFINITY;
#pragma unroll
            for (int ww = 0; ww < NW; ++ww) M = fmaxf(M, red[ww][row].x);
            float Z = 0.f;
            if (M > -INFINITY) {
#pragma unroll
                for (int ww = 0; ww < NW; ++ww) Z += red[ww][row].y * fast_exp2(red[ww][row].x - M);
            }
            stats[(((size_t)l * Hkv + g) * n_split + split) * rows_pad + rc0 + row] = make_float2(M, Z);
        }
    }
}

// Per row: merge the splits' (m, sum) pairs into a log2-sum-exp.
__global__ void score_merge(const float2* __restrict__ stats, int n_groups, int n_split,
                            int rows_pad, int n_rows, float* __restrict__ lse2) {
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= (long)n_groups * rows_pad) return;
    const long lg = i / rows_pad;
    const int row = (int)(i % rows_pad);
    if (row >= n_rows) {
        lse2[i] = INFINITY;     // padding rows contribute exp2(-inf) = 0
        return;
    }
    lse2[i] = merge_stats(stats + lg * n_split * rows_pad + row, n_split, rows_pad);
}

// ---------------------------------------------------------------- float32 path

// float32 MFMA (32x32x2: the products and sums of fp32 FMAs), operands straight from
// memory: lane l holds, of row or key l % 32 and of every 8 d values, the 4 at
// 4 (l / 32) (the contraction may take its index in any order, the same on both
// sides).  Against the VALU kernels before (one thread per key and all rows, one
// workgroup per row and all keys): 12 layers of 3000 keys, 64 query tokens, 32q/8kv
// heads, d 128, 8.06 -> 0.53 ms; 2 layers of 1024 keys, 4q/2kv heads 44 -> 23 us.
constexpr int kF32Waves = 8;            // of the column sums
constexpr int kF32StatsWaves = 16;
constexpr int kF32Round = kF32StatsWaves * 32;           // keys of a workgroup per round
constexpr int kF32Units = 64;                            // most units of the row statistics
constexpr int kF32Batch = 8;                             // units between two merges

template <int D>
__device__ __forceinline__ void load_row_f32(f32x4 (&dst)[D / 8], const float* p, int hf) {
#pragma unroll
    for (int j = 0; j < D / 8; ++j) dst[j] = *(const f32x4*)(p + 8 * j + 4 * hf);
}

template <int D>
__device__ __forceinline__ f32x16 dot_f32(const f32x4 (&a)[D / 8], const f32x4 (&b)[D / 8]) {
    f32x16 s = f32x16{};
#pragma unroll
    for (int j = 0; j < D / 8; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j][i], b[j][i], s, 0, 0, 0);
    return s;
}

// Row statistics over units of n_round rounds of 512 keys (one round up to 32768 keys, as
// many as make 64 units past that): a workgroup takes 32 (token, head) rows of a KV head
// of a layer and `per` consecutive units, one 32-key block per wave and round (S^T =
// K Q^T, one row per lane; Q staged in LDS, the next round's K loaded behind this one's
// products).  Every kF32Batch units the waves' (max, sum) of each unit are merged in wave
// order, a wave per unit; the units' pairs are merged in order, by the workgroup if it has
// them all, else by score_merge_f32.  The units depend on T only, so the bits are the same
// however they are spread over workgroups.
__device__ __forceinline__ float merge_units_f32(const float2* __restrict__ s, int n, size_t stride) {
    float M = -INFINITY, Z = 0.f;
#pragma unroll 8                                         // (loads in flight, in-order sum)
    for (int j = 0; j < n; ++j) M = fmaxf(M, s[j * stride].x);
#pragma unroll 8
    for (int j = 0; j < n; ++j) Z += s[j * stride].y * expf(s[j * stride].x - M);
    return M + logf(Z);
}

template <int D>
__global__ __launch_bounds__(kF32StatsWaves * 64) void score_stats_f32(
    const float* __restrict__ q, const float* __restrict__ kc, KvStrides ks, int T, int Qn, int H,
    int Hkv, int G, int n_rows, int rows_pad, int n_unit, int n_round, int per, float scale,
    float2* __restrict__ stats, float* __restrict__ lse_nat) {
    __shared__ f32x4 Qs[D / 8][64];
    __shared__ float2 red[kF32Batch][kF32StatsWaves][32], table[kF32Units][32];
    const int g = blockIdx.y, l = blockIdx.z;
    const int n_split = (n_unit + per - 1) / per;
    const int rb = blockIdx.x / n_split, u0 = (blockIdx.x - rb * n_split) * per;
    const int u1 = min(n_unit, u0 + per);
    const bool own = n_split == 1;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hf = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int row = rb * 32 + r32, rr = min(row, n_rows - 1);
    const size_t lg = (size_t)l * Hkv + g;
    const float* Kg = kc + l * ks.layer + g * ks.head;
    f32x4 kf[D / 8];
    auto load_k = [&](int k0) { load_row_f32<D>(kf, Kg + min(k0 + r32, T - 1) * ks.token, hf); };
    int k0 = u0 * n_round * kF32Round + w * 32;
    load_k(k0);
    const float* qrow = q + (((size_t)l * Qn + rr / G) * H + g * G + rr % G) * D;
    for (int j = w; j < D / 8; j += kF32StatsWaves) Qs[j][lane] = *(const f32x4*)(qrow + 8 * j + 4 * hf);
    __syncthreads();
    for (int u = u0; u < u1; ++u) {
        float m = -INFINITY, z = 0.f;
        for (int r = 0; r < n_round; ++r, k0 += kF32Round) {
            if (k0 >= T) continue;
            f32x16 s = f32x16{};
#pragma unroll
            for (int j = 0; j < D / 8; ++j) {
                const f32x4 qj = Qs[j][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[j][i], qj[i], s, 0, 0, 0);
            }
            if (r + 1 < n_round || u + 1 < u1) load_k(k0 + kF32Round);
            const int ex = T - 1 - k0 - 4 * hf;          // last key of the block
            float mx = m;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                s[v] = 8 * (v >> 2) + (v & 3) > ex ? -INFINITY : s[v] * scale;
                mx = fmaxf(mx, s[v]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));      // (the row's other half-wave)
            z *= expf(m - mx);
            m = mx;
#pragma unroll
            for (int v = 0; v < 16; ++v) z += expf(s[v] - m);
        }
        z += __shfl_xor(z, 32, 64);
        const int x = (u - u0) % kF32Batch;
        if (hf == 0) red[x][w][r32] = make_float2(m, z);
        if (x + 1 < kF32Batch && u + 1 < u1) continue;
        __syncthreads();
        if (w <= x && hf == 0) {
            float M = -INFINITY, Z = 0.f;
            for (int i = 0; i < kF32StatsWaves; ++i) M = fmaxf(M, red[w][i][r32].x);
            for (int i = 0; i < kF32StatsWaves; ++i)     // (a wave past the last key adds 0 * exp(-inf))
                Z += red[w][i][r32].y * expf(red[w][i][r32].x - M);
            const int uw = u - x + w;
            if (n_unit == 1) {
                if (row < n_rows) lse_nat[lg * rows_pad + row] = M + logf(Z);
            } else if (own) {
                table[uw][r32] = make_float2(M, Z);
            } else if (row < n_rows) {
                stats[(lg * n_unit + uw) * rows_pad + row] = make_float2(M, Z);
            }
        }
        __syncthreads();
    }
    if (own && n_unit > 1 && tid < 32 && row < n_rows)   // (one unit: see above)
        lse_nat[lg * rows_pad + row] = merge_units_f32(&table[0][r32], n_unit, 32);
}

__global__ void score_merge_f32(const float2* __restrict__ stats, int n_groups, int n_unit,
                                int rows_pad, int n_rows, float* __restrict__ lse_nat) {
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= (long)n_groups * rows_pad || i % rows_pad >= n_rows) return;
    lse_nat[i] = merge_units_f32(stats + i / rows_pad * n_unit * rows_pad + i % rows_pad, n_unit, rows_pad);
}

// Column sums: a workgroup takes 32 keys of a layer; its waves share out the (KV
// head, 32-row block) units in order (S = Q K^T, one key per lane).  Summed in
// double: a key's column takes H * Qn terms (thousands for long queries and wide
// GQA groups), and a float running sum of that many terms drifts by more than the
// 1e-5 the fp32 path has to meet after MinMax.
template <int D>
__global__ __launch_bounds__(kF32Waves * 64) void score_colsum_f32(
    const float* __restrict__ q, const float* __restrict__ kc, KvStrides ks, int T, int Qn, int H,
    int Hkv, int G, int n_rows, int rows_pad, float scale, const float* __restrict__ lse_nat,
    const float* __restrict__ q_lse, float* __restrict__ part) {
    __shared__ double red[kF32Waves][32];
    const int l = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hf = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int key = min((int)blockIdx.x * 32 + r32, T - 1);
    const int nrb = rows_pad / 32, units = Hkv * nrb, per = (units + kF32Waves - 1) / kF32Waves;
    const int u1 = min(units, (w + 1) * per);
    f32x4 qf[D / 8], kf[D / 8];
    int g_in = -1;                                       // the KV head whose keys are in kf
    double acc = 0.0;
    for (int u = w * per; u < u1; ++u) {
        const int g = u / nrb, row = (u - g * nrb) * 32 + r32, rr = min(row, n_rows - 1);
        const size_t th = ((size_t)l * Qn + rr / G) * H + g * G + rr % G;
        if (g != g_in) load_row_f32<D>(kf, kc + l * ks.layer + g * ks.head + key * ks.token, hf);
        g_in = g;
        load_row_f32<D>(qf, q + th * D, hf);
        const float lse = row >= n_rows ? INFINITY
                          : q_lse ? q_lse[th]
                                  : lse_nat[((size_t)l * Hkv + g) * rows_pad + row];
        const f32x16 s = dot_f32<D>(qf, kf);
#pragma unroll
        for (int v = 0; v < 16; ++v)
            acc += (double)expf(s[v] * scale - __shfl(lse, 8 * (v >> 2) + 4 * hf + (v & 3), 64));
    }
    acc += __shfl_xor(acc, 32, 64);
    if (hf == 0) red[w][r32] = acc;
    __syncthreads();
    const int i = blockIdx.x * 32 + tid;
    if (tid < 32 && i < T) {
        double p = 0.0;
        for (int ww = 0; ww < kF32Waves; ++ww) p += red[ww][tid];
        part[(size_t)l * T + i] = (float)p;
    }
}

// ---------------------------------------------------------------- finaliser

// Finaliser, two launches over (key block, layer):
//   score_pool: p_i = (1/(H Qn)) * sum over the n_part partial slices (fixed
//     order), written to scores, plus each block's (min, max) of p;
//   score_minmax: every block reduces its layer's block extrema (fixed order)
//     and rescales its keys to a = (p - min) / (max - min), or 0 when flat.
constexpr int kFinKeys = 1024;                 // keys per finaliser block (256 threads x 4)
// Longest context of the one-launch finaliser.  One-pass scores of one query token in
// us, two launches / one: 1024 keys 10.9 / 8.3 (one layer of 8 KV heads), 2048 keys 10.6
// / 8.9, 27.8 / 24.2 (40 layers), 24.6 / 19.1 (8 layers of 32 KV heads), 101 / 97 (200
// layers); 3000 keys 11.1 / 14.7, 33.8 / 36.9 (40 layers); 4096 keys 10.9 / 15.2.
constexpr int kFinishMaxT = 2048;

__global__ __launch_bounds__(256) void score_pool(const float* __restrict__ part, int n_part,
                                                  int T, float inv_hq, float* __restrict__ scores,
                                                  float2* __restrict__ mm, int n_blk) {
    __shared__ float red_lo[4], red_hi[4];
    const int blk = blockIdx.x, l = blockIdx.y, tid = threadIdx.x;
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = blk * kFinKeys + e * 256 + tid;
        if (i < T) {
            float p = 0.f;
            // eight independent loads in flight, summed in order: 15.8 -> 5.2 us at 32
            // layers of 8192 keys and 8 KV heads, 22.2 -> 10.5 us at 40 of 32768
#pragma unroll 8
            for (int j = 0; j < n_part; ++j) p += part[((size_t)l * n_part + j) * T + i];
            p *= inv_hq;
            scores[(size_t)l * T + i] = p;
            lo = fminf(lo, p);
            hi = fmaxf(hi, p);
        }
    }
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) {
        red_lo[tid >> 6] = lo;
        red_hi[tid >> 6] = hi;
    }
    __syncthreads();
    if (tid == 0) {
        float a = red_lo[0], b = red_hi[0];
        for (int i = 1; i < 4; ++i) {
            a = fminf(a, red_lo[i]);
            b = fmaxf(b, red_hi[i]);
        }
        mm[(size_t)l * n_blk + blk] = make_float2(a, b);
    }
}

__global__ __launch_bounds__(256) void score_minmax(const float2* __restrict__ mm, int n_blk, int T,
                                                    float* __restrict__ scores) {
    __shared__ float red_lo[4], red_hi[4];
    const int blk = blockIdx.x, l = blockIdx.y, tid = threadIdx.x;
    float lo = INFINITY, hi = -INFINITY;
    for (int b = tid; b < n_blk; b += 256) {
        const float2 v = mm[(size_t)l * n_blk + b];
        lo = fminf(lo, v.x);
        hi = fmaxf(hi, v.y);
    }
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) {
        red_lo[tid >> 6] = lo;
        red_hi[tid >> 6] = hi;
    }
    __syncthreads();
    lo = fminf(fminf(red_lo[0], red_lo[1]), fminf(red_lo[2], red_lo[3]));
    hi = fmaxf(fmaxf(red_hi[0], red_hi[1]), fmaxf(red_hi[2], red_hi[3]));
    const bool flat = !(hi > lo);
    const float span = hi - lo;
    float* a = scores + (size_t)l * T;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int i = blk * kFinKeys + e * 256 + tid;
        if (i < T) a[i] = flat ? 0.f : (a[i] - lo) / span;
    }
}

// Both steps in one launch for the contexts whose pooled mass one workgroup per layer
// holds in registers (E positions a thread): the same operations in the same order
// (extrema do not depend on it).  At 8 layers of 1531 positions 3.8 us against two
// launches of 4; one workgroup alone reads a layer's partial sums slowly, so at 8192
// positions and 8 KV heads it takes 28 us against 10 for the two.
template <int E>
__global__ __launch_bounds__(1024) void score_finish(const float* __restrict__ part, int n_part,
                                                     int T, float inv_hq,
                                                     float* __restrict__ scores) {
    __shared__ float red_lo[16], red_hi[16];
    const int l = blockIdx.x, tid = threadIdx.x;
    float p[E];
#pragma unroll
    for (int e = 0; e < E; ++e) p[e] = 0.f;
    const float* pl = part + (size_t)l * n_part * T;
#pragma unroll 4
    for (int j = 0; j < n_part; ++j)
#pragma unroll
        for (int e = 0; e < E; ++e) p[e] += pl[(size_t)j * T + min(e * 1024 + tid, T - 1)];
    float lo = INFINITY, hi = -INFINITY;
#pragma unroll
    for (int e = 0; e < E; ++e) {                        // (positions past T repeat the last one)
        p[e] *= inv_hq;
        lo = fminf(lo, p[e]);
        hi = fmaxf(hi, p[e]);
    }
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    if ((tid & 63) == 0) {
        red_lo[tid >> 6] = lo;
        red_hi[tid >> 6] = hi;
    }
    __syncthreads();
    lo = red_lo[0];
    hi = red_hi[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) {
        lo = fminf(lo, red_lo[i]);
        hi = fmaxf(hi, red_hi[i]);
    }
    const bool flat = !(hi > lo);
    const float span = hi - lo;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = e * 1024 + tid;
        if (i < T) scores[(size_t)l * T + i] = flat ? 0.f : (p[e] - lo) / span;
    }
}

void launch_finalize(const relaxkv_problem& p, const ScoreWorkspace& w, char* ws, float* scores,
                     hipStream_t st) {
    const float inv_hq = 1.0f / ((float)p.H * (float)p.n_query);
    auto finish = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(p.L), dim3(1024), 0, st, (const float*)(ws + w.part_off),
                           w.n_part, p.T_c, inv_hq, scores);
    };
    if (p.T_c <= kFinishMaxT) return finish(score_finish<kFinishMaxT / 1024>);
    const dim3 grid(w.n_blk, p.L);
    float2* mm = (float2*)(ws + w.mm_off);
    hipLaunchKernelGGL(score_pool, grid, dim3(256), 0, st, (const float*)(ws + w.part_off), w.n_part,
                       p.T_c, inv_hq, scores, mm, w.n_blk);
    hipLaunchKernelGGL(score_minmax, grid, dim3(256), 0, st, (const float2*)mm, w.n_blk, p.T_c, scores);
}

// Keys per workgroup of a scoring pass: the power of two in [512, max_split] that
// needs the fewest key-steps per CU, ceil(workgroups / 256) * (keys + 900), the
// larger one on a tie.  The 900 keys stand for what a workgroup costs before its
// first key (the start and the staging of its query rows, 6-9 us, against 3-5 us
// for 512 keys at 96-256 query rows).  Measured, self-contained scores in us with
// the statistics pass at 512 / 1024 / 2048 / 4096 keys: 4 layers of 3000 keys (8 KV
// heads, 64 query tokens) 68 / 72 / 82 / 93, 12 layers 100 / 95 / 87 / 95, 32 layers
// 167 / 140 / 141 / 124, 40 layers of 4096 (40 heads) 364 / 316 / 308 / 333; the
// column-sum pass runs in the same order.
int pass_split(const relaxkv_problem& p, int max_split) {
    constexpr long kCUs = 256, kStart = 900;
    long best = 0, best_cost = 0;
    for (long split = max_split; split >= 512; split /= 2) {
        const long wg = (p.T_c + split - 1) / split * (long)p.H_kv * p.L;
        const long keys = split < p.T_c ? split : (p.T_c + 511) / 512 * 512;
        const long cost = (wg + kCUs - 1) / kCUs * (keys + kStart);
        if (!best || cost < best_cost) {
            best = split;
            best_cost = cost;
        }
    }
    return (int)best;
}

// Column sums: each key's does not depend on the split, so neither do the scores.
int colsum_split(const relaxkv_problem& p) { return pass_split(p, 2 * kKeysPerSplit); }

// Statistics: the split sets the order in which a row's sum is merged, so it is
// fixed for the contexts of more than one full-size split (their scores are then
// the same bits whatever the number of layers) and chosen below.
int stats_split(const relaxkv_problem& p) {
    return p.T_c > kKeysPerSplit ? kKeysPerSplit : pass_split(p, kKeysPerSplit);
}

template <int D>
void launch_passes_bf16(const relaxkv_problem& p, const ScoreWorkspace& w, char* ws,
                        hipStream_t st, float sl2) {
    const int G = p.H / p.H_kv;
    const int n_rows = p.n_query * G;
    const uint16_t* q = (const uint16_t*)p.q;
    const uint16_t* kc = (const uint16_t*)p.k_cache;
    float* part = (float*)(ws + w.part_off);
    float* lse2 = (float*)(ws + w.lse_off);
    float2* stats = (float2*)(ws + w.stats_off);
    constexpr int KNW = RELAXKV_SCORE_KREG_NW, KNKB = RELAXKV_SCORE_KREG_NKB;
    constexpr int CNW = RELAXKV_SCORE_COLSUM_NW, CNKB = RELAXKV_SCORE_COLSUM_NKB;
    static_assert(kKeysPerSplit % (KNW * KNKB * 32) == 0 && kKeysPerSplit % (CNW * CNKB * 32) == 0,
                  "a full-size split is whole rounds of both passes");
    const int kps = stats_split(p);
    const dim3 kgrid((p.T_c + kps - 1) / kps, p.H_kv, p.L);
    const bool inline_merge = !p.q_lse && w.n_split <= kMergeInline && w.rows_pad <= kKregRowBlocks * 32;
    if (!p.q_lse) {
        hipLaunchKernelGGL((score_stats_kreg<D, KNW, KNKB>), kgrid, dim3(KNW * 64), 0, st, q, kc,
                           kv_strides(p), p.T_c, p.n_query, p.H, p.H_kv, G, n_rows, w.rows_pad, kps, w.n_split,
                           sl2, stats);
        const long n = (long)p.L * p.H_kv * w.rows_pad;
        if (!inline_merge)
            hipLaunchKernelGGL(score_merge, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                               (const float2*)stats, p.L * p.H_kv, w.n_split, w.rows_pad, n_rows, lse2);
    }
    const int cps = colsum_split(p);
    const dim3 cgrid((p.T_c + cps - 1) / cps, p.H_kv, p.L);
    hipLaunchKernelGGL((score_colsum_kreg<D, CNW, CNKB>), cgrid, dim3(CNW * 64), 0, st, q, kc,
                       kv_strides(p), p.T_c, p.n_query, p.H, p.H_kv, G, n_rows, w.rows_pad, cps, sl2,
                       inline_merge ? (const float*)stats : (const float*)lse2, p.q_lse,
                       inline_merge ? w.n_split : 0, part);
}

template <int D>
hipError_t launch_score_bf16(const relaxkv_problem& p, const ScoreWorkspace& w, char* ws,
                             float* scores, hipStream_t st, float scale) {
    launch_passes_bf16<D>(p, w, ws, st, scale * kLog2e);
    launch_finalize(p, w, ws, scores, st);
    return hipGetLastError();
}

// The float32 statistics' rounds per unit, units, and units per workgroup: as many splits as give each CU at most
// one workgroup, since a workgroup's units are a serial chain.  Self-contained scores
// in us, one workgroup per row and VALU / one per 32 rows and all keys / split: one
// layer of 30000 keys and 64 rows 286 / 422 / 34, of 8000 and 24 rows 185 / 189 / 40, 2
// of 2000 and 2 rows 29 / 37 / 21, 2 of 1024 and 32 rows 43 / 27 / 20, 4 of 3000 and
// 2048 rows (256 workgroups: not split) 4997 / 186 / 184.
struct F32Units {
    int n_round, n_unit, per;
};
F32Units f32_units(const relaxkv_problem& p) {
    constexpr long kCUs = 256;
    const int rounds = (p.T_c + kF32Round - 1) / kF32Round;
    F32Units u;
    u.n_round = (rounds + kF32Units - 1) / kF32Units;
    u.n_unit = (rounds + u.n_round - 1) / u.n_round;
    const long wg = (long)(round_up32(p.n_query * (p.H / p.H_kv)) / 32) * p.H_kv * p.L;
    const int split = wg >= kCUs ? 1 : (int)(kCUs / wg);
    u.per = (u.n_unit + split - 1) / split;
    return u;
}

template <int D>
hipError_t launch_score_f32(const relaxkv_problem& p, const ScoreWorkspace& w, char* ws,
                            float* scores, hipStream_t st, float scale) {
    const int G = p.H / p.H_kv;
    const float* q = (const float*)p.q;
    const float* kc = (const float*)p.k_cache;
    float* part = (float*)(ws + w.part_off);
    float* lse = (float*)(ws + w.lse_off);
    if (!p.q_lse) {
        float2* stats = (float2*)(ws + w.stats_off);
        const F32Units u = f32_units(p);
        hipLaunchKernelGGL(score_stats_f32<D>, dim3(w.rows_pad / 32 * w.n_split, p.H_kv, p.L),
                           dim3(kF32StatsWaves * 64), 0, st, q, kc, kv_strides(p), p.T_c, p.n_query,
                           p.H, p.H_kv, G, p.n_query * G, w.rows_pad, u.n_unit, u.n_round, u.per, scale,
                           stats, lse);
        const long n = (long)p.L * p.H_kv * w.rows_pad;
        if (w.n_split > 1)
            hipLaunchKernelGGL(score_merge_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                               (const float2*)stats, p.L * p.H_kv, u.n_unit, w.rows_pad, p.n_query * G,
                               lse);
    }
    hipLaunchKernelGGL(score_colsum_f32<D>, dim3((p.T_c + 31) / 32, p.L), dim3(kF32Waves * 64), 0, st,
                       q, kc, kv_strides(p), p.T_c, p.n_query, p.H, p.H_kv, G, p.n_query * G,
                       w.rows_pad, scale, lse, p.q_lse, part);
    launch_finalize(p, w, ws, scores, st);
    return hipGetLastError();
}

}  // namespace

ScoreWorkspace score_workspace_layout(const relaxkv_problem& p) {
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    ScoreWorkspace w;
    const int G = p.H / p.H_kv;
    const bool bf = p.dtype == RELAXKV_DTYPE_BF16;
    w.rows_pad = round_up32(p.n_query * G);
    const F32Units u = f32_units(p);
    const int kps = stats_split(p);
    w.n_split = bf ? (p.T_c + kps - 1) / kps : (u.n_unit + u.per - 1) / u.per;
    w.n_part = bf ? p.H_kv : 1;
    w.part_off = 0;
    size_t off = al((size_t)p.L * w.n_part * p.T_c * sizeof(float));
    w.stats_off = off;
    // (float32: a pair per unit, only where a merge launch reads them: below 256 row blocks)
    const int n_pair = bf ? w.n_split : w.n_split > 1 ? u.n_unit : 0;
    off += al((size_t)p.L * p.H_kv * n_pair * w.rows_pad * sizeof(float2));
    w.lse_off = off;
    off += al((size_t)p.L * p.H_kv * w.rows_pad * sizeof(float));
    w.n_blk = (p.T_c + kFinKeys - 1) / kFinKeys;
    w.mm_off = off;
    off += al((size_t)p.L * w.n_blk * sizeof(float2));
    w.total = off;
    return w;
}

hipError_t launch_score(const relaxkv_problem& p, const ScoreWorkspace& w, char* ws,
                        float* scores, hipStream_t st) {
    const float scale = p.softmax_scale > 0.f ? p.softmax_scale : 1.0f / sqrtf((float)p.d);
    if (p.dtype == RELAXKV_DTYPE_BF16) {
        return p.d == 128 ? launch_score_bf16<128>(p, w, ws, scores, st, scale)
                          : launch_score_bf16<64>(p, w, ws, scores, st, scale);
    }
    return p.d == 128 ? launch_score_f32<128>(p, w, ws, scores, st, scale)
                      : launch_score_f32<64>(p, w, ws, scores, st, scale);
}

}  // namespace relaxkv

// Sparse-context causal attention (Sec. 3.3-3.4, App. A.2; the attention step of
// Algorithm 1).  Target t of layer l (position p, compact index u_t in U)
// attends to the compact context c = 0 .. u_t (C_l(p) = U cap {j <= p}) or, for
// the Full-Prefix Control, to positions j = 0 .. p.  Key/value row j is the
// fresh row of j when j is in R_l (src[l][c] >= 0) and the naive cached row
// otherwise.
//
// bf16 kernel (bf16 MFMA 32x32x16, fp32 accumulation, flash-style online
// softmax in the exp2 domain):
// - a workgroup of NW = 12 waves owns NW*32 consecutive (target, head) rows (in
//   launches of few tiles a third of that, its waves split over the keys) of
//   one KV head g (row t*G + hh: target t, the hh-th of the G query heads that
//   share g), so every K/V row brought into LDS is used by NW*32 rows; a tile
//   may begin or end inside a target's group of heads, so no row is idle when
//   G does not divide NW*32;
// - context keys go in steps of 64 through a 4-deep ring of LDS buffers (a K
//   and a V tile per step, unpadded rows with an XOR swizzle), filled by direct
//   global->LDS loads that choose per key between the fresh rows
//   (k_new/v_new) and the cached layer; the keys' indices (U and src, or rank)
//   are staged into LDS the same way one step earlier, so the only vector
//   loads in flight are LDS fills, waited for by in-order counts;
// - each wave computes S^T = K Q^T with one query row per lane (Q stays in
//   registers), so row max and row sum are lane-local plus one exchange with
//   the lane 32 away; P^T stays in registers as the B operand of
//   O^T = V^T P^T, whose V^T operand comes from transposing LDS reads;
// - the mask is the staircase of the targets' limits: steps below the first
//   target's limit run unmasked, the rest compare each key with its row's limit,
//   and a wave skips the arithmetic of steps past all of its rows' limits;
// - tiles are taken heaviest-first (the last targets have the longest
//   contexts) from per-KV-head counters; a workgroup starts with the head tied
//   to its XCD, so the workgroups of one XCD share a KV head and its L2
//   working set, and takes the next head's tiles once its own are gone (the
//   XCDs run at different clocks, and a fixed map would wait for the slowest).
// fp32 kernel: the float32 MFMA core of attn_f32.h, 16 or 32 rows per workgroup; used for
// fp32 inputs, where bf16 MFMA would not meet fp32 accuracy.

#include <math.h>

#include "attn_f32.h"
#include "dev_common.h"
#include "internal.h"

namespace relaxkv {
namespace {

struct AttnArgs {
    const void* q_new;
    const void* k_new;
    const void* v_new;
    const void* kc;          // layer base: row i of KV head g at element g * kv_sh + i * kv_st
    const void* vc;
    const int32_t* U;
    const int32_t* cidx;
    const int32_t* src_l;    // src + layer * T
    const int32_t* rank_l;   // rank + layer * T
    const int32_t* R_off;
    const int32_t* R_idx;
    const int32_t* R_u;
    const int32_t* counts;
    int32_t* err;            // the error word counts[L+1]
    uint32_t* tiles;         // this layer's and mode's work counters: [Hkv] next tile, [Hkv] workgroups
    void* out;
    float* lse;
    int64_t kv_sh, kv_st;    // element strides of the cache's KV heads and tokens
    int H, Hkv, G, T, layer;
    int cap;                 // rows this launch may process (row capacity, host bound)
    float scale;             // softmax scale (natural units)
};

// ----------------------------------------------------------------- bf16 MFMA

template <int N> struct Int { static constexpr int value = N; };

constexpr float kRescaleSlack = 8.0f;      // log2 units the running max may lag the true max
constexpr int kXcds = 8;                   // XCDs of an MI355X (workgroup i runs on XCD i mod 8)
constexpr int kHwRegXccId = 20;            // hardware register holding the wave's XCD index

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// max / sum of a value and its copy in the lane 32 away (one VALU swap).
__device__ __forceinline__ float pair_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// NW waves as NW / KG groups of 32 rows times KG key groups; 64 keys per key group
// and step, one barrier per step.
// KG = 1 (12 waves; launches with tiles for every CU): a 4-deep ring.  The fills of
// step j+3 and the indices of step j+4 are issued right after the barrier of step
// j, so every fill has two steps of compute to land.
// KG = 2 (8 waves; launches with few tiles): a tile is a third of the rows, so
// there are three times as many workgroups, and each step brings 128 keys through a
// 2-deep ring, half for each key group (the fills of step j+1 go out after the
// barrier of step j; the rows of a KV head are shared by its workgroups, so most
// come from L2); the key groups keep their own running max, sum and output, which
// are combined through LDS after the last step like key splits.  The same fills
// serve a third of the rows, so a step costs more per row; it pays where CUs would
// stay idle (see attn_key_groups).
template <int D, bool FULL, int NW, int KG>
__global__ __launch_bounds__(NW * 64, 1) void attn_bf16(AttnArgs a) {
    static_assert(KG == 1 || KG == 2, "key groups");
    constexpr int NST = KG == 1 ? 4 : 2;   // ring depth
    constexpr int TKG = 64;                // keys per step of a key group
    constexpr int NKB = TKG / 32;          // 32-key blocks of it
    constexpr int TK = KG * TKG;           // keys per step
    constexpr int RG = NW / KG;            // row groups
    constexpr int IXP = TK / 64;           // index loads per step and list
    constexpr int NIX = 4;                 // index ring depth
    constexpr int IXA = KG == 1 ? NST : 2; // steps the indices are issued ahead of
    constexpr int KS = D / 16;             // k-steps of the QK^T contraction
    constexpr int DB = D / 32;             // 32-wide d blocks of O^T
    constexpr int ROWB = 2 * D;            // tile row bytes
    constexpr int CH = D / 8;              // 16-byte chunks per row
    constexpr int RPI = 64 / CH;           // rows per wave-wide load
    constexpr int NL = TK / RPI;           // wave-wide loads per step and tensor
    constexpr int PPW = (NL + NW - 1) / NW;   // K/V load pairs of the busiest wave
    constexpr int NWAIT = 2 * PPW;         // its fills per step
    constexpr int NWAIT_TAIL = 2 * (NL / NW);  // fills per step of the least busy wave
    __shared__ __attribute__((aligned(1024))) uint16_t Kt[NST][TK * D];
    __shared__ __attribute__((aligned(1024))) uint16_t Vt[NST][TK * D];
    __shared__ __attribute__((aligned(256))) int32_t Ix[NIX][2][IXP * 64];   // [U or rank, src]

    __shared__ int s_pick;

    const int Hkv = a.Hkv;
    const int nR_dev = a.counts[1 + a.layer];
    const int nR = min(nR_dev, a.cap);
    if (nR_dev > a.cap && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(a.err, RELAXKV_ERR_ROWS);
    constexpr int TR = RG * 32;            // (target, head) rows per tile
    const int nrows = nR * a.G;            // rows of one KV head (< 2^31: T_c <= 2^22, G <= kAttnRows)
    const int ntiles = (nrows + TR - 1) / TR;
    const int off = a.R_off[a.layer];
    const int idx_max = max((FULL ? a.T : a.counts[0]) - 1, 0);   // last entry of the context list
    // Tile choice, KG = 1.  Each KV head's tiles are handed out heaviest first from its
    // counter; a workgroup starts with a head tied to its XCD (so the
    // workgroups of one XCD share that head's K/V in their L2) and moves on to
    // the next head once that one is exhausted.  The XCDs run at different
    // clocks, so a fixed blockIdx -> tile map would make every launch wait for
    // the slowest; the grid carries spare workgroups for the faster ones.  The
    // last workgroup to finish returns the counters to zero for the next launch
    // of this layer and mode (it is counted after its pick was handed out, which
    // the pick's returned value proves, so every other pick happened before).
    // KG = 2: workgroup i takes head i mod Hkv, heaviest tiles first (also one head
    // per XCD at 8 heads); such a launch is one to three rounds of workgroups, so
    // the spread of the XCDs' clocks costs less than the counters' round trips.
    int pick = blockIdx.x;
    if constexpr (KG == 1) {
        if (threadIdx.x == 0) {
            const int xcc = (int)__builtin_amdgcn_s_getreg(kHwRegXccId | ((4 - 1) << 11));
            int h = (xcc + kXcds * (int)((blockIdx.x / kXcds) % ((Hkv + kXcds - 1) / kXcds))) % Hkv;
            int got = -1;
            for (int tried = 0; tried < Hkv; ++tried) {
                const int t = (int)atomicAdd(a.tiles + h, 1u);
                if (t < ntiles) {
                    got = t * Hkv + h;
                    break;
                }
                h = h + 1 == Hkv ? 0 : h + 1;
            }
            s_pick = got;
        }
        __syncthreads();
        pick = s_pick;
    } else if (pick >= ntiles * Hkv) {
        return;
    }
    // Counts this workgroup as done with the counters (KG = 1); the last one clears them.
    auto leave = [&] {
        if (KG == 1 && threadIdx.x == 0) {
            __threadfence();
            if (atomicAdd(a.tiles + Hkv, 1u) == gridDim.x - 1) {
                __threadfence();                   // every other pick happens before the resets
                for (int i = 0; i < Hkv; ++i) atomicExch(a.tiles + i, 0u);
                atomicExch(a.tiles + Hkv, 0u);
            }
        }
    };
    if (pick < 0) {
        leave();
        return;
    }
    const int g = pick % Hkv;
    const int tile = ntiles - 1 - pick / Hkv;        // heaviest tiles first
    const int r0 = tile * TR;                        // the tile's rows [r0, r1)
    const int r1 = min(r0 + TR, nrows);
    const int t0 = r0 / a.G, t1 = (r1 - 1) / a.G + 1;  // the targets they belong to
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, hf = lane >> 5;
    // The indices of step m.  KG = 2 clamps them to the list, which is known before
    // the tile's limits, so that the first ones travel with the limits and the queries
    // (the fills then clamp to cmax).
    const int32_t* srcmap = FULL ? a.rank_l : a.src_l;
    int idx_last = idx_max;
    auto issue_idx = [&](int m) {
        if (w < (FULL ? 1 : 2) * IXP) {
            int ww = w / IXP;
            asm volatile("" : "+s"(ww));
            const int part = IXP == 1 ? 0 : w % IXP * 64;
            const int c = min(m * TK + part + lane, idx_last);
            const int32_t* src = FULL ? srcmap + c : (ww == 0 ? a.U + c : srcmap + c);
            fill_lds4(src, lds_addr(&Ix[m & (NIX - 1)][ww][part]));
        }
    };
    if constexpr (KG > 1) {
#pragma unroll
        for (int m = 0; m < IXA; ++m) issue_idx(m);
    }
    const int32_t* lim_of = FULL ? a.R_idx + off : a.R_u + off;
    const int cmin = lim_of[t0];
    const int cmax = max(lim_of[t1 - 1], 0);
    if (KG == 1) idx_last = cmax;

    const float sl2 = a.scale * kLog2e;
    const int rg = KG == 1 ? w : w % RG, kg = KG == 1 ? 0 : w / RG;

    const int row = r0 + rg * 32 + r32;
    const bool valid = row < r1;
    const int t_row = valid ? row / a.G : t0;
    const int hh = valid ? row - t_row * a.G : 0;
    const int lim_v = lim_of[t_row];                 // value select: no pointer to cmax
    const int lim = valid ? lim_v : cmax;
    // The largest limit among the wave's rows (limits ascend with the row), -1
    // for a wave without rows: steps past it are masked for every row of the wave.
    const int w_first = r0 + rg * 32, w_last = min(w_first + 31, r1 - 1);
    const int wlim = __builtin_amdgcn_readfirstlane(w_last < w_first ? -1 : lim_of[w_last / a.G]);
    const int head = g * a.G + hh;
    bf16x8 qf[KS];
    {
        const uint16_t* qrow = (const uint16_t*)a.q_new + ((size_t)t_row * a.H + head) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(qrow + ks * 16 + hf * 8);
    }
    // Consumed before the loop, so the compiler's waits for these loads stay
    // there: inside it they would also wait for the K/V fills just issued.
    auto use_q = [&] {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qf[ks]));
    };
    if (KG == 1) use_q();
    f32x16 o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = f32x16{};
    float m_run = KG == 1 && lim < 0 ? 0.f : -INFINITY;   // empty context: every p is exp2(-inf) = 0
    float l_run = 0.f;

    // Row bases of the fresh rows (stride Hkv*D) and of the cached layer (stride D).
    const uint16_t* kng = (const uint16_t*)a.k_new + (size_t)g * D;
    const uint16_t* vng = (const uint16_t*)a.v_new + (size_t)g * D;
    const uint16_t* kcg = (const uint16_t*)a.kc + g * a.kv_sh;
    const uint16_t* vcg = (const uint16_t*)a.vc + g * a.kv_sh;
    const uint32_t kst = (uint32_t)a.kv_st;              // < 2^24 (checked on the host)
    const int S = cmax / TK + 1;                     // steps

    // The lane's tile row and swizzled chunk offset (elements) in each of its
    // fills: loop invariant.
    int f_row[PPW];
    uint32_t f_choff[PPW];
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
        f_row[i] = (w + i * NW) * RPI + lane / CH;
        f_choff[i] = (uint32_t)(((lane % CH) ^ tile_swz<D>(f_row[i])) << 3);
    }
    auto issue_rows = [&](int m) {
        const int st = m & (NST - 1), ix = m & (NIX - 1);
#pragma unroll
        for (int i = 0; i < PPW; ++i) {
            const int j = w + i * NW;
            if (NL % NW == 0 || j < NL) {
                int row = f_row[i];
                uint32_t choff = f_choff[i];
                asm volatile("" : "+v"(row), "+v"(choff));
                if (KG > 1) row = min(row, cmax - m * TK);
                const int c = m * TK + row;
                int pos = FULL ? min(c, cmax) : Ix[ix][0][row];
                int r = Ix[ix][FULL ? 0 : 1][row];
                asm volatile("" : "+v"(pos), "+v"(r));      // both read, then selected
                // (the empty asm statements keep the compiler from turning the
                // fresh/cached choice into a divergent branch)
                const bool fresh = r >= 0;
                // element offset of the row's chunk (< 2^31: (T_c - 1) * kst + D and
                // |R_l| * Hkv * D, both checked on the host, so 24-bit multiplies do)
                const uint32_t off = (fresh ? __umul24((uint32_t)r, (uint32_t)(Hkv * D))
                                            : __umul24((uint32_t)pos, kst)) + choff;
                const uint64_t kb = fresh ? (uint64_t)kng : (uint64_t)kcg;
                const uint64_t vb = fresh ? (uint64_t)vng : (uint64_t)vcg;
                const uint16_t* kp = (const uint16_t*)kb + off;
                const uint16_t* vp = (const uint16_t*)vb + off;
                fill_lds16(kp, lds_addr(Kt[st] + j * RPI * D));
                fill_lds16(vp, lds_addr(Vt[st] + j * RPI * D));
            }
        }
    };

    const int k_base = r32 * ROWB | ((hf ^ tile_swz<D>(r32)) << 4);
    const int rl = 4 * (lane >> 5) + ((lane & 15) >> 2);
    const int cl = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
    const int v_base0 = rl * ROWB | ((cl ^ tile_swz<D>(rl)) << 4) | ((lane & 1) << 3);
    const int v_base1 = (rl + 8) * ROWB | ((cl ^ tile_swz<D>(rl + 8)) << 4) | ((lane & 1) << 3);

    if constexpr (KG == 1) {
#pragma unroll
        for (int m = 0; m < IXA; ++m)
            if (m < S) issue_idx(m);
    }
    wait_loads_barrier<0>();
    if (KG > 1) use_q();
#pragma unroll
    for (int m = 0; m < NST - 1; ++m)
        if (m < S) issue_rows(m);

    for (int j = 0; j < S; ++j) {
        // The fills of step j and the indices of step j+3 are complete (only the
        // fills of step j+2 may be in flight), and every wave is done with step
        // j-1, whose buffers the fills of step j+3 reuse.  Loads complete in
        // order, so a wave's fills of step j are done once at most as many of
        // its loads are outstanding as it issued after them: the fills of steps
        // j+1 and j+2 (at least NWAIT loads while both steps exist), only those
        // of step j+1 near the end (at least NWAIT_TAIL), none in the last step.
        // (2-deep ring: nothing was issued after the fills of step j.)
        if (NST == 4 && j + 2 < S) wait_loads_barrier<NWAIT>();
        else if (NST == 4 && j + 1 < S) wait_loads_barrier<NWAIT_TAIL>();
        else wait_loads_barrier<0>();
        if (j + IXA < S) issue_idx(j + IXA);
        if (j + NST - 1 < S) issue_rows(j + NST - 1);
        // A step whose keys all lie past every limit of the wave's rows adds
        // exact zeros to them (p = 0): the wave only keeps the ring moving.
        const int c0 = j * TK + kg * TKG;              // the wave's first key of this step
        if (c0 > wlim) continue;
        // S^T = K Q^T: s[kb][v] = S[row][key c0 + 32 kb + 8(v/4) + 4 hf + v%4]
        f32x16 s[NKB];
        {
            // (the stage and key-group offsets leave the swizzled bits alone)
            int kbo = k_base + (j & (NST - 1)) * (TK * D * 2) + (KG == 1 ? 0 : kg * TKG * ROWB);
            asm volatile("" : "+v"(kbo));
            const char* kst = (const char*)Kt[0];
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) s[kb] = f32x16{};
            // K fragments x = NKB ks + kb, read KA ahead of their MFMA.
            constexpr int KA = RELAXKV_ATTN_KAHEAD < NKB * KS ? RELAXKV_ATTN_KAHEAD : NKB * KS;
            auto frag = [&](int x) {
                return *(const bf16x8*)(kst + (x % NKB) * 32 * ROWB + (kbo ^ ((x / NKB) << 5)));
            };
            bf16x8 kf[KA];
#pragma unroll
            for (int x = 0; x < KA; ++x) kf[x] = frag(x);
#if RELAXKV_ATTN_SETPRIO
            __builtin_amdgcn_s_setprio(2);
#endif
#pragma unroll
            for (int x = 0; x < NKB * KS; ++x) {
                const bf16x8 cur = kf[x % KA];
                if (x + KA < NKB * KS) kf[x % KA] = frag(x + KA);
                s[x % NKB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cur, qf[x / NKB], s[x % NKB], 0, 0, 0);
            }
#if RELAXKV_ATTN_SCHED
            __builtin_amdgcn_sched_group_barrier(0x100, KA, 0);
#pragma unroll
            for (int x = 0; x < NKB * KS; ++x) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (x + KA < NKB * KS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#endif
#if RELAXKV_ATTN_SETPRIO
            __builtin_amdgcn_s_setprio(0);
#endif
        }
        if (c0 + TKG - 1 > cmin) {                     // staircase step: mask
            const int ex = lim - c0 - 4 * hf;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    if (32 * kb + 8 * (v >> 2) + (v & 3) > ex) s[kb][v] = -INFINITY;
            }
        }
#if RELAXKV_ATTN_LEAN
        // Two chains of 3-input maxima (two new values per instruction).
        float m0 = fmaxf(s[0][0], s[0][1]), m1 = fmaxf(s[NKB - 1][0], s[NKB - 1][1]);
#pragma unroll
        for (int v = 2; v < 16; v += 2) {
            m0 = fmaxf(fmaxf(m0, s[0][v]), s[0][v + 1]);
            if (NKB == 2) m1 = fmaxf(fmaxf(m1, s[NKB - 1][v]), s[NKB - 1][v + 1]);
        }
        const float mx = pair_max(fmaxf(m0, m1)) * sl2;
#else
        float m = fmaxf(s[0][0], s[NKB - 1][0]);
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, fmaxf(s[0][v], s[NKB - 1][v]));
        const float mx = pair_max(m) * sl2;
#endif
        const bool need = mx > m_run + kRescaleSlack;
        if (__any(need)) {
            const float m_new = need ? mx : m_run;
            // (a key group's row may still be at -inf: -inf - -inf is no number)
            const float alpha = KG > 1 && !need ? 1.f : fast_exp2(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
            m_run = m_new;
        }
        // (a key group can meet steps whose keys are all masked for a row before the
        // row's first visible key: its reference is then 0, so they add exact zeros)
        const float m_ref = KG > 1 && m_run == -INFINITY ? 0.f : m_run;
        bf16x8 pb[NKB][2];
#if RELAXKV_ATTN_LEAN
        // The row sum adds the bf16 probabilities that the PV product uses, two
        // per dot2 instruction, in four chains.
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                pb[kb][v >> 3][v & 7] = (__bf16)fast_exp2(fmaf(s[kb][v], sl2, -m_ref));
        {
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            const bf16x2 one2 = {(__bf16)1.0f, (__bf16)1.0f};
            float ls0 = 0.f, ls1 = 0.f, ls2 = 0.f, ls3 = 0.f;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) {
                    const bf16x8 q8 = pb[kb][k2];
                    ls0 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(q8, q8, 0, 1), one2, ls0, false);
                    ls1 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(q8, q8, 2, 3), one2, ls1, false);
                    ls2 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(q8, q8, 4, 5), one2, ls2, false);
                    ls3 = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(q8, q8, 6, 7), one2, ls3, false);
                }
            l_run += (ls0 + ls1) + (ls2 + ls3);
        }
#else
        float ls = 0.f;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float p = fast_exp2(fmaf(s[kb][v], sl2, -m_ref));
                ls += p;
                pb[kb][v >> 3][v & 7] = (__bf16)p;
            }
        l_run += ls;
#endif
        // O^T += V^T P^T
        {
            // LDS byte addresses of the lane's two V rows in this step's tile: the
            // tile base and stage only set bits above the swizzled chunk bits.
            const uint32_t vstage = lds_addr(Vt[0]) + (uint32_t)(j & (NST - 1)) * (TK * D * 2) +
                                    (KG == 1 ? 0u : (uint32_t)(kg * TKG * ROWB));
            uint32_t vb0 = v_base0 + vstage, vb1 = v_base1 + vstage;
            asm volatile("" : "+v"(vb0), "+v"(vb1));
#if RELAXKV_ATTN_SETPRIO
            __builtin_amdgcn_s_setprio(2);
#endif
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int k2 = 0; k2 < 2; ++k2) {
                        const uint32_t rowo = (kb * 32 + k2 * 16) * ROWB;
                        const v4i16 a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_v4i16*)(uintptr_t)((vb0 ^ (db << 6)) + rowo));
                        const v4i16 a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_v4i16*)(uintptr_t)((vb1 ^ (db << 6)) + rowo));
                        const bf16x8 vv =
                            __builtin_bit_cast(bf16x8, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
                        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, pb[kb][k2], o[db], 0, 0, 0);
                    }
#if RELAXKV_ATTN_SETPRIO
            __builtin_amdgcn_s_setprio(0);
#endif
        }
    }

    float l_tot = pair_sum(l_run);
    const bool empty = lim < 0;
    // (t, head) row index: below T_c * H <= 2^32, and one register where a 64-bit
    // product held across the loop would take two
    const uint32_t orow = (uint32_t)t_row * (uint32_t)a.H + (uint32_t)head;
    // Blocks db0 .. db0 + NDB - 1 of the row, and with db0 = 0 its normaliser.
    auto store = [&](auto db0_t, auto ndb_t) {
        constexpr int DB0 = decltype(db0_t)::value, NDB = decltype(ndb_t)::value;
        if (!valid) return;
        const float inv = empty ? 0.f : 1.0f / l_tot;
        uint16_t* out = (uint16_t*)a.out + (size_t)orow * D;
#pragma unroll
        for (int db = DB0; db < DB0 + NDB; ++db) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int d0 = db * 32 + 8 * jj + 4 * hf;
                const uint32_t lo = (uint32_t)f32_to_bf16_bits(o[db][4 * jj] * inv) |
                                    ((uint32_t)f32_to_bf16_bits(o[db][4 * jj + 1] * inv) << 16);
                const uint32_t hi = (uint32_t)f32_to_bf16_bits(o[db][4 * jj + 2] * inv) |
                                    ((uint32_t)f32_to_bf16_bits(o[db][4 * jj + 3] * inv) << 16);
                *(u32x2*)(out + d0) = u32x2{lo, hi};
            }
        }
        if (DB0 == 0 && a.lse && hf == 0)
            a.lse[orow] = empty ? -INFINITY : (m_run + __log2f(l_tot)) * kLn2;
    };
    if constexpr (KG == 1) {
        leave();
        store(Int<0>{}, Int<DB>{});
    } else {
        // The two key groups of a row group exchange halves of O (and m, l) through the
        // ring's LDS (free: the last fills were waited for and read); each combines and
        // stores one half of the row.
        constexpr int HB = DB / 2, OW = HB * 16 * 64;      // blocks and floats of a half
        static_assert(2 * RG * OW * 4 <= (int)sizeof(Kt) && RG * 1024 <= (int)sizeof(Vt), "exchange");
        float* mine = (float*)&Kt[0][0] + (kg * RG + rg) * OW + lane;
        const float* other = (const float*)&Kt[0][0] + ((1 - kg) * RG + rg) * OW + lane;
        float* ml = (float*)&Vt[0][0] + rg * 256 + lane;
        auto give = [&](auto db0_t) {
            constexpr int DB0 = decltype(db0_t)::value;
#pragma unroll
            for (int db = 0; db < HB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) mine[(db * 16 + v) * 64] = o[DB0 + db][v];
            ml[kg * 128] = m_run;
            ml[kg * 128 + 64] = l_tot;
        };
        auto take = [&](auto db0_t) {
            constexpr int DB0 = decltype(db0_t)::value;
            const float m1 = ml[(1 - kg) * 128], l1 = ml[(1 - kg) * 128 + 64];
            const float m = fmaxf(m_run, m1);
            const float w0 = m_run == -INFINITY ? 0.f : fast_exp2(m_run - m);
            const float w1 = m1 == -INFINITY ? 0.f : fast_exp2(m1 - m);
#pragma unroll
            for (int db = 0; db < HB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    o[DB0 + db][v] = o[DB0 + db][v] * w0 + other[(db * 16 + v) * 64] * w1;
            l_tot = l_tot * w0 + l1 * w1;
            m_run = m;
            store(db0_t, Int<HB>{});
        };
        __syncthreads();
        if (kg == 0) give(Int<HB>{});
        else give(Int<0>{});
        __syncthreads();
        if (kg == 0) take(Int<0>{});
        else take(Int<HB>{});
    }
}


// ----------------------------------------------------------------- fp32 MFMA

// One workgroup per R (target, head) rows of a KV head (row t*G + hh), the last
// targets' tiles (the longest contexts) first.
template <int D, bool FULL, int R>
__global__ __launch_bounds__(MfmaF32<R>::waves * 64) void attn_f32(AttnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char f32_lds[];
    const int nR_dev = a.counts[1 + a.layer];
    const int nR = min(nR_dev, a.cap);
    if (nR_dev > a.cap && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        atomicOr(a.err, RELAXKV_ERR_ROWS);
    const long nrows = (long)nR * a.G;
    const long tile = (nrows + R - 1) / R - 1 - ((long)blockIdx.z * gridDim.x + blockIdx.x);
    if (tile < 0) return;
    const int g = blockIdx.y;
    const long row = tile * R + threadIdx.x % R;
    const bool valid = row < nrows;
    const int off = a.R_off[a.layer];
    const int32_t* lim_of = FULL ? a.R_idx + off : a.R_u + off;
    const long last = min(tile * R + R - 1, nrows - 1);
    const int t = (int)((valid ? row : last) / a.G);
    const int head = g * a.G + (int)((valid ? row : last) - (long)t * a.G);
    const int n_keys = max(lim_of[last / a.G], 0) + 1;   // limits ascend with the row
    const uint32_t orow = (uint32_t)t * (uint32_t)a.H + (uint32_t)head;   // below T_c * H <= 2^32
    auto id_of = [&](int c) {
        const int r = FULL ? a.rank_l[c] : a.src_l[c];
        return r >= 0 ? r : ~(FULL ? c : a.U[c]);
    };
    attn_f32_rows<D, R>(
        *(AttnF32Lds<D, R>*)f32_lds, (const float*)a.k_new + g * D, (const float*)a.v_new + g * D,
        (int64_t)a.Hkv * D, (const float*)a.kc + g * a.kv_sh, (const float*)a.vc + g * a.kv_sh, a.kv_st,
        id_of, n_keys, (const float*)a.q_new + (size_t)orow * D, lim_of[t], a.scale, valid,
        (float*)a.out, a.lse, orow);
}

constexpr int kNW = RELAXKV_ATTN_WAVES;
static_assert(kAttnRows == kNW * 32, "rows per workgroup");
constexpr int kNW2 = 8;                    // waves of the two-key-group kernel
constexpr int kAttnRows2 = kNW2 / 2 * 32;  // its rows per workgroup

// Key groups of a launch of `rows` (target, head) rows per KV head, by its count of
// 384-row tiles: two up to 5/4 of the chip's 256 CUs at d 128, up to 432 tiles at
// d 64 (whose smaller workgroups fit a CU twice) and there again from 600 to 768
// tiles; one otherwise.  While every tile has a CU to itself the launch lasts as long
// as the longest tile's steps, so a third of the rows and half of the steps per
// workgroup is shorter; past it the extra fills per row count, and at d 64 from 433
// to 600 tiles two rounds of the larger workgroups fit the chip about as well.
// Measured in us, one against two key groups, 8 KV heads: d 128: 24 tiles (1.5K
// context) 28.4 / 17.8, 104 (8K) 163 / 82, 264 (8K) 173 / 152, 264 (16K) 341 / 289, 312
// (8K) 181 / 174, 328 (9K) 199 / 200, 352 (8K) 186 / 199, 552 (16K) 493 / 576; d 64: 104
// (8K) 118 / 59, 264 (8K) 128 / 92, 592 (12K) 260 / 255, 624 (14K) 315 / 307, 752 (16K)
// 419 / 407, 1400 (32K) 1420 / 1466.  d 64 at other KV-head counts: 364 (2 heads, 10K)
// 156 / 136, 400 (1, 16K) 250 / 235, 416 (4, 16K) 250 / 241, 428 (4, 16K) 251 / 248, 440
// (2, 12K) 193 / 191 and over the full prefix 297 / 300, 452 (2, 16K) 258 / 263, 512 (2,
// 14K) 250 / 254, 539 (1, 24K) 428 / 449, 552 (2, 16K) 314 / 319, 598 (2, 16K) 343 / 339
// and 536 / 536, 668 (2, 24K) 558 / 548.
int attn_key_groups(long rows, int Hkv, int d) {
    constexpr long kCUs = 256;
    const long tiles = (rows + kAttnRows - 1) / kAttnRows * Hkv;
    if (d == 128) return tiles <= kCUs * 5 / 4 ? 2 : 1;
    return tiles <= 432 || (tiles >= 600 && tiles <= 768) ? 2 : 1;
}

template <int D, bool FULL>
void launch_one(const AttnArgs& a, bool bf16, int n_bound, hipStream_t st) {
    n_bound = n_bound > 0 ? n_bound : 1;                 // workgroup 0 still checks the count
    if (bf16) {
        const long rows = (long)n_bound * a.G;
        const int kg = attn_key_groups(rows, a.Hkv, D);
        const int tr = kg == 1 ? kAttnRows : kAttnRows2; // rows of a tile
        const int nwg = (int)((rows + tr - 1) / tr) * a.Hkv;
        // One workgroup per tile of the bound, plus an eighth spare where they take
        // their tiles from the counters (they exit once every one is exhausted).
        if (kg == 1)
            hipLaunchKernelGGL((attn_bf16<D, FULL, kNW, 1>), dim3(nwg + nwg / 8), dim3(kNW * 64), 0, st, a);
        else
            hipLaunchKernelGGL((attn_bf16<D, FULL, kNW2, 2>), dim3(nwg), dim3(kNW2 * 64), 0, st, a);
    } else {
        const long rows = (long)n_bound * a.G;
        auto go = [&](auto kernel, int r, int waves, size_t lds) {
            // A grid dimension times its threads stays below 2^32: 2^22 workgroups of at
            // most 512 threads in x (R = 32), the rest (up to 2^32 rows) in z.
            const long tiles = (rows + r - 1) / r, nx = tiles < (1L << 22) ? tiles : 1L << 22;
            hipLaunchKernelGGL(kernel, dim3((unsigned)nx, a.Hkv, (unsigned)((tiles + nx - 1) / nx)),
                               dim3(waves * 64), lds, st, a);
        };
        if (attn_f32_small(rows, a.Hkv))
            go(attn_f32<D, FULL, 16>, 16, MfmaF32<16>::waves, sizeof(AttnF32Lds<D, 16>));
        else
            go(attn_f32<D, FULL, 32>, 32, MfmaF32<32>::waves, sizeof(AttnF32Lds<D, 32>));
    }
}

}  // namespace

hipError_t launch_sparse_attn(const relaxkv_problem& p, const relaxkv_sets& s, int layer,
                              const void* q_new, const void* k_new, const void* v_new,
                              int n_rows, void* out, float* lse_out, int context_mode,
                              hipStream_t st) {
    const bool bf16 = p.dtype == RELAXKV_DTYPE_BF16;
    const size_t esz = bf16 ? 2 : 4;
    const KvStrides ks = kv_strides(p);
    AttnArgs a;
    a.q_new = q_new;
    a.k_new = k_new;
    a.v_new = v_new;
    a.kc = (const char*)p.k_cache + (size_t)(layer * ks.layer) * esz;
    a.vc = (const char*)p.v_cache + (size_t)(layer * ks.layer) * esz;
    a.kv_sh = ks.head;
    a.kv_st = ks.token;
    // The layer's context list: the union, or a construction variant's list.
    a.U = s.context_sets == RELAXKV_CONTEXT_SETS_GLOBAL      ? s.ctx
          : s.context_sets == RELAXKV_CONTEXT_SETS_LAYERWISE ? s.ctx + (size_t)layer * p.T_c
                                                             : s.U;
    a.cidx = s.cidx;
    a.src_l = s.src + (size_t)layer * p.T_c;
    a.rank_l = s.rank + (size_t)layer * p.T_c;
    a.R_off = s.R_off;
    a.R_idx = s.R_idx;
    a.R_u = s.R_u;
    a.counts = s.counts;
    a.err = s.counts + p.L + 1;
    a.tiles = s.tiles + ((size_t)(context_mode == RELAXKV_CONTEXT_FULL ? p.L : 0) + layer) *
                            (size_t)(p.H_kv + 1);
    a.out = out;
    a.lse = lse_out;
    a.H = p.H;
    a.Hkv = p.H_kv;
    a.G = p.H / p.H_kv;
    a.T = p.T_c;
    a.layer = layer;
    a.scale = p.softmax_scale > 0.f ? p.softmax_scale : 1.0f / sqrtf((float)p.d);
    // The grid covers the row cap; the device count (clamped to it) decides
    // which workgroups run.
    a.cap = row_cap(p, s, layer, n_rows);
    const int n_bound = a.cap;
    const bool full = context_mode == RELAXKV_CONTEXT_FULL;
    if (p.d == 128) {
        full ? launch_one<128, true>(a, bf16, n_bound, st) : launch_one<128, false>(a, bf16, n_bound, st);
    } else {
        full ? launch_one<64, true>(a, bf16, n_bound, st) : launch_one<64, false>(a, bf16, n_bound, st);
    }
    return hipGetLastError();
}

}  // namespace relaxkv

// Repair schedule and compact context (Sec. 3.2 set equations, App. A.1-A.2):
//   h_i = max{l : i in S_l},  U = union_l S_l (sorted),  R_l = {i in U : h_i >= l},
// the compact index of every union position, the per-layer source map
// (rank within R_l, or -1 for a cached row), the CSR lists of R_l and the
// edge counts sum_{p in R_l} |C_l(p)| and sum_{p in R_l} (p + 1).
//
// Two launches.  The positions are cut into blocks (256 to 16384 positions, at
// most 256 blocks).  sets_blocks, one workgroup per block, finds each layer's
// anchors inside its block by search (anchor rows ascend), takes the maximum
// layer per position in LDS and counts |R_l| within the block.  sets_emit, one
// wave per (block, layer), adds up the counts of the blocks and layers before it
// and writes its part of every list, ranking positions by ballots.  Every output
// is a count or a prefix count of integers, so all are deterministic.
//
// Why this split: the lists are a few MB and the work per entry is a handful of
// instructions, so the time is the length of the dependent chain.  One workgroup
// for U and one per layer for R_l (with h reset and marked by two launches more)
// walked the positions in 8192-entry turns: 54 us at 40 layers of 16384 positions
// and 96 us at 32768, against 16.6 and 19.2 us for these two.
//
// Matched-target variants (RelaxKV^G, Sec. 4.1 / App. A.3; the global target
// sweep of App. B): U comes from the anchors the same way, then every layer
// takes the same caller-given target list P.  The first launch leaves each
// position's count of union positions within its block, which gives every
// target its compact limit |U cap {j <= p}| - 1; targets need not lie in U.
//
// Context-construction variants (Sec. 4.4): the same anchors and targets R_l;
// the context list of a layer is replaced by a top-|U| list (of the layer-mean
// score, shared, or of the layer's score), written to ctx; the compact limits,
// source map and edge counts are recomputed against it.

#include "dev_common.h"
#include "internal.h"

namespace relaxkv {
namespace {

constexpr int kSetThreads = 1024;
constexpr int kEmitThreads = 256;              // one wave per layer
constexpr int kEmitWaves = kEmitThreads / 64;

// First index of the ascending list a[0..n) whose entry is >= v, searched by
// groups of 16 lanes (16 probes a round, so 3 rounds for 4913 entries); every
// lane of the wave calls, the lanes of a group with the same arguments.  For a
// list that does not ascend the result is some index in [0, n].
__device__ __forceinline__ int lower_bound16(const int32_t* __restrict__ a, int n, int v) {
    const int j = threadIdx.x & 15, shift = threadIdx.x & 48;
    int lo = 0, hi = n;
    while (__any(lo < hi)) {
        const bool open = lo < hi;
        const int m = hi - lo;
        const int p = lo + (j + 1) * m / 17;             // < hi for an open interval
        const bool less = open && a[open ? p : 0] < v;
        const int c = __popc((uint32_t)(__ballot(less) >> shift) & 0xffffu);
        if (open) {
            const int base = lo;
            if (c > 0) lo = base + c * m / 17 + 1;
            if (c < 16) hi = base + (c + 1) * m / 17;
        }
    }
    return lo;
}

// Past this many layers sets_blocks finds and marks the anchors of several layers at a
// time (MANY: their searches and loads together), and sums the positions by h (LDS
// atomics) and then over the layers, instead of once per layer.  One workgroup per
// block goes through all layers, so with many of them and few blocks these chains
// were longer than the four launches before (16.5 us at 128 layers of 64 positions, 54
// at 1024 of 1024).  Both launches in us, without / with it: 40 layers of 32768 positions
// 18.1 / 18.6, 80 of 16384 23.8 / 25.5, 96 of 4096 20.2 / 20.7, 128 of 1024 19.3 / 16.1,
// 256 of 16384 60 / 46, 1024 of 64 69 / 22, 1024 of 1024 107 / 48; a global list, which
// has no counts per layer: 80 of 65536 32.7 / 37.7, 128 of 16384 22.7 / 25.3, 256 of 1024
// 18.5 / 18.0, of 16384 36.8 / 35.5, 1024 of 64 34 / 22, of 1024 47.9 / 44.2.
constexpr int kFewLayers = 96, kFewLayersGlobal = 192;
static_assert(RELAXKV_MAX_LAYERS <= kSetThreads, "one layer per thread");

// lower_bound16 of N lists at once.
template <int N>
__device__ __forceinline__ void lower_bounds16(const int32_t* const (&a)[N], int n, const int (&v)[N],
                                               int (&lo)[N]) {
    const int j = threadIdx.x & 15, shift = threadIdx.x & 48;
    int hi[N];
    bool any_open = n > 0;
#pragma unroll
    for (int x = 0; x < N; ++x) {
        lo[x] = 0;
        hi[x] = n;
    }
    while (__any(any_open)) {
        int e[N];
#pragma unroll
        for (int x = 0; x < N; ++x)
            e[x] = lo[x] < hi[x] ? a[x][lo[x] + (j + 1) * (hi[x] - lo[x]) / 17] : 0;
        any_open = false;
#pragma unroll
        for (int x = 0; x < N; ++x) {
            const bool open = lo[x] < hi[x];
            const int m = hi[x] - lo[x], base = lo[x];
            const int c = __popc((uint32_t)(__ballot(open && e[x] < v[x]) >> shift) & 0xffffu);
            if (open) {
                if (c > 0) lo[x] = base + c * m / 17 + 1;
                if (c < 16) hi[x] = base + (c + 1) * m / 17;
            }
            any_open |= lo[x] < hi[x];
        }
    }
}

// The parts of the ascending anchor rows that lie in [v0, v1), four layers per group
// of 16 lanes at a time.
__device__ __forceinline__ void block_segments(const int32_t* __restrict__ anchors, int L, int k,
                                               int v0, int v1, int* seg_lo, int* seg_hi) {
    constexpr int NG = kSetThreads / 16, NL = 4;
    for (int l0 = threadIdx.x / 16; l0 < (L + NG - 1) / NG * NG; l0 += NL * NG) {
        const int32_t* rows[2 * NL];
        int v[2 * NL], at[2 * NL];
#pragma unroll
        for (int x = 0; x < NL; ++x) {
            rows[2 * x] = rows[2 * x + 1] = anchors + (size_t)min(l0 + x * NG, L - 1) * k;
            v[2 * x] = v0;
            v[2 * x + 1] = v1;
        }
        lower_bounds16<2 * NL>(rows, k, v, at);
#pragma unroll
        for (int x = 0; x < NL; ++x)
            if (l0 + x * NG < L && (threadIdx.x & 15) == 0) {
                seg_lo[l0 + x * NG] = at[2 * x];
                seg_hi[l0 + x * NG] = at[2 * x + 1];
            }
    }
}

// Per-block counts the first launch leaves for the second, in the scratch array of
// the sets buffer, which no caller is given (a caller may pass one of the sets' lists
// as the targets, or keep using them after the build).  Anchor targets: n, e, f
// of (layer, block) at [l * n_blk + b], with n = |R_l| in the block, e the sum of
// the targets' 1-based union ranks within the block and f that of their 1-based
// positions within it.  Global targets: last[i], the number of union positions of i's
// block up to i, minus one, and n, e, f of the block's targets.  e and f are kept
// only for more than one block; a single block writes its sums itself.
struct BlockScratch {
    int32_t* n;
    int32_t* e;
    int32_t* f;
    int16_t* last;
};
static_assert((long)kMaxSetBlock * (kMaxSetBlock + 1) / 2 <= INT32_MAX && kMaxSetBlock - 1 <= INT16_MAX,
              "a block's e and f fit 32 bits, its counts 16");

// One workgroup per block of positions: h of the block and the counts above (GT:
// of the targets P instead of R_l; h is written by the second launch).  Also
// zeroes the attention's work counters.
template <bool GT, bool MANY>
__global__ __launch_bounds__(kSetThreads) void sets_blocks(
    const int32_t* __restrict__ anchors, int L, int k, int T, int pb,
    const int32_t* __restrict__ P, const int32_t* __restrict__ n_P, int32_t* __restrict__ h,
    BlockScratch sc, uint32_t* __restrict__ tiles, int n_tiles) {
    extern __shared__ int hl[];                          // [pb]
    __shared__ int seg_lo[RELAXKV_MAX_LAYERS], seg_hi[RELAXKV_MAX_LAYERS];
    __shared__ int wave_n[kSetThreads / 64];
    __shared__ int sums[3], seg[2];
    const int b = blockIdx.x, n_blk = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int b0 = b * pb, len = min(pb, T - b0);
    for (int i = b * kSetThreads + tid; i < n_tiles; i += n_blk * kSetThreads) tiles[i] = 0u;
    for (int i = tid; i < pb; i += kSetThreads) hl[i] = -1;
    if (MANY && n_blk == 1) {
        for (int l = tid; l < L; l += kSetThreads) {
            seg_lo[l] = 0;
            seg_hi[l] = k;
        }
    } else if (MANY) {
        block_segments(anchors, L, k, b0, b0 + len, seg_lo, seg_hi);
    } else {
        for (int l0 = 0; l0 < L; l0 += kSetThreads / 16) {
            const int l = l0 + tid / 16;
            const int32_t* row = anchors + (size_t)min(l, L - 1) * k;
            const int lo = lower_bound16(row, k, b0), hi = lower_bound16(row, k, b0 + len);
            if (l < L && (tid & 15) == 0) {
                seg_lo[l] = lo;
                seg_hi[l] = hi;
            }
        }
    }
    if (GT && w == 0) {                                  // lanes 0-15: b0, the others: b0 + len
        const int x = lower_bound16(P, min(max(n_P[0], 0), T), lane < 16 ? b0 : b0 + len);
        if (lane == 0) seg[0] = x;
        if (lane == 16) seg[1] = x;
        if (lane < 3) sums[lane] = 0;
    }
    __syncthreads();
    if constexpr (MANY) {
        constexpr int NX = 4, NWV = kSetThreads / 64;    // NX layers of a wave in flight
        for (int l0 = w; l0 < L; l0 += NX * NWV) {
            int at[NX];
#pragma unroll
            for (int x = 0; x < NX; ++x) {               // (past the last layer it is marked again)
                const int l = min(l0 + x * NWV, L - 1), j = seg_lo[l] + lane;
                at[x] = j < seg_hi[l] ? anchors[(size_t)l * k + j] - b0 : -1;
            }
#pragma unroll
            for (int x = 0; x < NX; ++x) {
                const int l = min(l0 + x * NWV, L - 1);
                if (at[x] >= 0 && at[x] < len) atomicMax(&hl[at[x]], l);
                for (int j = seg_lo[l] + 64 + lane; j < seg_hi[l]; j += 64) {
                    const int i = anchors[(size_t)l * k + j] - b0;
                    if (i >= 0 && i < len) atomicMax(&hl[i], l);
                }
            }
        }
    } else {
        for (int l = w; l < L; l += kSetThreads / 64) {
            const int32_t* row = anchors + (size_t)l * k;
            for (int j = seg_lo[l] + lane; j < seg_hi[l]; j += 64) {
                const int i = row[j] - b0;
                if (i >= 0 && i < len) atomicMax(&hl[i], l);
            }
        }
    }
    __syncthreads();
    if constexpr (!GT) {
        for (int i = tid; i < len; i += kSetThreads) h[b0 + i] = hl[i];
        if constexpr (MANY) {
            __shared__ int by_f[RELAXKV_MAX_LAYERS];     // (the other sums in the segments' arrays)
            int *by_n = seg_lo, *by_e = seg_hi;
            for (int l = tid; l < L; l += kSetThreads) by_n[l] = by_e[l] = by_f[l] = 0;
            const int per = max(64, pb / (kSetThreads / 64)), s0 = w * per;   // positions of a wave
            int u = 0;
            if (s0 < pb)
                for (int c = s0; c < s0 + per; c += 64) u += __popcll(__ballot(hl[c + lane] >= 0));
            if (lane == 0) wave_n[w] = u;
            __syncthreads();
            u = 0;
            for (int ww = 0; ww < w; ++ww) u += wave_n[ww];
            if (s0 < pb)
                for (int c = s0; c < s0 + per; c += 64) {
                    const int hv = hl[c + lane];
                    const uint64_t mu = __ballot(hv >= 0);
                    if (hv >= 0) {
                        atomicAdd(&by_n[hv], 1);
                        if (n_blk > 1) {
                            atomicAdd(&by_e[hv], u + lanes_below(mu) + 1);
                            atomicAdd(&by_f[hv], c + lane + 1);
                        }
                    }
                    u += __popcll(mu);
                }
            __syncthreads();
            const int l = L - 1 - tid;
            int32_t* const to[3] = {sc.n, sc.e, sc.f};
            const int* const by[3] = {by_n, by_e, by_f};
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                if (x > 0 && n_blk == 1) break;
                int tot;
                const int v = l >= 0 ? by[x][l] : 0;
                const int sum = block_exclusive_scan<kSetThreads>(v, wave_n, tot) + v;
                if (l >= 0) to[x][(size_t)l * n_blk + b] = sum;
            }
            return;
        }
        for (int l = w; l < L; l += kSetThreads / 64) {
            int n = 0, u = 0, e = 0, f = 0;
            for (int c = 0; c < pb; c += 64) {
                const int hv = hl[c + lane];
                const uint64_t mu = __ballot(hv >= 0);
                if (hv >= l) {
                    e += u + lanes_below(mu) + 1;
                    f += c + lane + 1;
                    n += 1;
                }
                u += __popcll(mu);
            }
            n = wave_sum(n);
            if (n_blk > 1) {
                e = wave_sum(e);
                f = wave_sum(f);
            }
            if (lane == 0) {
                sc.n[(size_t)l * n_blk + b] = n;
                if (n_blk > 1) {
                    sc.e[(size_t)l * n_blk + b] = e;
                    sc.f[(size_t)l * n_blk + b] = f;
                }
            }
        }
    } else {
        const int per = max(64, pb / (kSetThreads / 64));    // positions of a wave
        const int s0 = w * per;
        int n = 0;
        if (s0 < pb)
            for (int c = s0; c < s0 + per; c += 64) n += __popcll(__ballot(hl[c + lane] >= 0));
        if (lane == 0) wave_n[w] = n;
        __syncthreads();
        int run = 0;
        for (int ww = 0; ww < w; ++ww) run += wave_n[ww];
        if (s0 < pb)
            for (int c = s0; c < s0 + per; c += 64) {
                const bool in = hl[c + lane] >= 0;
                const uint64_t m = __ballot(in);
                const int v = run + lanes_below(m) + in - 1;
                hl[c + lane] = v;                        // (this lane's own entry)
                if (c + lane < len) sc.last[b0 + c + lane] = (int16_t)v;
                run += __popcll(m);
            }
        if (n_blk == 1) return;
        __syncthreads();
        int tn = 0, te = 0, tf = 0;
        for (int t = seg[0] + tid; t < seg[1]; t += kSetThreads) {
            const int i = P[t] - b0;
            if (i >= 0 && i < len) {
                tn += 1;
                te += hl[i] + 1;
                tf += i + 1;
            }
        }
        tn = wave_sum(tn);
        te = wave_sum(te);
        tf = wave_sum(tf);
        if (lane == 0 && tn) {
            atomicAdd(&sums[0], tn);
            atomicAdd(&sums[1], te);
            atomicAdd(&sums[2], tf);
        }
        __syncthreads();
        if (tid == 0) {
            sc.n[b] = sums[0];
            sc.e[b] = sums[1];
            sc.f[b] = sums[2];
        }
    }
}

// The edge counts of a layer from its blocks' n, e, f and the union positions of
// each block (one wave; u_of(j) is block j's union count): (sum of union ranks,
// sum of positions), both 1-based, in every lane.
template <typename UnionOf>
__device__ __forceinline__ void block_edges(const int32_t* n, const int32_t* e, const int32_t* f,
                                            int n_blk, int pb, UnionOf u_of, long long& e_sum,
                                            long long& f_sum) {
    const int lane = threadIdx.x & 63;
    long long es = 0, fs = 0;
    int u0 = 0;                                          // union positions before this turn's blocks
    for (int j0 = 0; j0 < n_blk; j0 += 64) {
        const int j = j0 + lane;
        const int u = j < n_blk ? u_of(j) : 0;
        const int inc = wave_inclusive_scan(u);
        if (j < n_blk) {
            es += e[j] + (long long)(u0 + inc - u) * n[j];
            fs += f[j] + (long long)j * pb * n[j];
        }
        u0 += __shfl(inc, 63, 64);
    }
    e_sum = wave_sum(es);
    f_sum = wave_sum(fs);
}

// One wave per (block, layer): the block's part of U, cidx (layer 0's wave), R_l,
// its compact indices, the source map, the rank map and the edge counts; without
// LISTS only U, cidx, R_off and the counts.
template <bool LISTS>
__global__ __launch_bounds__(kEmitThreads) void sets_emit(
    const int32_t* __restrict__ h, int T, int L, int pb, BlockScratch sc,
    int32_t* __restrict__ U, int32_t* __restrict__ cidx, int32_t* __restrict__ R_off,
    int32_t* __restrict__ R_idx, int32_t* __restrict__ R_u, int32_t* __restrict__ src,
    int32_t* __restrict__ rank, int32_t* __restrict__ counts, int64_t* __restrict__ edges) {
    const int32_t* cnt = sc.n;
    __shared__ int red[kEmitWaves], tot_sh[kEmitWaves];
    const int b = blockIdx.x, n_blk = gridDim.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int l0 = blockIdx.y * kEmitWaves, l = l0 + w;
    const int b0 = b * pb;
    // Entries of the layers before this workgroup's, of this layer (all blocks and
    // the blocks before this one), and union positions before this block.
    int before = 0;
    for (int i = tid; i < l0 * n_blk; i += kEmitThreads) before += cnt[i];
    int tot = 0, pre = 0, u_base = 0;
    for (int j = lane; j < n_blk; j += 64) {
        const int c = l < L ? cnt[(size_t)l * n_blk + j] : 0;
        tot += c;
        if (j < b) {
            pre += c;
            u_base += cnt[j];
        }
    }
    before = wave_sum(before);
    tot = wave_sum(tot);
    pre = wave_sum(pre);
    u_base = wave_sum(u_base);
    if (lane == 0) {
        red[w] = before;
        tot_sh[w] = tot;
    }
    __syncthreads();
    if (l >= L) return;
    int off = 0;
    for (int ww = 0; ww < kEmitWaves; ++ww) off += red[ww];
    for (int ww = 0; ww < w; ++ww) off += tot_sh[ww];
    if (b == 0 && lane == 0) {
        R_off[l] = off;
        counts[1 + l] = tot;
        if (l == 0) counts[0] = tot;                     // R_0 = U
        if (l == L - 1) R_off[L] = off + tot;
    }
    if (!LISTS && l > 0) return;
    int32_t* src_l = src + (size_t)l * T;
    int32_t* rank_l = rank + (size_t)l * T;
    int u = u_base, r = pre;
    long long e_sum = 0, ef_sum = 0;
    constexpr int NC = 4;                                // 64-position chunks loaded at once
    for (int c = 0; c < pb && b0 + c < T; c += NC * 64) {
        int hv[NC];
#pragma unroll
        for (int x = 0; x < NC; ++x) {
            const int i = b0 + c + x * 64 + lane;
            hv[x] = i < T ? h[i] : -1;
        }
#pragma unroll
        for (int x = 0; x < NC; ++x) {
            const int i = b0 + c + x * 64 + lane;
            const bool in = hv[x] >= 0, act = hv[x] >= l;    // (l >= 0, so act implies in)
            const uint64_t mu = __ballot(in), ma = __ballot(act);
            const int uc = u + lanes_below(mu), rc = r + lanes_below(ma);
            if (LISTS && i < T) rank_l[i] = act ? rc : -1;
            if (LISTS && in) src_l[uc] = act ? rc : -1;
            if (LISTS && act) {
                R_idx[off + rc] = i;
                R_u[off + rc] = uc;
                e_sum += uc + 1;                         // |C_l(p)| = compact index of p + 1
                ef_sum += i + 1;                         // full causal prefix
            }
            if (l == 0 && i < T) {
                cidx[i] = in ? uc : -1;
                if (in) U[uc] = i;
            }
            u += __popcll(mu);
            r += __popcll(ma);
        }
    }
    if (!LISTS || b > 0) return;
    if (n_blk > 1) {
        const size_t at = (size_t)l * n_blk;
        block_edges(cnt + at, sc.e + at, sc.f + at, n_blk, pb, [&](int j) { return cnt[j]; }, e_sum, ef_sum);
    } else {
        e_sum = wave_sum(e_sum);
        ef_sum = wave_sum(ef_sum);
    }
    if (lane == 0) {
        edges[l] = e_sum;
        edges[L + l] = ef_sum;
    }
}

// ------------------------------------------------------ global target lists

// One wave per (block, layer), every layer with the same targets R_l = P: the
// block's part of the rank and source maps (layer 0's wave: also U, cidx and h =
// L - 1 for targets), and the block's share of the target list: positions, compact
// limits and edge counts.  The first layer group's waves check the list.
__global__ __launch_bounds__(kEmitThreads) void sets_emit_global(
    BlockScratch sc, int T, int L, int pb, const int32_t* __restrict__ P,
    const int32_t* __restrict__ n_P, int32_t* __restrict__ h, int32_t* __restrict__ U,
    int32_t* __restrict__ cidx, int32_t* __restrict__ R_off, int32_t* __restrict__ R_idx,
    int32_t* __restrict__ R_u, int32_t* __restrict__ src, int32_t* __restrict__ rank,
    int32_t* __restrict__ counts, int64_t* __restrict__ edges) {
    extern __shared__ int trank[];                       // [pb] rank of each position in P
    const int16_t* last_loc = sc.last;
    __shared__ int u_base[kEmitThreads];                 // union positions before each block
    __shared__ int scan_scratch[kEmitWaves];
    __shared__ int seg[2];
    const int b = blockIdx.x, n_blk = gridDim.x;         // n_blk <= kEmitThreads
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int l = blockIdx.y * kEmitWaves + w;
    const int b0 = b * pb, len = min(pb, T - b0);
    const int n_raw = n_P[0];
    const int n = min(max(n_raw, 0), T);
    const int in_blk = tid < n_blk ? last_loc[min(T, (tid + 1) * pb) - 1] + 1 : 0;
    for (int i = tid; i < pb; i += kEmitThreads) trank[i] = -1;
    if (w == 0) {                                        // lanes 0-15: b0, the others: b0 + len
        const int x = lower_bound16(P, n, lane < 16 ? b0 : b0 + len);
        if (lane == 0) seg[0] = x;
        if (lane == 16) seg[1] = x;
    }
    int n_u;
    const int ub = block_exclusive_scan<kEmitThreads>(in_blk, scan_scratch, n_u);
    u_base[tid] = ub;
    __syncthreads();
    for (int t = seg[0] + tid; t < seg[1]; t += kEmitThreads) {
        const int i = P[t] - b0;
        if (i >= 0 && i < len) trank[i] = t;
    }
    // The block's share of the target list.
    const int share = (n + n_blk - 1) / n_blk;
    const int ta = min(n, b * share), tb = min(n, ta + share);
    if (blockIdx.y == 0) {                               // 0 <= |P| <= T, ascending within [0, T)
        bool bad = n_raw < 0 || n_raw > T;
        for (int t = ta + tid; t < tb; t += kEmitThreads) {
            const int p = P[t];
            bad |= p < 0 || p >= T || (t > 0 && P[t - 1] >= p);
        }
        if (__any(bad) && lane == 0) atomicOr(&counts[L + 1], RELAXKV_ERR_BAD_TARGETS);
        if (b == 0 && tid == 0) counts[0] = n_u;
    }
    __syncthreads();
    if (l >= L) return;
    if (b == 0 && lane == 0) {
        R_off[l] = l * n;
        counts[1 + l] = n;
        if (l == L - 1) R_off[L] = L * n;
    }
    long long e_sum = 0, ef_sum = 0;
    for (int t = ta + lane; t < tb; t += 64) {
        const int p = min(max(P[t], 0), T - 1);          // in range even for a rejected list
        const int ul = u_base[p / pb] + last_loc[p];     // |U cap {j <= p}| - 1
        R_idx[l * n + t] = p;
        R_u[l * n + t] = ul;
        e_sum += ul + 1;
        ef_sum += p + 1;
    }
    if (b == 0) {
        if (n_blk > 1) {
            block_edges(sc.n, sc.e, sc.f, n_blk, pb,
                        [&](int j) { return last_loc[min(T, (j + 1) * pb) - 1] + 1; }, e_sum, ef_sum);
        } else {
            e_sum = wave_sum(e_sum);
            ef_sum = wave_sum(ef_sum);
        }
        if (lane == 0) {
            edges[l] = e_sum;
            edges[L + l] = ef_sum;
        }
    }
    int32_t* src_l = src + (size_t)l * T;
    int32_t* rank_l = rank + (size_t)l * T;
    int carry = -1;                                      // last_loc before this chunk
    for (int c = 0; c < len; c += 64) {
        const int i = c + lane;
        const int ll = i < len ? last_loc[b0 + i] : 0;
        int prev = __shfl_up(ll, 1, 64);
        if (lane == 0) prev = carry;
        carry = __shfl(ll, 63, 64);                      // (only read again after a full chunk)
        if (i >= len) continue;
        const bool in = ll != prev;                      // a union position raises the count
        const int t = trank[i], uc = u_base[b] + ll;
        rank_l[b0 + i] = t;
        if (in) src_l[uc] = t;
        if (l == 0) {
            cidx[b0 + i] = in ? uc : -1;
            if (in) U[uc] = b0 + i;
            h[b0 + i] = t >= 0 ? L - 1 : -1;
        }
    }
}

// A copy of the target list and its length.
__global__ void sets_copy_list(const int32_t* P, const int32_t* n_P, int T, int32_t* to, int32_t* n_to) {
    const int n = n_P[0], i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < min(max(n, 0), T)) to[i] = P[i];
    if (i == 0) n_to[0] = n;
}

// ------------------------------------------------ context-construction variants

// One workgroup per layer: compact limits of RelaxKV's targets R_l within the
// layer's context list U_l (upper bound by binary search: both are ascending),
// the source map over U_l and the edge counts.
__global__ __launch_bounds__(kSetThreads) void ctx_layers(
    const int32_t* __restrict__ ctx, int ctx_stride, int T, const int32_t* __restrict__ R_off,
    const int32_t* __restrict__ R_idx, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ rank, int32_t* __restrict__ R_u, int32_t* __restrict__ src,
    int64_t* __restrict__ edges) {
    __shared__ long long red[kSetThreads / 64];
    const int l = blockIdx.x, tid = threadIdx.x;
    const int32_t* ctx_l = ctx + (size_t)l * ctx_stride;
    const int n = counts[0];                           // every context list has |U| entries
    const int off = R_off[l], nR = counts[1 + l];
    const int32_t* rank_l = rank + (size_t)l * T;
    int32_t* src_l = src + (size_t)l * T;
    long long e_sum = 0;
    for (int t = tid; t < nR; t += kSetThreads) {
        const int p = R_idx[off + t];
        int lo = 0, hi = n;                            // first entry > p
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (ctx_l[mid] <= p) lo = mid + 1;
            else hi = mid;
        }
        R_u[off + t] = lo - 1;
        e_sum += lo;                                   // |U_l cap {j <= p}|
    }
    for (int c = tid; c < n; c += kSetThreads) src_l[c] = rank_l[ctx_l[c]];
    e_sum = wave_sum(e_sum);
    if ((tid & 63) == 0) red[tid >> 6] = e_sum;
    __syncthreads();
    if (tid == 0) {
        long long a = 0;
        for (int i = 0; i < kSetThreads / 64; ++i) a += red[i];
        edges[l] = a;
    }
}

// The same with the context list as a bitmap in LDS and a prefix count per
// 32-position word, so a target's compact limit is two LDS reads instead of a
// chain of log2 |U| dependent loads.
__global__ __launch_bounds__(kSetThreads) void ctx_layers_bits(
    const int32_t* __restrict__ ctx, int ctx_stride, int T, const int32_t* __restrict__ R_off,
    const int32_t* __restrict__ R_idx, const int32_t* __restrict__ counts,
    const int32_t* __restrict__ rank, int32_t* __restrict__ R_u, int32_t* __restrict__ src,
    int64_t* __restrict__ edges) {
    extern __shared__ uint32_t bits[];                   // [words] membership, [words] prefix counts
    __shared__ int scan_scratch[kSetThreads / 64];
    __shared__ long long red[kSetThreads / 64];
    const int l = blockIdx.x, tid = threadIdx.x;
    const int words = (T + 31) / 32;
    uint32_t* pre = bits + words;
    const int32_t* ctx_l = ctx + (size_t)l * ctx_stride;
    const int n = counts[0];                             // every context list has |U| entries
    const int off = R_off[l], nR = counts[1 + l];
    const int32_t* rank_l = rank + (size_t)l * T;
    int32_t* src_l = src + (size_t)l * T;
    for (int i = tid; i < words; i += kSetThreads) bits[i] = 0u;
    __syncthreads();
#pragma unroll 4
    for (int c = tid; c < n; c += kSetThreads) {
        const int p = ctx_l[c];
        atomicOr(&bits[p >> 5], 1u << (p & 31));
        src_l[c] = rank_l[p];
    }
    __syncthreads();
    const int per = (words + kSetThreads - 1) / kSetThreads;
    const int w0 = min(words, tid * per), w1 = min(words, w0 + per);
    int sum = 0;
    for (int i = w0; i < w1; ++i) sum += __popc(bits[i]);
    int tot;
    int run = block_exclusive_scan<kSetThreads>(sum, scan_scratch, tot);
    for (int i = w0; i < w1; ++i) {
        pre[i] = (uint32_t)run;
        run += __popc(bits[i]);
    }
    __syncthreads();
    long long e_sum = 0;
#pragma unroll 4
    for (int t = tid; t < nR; t += kSetThreads) {
        const int p = R_idx[off + t];
        const int m = (int)pre[p >> 5] + __popc(bits[p >> 5] & (0xffffffffu >> (31 - (p & 31))));
        R_u[off + t] = m - 1;
        e_sum += m;                                      // |U_l cap {j <= p}|
    }
    e_sum = wave_sum(e_sum);
    if ((tid & 63) == 0) red[tid >> 6] = e_sum;
    __syncthreads();
    if (tid == 0) {
        long long a = 0;
        for (int i = 0; i < kSetThreads / 64; ++i) a += red[i];
        edges[l] = a;
    }
}

constexpr int kCtxBitsMaxT = 1 << 18;                    // 64 KB of LDS; longer contexts search

int set_blocks(const relaxkv_problem& p, int pb) { return (p.T_c + pb - 1) / pb; }

BlockScratch block_scratch(const relaxkv_problem& p, const relaxkv_sets& s, int n_blk, bool global) {
    const size_t words = sets_scratch_words(p.L, p.T_c), per = global ? n_blk : (size_t)p.L * n_blk;
    int32_t* base = (int32_t*)s.tiles - (words * 4 + 255) / 256 * 64;
    BlockScratch sc;
    sc.last = (int16_t*)base;                            // 2 T bytes, rounded up to whole words
    sc.n = base + (global ? ((size_t)p.T_c + 1) / 2 : 0);
    sc.e = sc.n + per;
    sc.f = sc.e + per;
    return sc;
}

template <bool GT>
void launch_blocks(const relaxkv_problem& p, const relaxkv_sets& s, int pb, const BlockScratch& sc,
                   const int32_t* P, const int32_t* n_P, hipStream_t st) {
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(set_blocks(p, pb)), dim3(kSetThreads), pb * sizeof(int), st,
                           s.anchors, p.L, s.k, p.T_c, pb, P, n_P, s.h, sc, s.tiles,
                           (int)attn_tile_words(p));
    };
    if (p.L > (GT ? kFewLayersGlobal : kFewLayers)) go(sets_blocks<GT, true>);
    else go(sets_blocks<GT, false>);
}

// The anchors' union and targets; without LISTS only U, cidx, R_off and the counts.
template <bool LISTS>
void launch_anchor_sets(const relaxkv_problem& p, const relaxkv_sets& s, hipStream_t st) {
    const int T = p.T_c, L = p.L, pb = set_block_positions(T), n_blk = set_blocks(p, pb);
    const BlockScratch sc = block_scratch(p, s, n_blk, false);
    launch_blocks<false>(p, s, pb, sc, nullptr, nullptr, st);
    hipLaunchKernelGGL(sets_emit<LISTS>, dim3(n_blk, (L + kEmitWaves - 1) / kEmitWaves),
                       dim3(kEmitThreads), 0, st, (const int32_t*)s.h, T, L, pb, sc, s.U, s.cidx,
                       s.R_off, s.R_idx, s.R_u, s.src, s.rank, s.counts, s.edges);
}

// Whether the n words at a overlap an array that a build of target lists writes.
bool in_outputs(const relaxkv_problem& p, const relaxkv_sets& s, const int32_t* a, size_t n) {
    const size_t L = p.L, T = p.T_c;
    const struct { const void* at; size_t words; } outs[] = {
        {s.h, T}, {s.U, T}, {s.cidx, T}, {s.R_off, L + 1}, {s.R_idx, L * T}, {s.R_u, L * T},
        {s.src, L * T}, {s.rank, L * T}, {s.counts, L + 2}, {s.edges, 4 * L}};
    const uintptr_t a0 = (uintptr_t)a;
    for (const auto& o : outs)
        if (a0 < (uintptr_t)o.at + 4 * o.words && (uintptr_t)o.at < a0 + 4 * n) return true;
    return false;
}

}  // namespace

hipError_t launch_build_sets_context(const relaxkv_problem& p, const float* scores,
                                     int construction, const relaxkv_sets& s, hipStream_t st) {
    const int T = p.T_c, L = p.L;
    hipError_t e = launch_build_sets(p, s, st);       // anchors -> h, U, R_l, rank (+ union maps)
    if (e != hipSuccess || construction == RELAXKV_CONTEXT_SETS_UNION) return e;
    // Top-|U| context lists, ascending (the k cap |U| is read on the device).
    if (construction == RELAXKV_CONTEXT_SETS_GLOBAL) {
        e = launch_global_mean(scores, L, T, s.g, st);
        if (e == hipSuccess) e = launch_select_rows(s.g, 1, T, T, s.counts, s.ctx, 0, s.counts, L, st);
    } else {
        e = launch_select_rows(scores, L, T, T, s.counts, s.ctx, T, s.counts, L, st);
    }
    if (e != hipSuccess) return e;
    const int stride = construction == RELAXKV_CONTEXT_SETS_GLOBAL ? 0 : T;
    if (T <= kCtxBitsMaxT)
        hipLaunchKernelGGL(ctx_layers_bits, dim3(L), dim3(kSetThreads), (size_t)(T + 31) / 32 * 8, st,
                           (const int32_t*)s.ctx, stride, T, s.R_off, s.R_idx, s.counts, s.rank,
                           s.R_u, s.src, s.edges);
    else
        hipLaunchKernelGGL(ctx_layers, dim3(L), dim3(kSetThreads), 0, st, (const int32_t*)s.ctx,
                           stride, T, s.R_off, s.R_idx, s.counts, s.rank, s.R_u, s.src, s.edges);
    return hipGetLastError();
}

hipError_t launch_build_sets_global(const relaxkv_problem& p, const relaxkv_sets& s,
                                    const int32_t* targets, const int32_t* n_targets,
                                    hipStream_t st) {
    const int T = p.T_c, L = p.L, pb = set_block_positions(T), n_blk = set_blocks(p, pb);
    const BlockScratch sc = block_scratch(p, s, n_blk, true);
    // A list (or its length) in an array that this build writes, for instance U with
    // counts[0], stands for what the array holds once the union is rebuilt from the
    // anchors: the union comes first, and the build then reads a copy of the list.
    if (in_outputs(p, s, targets, T) || in_outputs(p, s, n_targets, 1)) {
        launch_anchor_sets<false>(p, s, st);
        int32_t* copy = sc.f + n_blk;
        hipLaunchKernelGGL(sets_copy_list, dim3((T + 255) / 256), dim3(256), 0, st, targets, n_targets,
                           T, copy, copy + T);
        targets = copy;
        n_targets = copy + T;
    }
    launch_blocks<true>(p, s, pb, sc, targets, n_targets, st);
    hipLaunchKernelGGL(sets_emit_global, dim3(n_blk, (L + kEmitWaves - 1) / kEmitWaves),
                       dim3(kEmitThreads), pb * sizeof(int), st, sc, T, L, pb, targets, n_targets,
                       s.h, s.U, s.cidx, s.R_off, s.R_idx, s.R_u, s.src, s.rank, s.counts, s.edges);
    return hipGetLastError();
}

hipError_t launch_build_sets(const relaxkv_problem& p, const relaxkv_sets& s, hipStream_t st) {
    launch_anchor_sets<true>(p, s, st);
    return hipGetLastError();
}

}  // namespace relaxkv

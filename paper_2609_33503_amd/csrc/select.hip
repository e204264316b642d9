// Per-layer top-k anchor selection (Sec. 3.2 / App. A.1: S_l = TopK_i(a_{l,i}, k)),
// and the global target list of the target-capacity sweep (App. B equation:
// g_i = (1/L) sum_l a_{l,i}, P = TopK_i(g_i, min(floor(r_g T_c), |U|))), which
// runs the same selection on the single row g with the count capped on the
// device by |U|.
//
// One 1024-thread workgroup per selected row.  Scores are mapped to order-preserving
// unsigned keys (-0.0 folded onto +0.0), an MSB-first radix select finds the
// k-th largest key T and how many keys equal to T must be taken, and a stable
// compaction in position order writes the anchors: every key above T, plus the
// lowest-position keys equal to T.  Because the compaction walks positions in
// ascending order, each S_l comes out sorted.  Histograms use integer LDS
// atomics and every reduction is a scan, so the result is deterministic and
// unique.  Rows of up to 49152 entries stay in registers (select_topk_reg);
// longer rows are read again in each pass (select_topk).

#include "dev_common.h"
#include "internal.h"

namespace relaxkv {
namespace {

constexpr int kSelThreads = 1024;
constexpr int kSelPerThread = 8;   // contiguous elements per thread per compaction chunk

__device__ __forceinline__ uint32_t order_key(float f, int& nan_seen) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) nan_seen = 1;
    if (u == 0x80000000u) u = 0u;                       // -0.0 ties +0.0
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending key == ascending value
}

__global__ void clear_error_word(int32_t* counts, int L) {
    if (threadIdx.x == 0 && blockIdx.x == 0) counts[L + 1] = 0;
}

// Rows of up to E * 1024 entries: every key is read once and kept in registers.
// Wave w owns the n_e * 64 consecutive positions from w * n_e * 64 (n_e =
// ceil(T / 1024) <= E), lane by lane, so loads are coalesced and the compaction
// ranks come from ballots (position order is (wave, e, lane)).  Positions past T
// hold key 0, the smallest; they come after every real position, so with k <= T
// the tie rule never takes one.
// The bound is latency: one workgroup per row, so a chain of one load, three
// histogram passes and the compaction, each a few barriers long.  Digits of
// 11/11/10 bits give three passes instead of four.  MinMax-normalised scores
// share few exponents, so in the first pass most lanes of a wave want the same
// few bins and an LDS atomic takes a turn per lane: eight copies of the first
// histogram (copy = lane % 8) cut that to an eighth (later digits are mantissa
// bits, spread over the bins, one copy).
template <int E>
__global__ __launch_bounds__(kSelThreads) void select_topk_reg(
    const float* __restrict__ scores, int T, int k, const int32_t* __restrict__ k_cap,
    int32_t* __restrict__ out_base, int out_stride, int32_t* __restrict__ n_out,
    int32_t* __restrict__ counts, int L) {
    constexpr int NW = kSelThreads / 64;
    constexpr int BINS = 2048, COPIES = 8;
    __shared__ __attribute__((aligned(16))) int hist[BINS * COPIES];
    __shared__ int scan_scratch[NW];
    __shared__ int digit_sh, above_sh;
    __shared__ int w_gt[NW], w_eq[NW];
    const int l = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* a = scores + (size_t)l * T;
    if (k_cap) k = min(k, k_cap[0]);
    if (n_out && tid == 0) n_out[0] = max(k, 0);
    if (k <= 0) return;                                  // nothing to select

    const int n_e = (T + kSelThreads - 1) / kSelThreads;
    const int i0 = w * n_e * 64 + lane;
    uint32_t key[E];
    int nan_seen = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = i0 + e * 64;
        key[e] = e < n_e && i < T ? __float_as_uint(a[i]) : 0xffffffffu;
    }
    for (int i = tid; i < BINS * COPIES / 4; i += kSelThreads) ((u32x4*)hist)[i] = u32x4{0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < E; ++e) {
        int bad = 0;
        key[e] = order_key(__uint_as_float(key[e]), bad);   // 0xffffffff -> key 0
        if (i0 + e * 64 < T && e < n_e) nan_seen |= bad;
    }
    if (__any(nan_seen) && lane == 0) atomicOr(&counts[L + 1], 1);
    __syncthreads();

    uint32_t prefix = 0, mask = 0;
    int k_rem = k;
#pragma unroll
    for (int pass = 0; pass < 3; ++pass) {
        const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
        const uint32_t dmask = pass == 2 ? 1023u : 2047u;
        const int copies = pass == 0 ? COPIES : 1;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e < n_e && (key[e] & mask) == prefix)
                atomicAdd(&hist[((key[e] >> shift) & dmask) * copies + (pass == 0 ? lane % COPIES : 0)], 1);
        __syncthreads();
        // Descending digits: thread t takes bins 2047 - 2t and 2046 - 2t.
        const int b0 = BINS - 2 - 2 * tid;
        int c1 = 0, c0 = 0;                              // bins b0 + 1 and b0
        if (pass == 0) {
#pragma unroll
            for (int q = 0; q < COPIES; q += 4) {
                const u32x4 x = *(const u32x4*)&hist[b0 * COPIES + q];
                const u32x4 y = *(const u32x4*)&hist[(b0 + 1) * COPIES + q];
                c0 += (int)(x[0] + x[1] + x[2] + x[3]);
                c1 += (int)(y[0] + y[1] + y[2] + y[3]);
            }
        } else {
            c0 = hist[b0];
            c1 = hist[b0 + 1];
        }
        int tot;
        const int above = block_exclusive_scan<kSelThreads>(c0 + c1, scan_scratch, tot);
        if (above < k_rem && k_rem <= above + c1) {
            digit_sh = b0 + 1;
            above_sh = above;
        } else if (above + c1 < k_rem && k_rem <= above + c1 + c0) {
            digit_sh = b0;
            above_sh = above + c1;
        }
        if (pass < 2) {
            hist[tid] = 0;                               // the next pass's bins
            hist[tid + kSelThreads] = 0;
        }
        __syncthreads();
        prefix |= (uint32_t)digit_sh << shift;
        mask |= dmask << shift;
        k_rem -= above_sh;
    }

    // prefix = the k-th largest key; k_rem = how many keys equal to it to take.
    const uint32_t thr = prefix;
    int n_gt = 0, n_eq = 0;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e < n_e) {
            n_gt += __popcll(__ballot(key[e] > thr));
            n_eq += __popcll(__ballot(key[e] == thr));
        }
    if (lane == 0) {
        w_gt[w] = n_gt;
        w_eq[w] = n_eq;
    }
    __syncthreads();
    int gt_base = 0, eq_base = 0;                        // of the earlier waves
    for (int ww = 0; ww < w; ++ww) {
        gt_base += w_gt[ww];
        eq_base += w_eq[ww];
    }
    int pos = gt_base + min(eq_base, k_rem);
    int32_t* out = out_base + (size_t)l * out_stride;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (e < n_e) {
            const uint64_t eq = __ballot(key[e] == thr);
            const bool take = key[e] > thr || (key[e] == thr && eq_base + lanes_below(eq) < k_rem);
            const uint64_t tk = __ballot(take);
            if (take) out[pos + lanes_below(tk)] = i0 + e * 64;
            pos += __popcll(tk);
            eq_base += __popcll(eq);
        }
}

// Row blockIdx.x of `scores` [rows][T]: its k largest entries (k capped by
// *k_cap when given), ascending positions into out + row * out_stride; the
// count taken into *n_out when given.
__global__ __launch_bounds__(kSelThreads) void select_topk(const float* __restrict__ scores,
                                                           int T, int k,
                                                           const int32_t* __restrict__ k_cap,
                                                           int32_t* __restrict__ out_base,
                                                           int out_stride,
                                                           int32_t* __restrict__ n_out,
                                                           int32_t* __restrict__ counts, int L) {
    __shared__ int hist[256];
    __shared__ int scan_scratch[kSelThreads / 64];
    __shared__ int digit_sh, above_sh, nan_sh;
    const int l = blockIdx.x;
    const int tid = threadIdx.x;
    const float* a = scores + (size_t)l * T;
    if (k_cap) k = min(k, k_cap[0]);
    if (n_out && tid == 0) n_out[0] = max(k, 0);
    if (k <= 0) return;                                  // nothing to select

    if (tid == 0) nan_sh = 0;
    int nan_seen = 0;
    uint32_t prefix = 0, mask = 0;
    int k_rem = k;

    for (int pass = 0; pass < 4; ++pass) {
        const int shift = 24 - 8 * pass;
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
        for (int i = tid; i < T; i += kSelThreads) {
            uint32_t key = order_key(a[i], nan_seen);
            if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1);
        }
        __syncthreads();
        // Suffix sums over digits: threads 0..255 take digit 255 - tid, so an
        // inclusive prefix scan gives sum_{b' >= b} hist[b'].  The first four
        // waves hold those 256 threads; the other waves add zeros.
        const int b = 255 - tid;
        const int cnt = tid < 256 ? hist[b] : 0;
        int tot;
        const int excl = block_exclusive_scan<kSelThreads>(cnt, scan_scratch, tot);
        if (tid < 256) {
            const int above = excl;                 // keys whose digit exceeds b
            if (above < k_rem && k_rem <= above + cnt) {
                digit_sh = b;
                above_sh = above;
            }
        }
        __syncthreads();
        prefix |= (uint32_t)digit_sh << shift;
        mask |= 255u << shift;
        k_rem -= above_sh;
        __syncthreads();
    }
    if (nan_seen) nan_sh = 1;   // benign race: every writer stores 1

    // prefix = the k-th largest key; k_rem = how many keys equal to it to take.
    const uint32_t thr = prefix;
    int eq_base = 0, sel_base = 0;
    int32_t* out = out_base + (size_t)l * out_stride;
    for (int base = 0; base < T; base += kSelThreads * kSelPerThread) {
        const int i0 = base + tid * kSelPerThread;
        uint32_t keys[kSelPerThread];
        int n_eq = 0;
#pragma unroll
        for (int e = 0; e < kSelPerThread; ++e) {
            const int i = i0 + e;
            keys[e] = i < T ? order_key(a[i], nan_seen) : 0u;
            n_eq += (i < T && keys[e] == thr);
        }
        int eq_tot;
        int eq_rank = block_exclusive_scan<kSelThreads>(n_eq, scan_scratch, eq_tot) + eq_base;
        bool sel[kSelPerThread];
        int n_sel = 0;
#pragma unroll
        for (int e = 0; e < kSelPerThread; ++e) {
            const int i = i0 + e;
            bool s = false;
            if (i < T) {
                if (keys[e] > thr) s = true;
                else if (keys[e] == thr) s = (eq_rank++ < k_rem);
            }
            sel[e] = s;
            n_sel += s;
        }
        int sel_tot;
        int pos = block_exclusive_scan<kSelThreads>(n_sel, scan_scratch, sel_tot) + sel_base;
#pragma unroll
        for (int e = 0; e < kSelPerThread; ++e)
            if (sel[e] && pos < k) out[pos++] = i0 + e;
        eq_base += eq_tot;
        sel_base += sel_tot;
    }
    __syncthreads();
    if (tid == 0 && nan_sh) atomicOr(&counts[L + 1], 1);
}

// g_i = (sum_l a_{l,i}) / L, the sum in layer order.
__global__ void global_mean(const float* __restrict__ scores, int L, int T, float* __restrict__ g) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= T) return;
    float acc = 0.f;
#pragma unroll 8                                         // (independent loads, in-order sum)
    for (int l = 0; l < L; ++l) acc += scores[(size_t)l * T + i];
    g[i] = acc / (float)L;
}

// Rows that fit the registers of one workgroup take select_topk_reg with the
// smallest register tile that holds them; longer ones the streaming kernel.
// Measured (kernel time, registers vs streaming): 11.5 vs 32.5 us at 40 rows of 16384,
// 20.1 vs 60.7 us at 40 rows of 32768, 7.0 vs 10.4 us at 8 rows of 1531.
void launch_topk(const float* scores, int n_rows, int T, int k, const int32_t* k_cap, int32_t* out,
                 int out_stride, int32_t* n_out, int32_t* counts, int L, hipStream_t st) {
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(n_rows), dim3(kSelThreads), 0, st, scores, T, k, k_cap, out,
                           out_stride, n_out, counts, L);
    };
    const int n_e = (T + kSelThreads - 1) / kSelThreads;
    if (n_e <= 2) go(select_topk_reg<2>);
    else if (n_e <= 8) go(select_topk_reg<8>);
    else if (n_e <= 16) go(select_topk_reg<16>);
    else if (n_e <= 32) go(select_topk_reg<32>);
    else if (n_e <= 48) go(select_topk_reg<48>);
    else go(select_topk);
}

}  // namespace

hipError_t launch_select(const relaxkv_problem& p, const float* scores, const relaxkv_sets& s,
                         hipStream_t st) {
    hipLaunchKernelGGL(clear_error_word, dim3(1), dim3(64), 0, st, s.counts, p.L);
    launch_topk(scores, p.L, p.T_c, s.k, nullptr, s.anchors, s.k, nullptr, s.counts, p.L, st);
    return hipGetLastError();
}

hipError_t launch_select_rows(const float* scores, int n_rows, int T, int k, const int32_t* k_cap,
                              int32_t* out, int out_stride, int32_t* counts, int L,
                              hipStream_t st) {
    launch_topk(scores, n_rows, T, k, k_cap, out, out_stride, nullptr, counts, L, st);
    return hipGetLastError();
}

hipError_t launch_global_mean(const float* scores, int L, int T, float* g, hipStream_t st) {
    hipLaunchKernelGGL(global_mean, dim3((T + 255) / 256), dim3(256), 0, st, scores, L, T, g);
    return hipGetLastError();
}

hipError_t launch_select_global(const relaxkv_problem& p, const float* scores, int k_target,
                                const relaxkv_sets& s, float* g, int32_t* targets,
                                int32_t* n_targets, hipStream_t st) {
    hipLaunchKernelGGL(global_mean, dim3((p.T_c + 255) / 256), dim3(256), 0, st, scores, p.L,
                       p.T_c, g);
    // |P| = min(floor(r_g T_c), |U|) with |U| = counts[0] on the device.
    launch_topk(g, 1, p.T_c, k_target, s.counts, targets, 0, n_targets, s.counts, p.L, st);
    return hipGetLastError();
}

}  // namespace relaxkv

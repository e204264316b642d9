// The float32 attention core shared by the sparse-context attention and the
// query-side completion: R = 32 or 16 (token, head) rows of one KV head against the
// keys 0 .. n_keys-1, each row up to its own limit.
//
// float32 MFMA (32x32x2 or 16x16x4: the products and sums of fp32 FMAs, no reduced
// precision), expf for the probabilities.  The NW waves of a workgroup take the
// R-key blocks in turn (wave w: blocks w, w + NW, ...), each with its own running
// max, sum and output, combined through LDS at the end in wave order, so small
// row sets still spread over the waves.  K and V go from memory straight into
// registers as MFMA operands (NG = 64 / R lane groups; grp = lane / R):
// - S^T = K Q^T: a lane holds key lane % R and, of every 4 NG d values, the 4 at
//   4 grp (one float4; the contraction may take its index in any order as long as
//   Q, staged in LDS, uses the same one); element v of the result is key
//   4 (NG (v/4) + grp) + v%4 of row lane % R, so the softmax is lane-local plus an
//   exchange between the lane groups;
// - O^T = V^T P^T: contraction step v takes that key's row of V, lane m holding
//   its D/R consecutive d values from D/R m, one MFMA for each.
// The next block's K is loaded during this block's softmax and PV product, its key
// ids a block earlier.
//
// The kernels before took one wave per (token, head) row, with VALU dot products
// that read 64 K rows side by side.  Per launch, before and now: 2.5K context, 1100
// targets, 32q/8kv heads, d 128: 1522 -> 148 us (47 TFLOP/s); 64 query tokens over
// it 900 -> 80 us; 16 query tokens over 1K keys, 4q/2kv heads, d 64: 154 -> 20 us
// (four workgroups, so latency: 37 us as 32-row tiles of 8 waves).  With all V loads
// of half a block ahead of its products, as the test for non-finite V needs them:
// 75 -> 68 us for the 64 query tokens, 700 targets' full prefix there 262 -> 221 us,
// the 16-row launches within 2% (d 64) or 7% faster (d 128).
#pragma once

#include <math.h>

#include "dev_common.h"

namespace relaxkv {

// Rows that no caller promises more than 4-byte alignment for.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_u __attribute__((ext_vector_type(2), aligned(4)));

// A launch that gives each CU at most one 16-row workgroup takes those (half the
// work per workgroup, 16 waves); larger ones take 32 rows, which read K and V half
// as often.
inline bool attn_f32_small(long rows, int Hkv) { return (rows + 15) / 16 * Hkv <= 256; }

// Inf or NaN, from the bits, which are hidden from the compiler: the files of these
// kernels are built without NaN semantics, so it would fold a test for NaN away.
__device__ __forceinline__ bool not_finite(float x) {
    uint32_t u = __float_as_uint(x);
    asm("" : "+v"(u));
    return (u & 0x7fffffffu) >= 0x7f800000u;
}

// The bits of z + 0 * x: 0 while every x is finite, a NaN's afterwards.
__device__ __forceinline__ uint32_t zero_or_nan(float x, uint32_t z) {
    asm("v_fmac_f32_e32 %0, 0, %1" : "+v"(z) : "v"(x));
    return z;
}

template <int R> struct MfmaF32;
template <> struct MfmaF32<32> {
    typedef f32x16 Acc;
    static constexpr int waves = 8;
    static __device__ __forceinline__ Acc mac(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
    }
};
template <> struct MfmaF32<16> {
    typedef f32x4 Acc;
    static constexpr int waves = 16;
    static __device__ __forceinline__ Acc mac(float a, float b, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
};

template <int D, int R>
struct AttnF32Lds {
    static constexpr int NW = MfmaF32<R>::waves;
    f32x4 q[D * R / 256][64];        // Q fragments: lane l's float4 of d block j
    float o[NW][D][R];               // the waves' outputs, [d][row]
    float m[NW][R], l[NW][R];
};

// Called by every thread of a workgroup of MfmaF32<R>::waves waves; the lane's row
// is lane % R.  id_of(c) is the source of key c: a row index of kn/vn (row stride
// fs) when >= 0, else the cached position ~id of kc/vc (row stride cs); all four
// point at the KV head's first element.  q_row: the lane's query row; lim: its last
// visible key, -1 for none (the row is then the empty sum: O = 0, lse = -inf).
// A row's result depends on no K or V it does not see, not even on a NaN there.
// n_keys > every row's limit.  The lane's row is row orow of out [][D] and lse_out
// (may be null); written only if `valid`.
template <int D, int R, typename IdOf>
__device__ __forceinline__ void attn_f32_rows(AttnF32Lds<D, R>& sm, const float* kn,
                                              const float* vn, int64_t fs, const float* kc,
                                              const float* vc, int64_t cs, IdOf id_of, int n_keys,
                                              const float* q_row, int lim, float scale, bool valid,
                                              float* out, float* lse_out, uint32_t orow) {
    typedef MfmaF32<R> M32;
    typedef typename M32::Acc Acc;
    constexpr int NW = M32::waves, NG = 64 / R, NV = sizeof(Acc) / 4;
    constexpr int J = D / (4 * NG), DB = D / R;
    const int tid = threadIdx.x, lane = tid & 63, rl = lane % R, grp = lane / R;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int j = w; j < J; j += NW) sm.q[j][lane] = *(const f32x4_u*)(q_row + 4 * NG * j + 4 * grp);
    __syncthreads();

    auto key_of = [&](int v) { return 4 * (NG * (v >> 2) + grp) + (v & 3); };
    Acc o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = Acc{};
    float m_run = -INFINITY, l_run = 0.f;
    auto id_at = [&](int b) { return id_of(min(b * R + rl, n_keys - 1)); };
    f32x4 kf[J];
    auto load_k = [&](int id) {
        const float* kp = (id >= 0 ? kn + id * fs : kc + ~id * cs) + 4 * grp;
#pragma unroll
        for (int j = 0; j < J; ++j) kf[j] = *(const f32x4_u*)(kp + 4 * NG * j);
    };
    // What is not finite in a block's V, added to the rows that see its key (rare; the
    // wave's part of the output area holds P meanwhile).
    auto add_odd = [&](const Acc& p, int id, int ex) {
#pragma unroll
        for (int v = 0; v < NV; ++v) sm.o[w][key_of(v)][rl] = p[v];
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int kk = 0; kk < R; ++kk) {
            const int vid = __shfl(id, kk, 64);
            const float* vp = vid >= 0 ? vn + vid * fs : vc + ~vid * cs;
            const float pk = sm.o[w][kk][rl];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const float x = vp[DB * key_of(v) + db];
                    if (kk <= ex && not_finite(x)) o[db][v] = fmaf(pk, x, o[db][v]);
                }
                __builtin_amdgcn_sched_barrier(0);       // (few loads live at once)
            }
        }
        __builtin_amdgcn_wave_barrier();
    };
    int b = w, id = 0;
    if (b * R < n_keys) {
        id = id_at(b);
        load_k(id);
    }
    while (b * R < n_keys) {
        const int bn = b + NW;
        const bool more = bn * R < n_keys;
        const int id_n = more ? id_at(bn) : 0;
        Acc s = Acc{};
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const f32x4 qj = sm.q[j][lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) s = M32::mac(kf[j][i], qj[i], s);
        }
        if (more) load_k(id_n);
        const int ex = lim - b * R;
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            s[v] = key_of(v) > ex ? -INFINITY : s[v] * scale;
            mx = fmaxf(mx, s[v]);
        }
#pragma unroll
        for (int x = R; x < 64; x <<= 1) mx = fmaxf(mx, __shfl_xor(mx, x, 64));
        const float m_new = fmaxf(m_run, mx);
        const float m_ref = m_new == -INFINITY ? 0.f : m_new;   // no visible key yet: exact zeros
        if (__any(m_new > m_run)) {
            const float alpha = expf(m_run - m_ref);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
            m_run = m_new;
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            s[v] = expf(s[v] - m_ref);
            l_run += s[v];
        }
        // O^T += V^T P^T, at d 128 half of the V rows at a time (for the registers).  A
        // masked key's probability is 0, but 0 * Inf is no number: in a block with a
        // masked key, what is not finite in V (found by one multiply-add per value) is
        // left out of the product, and the rows that see it get it afterwards.
        constexpr int NH = D / 64, VH = NV / NH;
        const bool masked = __any(ex < R - 1);
        bool odd = false;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            if (h) __builtin_amdgcn_sched_barrier(0);
            float vv[VH][DB];
#pragma unroll
            for (int v = 0; v < VH; ++v) {
                const int vid = __shfl(id, key_of(h * VH + v), 64);
                const float* vp = (vid >= 0 ? vn + vid * fs : vc + ~vid * cs) + DB * rl;
                if constexpr (DB == 2) {
                    const f32x2_u x = *(const f32x2_u*)vp;
                    vv[v][0] = x[0];
                    vv[v][1] = x[1];
                } else {
#pragma unroll
                    for (int q = 0; q < DB / 4; ++q) {
                        const f32x4 x = *(const f32x4_u*)(vp + 4 * q);
#pragma unroll
                        for (int i = 0; i < 4; ++i) vv[v][4 * q + i] = x[i];
                    }
                }
            }
            if (masked) {
                uint32_t z = 0;
#pragma unroll
                for (int v = 0; v < VH; ++v)
#pragma unroll
                    for (int db = 0; db < DB; ++db) z = zero_or_nan(vv[v][db], z);
                if (__any(z != 0)) {
                    odd = true;
#pragma unroll
                    for (int v = 0; v < VH; ++v)
#pragma unroll
                        for (int db = 0; db < DB; ++db) vv[v][db] = not_finite(vv[v][db]) ? 0.f : vv[v][db];
                }
            }
#pragma unroll
            for (int v = 0; v < VH; ++v)
#pragma unroll
                for (int db = 0; db < DB; ++db) o[db] = M32::mac(vv[v][db], s[h * VH + v], o[db]);
        }
        if (odd) add_odd(s, id, ex);
        id = id_n;
        b = bn;
    }
#pragma unroll
    for (int x = R; x < 64; x <<= 1) l_run += __shfl_xor(l_run, x, 64);
    // Combine the waves: element v of block db is d = DB key_of(v) + db.
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int v = 0; v < NV; ++v) sm.o[w][DB * key_of(v) + db][rl] = o[db][v];
    if (grp == 0) {
        sm.m[w][rl] = m_run;
        sm.l[w][rl] = l_run;
    }
    __syncthreads();
    if (!valid) return;
    float M = -INFINITY, wt[NW], z = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) M = fmaxf(M, sm.m[ww][rl]);
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
        wt[ww] = sm.m[ww][rl] == -INFINITY ? 0.f : expf(sm.m[ww][rl] - M);
        z += wt[ww] * sm.l[ww][rl];
    }
    const float inv = lim < 0 ? 0.f : 1.0f / z;
    constexpr int PER = D * R / (64 * NW);               // d values a thread writes
    const int d0 = tid / R * PER;
    float* out_row = out + (size_t)orow * D;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        float acc = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) acc += wt[ww] * sm.o[ww][d0 + e][rl];
        out_row[d0 + e] = acc * inv;
    }
    if (lse_out && tid < R) lse_out[orow] = lim < 0 ? -INFINITY : M + logf(z);
}

}  // namespace relaxkv

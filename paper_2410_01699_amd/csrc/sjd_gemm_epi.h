// Pieces shared by the bf16 projection kernels (skinny, span and wide): MFMA operand types, the hi / lo split, and the epilogues
// that see final fp32 sums (plain store, residual add + operands of the next normalisation, SiLU(gate) * up, RoPE + KV-cache write;
// paper Sec. 4.1 Step 2).  Included by those files only.
#pragma once
#include "sjd_internal.h"

// what a projection does with its activations before the product
#define SJD_PRO_PLAIN 0     // fp32 activations as they are
#define SJD_PRO_NORM 1      // planes of x * gain; the token factors rsqrt(mean(x^2) + eps) come from partial sums
#define SJD_PRO_A24 2       // activations in hi / lo planes, as they are
#define SJD_PRO_A16 3       // as SJD_PRO_A24, the lo plane in its 2-byte form (the second operand ready made; sjd_gemm_bench only)

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// hi = bf16(x) (round to nearest even), lo = bf16(x - hi)
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 &hi, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 h = (__bf16)x[e];
        hi[e] = h;
        lo[e] = (__bf16)(x[e] - (float)h);
    }
}

__device__ __forceinline__ uint32_t pack_hi2(float a, float b, float &ra, float &rb)
{
    const bf16_t ha = f32_to_bf16(a), hb = f32_to_bf16(b);
    ra = a - bf16_to_f32(ha); rb = b - bf16_to_f32(hb);
    return (uint32_t)ha | ((uint32_t)hb << 16);
}

// What an epilogue needs from memory besides the sums; fetched while the weights stream.
struct EpiPre {
    f32x4 x;                  // RESID: current residual values
    uint2 gn;                 // RESID: 4 bf16 gains of the normalisation that follows
    float c0, s0, c1, s1;     // QKV: RoPE factors of this thread's two pairs
    int pos;                  // QKV: absolute position of row m in its stream's cache
    int row;                  // QKV: row index inside the stream
    SJD_GLOBAL bf16_t *cache; // QKV: this layer of the stream's cache (NULL: the row belongs to no stream)
};

// ... of NF fragments (row m[i], features n0[i] .. + 3 of this lane)
template <int EPI, int NF>
__device__ __forceinline__ void preload_epilogue(const SjdGemmEpi &ep, int N, const int (&m)[NF], const int (&n0)[NF], EpiPre (&pre)[NF])
{
    if (EPI == SJD_EPI_RESID) {
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            pre[f].x = *reinterpret_cast<const f32x4 *>(ep.out + act_off(m[f], n0[f], N / 32));
            pre[f].gn = ep.out24 ? *reinterpret_cast<const uint2 *>(ep.gain_next + n0[f]) : make_uint2(0u, 0u);
        }
    } else if (EPI == SJD_EPI_QKV) {
        const int half = ep.hd >> 1;
        int n_s[NF];
        // the stream that owns row m: its cache length and cache.  What this costs is round trips to memory in front of
        // the stores, so it is two scalar loads in a row whatever the number of streams (walking the table entry by entry
        // made the 775M forward of 4 images 1576 us, now 1565), and the same two for all fragments.
#pragma unroll
        for (int f = 0; f < NF; ++f) { n_s[f] = 0; pre[f].cache = nullptr; pre[f].row = m[f] & ((1 << ep.sm.shift) - 1); }
        if (ep.sm.shift >= 4) {
            // a stream owns whole 16-row tiles: one owner per fragment
            if (ep.sm.count > 0) {
                SjdStreamEntry e[NF];
#pragma unroll
                for (int f = 0; f < NF; ++f) e[f] = ep.sm.first;
                if (ep.sm.count > 1) {
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const int su = __builtin_amdgcn_readfirstlane(m[f] >> ep.sm.shift);
                        const SJD_GLOBAL SjdStreamEntry *t = as_global(ep.sm.table) + min(su, ep.sm.count - 1);
                        e[f].n = t->n; e[f].kvc = t->kvc;
                    }
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) n_s[f] = *as_global(e[f].n);
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    if (m[f] >> ep.sm.shift < ep.sm.count) pre[f].cache = as_global(e[f].kvc) + ep.layer_off;
            }
        } else {
            // several owners in a tile: every entry, then every length, requested together; each lane picks its own
            // (count > 1 here: a lone stream has all rows)
            SjdStreamEntry e[SJD_MAX_STREAMS];
            int n_e[SJD_MAX_STREAMS];
            if (ep.sm.count > 0) {
#pragma unroll
                for (int i = 0; i < SJD_MAX_STREAMS; ++i) e[i] = stream_entry(ep.sm, min(i, ep.sm.count - 1));
#pragma unroll
                for (int i = 0; i < SJD_MAX_STREAMS; ++i) n_e[i] = *as_global(e[i].n);
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int i = 0; i < SJD_MAX_STREAMS; ++i)
                        if (i == m[f] >> ep.sm.shift && i < ep.sm.count) { n_s[f] = n_e[i]; pre[f].cache = as_global(e[i].kvc) + ep.layer_off; }
            }
        }
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            pre[f].pos = min(n_s[f] + pre[f].row, ep.max_seq - 1);   // rows past the window are computed but never stored
            // (V fragments fetch factors they do not use: no branch around the loads)
            const int j = (n0[f] & (ep.hd - 1)) >> 1;        // (hd is a power of two and divides d)
            const float2 cc = *reinterpret_cast<const float2 *>(ep.cosT + (size_t)pre[f].pos * half + j);
            const float2 ss = *reinterpret_cast<const float2 *>(ep.sinT + (size_t)pre[f].pos * half + j);
            pre[f].c0 = cc.x; pre[f].c1 = cc.y; pre[f].s0 = ss.x; pre[f].s1 = ss.y;
        }
    }
}
template <int EPI>
__device__ __forceinline__ void preload_epilogue(const SjdGemmEpi &ep, int N, int m, int n0, EpiPre &pre)
{
    const int m_[1] = {m}, n_[1] = {n0};
    EpiPre p_[1];
    preload_epilogue<EPI, 1>(ep, N, m_, n_, p_);
    pre = p_[0];
}

// One accumulator fragment: lane l of the MFMA result holds features n0..n0+3 (packed order) of
// token m.  v = final sums.
template <int EPI>
__device__ __forceinline__ void apply_epilogue(const SjdGemmEpi &ep, int N, int m, int n0, f32x4 v, const EpiPre &pre)
{
    if (EPI == SJD_EPI_STORE) {
        if (m < ep.rows_out) *reinterpret_cast<f32x4 *>(ep.out + (size_t)m * N + n0) = v;
    } else if (EPI == SJD_EPI_RESID) {
        const f32x4 y = pre.x + v;
        *reinterpret_cast<f32x4 *>(ep.out + act_off(m, n0, N / 32)) = y;
        if (ep.out24) {
            // what the projection behind the next normalisation reads: x * gain in planes, and this
            // tile's share of sum(x^2) of token m (lanes l, l^16, l^32, l^48 hold its 16 features)
            act24_store4(ep.out24, m, n0, N / 32, y[0] * __uint_as_float(pre.gn.x << 16),
                         y[1] * __uint_as_float(pre.gn.x & 0xFFFF0000u), y[2] * __uint_as_float(pre.gn.y << 16),
                         y[3] * __uint_as_float(pre.gn.y & 0xFFFF0000u), ep.lo16 != 0);
            float sq = fmaf(y[0], y[0], fmaf(y[1], y[1], fmaf(y[2], y[2], y[3] * y[3])));
            sq += __shfl_xor(sq, 16);
            sq += __shfl_xor(sq, 32);
            if ((threadIdx.x & 48) == 0) ep.ssq_out[(size_t)m * ssq_stride(N) + (n0 >> 4)] = sq;
        }
    } else if (EPI == SJD_EPI_SILU) {
        // packed rows: (gate f, up f, gate f+1, up f+1)
        const int f = n0 >> 1;
        act24_store2(ep.ffn, m, f, ep.F / 32, v[0] / (1.0f + __expf(-v[0])) * v[1], v[2] / (1.0f + __expf(-v[2])) * v[3], ep.lo16 != 0);
    } else {   // SJD_EPI_QKV
        const int d = ep.d, hd = ep.hd, half = hd >> 1;
        const int pos = pre.pos;
        if (n0 < 2 * d) {
            // Q or K: packed order inside a head is (j, j+half, j+1, j+1+half, ...)
            const int is_k = n0 >= d;
            const int c = n0 - (is_k ? d : 0);
            const int head = c >> ep.hd_shift, j = (c & (hd - 1)) >> 1;
            const float c0 = pre.c0, s0 = pre.s0, c1 = pre.c1, s1 = pre.s1;
            const float r0 = v[0] * c0 - v[1] * s0, r0p = v[1] * c0 + v[0] * s0;   // dims j, j+half
            const float r1 = v[2] * c1 - v[3] * s1, r1p = v[3] * c1 + v[2] * s1;   // dims j+1, j+1+half
            if (!is_k) {
                float *q = ep.qact + (size_t)m * d + head * hd + j;
                *reinterpret_cast<float2 *>(q) = make_float2(r0, r1);
                *reinterpret_cast<float2 *>(q + half) = make_float2(r0p, r1p);
            } else if (pre.row < ep.rows_valid && pre.cache) {
                SJD_GLOBAL bf16_t *rec = pre.cache + kv_block_off(head, pos >> 5, ep.nblk, hd);
                const int kk = pos & 31;
                float la, lb, dummy0, dummy1;
                uint32_t hi = pack_hi2(r0, r1, la, lb);
                *reinterpret_cast<SJD_GLOBAL uint32_t *>(rec + kv_k_off(kk, j, hd, 0)) = hi;
                *reinterpret_cast<SJD_GLOBAL uint32_t *>(rec + kv_k_off(kk, j, hd, 1)) = pack_hi2(la, lb, dummy0, dummy1);
                hi = pack_hi2(r0p, r1p, la, lb);
                *reinterpret_cast<SJD_GLOBAL uint32_t *>(rec + kv_k_off(kk, j + half, hd, 0)) = hi;
                *reinterpret_cast<SJD_GLOBAL uint32_t *>(rec + kv_k_off(kk, j + half, hd, 1)) = pack_hi2(la, lb, dummy0, dummy1);
            }
        } else if (pre.row < ep.rows_valid && pre.cache) {
            // V: natural feature order
            const int col = n0 - 2 * d;
            const int head = col >> ep.hd_shift, dim = col & (hd - 1);
            SJD_GLOBAL bf16_t *rec = pre.cache + kv_block_off(head, pos >> 5, ep.nblk, hd);
            const int kk = pos & 31;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bf16_t h = f32_to_bf16(v[r]);
                rec[kv_v_off(kk, dim + r, hd, 0)] = h;
                rec[kv_v_off(kk, dim + r, hd, 1)] = f32_to_bf16(v[r] - bf16_to_f32(h));
            }
        }
    }
}


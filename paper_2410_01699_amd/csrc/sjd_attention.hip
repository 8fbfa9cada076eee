// Window attention (paper Sec. 4.1 Step 2 "forward pass ... with a causal mask"): the `rows` window
// queries attend the n cached positions plus the window positions up to their own.  The key range
// is cut into `splits` chunks so that heads x splits workgroups cover the chip; every workgroup keeps
// an online-softmax state (running max, denominator, unnormalised output) for its chunk and a small
// second kernel merges the chunks in a fixed order.
//
// Two implementations: a generic one for the fp32 models (key/value tiles of 64 positions staged in
// LDS as fp32, plain FMA arithmetic) and an MFMA one for the blocked hi/lo cache of bf16 models.
#include "sjd_internal.h"

#include <algorithm>
#include <type_traits>

#define ATT_TILE 64
#define ATT_THREADS 256

template <typename T> __device__ __forceinline__ float ld(const T *p, size_t i);
template <> __device__ __forceinline__ float ld<float>(const float *p, size_t i) { return p[i]; }
template <typename T> __device__ __forceinline__ void st_act(T *p, int r, int c, int d, float v);
template <> __device__ __forceinline__ void st_act<float>(float *p, int r, int c, int d, float v) { p[(size_t)r * d + c] = v; }

// part layout per (head, split): [rows][hd] unnormalised output, then m[rows], then l[rows]
template <typename T, int HD>
__global__ __launch_bounds__(ATT_THREADS) void attn_partial_kernel(const float *__restrict__ qact, const T *__restrict__ kc,
                                                                   const T *__restrict__ vc, int d, int rows, int splits,
                                                                   float *__restrict__ part, int stream,
                                                                   const SjdState *st)
{
    if (st->done) return;
    constexpr int ROWS = SJD_ROWS_F32;
    constexpr int RG = ATT_THREADS / HD;          // row groups in the PV phase
    constexpr int RPT = (ROWS + RG - 1) / RG;     // rows per thread there
    __shared__ float qs[ROWS][HD + 1];
    __shared__ float ks[ATT_TILE][HD + 1];        // reused for V
    __shared__ float sc[ROWS][ATT_TILE + 1];
    __shared__ float m_run[ROWS], l_run[ROWS], scale_old[ROWS];

    const int head = blockIdx.x, split = blockIdx.y, tid = threadIdx.x;
    const int n = state_n(st, stream);
    const int total = n + rows;
    int chunk = (total + splits - 1) / splits;
    chunk = (chunk + ATT_TILE - 1) / ATT_TILE * ATT_TILE;
    const int k_beg = split * chunk, k_end = min(total, k_beg + chunk);
    const float inv_sqrt = rsqrtf((float)HD);

    for (int e = tid; e < ROWS * HD; e += ATT_THREADS) {
        int r = e / HD, j = e % HD;
        qs[r][j] = r < rows ? qact[(size_t)r * d + head * HD + j] * inv_sqrt : 0.f;
    }
    if (tid < ROWS) { m_run[tid] = -INFINITY; l_run[tid] = 0.f; }
    float acc[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) acc[i] = 0.f;
    const int pv_j = tid % HD, pv_g = tid / HD;
    __syncthreads();

    // A launch of these models is a chain of latencies: a tile's keys, then its values, are requested together (positions
    // behind the end repeat the last one and count as zero), the rows behind the window are left out, the exponentials of a
    // row are made by eight threads.  Their sum stays one chain in key order.  (8 rows over 88 positions: 12.8 -> 6.1 us, an 8 x 8 image 5436 -> 4776.)
    constexpr int LPT = ATT_TILE * HD / ATT_THREADS;
    for (int t0 = k_beg; t0 < k_end; t0 += ATT_TILE) {
        const int tl = min(ATT_TILE, k_end - t0);
        float kv[LPT];
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int e = tid + i * ATT_THREADS, kk = e / HD, j = e % HD;
            kv[i] = ld<T>(kc, (size_t)(t0 + min(kk, tl - 1)) * d + head * HD + j);
        }
        float vv[LPT];
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int e = tid + i * ATT_THREADS, kk = e / HD, j = e % HD;
            vv[i] = ld<T>(vc, (size_t)(t0 + min(kk, tl - 1)) * d + head * HD + j);
        }
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int e = tid + i * ATT_THREADS, kk = e / HD, j = e % HD;
            ks[kk][j] = kk < tl ? kv[i] : 0.f;
        }
        __syncthreads();
        for (int e = tid; e < rows * ATT_TILE; e += ATT_THREADS) {
            int r = e / ATT_TILE, kk = e % ATT_TILE;
            float s = -INFINITY;
            if (kk < tl && t0 + kk <= n + r) {     // causal inside the window
                s = 0.f;
#pragma unroll 8
                for (int j = 0; j < HD; ++j) s = fmaf(qs[r][j], ks[kk][j], s);
            }
            sc[r][kk] = s;
        }
        __syncthreads();
        // online softmax bookkeeping: eight threads per row, eight keys each
        {
            static_assert(ROWS * 8 == ATT_THREADS && ATT_TILE == 64, "");
            const int r = tid >> 3, k8 = (tid & 7) * 8;
            if (r < rows) {
                float mx = m_run[r];
                const float m_old = mx;
#pragma unroll
                for (int k = 0; k < 8; ++k) mx = fmaxf(mx, sc[r][k8 + k]);
#pragma unroll
                for (int o = 1; o < 8; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
#pragma unroll
                for (int k = 0; k < 8; ++k) sc[r][k8 + k] = (sc[r][k8 + k] == -INFINITY) ? 0.f : expf(sc[r][k8 + k] - mx);
                if ((tid & 7) == 0) { scale_old[r] = (mx == -INFINITY) ? 1.f : expf(m_old - mx); m_run[r] = mx; }
            }
        }
        // V tile into ks
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int e = tid + i * ATT_THREADS, kk = e / HD, j = e % HD;
            ks[kk][j] = kk < tl ? vv[i] : 0.f;
        }
        __syncthreads();
        if (tid < rows) {
            float sum = 0.f;
#pragma unroll 16
            for (int kk = 0; kk < ATT_TILE; ++kk) sum += sc[tid][kk];
            l_run[tid] = l_run[tid] * scale_old[tid] + sum;
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int r = pv_g + i * RG;
            if (r < rows) {
                float a = acc[i] * scale_old[r];
#pragma unroll 16
                for (int kk = 0; kk < ATT_TILE; ++kk) a = fmaf(sc[r][kk], ks[kk][pv_j], a);
                acc[i] = a;
            }
        }
        __syncthreads();
    }
    float *dst = part + (size_t)(head * splits + split) * (ROWS * HD + 2 * ROWS);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int r = pv_g + i * RG;
        if (r < ROWS) dst[r * HD + pv_j] = acc[i];
    }
    if (tid < ROWS) { dst[ROWS * HD + tid] = m_run[tid]; dst[ROWS * HD + ROWS + tid] = l_run[tid]; }
}

template <typename T, int HD>
__global__ void attn_combine_kernel(const float *__restrict__ part, int splits, int d, int rows, T *__restrict__ out,
                                    const SjdState *st)
{
    if (st->done) return;
    constexpr int ROWS = SJD_ROWS_F32;
    const int head = blockIdx.x;
    for (int e = threadIdx.x; e < rows * HD; e += blockDim.x) {
        const int r = e / HD, j = e % HD;
        float mx = -INFINITY;
        for (int s = 0; s < splits; ++s)
            mx = fmaxf(mx, part[(size_t)(head * splits + s) * (ROWS * HD + 2 * ROWS) + ROWS * HD + r]);
        float num = 0.f, den = 0.f;
        for (int s = 0; s < splits; ++s) {
            const float *p = part + (size_t)(head * splits + s) * (ROWS * HD + 2 * ROWS);
            const float ms = p[ROWS * HD + r];
            if (ms == -INFINITY) continue;
            const float w = expf(ms - mx);
            num += w * p[r * HD + j];
            den += w * p[ROWS * HD + ROWS + r];
        }
        st_act<T>(out, r, head * HD + j, d, num / den);
    }
}

// ---------------------------------------------------------------------------------------------
// bf16 models: MFMA kernels over the blocked hi/lo cache.  Per block of 32 positions
//   S^T[key][query] = K[key][:] . Q[query][:]       A = K tile (16 keys x 32 dims), B = Q
//   O^T[dim][query] += V^T[dim][key] * P[key][query] A = V^T tile (16 dims x 32 keys), B = P
// Both cache operands are stored exactly as the lanes consume them, so a wave fetches a block's K and
// V tiles as contiguous 1 KiB loads.  Every operand is a hi + lo bf16 pair; a product keeps the
// three leading terms hi*hi + hi*lo + lo*hi (about 16 significant bits).  The two 16-key score tiles
// of a block leave lane l (query l%16, group g = l/16) with the keys {4g..4g+3} and {16+4g..16+4g+3};
// the V^T tiles use the same key order, which makes the probabilities the B operand of the second
// product without any cross-lane movement.
//
// attn_split_kernel: workgroup (head, split) of AW waves (4 or 8) takes a contiguous range of blocks; wave w
// handles every AW-th block of it with an online softmax (running max, denominator, unnormalised
// O^T per query); the waves are merged through LDS in wave order and the workgroup writes one
// partial result.  attn_merge_kernel combines the splits of a head in split order.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 &hi, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const __bf16 h = (__bf16)x[e];
        hi[e] = h;
        lo[e] = (__bf16)(x[e] - (float)h);
    }
}

// The workgroup barrier as gfx950 has it: an s_barrier lets the waves of a workgroup go on when each of them has arrived
// at an s_barrier, at whichever address.  __syncthreads() promises this only where all threads come to the same call.
// Every wave has to arrive equally often, and the branch around it has to be uniform in the wave.
__device__ __forceinline__ void arrive_and_wait()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Up to about 1000 positions a launch is one round of latencies (arguments, cache length, K and V, merge); above, what the
// workgroups in flight can request bounds it.  Hence:
//  - two waves per SIMD, at most 256 registers each (left alone the compiler took 316 for heads of 128 and 32 queries, one
//    workgroup per CU): the scores of every query tile come first, so that the key tiles' registers are free before the
//    probabilities are made (1240 positions x 2 contexts of 32 queries: 35.7 -> 27.1 us, 23.1 with what follows);
//  - keys and values as non-temporal loads (NT: a plain read of this chip runs at 6.4 TB/s with them and at 5.9 without) where one
//    query group reads them and the forward's caches are more than the last-level cache can keep (sjd_kv_streams).  Plain loads
//    and non-temporal ones, us a forward: 7B, eight images of 16 drafts at 1239 positions (10 GB) 7204 and 6888, at 583
//    6262 and 6192, one at 583 (0.6 GB) 2756 and 2736.  Smaller caches are still there when the next forward reads them, and when
//    the QKV epilogue writes into their lines, unless they were read so: 775M, one image at 633 positions (0.19 GB) 773 and 789, eight
//    at 200 1628 and 1649, 7B at 100 (0.1 GB) 2632 and 2648; 775M whole images 1948 and 1924 tokens/s.  (Forwards that take turns between
//    caches keep none of them: 775M at 633 positions 803 and 798.)  Two query groups, 775M window of 64 at 1100 positions 1190 and 1215;
//  - loads in the order of their use (Q, K, V; the next block's K during the probabilities), as global accesses with
//    nothing conditional between a load and its use, so that each wait is for its own loads only; and the arguments of the
//    first loads in registers (16 queries at 600 positions: 8.3 -> 6.7 us; 7B forward of 16 drafts there 2998 -> 2942).
// partial record of (head, split): O[MT*16][HD] unnormalised, then m[MT*16], then l[MT*16]
template <int HD, int MT, int AW, bool NT>
__global__ __launch_bounds__(64 * AW, 2) void attn_split_kernel(const int32_t *n0, const int32_t *done0, const bf16_t *kvc0,
                                                            const float *__restrict__ qact, int d, int nblk_cache,
                                                            int rows, int splits, int qgroups, int shift,
                                                            float *__restrict__ part, const SjdStreamEntry *table,
                                                            size_t layer_off, void *__restrict__ out, int lo16)
{
    // (n0, done0, kvc0: stream 0, its cache at this layer; they and all that every workgroup needs at once are the
    // 14 registers of arguments that arrive with the dispatch, in front of the first dependent load)
    // blockIdx.z = (stream, query group): the stream has its own cache and cache length and its queries in
    // rows (stream << shift)..; a stream with more than MT * 16 rows is covered by several groups of
    // MT * 16 consecutive queries, each walking the keys on its own
    const int stream = qgroups == 1 ? (int)blockIdx.z : (int)blockIdx.z / qgroups;
    const int qbase = ((int)blockIdx.z - stream * qgroups) * (MT * 16);
    const SJD_GLOBAL int32_t *np = as_global(n0), *dp = as_global(done0);
    const SJD_GLOBAL bf16_t *kvc = as_global(kvc0);
    if (stream) {
        const SJD_GLOBAL SjdStreamEntry *e = as_global(table) + stream;
        np = as_global(e->n); dp = as_global(e->done); kvc = as_global((const bf16_t *)e->kvc) + layer_off;
    }
    const int done = *dp, n = *np;
    asm volatile("" ::"s"(done), "s"(n));         // (one round trip for both: the length is not fetched behind the branch)
    if (done) return;
    const int row0 = (stream << shift) + qbase;
    part += (size_t)blockIdx.z * gridDim.x * splits * (MT * 16 * HD + 2 * MT * 16);
    constexpr int KS = HD / 32;      // k-steps of the score product
    constexpr int DT = HD / 16;      // output dim tiles
    constexpr int REC = MT * 16 * HD + 2 * MT * 16;
    __shared__ float m_all[AW][MT * 16], l_all[AW][MT * 16];
    __shared__ f32x4 o_slot[AW][DT][64];
    __shared__ bf16x8 q_lds[MT][KS][2][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, c = lane & 15;
    const int head = blockIdx.x, split = blockIdx.y;
    const int total = n + rows;
    const int nblk = (total + 31) >> 5;
    const int bps = (nblk + splits - 1) / splits;
    const int b_beg = split * bps, b_end = min(nblk, b_beg + bps);
    const float scale = rsqrtf((float)HD);

    // Loads return in order: Q first (it does not wait for the cache length either), so that it is staged while the
    // first block's tiles are on their way, then K, then V.
    constexpr int QU = (MT * KS + AW - 1) / AW;          // (tile, lane) units of Q a thread stages
    float4 qx[QU][2];
#pragma unroll
    for (int i = 0; i < QU; ++i) {
        const int u = min((int)threadIdx.x + i * 64 * AW, MT * KS * 64 - 1), l = u & 63, ks = (u >> 6) % KS, mt = (u >> 6) / KS;
        // (query rows past the stream's `rows` are masked below; the clamp keeps their loads inside qact)
        const int qr = min(row0 + mt * 16 + (l & 15), SJD_ROWS_MAX - 1);
        const float4 *src = reinterpret_cast<const float4 *>(qact + (size_t)qr * d + head * HD + ks * 32 + (l >> 4) * 8);
        qx[i][0] = src[0]; qx[i][1] = src[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 ka[2][KS][2], va[DT][2];
    auto load_once = [](const SJD_GLOBAL bf16x8 *p) -> bf16x8 { if constexpr (NT) return __builtin_nontemporal_load(p); else return *p; };
    auto load_k = [&](int blk) {
        const SJD_GLOBAL bf16x8 *rec = reinterpret_cast<const SJD_GLOBAL bf16x8 *>(kvc + kv_block_off(head, blk, nblk_cache, HD)) + lane;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int pl = 0; pl < 2; ++pl) ka[h][ks][pl] = load_once(rec + ((h * KS + ks) * 2 + pl) * 64);
    };
    auto load_v = [&](int blk) {
        const SJD_GLOBAL bf16x8 *rec = reinterpret_cast<const SJD_GLOBAL bf16x8 *>(kvc + kv_block_off(head, blk, nblk_cache, HD)) + lane;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl) va[t][pl] = load_once(rec + (2 * KS * 2 + t * 2 + pl) * 64);
    };
    // Q as B operand, shared by the waves: entry [mt][ks][plane][lane] holds
    // Q[query c (+16 mt)][32 ks + 8 g .. +8], scaled by 1/sqrt(HD), as hi and lo bf16 planes
    auto stage_q = [&]() {
#pragma unroll
        for (int i = 0; i < QU; ++i) {
            const int u = threadIdx.x + i * 64 * AW;
            if (u >= MT * KS * 64) break;
            const float x[8] = {qx[i][0].x * scale, qx[i][0].y * scale, qx[i][0].z * scale, qx[i][0].w * scale,
                                qx[i][1].x * scale, qx[i][1].y * scale, qx[i][1].z * scale, qx[i][1].w * scale};
            bf16x8 hi, lo;
            split8(x, hi, lo);
            q_lds[(u >> 6) / KS][(u >> 6) % KS][0][u & 63] = hi; q_lds[(u >> 6) / KS][(u >> 6) % KS][1][u & 63] = lo;
        }
    };

    f32x4 o[MT][DT];
    float m_run[MT], l_run[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        m_run[mt] = -INFINITY; l_run[mt] = 0.f;
#pragma unroll
        for (int t = 0; t < DT; ++t) o[mt][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
    int blk = b_beg + wave;
    // One block.  The next block's K tiles are requested as soon as the scores have left their registers, its V tiles
    // as soon as this block's output has left theirs; the wave's last block has a copy of the code of its own (loads
    // behind a branch would make every wait drain them all).
    // (Not with 32 queries on heads of 128: 256 registers do not hold it.)
    constexpr bool AHEAD = MT * HD < 256;
    auto block = [&](auto more) {
        const int k0 = blk * 32;
        // scores of all query tiles first: the K tiles' registers are free before the probabilities are made
        f32x4 sc[MT][2];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                sc[mt][h] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 qh = q_lds[mt][ks][0][lane], ql = q_lds[mt][ks][1][lane];
                    sc[mt][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[h][ks][1], qh, sc[mt][h], 0, 0, 0);
                    sc[mt][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[h][ks][0], ql, sc[mt][h], 0, 0, 0);
                    sc[mt][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[h][ks][0], qh, sc[mt][h], 0, 0, 0);
                }
            }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (more.value && AHEAD) { load_k(blk + AW); __builtin_amdgcn_sched_barrier(0); }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const f32x4 (&s_)[2] = sc[mt];
            const int qrow = qbase + mt * 16 + c;    // row inside the stream's window
            float p_[8];
            float mx = m_run[mt];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int key = k0 + (e >> 2) * 16 + g * 4 + (e & 3);
                const bool ok = key <= n + qrow && qrow < rows;     // causal inside the window
                p_[e] = ok ? s_[e >> 2][e & 3] : -INFINITY;
                mx = fmaxf(mx, p_[e]);
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float so = (mx == -INFINITY) ? 1.f : __expf(m_run[mt] - mx);
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                p_[e] = (p_[e] == -INFINITY) ? 0.f : __expf(p_[e] - mx);
                sum += p_[e];
            }
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            l_run[mt] = l_run[mt] * so + sum;
            m_run[mt] = mx;
            bf16x8 ph, pl;
            split8(p_, ph, pl);
#pragma unroll
            for (int t = 0; t < DT; ++t) {
                o[mt][t] *= so;
                o[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t][1], ph, o[mt][t], 0, 0, 0);
                o[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t][0], pl, o[mt][t], 0, 0, 0);
                o[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[t][0], ph, o[mt][t], 0, 0, 0);
            }
        }
        if constexpr (more.value) {
            __builtin_amdgcn_sched_barrier(0);
            if (!AHEAD) load_k(blk + AW);
            load_v(blk + AW);
        }
    };
    // A wave without a block (short caches) arrives from the other side of the branch.  With one barrier behind the branch
    // every wait for Q has to hold for a wave that requested nothing after Q as well, and so drains the first block's tiles:
    // 775M forward of 16 drafts 818 us as it is, 829 so; 7B 2899 and 2920.
    if (blk < b_end) {
        load_k(blk);
        __builtin_amdgcn_sched_barrier(0);
        load_v(blk);
        __builtin_amdgcn_sched_barrier(0);
        stage_q();
        arrive_and_wait();                        // q_lds ready
        for (; blk + AW < b_end; blk += AW) block(std::true_type{});
        block(std::false_type{});
    } else {
        stage_q();
        arrive_and_wait();
    }

    // ---- merge the AW waves (wave order) and write the partial record -----------------------------
    if (g == 0) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) { m_all[wave][mt * 16 + c] = m_run[mt]; l_all[wave][mt * 16 + c] = l_run[mt]; }
    }
    __syncthreads();
    float *dst = part + (size_t)(head * splits + split) * REC;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < AW; ++w) M = fmaxf(M, m_all[w][mt * 16 + c]);
        const float mine = (m_run[mt] == -INFINITY) ? 0.f : __expf(m_run[mt] - M);
        float den = 0.f;
#pragma unroll
        for (int w = 0; w < AW; ++w) {
            const float mw = m_all[w][mt * 16 + c];
            den += (mw == -INFINITY) ? 0.f : __expf(mw - M) * l_all[w][mt * 16 + c];
        }
        if (mt) __syncthreads();                  // o_slot is reused
#pragma unroll
        for (int t = 0; t < DT; ++t) o_slot[wave][t][lane] = o[mt][t] * mine;
        __syncthreads();
        for (int u = threadIdx.x; u < DT * 64; u += 64 * AW) {
            const int t = u >> 6, l = u & 63;
            f32x4 v = o_slot[0][t][l];
#pragma unroll
            for (int w = 1; w < AW; ++w) v += o_slot[w][t][l];
            // lane l holds dims 16 t + 4 (l/16) .. +4 of query l%16
            if (splits > 1) {
                *reinterpret_cast<f32x4 *>(dst + (size_t)(mt * 16 + (l & 15)) * HD + t * 16 + (l >> 4) * 4) = v;
            } else if (qbase + mt * 16 + c < rows) {
                // all keys were this workgroup's: what the merge kernel would do with the only record
                const f32x4 y = v * (1.0f / den);
                act24_store4(out, row0 + mt * 16 + c, head * HD + t * 16 + (l >> 4) * 4, d / 32, y[0], y[1], y[2], y[3], lo16 != 0);
            }
        }
        if (splits > 1 && wave == 0 && g == 0) {
            dst[MT * 16 * HD + mt * 16 + c] = M;
            dst[MT * 16 * HD + MT * 16 + mt * 16 + c] = den;
        }
    }
}

// out[q][head*HD + :] = sum_s w_s O_s[q][:] / sum_s w_s l_s,  w_s = exp(m_s - max_s m_s), written as
// the hi / lo operand planes the O projection streams (act24_idx).  All loads of a thread are issued before anything
// depends on them (splits <= ATT_MAX_SPLITS), four splits at a time; one wave per workgroup, so that the records are read
// by as many CUs as there are waves (four waves each, and the loads of all 16 splits whatever their number: 7B forward
// of 16 drafts 2945 us, now 2893; 775M 838, now 821; in a kernel trace the kernel itself is 5.1 and 4.9).
#define ATT_MAX_SPLITS 16
#define ATT_MERGE_THREADS 64
template <int HD, int MT>
__global__ __launch_bounds__(ATT_MERGE_THREADS) void attn_merge_kernel(const float *__restrict__ part, int splits, int d, int rows,
                                                        void *__restrict__ out, int shift, int qgroups, int lo16)
{
    constexpr int REC = MT * 16 * HD + 2 * MT * 16;
    constexpr int Q4 = HD / 4;
    const int head = blockIdx.x, stream = blockIdx.z / qgroups, qbase = (blockIdx.z % qgroups) * (MT * 16);
    const float *base = part + ((size_t)blockIdx.z * gridDim.x + head) * splits * REC;
    const int u = blockIdx.y * ATT_MERGE_THREADS + threadIdx.x;
    if (u >= min(rows - qbase, MT * 16) * Q4) return;
    const int q = u / Q4, j4 = u % Q4;
    float ms[ATT_MAX_SPLITS], ls[ATT_MAX_SPLITS];
    f32x4 os[ATT_MAX_SPLITS];
#pragma unroll
    for (int s = 0; s < ATT_MAX_SPLITS; ++s) { ms[s] = -INFINITY; ls[s] = 0.f; os[s] = (f32x4){0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
    for (int s0 = 0; s0 < ATT_MAX_SPLITS; s0 += 4) {
        if (s0 >= splits) break;
#pragma unroll
        for (int s = s0; s < s0 + 4; ++s) {
            const float *p = base + (size_t)(s < splits ? s : 0) * REC;
            ms[s] = p[MT * 16 * HD + q];
            ls[s] = p[MT * 16 * HD + MT * 16 + q];
            os[s] = *reinterpret_cast<const f32x4 *>(p + (size_t)q * HD + j4 * 4);
        }
    }
    float M = -INFINITY;
#pragma unroll
    for (int s = 0; s < ATT_MAX_SPLITS; ++s) if (s < splits) M = fmaxf(M, ms[s]);
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
#pragma unroll
    for (int s = 0; s < ATT_MAX_SPLITS; ++s) {
        const float w = (s < splits && ms[s] != -INFINITY) ? __expf(ms[s] - M) : 0.f;   // an empty split holds zeros
        num += w * os[s];
        den += w * ls[s];
    }
    const f32x4 o = num * (1.0f / den);
    act24_store4(out, (stream << shift) + qbase + q, head * HD + j4 * 4, d / 32, o[0], o[1], o[2], o[3], lo16 != 0);
}

int32_t sjd_attention_splits(const sjd_model *m)
{
    const int H = m->cfg.n_heads;
    if (m->cfg.dtype == 1) {
        // about two workgroups per CU, but at least four 32-position blocks per split at full length
        int s = (512 + H - 1) / H;
        int max_s = ((m->cfg.max_seq + 31) / 32 + 3) / 4;
        if (s > max_s) s = max_s;
        if (s > 16) s = 16;              // ATT_MAX_SPLITS of the merge kernel
        return s < 1 ? 1 : s;
    }
    int s = (512 + H - 1) / H;   // about two workgroups per CU
    int max_s = (m->cfg.max_seq + ATT_TILE - 1) / ATT_TILE;
    if (s > max_s) s = max_s;
    return s < 1 ? 1 : s;
}

size_t sjd_attention_part_elems(const sjd_model *m)
{
    if (m->cfg.dtype == 0) return (size_t)m->cfg.n_heads * sjd_attention_splits(m) * (SJD_ROWS_F32 * m->hd + 2 * SJD_ROWS_F32);
    // (stream, query group) pairs of up to 32 rows each: one or two of them run at the full number of key
    // splits, more of them (up to SJD_MAX_STREAMS) split their keys less finely (never below one split
    // each), so that pairs x splits stays within 2 x the full number
    const int splits = std::max(sjd_attention_splits(m), SJD_MAX_STREAMS / 2);
    return (size_t)m->cfg.n_heads * 2 * splits * (32 * m->hd + 2 * 32);
}

template <typename T, int HD>
static int launch_t(const sjd_model *m, sjd_kv *kv, int32_t layer, int32_t rows, int32_t stream, hipStream_t s)
{
    const int d = m->cfg.d_model, H = m->cfg.n_heads;
    const T *kc = (const T *)(stream ? kv->k_u : kv->k), *vc = (const T *)(stream ? kv->v_u : kv->v);
    SJD_LAUNCH((attn_partial_kernel<T, HD>), dim3(H, kv->att_splits), dim3(ATT_THREADS), 0, s,
                       kv->qact, kc + (size_t)layer * kv->k_layer_stride,
                       vc + (size_t)layer * kv->v_layer_stride, d, rows, kv->att_splits,
                       kv->att_part, stream, kv->state);
    HIP_TRY(hipGetLastError());
    SJD_LAUNCH((attn_combine_kernel<T, HD>), dim3(H), dim3(256), 0, s, kv->att_part, kv->att_splits, d, rows,
                       (T *)kv->att_out, kv->state);
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

// Key splits of a launch over `pairs` (stream, query group) pairs of `heads` heads.  The partial-record buffer holds two
// pairs at att_splits splits; more of them share it by splitting their keys less finely.  Heads of 128 take the count, up to
// that, with the least work in a row: 512 workgroups run at once (two fit a CU by their registers), so the launch is
// ceil(workgroups / 512) rounds of 1 / splits of the keys each, and of equal counts the smallest (fewer records to merge).
// Without and with it, 7B forwards over 3967 positions: two contexts of 16 drafts 16 splits (two rounds) 4820 us, 8 splits
// 4757; of 32 drafts 5780 and 5713; five of 16 6 and 3 splits 8858 and 8698; eight 4 and 2 splits 11750 and 11646; six keep
// their 5 (two rounds; 2 splits, one round, 9571 us, 5 splits 9518).  At 1239 positions two of 32: 4761 and 4702.
static int most_splits(int pairs, int att_splits) { return pairs <= 2 ? att_splits : std::max(1, 2 * att_splits / pairs); }
static int key_splits(int hd, int heads, int pairs, int att_splits)
{
    const int most = most_splits(pairs, att_splits);
    if (hd != 128) return most;
    int best = 1, best_rounds = (heads * pairs + 511) / 512;
    for (int s = 2; s <= most; ++s) {
        const int rounds = (heads * pairs * s + 511) / 512;
        if (rounds * best < best_rounds * s) { best = s; best_rounds = rounds; }
    }
    return best;
}

// Workgroups of eight waves instead of four, one per CU instead of two: as many waves and half as many records, which cost a
// launch 4-6 us at its end where they are 4-8 MB, and none where one workgroup has all keys of a head (then it writes the
// operand planes itself and no merge kernel runs).  Only where such workgroups cover the 256 CUs exactly: with three, five, six or
// seven pairs of 32 heads they would leave CUs idle or need a second round, and nothing overlaps a round's start.  Four waves
// and eight, us a forward: one context of 32 drafts at 1239 positions 3422 -> 3391, two 4344 -> 4288, eight of 16 at 583
// (one split) 6330 -> 6200, prompt of 64 3998 -> 3937, one of 16 at 3967 3348 -> 3326, at 583 2778 -> 2780.
static bool eight_waves(int hd, int heads, int pairs, int att_splits)
{
    return hd == 128 && 256 % (heads * pairs) == 0 && 256 / (heads * pairs) <= most_splits(pairs, att_splits);
}

template <int HD, int MT>
static int launch_mfma_t(const sjd_model *m, sjd_kv *kv, int32_t layer, int32_t rows, const SjdStreams &sm, bool lo16,
                         bool kv_streams, hipStream_t s)
{
    const int d = m->cfg.d_model, H = m->cfg.n_heads;
    const size_t off = (size_t)layer * kv->k_layer_stride;
    const int qgroups = (rows + MT * 16 - 1) / (MT * 16), pairs = sm.count * qgroups;
    const bool eight = eight_waves(HD, H, pairs, kv->att_splits);
    const int splits = eight ? 256 / (H * pairs) : key_splits(HD, H, pairs, kv->att_splits);
    if (pairs * splits > 2 * std::max(kv->att_splits, SJD_MAX_STREAMS / 2)) return SJD_EINVAL;    // (what att_part holds)
    const int grows = std::min(rows, MT * 16);
#define GO(W, NT) SJD_LAUNCH((attn_split_kernel<HD, MT, W, NT>), dim3(H, splits, pairs), dim3(64 * W), 0, s, sm.first.n, sm.first.done, \
                       sm.first.kvc + off, kv->qact, d, kv->nblk, rows, splits, qgroups, sm.shift, kv->att_part, sm.table, off, \
                       kv->att_out, lo16 ? 1 : 0)
    const bool nt = kv_streams && qgroups == 1;
    if constexpr (HD == 128) {
        if (eight && nt) GO(8, true);
        else if (eight) GO(8, false);
    }
    if (!eight && nt) GO(4, true);
    else if (!eight) GO(4, false);
#undef GO
    HIP_TRY(hipGetLastError());
    if (splits == 1) return SJD_OK;               // (written in place)
    SJD_LAUNCH((attn_merge_kernel<HD, MT>), dim3(H, (grows * (HD / 4) + ATT_MERGE_THREADS - 1) / ATT_MERGE_THREADS, pairs), dim3(ATT_MERGE_THREADS), 0, s, kv->att_part,
                       splits, d, rows, kv->att_out, sm.shift, qgroups, lo16 ? 1 : 0);
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

template <int HD>
static int launch_mfma(const sjd_model *m, sjd_kv *kv, int32_t layer, int32_t rows, const SjdStreams &sm, bool lo16,
                       bool kv_streams, hipStream_t s)
{
    if (sm.count < 1 || sm.count > SJD_MAX_STREAMS || rows > (1 << sm.shift) || (sm.count << sm.shift) > SJD_ROWS_MAX)
        return SJD_EINVAL;
    if (rows <= 16) return launch_mfma_t<HD, 1>(m, kv, layer, rows, sm, lo16, kv_streams, s);
    return launch_mfma_t<HD, 2>(m, kv, layer, rows, sm, lo16, kv_streams, s);     // 32 queries per (stream, query group)
}

int sjd_launch_attention(const sjd_model *m, sjd_kv *kv, int32_t layer, int32_t rows, const SjdStreams &sm, bool lo16,
                         bool kv_streams, hipStream_t s)
{
    const int hd = m->hd;
    if (m->cfg.dtype != 1) return SJD_EINVAL;
    if (hd == 32) return launch_mfma<32>(m, kv, layer, rows, sm, lo16, kv_streams, s);
    if (hd == 64) return launch_mfma<64>(m, kv, layer, rows, sm, lo16, kv_streams, s);
    if (hd == 128) return launch_mfma<128>(m, kv, layer, rows, sm, lo16, kv_streams, s);
    return SJD_EINVAL;
}

int sjd_launch_attention_f32(const sjd_model *m, sjd_kv *kv, int32_t layer, int32_t rows, int32_t stream, hipStream_t s)
{
    const int hd = m->hd;
    if (m->cfg.dtype != 0 || stream < 0 || stream > 1) return SJD_EINVAL;
    if (hd == 16) return launch_t<float, 16>(m, kv, layer, rows, stream, s);
    if (hd == 32) return launch_t<float, 32>(m, kv, layer, rows, stream, s);
    if (hd == 64) return launch_t<float, 64>(m, kv, layer, rows, stream, s);
    if (hd == 128) return launch_t<float, 128>(m, kv, layer, rows, stream, s);
    return SJD_EINVAL;
}

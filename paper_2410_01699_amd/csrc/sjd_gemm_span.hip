// bf16 projections whose workgroups own a span of output features for the whole reduction, at any row count (paper
// Sec. 4.1 Step 2): C[M x N] = A[M x K] * W^T, M = 1 .. 128.
//
// Like the skinny kernel, the waves of a workgroup split K, each streams its own weights and its own activation tiles
// straight into registers (nothing is shared, so nothing is staged and no barrier stands in the loop) and the fp32 sums
// meet once, through LDS, in wave order; the epilogue sees final values, so there are no K-slices in memory and no second
// kernel.  Three things differ:
//  - a workgroup owns G packed weight groups (up to six 16-feature tiles), so many that one workgroup per CU covers N.
//    Every workgroup reads all M x K activations from L2; with the skinny kernel's two tiles the 7B gate/up projection had
//    688 workgroups, 2.7 reads of the activations per CU.
//  - K may be cut across gridDim.y workgroups as well, where all of it would make a workgroup read far more activations than
//    weights or leave CUs without one: the slices' sums meet in the workgroup of a column that arrives last.
//  - up to eight row tiles.  A wave's activation tiles are refilled in place as soon as their products are issued, the
//    weights of the next k-step are requested one k-step ahead.
//
// What bounds it, 7B gate/up (180 MB) alone on cold weights: up to 32 rows the weight stream (16 rows 29.7 us, 32 rows 31.5;
// a kernel that only reads these bytes 26 to 32; the skinny kernel was at 32.3 and 39.2).  Above, the activation loads in between,
// 64 rows 38.5 us, 128 rows 56.4: without these loads 32.9 and 45.5, but 33.8 and 53.9 with loads of no bytes in their place, so at 128 rows
// it is less the bytes from L2 than the loads themselves (they return in order, behind weights from HBM) and the products (without them
// 34.7 and 50.0).  QKV at 128 rows 38.0: 25.5, 34.8 and 35.4.  The wide kernel and its second kernel need 42.5 and 62.7 us.  Inside a forward, per launch: 29.2 us at 16 rows (skinny 32.2), 31.0 at 32 (the wide
// kernel with final sums in it 38.5), 37.6 at 64 (wide 40.7 + 5.3), 58.7 at 128 (wide 55.8 + 9.5).
#include "sjd_gemm_epi.h"

#include <algorithm>

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

constexpr int pow2_floor(int x) { int p = 1; while (p * 2 <= x) p *= 2; return p; }

// second operand of 8 values from their hi plane entry (8 bf16) and their byte plane entry (8 bytes): value = hi bits | lo byte << 8
// (as fp32); second operand = bf16(value - hi)
__device__ __forceinline__ bf16x8 lo_by_perm(bf16x8 hi, u32x2_t lo8)
{
    const u32x4_t hw = __builtin_bit_cast(u32x4_t, hi);
    u32x4_t r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t lw = lo8[p >> 1], b = (2 * p) & 3;
        const uint32_t v0 = __builtin_amdgcn_perm(hw[p], lw, 0x0504000Cu | (b << 8));          // (hi bits, lo byte, 0)
        const uint32_t v1 = __builtin_amdgcn_perm(hw[p], lw, 0x0706000Cu | ((b + 1) << 8));
        const float d0 = __uint_as_float(v0) - __uint_as_float(hw[p] << 16);
        const float d1 = __uint_as_float(v1) - __uint_as_float(hw[p] & 0xFFFF0000u);
        r[p] = __builtin_amdgcn_perm(__float_as_uint(d1), __float_as_uint(d0), 0x07060302u);   // (exact: 8 significant bits)
    }
    return __builtin_bit_cast(bf16x8, r);
}

#define SPAN_AGENT 16             // cache policy sc1: stores go through to memory, loads come from there, whichever XCD asks
#define SPAN_OOB 0x40000000u      // a byte offset behind every buffer: the load returns zeros and costs no memory access
#define SPAN_K_MAX (1 << 21)      // (a buffer is at most 384 K bytes)

template <int MT, int TN, int G, int WK, int EPI, bool NORM, int KSM>
__global__ __launch_bounds__(64 * WK) void gemm_span_kernel(const bf16_t *__restrict__ Wp, const void *__restrict__ Xv,
                                                            const float *__restrict__ ssq_in, float eps, int N, int K, int kslice,
                                                            float *part, uint32_t *tickets, SjdGemmEpi ep)
{
    constexpr bool SLICED = KSM > 1;                      // K cut across gridDim.y <= KSM workgroups
    constexpr int TNE = TN * G, F = MT * TNE;             // tiles, accumulator fragments of a wave
    // the sums meet in LDS in passes of FC fragments, of which every wave finishes FPW
    constexpr int FPW = WK == 8 ? 1 : 4, FC = F < WK * FPW ? F : WK * FPW, NCH = (F + FC - 1) / FC;
    __shared__ f32x4 red[WK][FC][64];
    __shared__ float rs[MT * 16];
    __shared__ uint32_t arrived;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, c = lane & 15;
    const int KT = K / 32, NT = N / 16, groups = NT / TN;
    const int s0 = SLICED ? (int)blockIdx.y * kslice : 0, s1 = SLICED ? min(KT, s0 + kslice) : KT;      // this K-slice
    const int kps = (s1 - s0 + WK - 1) / WK;
    const int kt0 = min(s1, s0 + wave * kps), klen = min(s1, kt0 + kps) - kt0;
    // workgroups start their walk at different k-steps (as in the skinny kernel), from 8 k-steps a wave on: 16384 x 2048, whose
    // workgroups' weights lie 256 KB apart, 15.7 us at 16 rows and 20.2 at 64 without, 13.0 and 17.1 with (skinny kernel at 16: 12.3)
    const int rot = klen >= 8 ? (int)((((blockIdx.x >> 3) & 31u) * (unsigned)klen) >> 5) : 0;

    f32x4 acc[MT][TNE];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < TNE; ++t) acc[mt][t] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // Both operands through buffer descriptors: scalar offsets, one vector register of addresses for each.
    const int g0 = blockIdx.x * G, gv = min(G, groups - g0);
    const uint32_t gstride = (uint32_t)(KT * TN) << 10, lo_base = (uint32_t)act24_lo_base(KT);
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(Wp) + (size_t)g0 * KT * TN * 512, 0, gstride * gv, 0x00020000);
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(Xv), 0,
                                                                        lo_base + ((uint32_t)(SJD_MTILES * KT) << 9), 0x00020000);
    uint32_t goff[G];                                     // (a group behind the last one: the last one again, not written)
#pragma unroll
    for (int j = 0; j < G; ++j) goff[j] = gstride * min(j, gv - 1);

    // sum(x^2) of every token from the partial sums its writer left: TPT threads a token, requested before the first tiles
    // (loads return in order) and added up while those are on their way
    constexpr int TPT = pow2_floor(4 * WK / MT), PJ = 64 / TPT;
    const int NQ = ssq_stride(K) / 4, tok = threadIdx.x / TPT, sl = threadIdx.x % TPT;
    const SJD_GLOBAL f32x4 *pp = as_global(reinterpret_cast<const f32x4 *>(ssq_in)) + (size_t)min(tok, MT * 16 - 1) * NQ;
    f32x4 pr[NORM ? PJ : 1];
    if constexpr (NORM) {
#pragma unroll
        for (int j = 0; j < PJ; ++j) pr[j] = pp[min(sl + j * TPT, NQ - 1)];     // (past the row's end: a duplicate, dropped below)
    }

    // Up to two row tiles: two sets of activation tiles, the next one requested with the next weights.  More: one set,
    // each tile requested again when its products are issued (MT - 1 tiles' products ahead of its next use).
    constexpr int AB = MT <= 2 ? 2 : 1;
    bf16x8 w[2][TNE], h[AB][MT];
    u32x2_t l[AB][MT];
    auto kpos = [&](int i) {
        const int r = i + rot, kq = kt0 + (r >= klen ? r - klen : r);
        return (uint32_t)min(kq, KT - 1);                 // (offsets stay inside the buffers also where the walk has ended)
    };
    auto load_w = [&](bf16x8 (&d)[TNE], uint32_t kq, uint32_t oob) {
#pragma unroll
        for (int j = 0; j < G; ++j)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
                d[j * TN + tn] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                    wr, lane * 16 + oob, goff[j] + ((kq * TN + tn) << 10), 2));         // (2: non-temporal)
    };
    auto load_a = [&](int b, int mt, uint32_t kq, uint32_t oob) {
        const uint32_t tix = mt * KT + kq;
        h[b][mt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(xr, lane * 16 + oob, tix << 10, 0));
        l[b][mt] = __builtin_amdgcn_raw_buffer_load_b64(xr, lane * 8 + oob, lo_base + (tix << 9), 0);
    };
    auto step = [&](int i, int cur) {
        const uint32_t kn = kpos(i + 1), oob = i + 1 < klen ? 0u : SPAN_OOB;
        load_w(w[cur ^ 1], kn, oob);
        if constexpr (AB == 2) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) load_a(cur ^ 1, mt, kn, oob);
        }
        __builtin_amdgcn_sched_barrier(0);
        const int b = AB == 2 ? cur : 0;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            const bf16x8 bh = h[b][mt], bl = lo_by_perm(h[b][mt], l[b][mt]);
#pragma unroll
            for (int t = 0; t < TNE; ++t) acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[cur][t], bh, acc[mt][t], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < TNE; ++t) acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[cur][t], bl, acc[mt][t], 0, 0, 0);
            if constexpr (AB == 1) { __builtin_amdgcn_sched_barrier(0); load_a(0, mt, kn, oob); __builtin_amdgcn_sched_barrier(0); }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    {
        const uint32_t k0 = kpos(0), oob = klen > 0 ? 0u : SPAN_OOB;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) load_a(0, mt, k0, oob);
        load_w(w[0], k0, oob);
    }
    __builtin_amdgcn_sched_barrier(0);
    // what the epilogue needs of this wave's fragments besides their sums: requested here, or pass by pass where there
    // are too many of them to hold
    constexpr bool EARLY = !SLICED && NCH * FPW <= 4;
    constexpr int NPRE = (EARLY ? NCH : 1) * FPW;
    EpiPre pre[NPRE];
    auto load_pre = [&](int ch0) {
        int pm[NPRE], pn[NPRE];
#pragma unroll
        for (int i = 0; i < NPRE; ++i) {
            const int f = min((ch0 + i / FPW) * FC + wave * FPW + i % FPW, F - 1);
            pm[i] = f / TNE * 16 + c; pn[i] = min((int)blockIdx.x * TNE + f % TNE, NT - 1) * 16 + g * 4;
        }
        preload_epilogue<EPI, NPRE>(ep, N, pm, pn, pre);
    };
    if constexpr (EARLY) load_pre(0);
    if constexpr (NORM) {
        float t = 0.f;
#pragma unroll
        for (int j = 0; j < PJ; ++j)
            t += sl + j * TPT < NQ ? (pr[j][0] + pr[j][1]) + (pr[j][2] + pr[j][3]) : 0.f;
        for (int i = sl + PJ * TPT; i < NQ; i += TPT) { const f32x4 v = pp[i]; t += (v[0] + v[1]) + (v[2] + v[3]); }
#pragma unroll
        for (int o = TPT / 2; o > 0; o >>= 1) t += __shfl_xor(t, o);
        if (sl == 0 && tok < MT * 16) rs[tok] = rsqrtf(t / (float)K + eps);
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int i = 0; i < klen; i += 2) { step(i, 0); step(i + 1, 1); }           // (an odd walk ends with a step of zeros)

    // add the waves' sums in wave order
    f32x4 own[SLICED ? NCH * FPW : 1];
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
        if (ch) __syncthreads();
        if constexpr (!EARLY && !SLICED) load_pre(ch);
#pragma unroll
        for (int i = 0; i < FC; ++i)
            if (ch * FC + i < F) red[wave][i][lane] = acc[(ch * FC + i) / TNE][(ch * FC + i) % TNE];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FPW; ++i) {
            const int fi = wave * FPW + i, f = ch * FC + fi, tile = blockIdx.x * TNE + f % TNE;
            if (fi < FC && f < F && tile < NT) {
                f32x4 v = red[0][fi][lane];
#pragma unroll
                for (int k = 1; k < WK; ++k) v += red[k][fi][lane];
                if constexpr (SLICED) {
                    own[ch * FPW + i] = v;
                } else {
                    const int m = f / TNE * 16 + c;
                    if constexpr (NORM) v *= rs[m];
                    apply_epilogue<EPI>(ep, N, m, tile * 16 + g * 4, v, pre[(EARLY ? ch : 0) * FPW + i]);
                }
            }
        }
    }
    if constexpr (SLICED) {
        // The slices' sums meet in the workgroup of a column that arrives last.  Records are written through to memory and
        // read from there (no fence: a write-back of the XCD's L2 costs 20 us), each wave waits for its own stores, then the
        // workgroup takes a ticket; nobody waits for anybody.  Slices are added in slice order, whoever is last.
        constexpr int NV = NCH * FPW;
        const int KS = gridDim.y, me = blockIdx.y;
        const __amdgpu_buffer_rsrc_t pb = __builtin_amdgcn_make_buffer_rsrc(part + (size_t)blockIdx.x * KS * F * 256, 0, KS * F << 10, 0x00020000);
        int vf[NV];                               // this wave's fragments (F: none)
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int fi = wave * FPW + i % FPW, f = i / FPW * FC + fi;
            vf[i] = fi < FC && f < F && (int)blockIdx.x * TNE + f % TNE < NT ? f : F;
            if (vf[i] < F) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, own[i]), pb, lane * 16, (me * F + f) << 10, SPAN_AGENT);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);            // this wave's records have reached memory
        __syncthreads();
        if (threadIdx.x == 0) arrived = __hip_atomic_fetch_add(tickets + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (arrived != (uint32_t)KS - 1) return;
        f32x4 q[NV][KSM];
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int k = 0; k < KSM; ++k)
                q[i][k] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                    pb, lane * 16 + (k < KS && k != me && vf[i] < F ? 0u : SPAN_OOB), (min(k, KS - 1) * F + min(vf[i], F - 1)) << 10, SPAN_AGENT));
        int pm[NV], pn[NV];
        EpiPre e[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int f = min(vf[i], F - 1);
            pm[i] = f / TNE * 16 + c; pn[i] = min((int)blockIdx.x * TNE + f % TNE, NT - 1) * 16 + g * 4;
        }
        preload_epilogue<EPI, NV>(ep, N, pm, pn, e);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (vf[i] == F) continue;
            f32x4 v = me == 0 ? own[i] : q[i][0];
#pragma unroll
            for (int k = 1; k < KSM; ++k) v += k == me ? own[i] : q[i][k];      // (slices behind the last one: zeros)
            if constexpr (NORM) v *= rs[pm[i]];
            apply_epilogue<EPI>(ep, N, pm[i], pn[i], v, e[i]);
        }
        if (threadIdx.x == 0) __hip_atomic_store(tickets + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------------------------
template <int MT, int TN, int G>
static int launch_span_t(const SjdLinear *lin, const void *act, const float *ssq_in, float eps, const SjdGemmEpi &ep, hipStream_t s)
{
    constexpr int WK = MT * TN * G <= 24 ? 8 : 4;         // (eight waves of 256 registers or four of 512)
    const int NT = lin->N / 16;
    const dim3 grid((NT + TN * G - 1) / (TN * G)), block(64 * WK);
    const bf16_t *W = (const bf16_t *)lin->w;
#define GO(EPI, NORM) SJD_LAUNCH((gemm_span_kernel<MT, TN, G, WK, EPI, NORM, 1>), grid, block, 0, s, W, act, ssq_in, eps, lin->N, lin->K, 0, (float *)nullptr, (uint32_t *)nullptr, ep)
    if (ssq_in) {
        switch (ep.kind) {
            case SJD_EPI_STORE: GO(SJD_EPI_STORE, true); break;
            case SJD_EPI_SILU: GO(SJD_EPI_SILU, true); break;
            case SJD_EPI_QKV: GO(SJD_EPI_QKV, true); break;
            default: return SJD_EINVAL;
        }
    } else {
        switch (ep.kind) {
            case SJD_EPI_STORE: GO(SJD_EPI_STORE, false); break;
            case SJD_EPI_RESID: GO(SJD_EPI_RESID, false); break;
            default: return SJD_EINVAL;
        }
    }
#undef GO
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

template <int MT, int G, int KSM>
static int launch_sliced_t(const SjdLinear *lin, const void *act, const SjdGemmEpi &ep, int ks, const SjdPartials &part, hipStream_t s)
{
    const int cols = (lin->N / 16 + G - 1) / G, kps = (lin->K / 32 + ks - 1) / ks;
    ks = (lin->K / 32 + kps - 1) / kps;
    if (ks > KSM || cols > SJD_TICKETS || !part.sums || !part.tickets || (size_t)cols * ks * MT * G * 256 > part.elems) return SJD_EINVAL;
#define GO(EPI) SJD_LAUNCH((gemm_span_kernel<MT, 1, G, 8, EPI, false, KSM>), dim3(cols, ks), dim3(512), 0, s, (const bf16_t *)lin->w, act, \
                           (const float *)nullptr, 0.f, lin->N, lin->K, kps, part.sums, part.tickets, ep)
    switch (ep.kind) {
        case SJD_EPI_STORE: GO(SJD_EPI_STORE); break;      // (test hooks)
        case SJD_EPI_RESID: GO(SJD_EPI_RESID); break;
        default: return SJD_EINVAL;
    }
#undef GO
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

int sjd_launch_gemm_sliced(const SjdLinear *lin, const void *act, int32_t rows, const SjdGemmEpi &ep, int g, int ks,
                           const SjdPartials &part, hipStream_t s)
{
    if (rows < 1 || rows > SJD_ROWS_MAX || lin->tn != 1 || lin->N % 16 || lin->K % 32 || lin->K > SPAN_K_MAX || ks < 1) return SJD_EINVAL;
    if (ep.kind == SJD_EPI_RESID && ep.out24 && (!ep.gain_next || !ep.ssq_out)) return SJD_EINVAL;
    int mt = (rows + 15) / 16;
    if (mt > 4) mt = (mt + 1) & ~1;
#define CASE(MT, G, KSM) if (mt == MT && g == G && ks <= KSM) return launch_sliced_t<MT, G, KSM>(lin, act, ep, ks, part, s)
    CASE(1, 2, 8); CASE(2, 2, 8); CASE(3, 2, 8); CASE(4, 2, 8); CASE(6, 2, 8); CASE(8, 2, 8);
    CASE(3, 4, 4); CASE(4, 4, 4);
    CASE(1, 8, 8); CASE(2, 8, 8);
#undef CASE
    return SJD_EINVAL;
}

// packed weight groups per workgroup: one workgroup per CU where six tiles a workgroup allow it (eight waves hold the sums of
// 24 fragments and two k-steps of operands in 256 registers each, four waves 48 in 512)
int sjd_span_groups(const SjdLinear *lin)
{
    const int groups = lin->N / 16 / lin->tn;
    return std::max(1, std::min((groups + 255) / 256, 6 / lin->tn > 3 ? 3 : 6 / lin->tn));
}

// Which projections are cut into K-slices here, and how: G groups of one tile a workgroup, KS slices.  O and down only (their
// output is added to the residual stream), where a workgroup with all of K reads more activations than weights or CUs stay
// without a workgroup:
//  - 256 tiles and more, long K (7B down), up to 32 rows: 8 x 8 cuts the activations a workgroup reads to an eighth.  16 rows inside
//    a forward 20.7 us (skinny kernel) -> 19.0, 32 rows 19.4 + 5.3 (wide kernel and its second) -> 21.9.  At 64 rows the last
//    workgroup's share grows: 22 + 5.2 -> 27.9, so the wide kernel keeps those.
//  - 256 tiles and more, other K (7B O), 33 to 64 rows: 4 x 4; forward of 2 x 32 rows 4251 -> 4202 us, prompt of 64 3880 -> 3808.
//    At 128 rows it loses (5962 -> 5994), up to 32 the skinny kernel alone needs 8.2 and 10.8 us, sliced 9.9 and 11.1.
//  - fewer tiles (775M, 96 of them for 256 CUs): 2 x 4.  down at 16, 64, 121 rows 8.1 -> 7.0, 7.4 + 4.1 -> 8.3, 10.1 + 5.1 -> 12.4 us, O at
//    64 rows 8.7 -> 8.3; O up to 32 rows is faster whole (4.3 us alone against 5.0), and so is what has fewer than 72 k-steps:
//    512 x 2048 at 16 rows alone skinny 4.8, sliced 5.5, x 2304 5.4 and 5.3.
//  - more than 128 of them leave two slices, 2 x 2, and a long share of the activations for each: alone, wide kernel and sliced, 3072 x
//    3072 10.7 and 10.7 us at 64 rows, 12.2 and 13.8 at 96; long K, 3072 x 8192 20.8 and 18.7 at 48 rows, 20.8 and 21.4 at 64, 25.3 and 32.6
//    at 128, 3584 x 18944 44.9 and 40.0, 45.0 and 46.8, 46.4 and 72.4.  So up to 64 rows, with a long K up to 48.
bool sjd_sliced_plan(const SjdLinear *lin, int32_t rows, int *g, int *ks)
{
    const int tiles = lin->N / 16, KT = lin->K / 32;
    const bool longk = lin->K >= 2 * lin->N, few = rows <= SJD_ROWS_SKINNY;
    *g = *ks = 1;
    if (!lin->resid || lin->tn != 1 || lin->K > SPAN_K_MAX) return false;
    if (tiles >= 256) {
        if (longk ? !few : few || rows > 64) return false;
        *g = *ks = longk ? 8 : 4;
    } else {
        if (few ? !longk || KT < 72 : tiles > 128 && rows > (longk ? 48 : 64)) return false;
        *g = 2;
        *ks = 512 / tiles >= 8 ? 8 : 512 / tiles >= 4 ? 4 : 2;
    }
    while (*ks > 1 && KT / *ks < 8) *ks /= 2;             // (a k-step for every wave)
    return *ks > 1 && (tiles + *g - 1) / *g <= SJD_TICKETS;
}

// floats of slices' sums of such a projection at most, over all row counts
size_t sjd_sliced_elems(const SjdLinear *lin)
{
    size_t most = 0;
    for (int rows = 16; rows <= SJD_ROWS_MAX; rows += 16) {
        int g, ks;
        if (sjd_sliced_plan(lin, rows, &g, &ks)) most = std::max(most, (size_t)((lin->N / 16 + g - 1) / g) * ks * (rows / 16 + 1) * g * 256);       // (row tiles in pairs)
    }
    return most;
}

// Which projections come here.  Up to 32 rows: those that leave the skinny kernel with two or more workgroups per CU (7B
// gate/up above; the LM head of the 775M model 10.5 -> 10.7 us alone at 16 rows, 13.4 -> 12.0 at 32).  More rows: the
// alternative is the wide kernel, which reads the activations once for eight tiles but pays a second kernel (4-5 us) and the
// slices' traffic.  With three tiles or more per workgroup reading all activations is the smaller price (7B QKV inside a forward: 64 rows
// 28.6 us against 23.3 + 8.2, 128 rows 43.8 against 30.4 + 12.3; forwards of 64 and 128 rows 1.2 % and 1.1 % faster);
// with fewer, as long as they are few bytes: all 775M projections but down (K = 1536; 295 KB at 64 rows, 590 at 128) gain
// 14 % of a forward of 64 rows and 5 % of one of 121; 7B O at 64 rows (786 KB) makes its forward 1.7 % slower.
//
// Only with one workgroup per CU: more of them are a second round that is mostly empty, each reading all activations again.
// One projection alone on cold weights, skinny or wide kernel and span:
//  - 32768 x 4096, 342 workgroups: 16 rows 42.9 and 50.3 us, 64 rows 58.9 and 67.2, 128 rows 73.9 and 102.7
//  - 27648 x 5120 in one-tile groups, 576: 64 rows 69.3 and 81.7, 128 rows 93.9 and 124.8; forwards of two such layers (d = 5120,
//    8192 logits) of 64, 96 and 128 rows had become 449, 570 and 701 us, 437, 531 and 626 before
// Two-tile groups at 17 to 32 rows are the exception: 32768 x 4096 53.3 and 55.2, x 7168 100.8 and 94.7, 57344 x 8192 187.7 and 172.3.
// Nor above 64 rows of 8192 features and more (2.4 MB of activations for every workgroup at 96 rows): 24576 x 8192 alone 72.3 and 73.1 us at 64 rows, 79.7 and 86.5 at 96, 95.5 and 101.1 at 128; 16384 x 8192 at 128 73.6 and 86.6; 21504 x 7168 97.1 and 86.4.
// Nor, above 96 rows, four tiles a workgroup with 3072 features and more: their 32 fragments leave four waves a workgroup, for two thirds of
// the weights that six tiles give it.  Forwards of two layers at 128 rows, wide kernel and span: d = 3072 (gate/up) 289 and 294 us, with 16384
// logits 301 and 310; d = 4096 with 16384 logits 399 and 406; d = 5120 (QKV) 592 and 600.  At 80 and 96 rows (eight waves) the
// span kernel is up to 3 % of such a forward ahead; alone 16384 x 2048 at 128 rows 30.4 and 25.6.
bool sjd_span_takes(const SjdLinear *lin, int32_t rows)
{
    const int groups = lin->N / 16 / lin->tn, g = sjd_span_groups(lin), tiles = g * lin->tn;
    const bool one_round = (groups + g - 1) / g <= 256;
    if (lin->K > SPAN_K_MAX) return false;
    if (rows <= SJD_ROWS_SKINNY) return groups >= 512 && tiles >= 4 && (one_round || (rows > 16 && lin->tn == 2));
    if (rows > 96 && tiles == 4 && lin->K >= 3072) return false;
    const int64_t act = (int64_t)((rows + 15) / 16 * 16) * lin->K * 3;
    return one_round && (rows <= 64 || lin->K < 8192) && (tiles >= 3 || act <= 600 * 1024);
}

int sjd_launch_gemm_span(const SjdLinear *lin, const void *act, const float *ssq_in, float eps, int32_t rows,
                         const SjdGemmEpi &ep, hipStream_t s)
{
    if (rows < 1 || rows > SJD_ROWS_MAX || lin->tn < 1 || lin->tn > 3 || lin->N % (16 * lin->tn) || lin->K % 32 || lin->K > SPAN_K_MAX) return SJD_EINVAL;
    if (ep.kind == SJD_EPI_RESID && ep.out24 && (!ep.gain_next || !ep.ssq_out)) return SJD_EINVAL;
    const int tn = lin->tn, g = sjd_span_groups(lin);
    int mt = (rows + 15) / 16;
    if (mt > 4) mt = (mt + 1) & ~1;                       // variants for 16, 32, 48, 64, 96 and 128 rows
#define CASE(MT, TN, G) if (mt == MT && tn == TN && g == G) return launch_span_t<MT, TN, G>(lin, act, ssq_in, eps, ep, s)
#define FEW(TN, G) CASE(1, TN, G); CASE(2, TN, G)        // (what sjd_span_takes lets through up to 32 rows)
#define MORE(TN, G) CASE(3, TN, G); CASE(4, TN, G); CASE(6, TN, G); CASE(8, TN, G)
    FEW(2, 2); FEW(2, 3); FEW(3, 2);
    MORE(1, 1); MORE(1, 2); MORE(1, 3);
    MORE(2, 1); MORE(2, 2); MORE(2, 3);
    MORE(3, 1); MORE(3, 2);
#undef FEW
#undef MORE
#undef CASE
    return SJD_EINVAL;
}

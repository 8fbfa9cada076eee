// bf16 projections of a window forward with MORE than 32 rows (paper Sec. 4.1 Step 2 for windows of 64
// tokens, for guided windows of 32 -- two contexts -- and for batches of images that share one pass
// over the weights): C[M x N] = A[M x K] * W^T, M = 33 .. 128, for the shapes and rows that the span kernel does not take, whole
// or in slices (of the 7B model down above 32 rows, the LM head above 48, O above 64; of wider models QKV and gate/up too).
//
// With this many rows a workgroup can no longer afford a private copy of the activations per wave (M
// rows cost M * 96 bytes of activations per KiB of weights), so the roles inside a workgroup change
// with respect to the skinny kernel:
//  - the four waves of a workgroup split N: each streams its own packed
//    weight groups (the same layout the skinny kernel reads: every weight byte still leaves HBM once and
//    goes straight into the registers of the one wave that uses it);
//  - all of them walk the SAME k-steps, and the activation tiles of a stage of k-steps are staged in LDS by
//    the workgroup and read from there by every wave: L2 -> CU activation traffic drops by the number of
//    waves.  The producers of a wide forward's activations write the second operand ready made (2-byte lo
//    plane), so staging is a copy;
//  - K is split across workgroups (grid.y) wherever N alone gives too few of them; every workgroup
//    writes its fp32 sums as whole accumulator fragments, and a second kernel adds the K-slices in
//    slice order (deterministic), applies the token factors of a folded RMSNorm and runs the same
//    epilogues as the skinny kernel (residual, SiLU * up, RoPE + cache write, plain store).  (Adding the
//    slices in the last workgroup to arrive behind device-scope fences was measured 3x slower: they write back and
//    invalidate the L2 of the XCD.  The sliced spans do it without a fence, where few slices of few rows meet.)
// At M = 128 the two MFMAs per weight tile and M-tile price the matrix cores at about 9.8 TB/s of
// weights; measured, the kernel runs at about 30 % of the bf16 MFMA peak there: the one regime of this path where
// matrix-core utilisation is a meaningful number.  What bounds it is known in part only: at 128 rows the CUs fill their
// L1s from L2 with 10.1 TB/s, as the skinny kernel does at 32, but half the activation traffic (eight waves per
// workgroup) gained 3 % on gate/up and lost elsewhere; at 64 rows they fill with 6.2, and LDS waits are 1 and 6 % of wave time.
#include "sjd_gemm_epi.h"

#include <algorithm>
#include <mutex>

// one pipeline stage = KU k-steps; LDS holds two stages of MT activation tiles as hi and lo operands
#define WIDE_WAVES 4

template <int MT, int TN, int G, int KU, int NW>
__global__ __launch_bounds__(64 * NW, 2) void gemm_wide_kernel(const bf16_t *__restrict__ Wp,
                                                            const void *__restrict__ Xv, int N, int K, int kps,
                                                            f32x4 *__restrict__ part)
{
    constexpr int TNE = TN * G;               // 16-feature tiles per wave
    constexpr int TPS = KU * MT;              // activation tiles per stage
    constexpr int APT = TPS / NW;             // of which each wave fetches
    static_assert(TPS % NW == 0 && APT >= 1, "the waves share the staging of a stage evenly");
    extern __shared__ bf16x8 act_lds[];       // [2 stages][KU][MT][plane][64 lanes]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int KT = K / 32, NT = N / 16, groups = NT / TN;
    const int k0 = blockIdx.y * kps, k1 = min(KT, k0 + kps);

    const bf16x8 *xp = reinterpret_cast<const bf16x8 *>(Xv) + lane;
    const bf16x8 *xl = reinterpret_cast<const bf16x8 *>(reinterpret_cast<const char *>(Xv) + act24_lo_base(KT)) + lane;   // 2-byte lo plane
    const size_t ztile = (size_t)SJD_MTILES * KT;        // the all-zero tile behind every activation matrix
    const bf16x8 *zw = xp + ztile * 64;
    if ((int)blockIdx.x * NW * G >= groups) return;      // (a column group added by rounding the grid up)
    // this wave's packed weight groups (a group past the end reads the zero tile and stores nothing)
    const bf16x8 *wp[G];
    int grp[G];
#pragma unroll
    for (int j = 0; j < G; ++j) {
        grp[j] = (blockIdx.x * NW + wave) * G + j;
        wp[j] = grp[j] < groups ? reinterpret_cast<const bf16x8 *>(Wp) + (size_t)grp[j] * KT * TN * 64 + lane : nullptr;
    }

    f32x4 acc[MT][TNE];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int t = 0; t < TNE; ++t) acc[mt][t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // Weights: a ring of WD stages in registers, requested WD - 1 stages ahead of their use (a stage is
    // KU k-steps; HBM latency under load is several stages long).  Activations: both operand planes come
    // ready made (the forward's producers write the 2-byte lo plane), so a stage is requested from L2 one
    // stage ahead into registers and parked in LDS, tile by tile, between the products of the stage before.
    // stages of weights in registers: four, three or two, at most 32 weight tiles (128 registers) in all
    constexpr int WD = KU * TNE <= 4 ? 4 : KU * TNE <= 8 ? 3 : 2;
    bf16x8 a_[WD][KU][TNE];
    bf16x8 sh_[APT], sl_[APT];

    // All loads are unconditional: a k-step past this workgroup's slice fetches the zero tile.
#define LOAD_ACT(kbase)                                                                               \
    _Pragma("unroll") for (int i = 0; i < APT; ++i) {                                                 \
        const int ti_ = i * NW + wave, u_ = ti_ / MT, mt_ = ti_ % MT, kk_ = (kbase) + u_;             \
        const size_t tix_ = kk_ < k1 ? (size_t)mt_ * KT + kk_ : ztile;                                \
        sh_[i] = xp[tix_ * 64];                                                                       \
        sl_[i] = xl[tix_ * 64];                                                                       \
    }
#define PARK_TILE(buf, i)                                                                             \
    {                                                                                                 \
        const int ti_ = (i) * NW + wave, u_ = ti_ / MT, mt_ = ti_ % MT;                               \
        bf16x8 *dst_ = act_lds + ((((buf) * KU + u_) * MT + mt_) * 2) * 64 + lane;                    \
        dst_[0] = sh_[i];                                                                             \
        dst_[64] = sl_[i];                                                                            \
    }
#define STORE_ACT(buf) _Pragma("unroll") for (int i = 0; i < APT; ++i) PARK_TILE(buf, i)
#define LOAD_W(a, kbase)                                                                              \
    _Pragma("unroll") for (int u = 0; u < KU; ++u) {                                                  \
        const int kk_ = (kbase) + u;                                                                  \
        _Pragma("unroll") for (int j = 0; j < G; ++j)                                                 \
            _Pragma("unroll") for (int tn = 0; tn < TN; ++tn)                                         \
                a[u][j * TN + tn] = __builtin_nontemporal_load(                                       \
                    (kk_ < k1 && wp[j]) ? wp[j] + ((size_t)kk_ * TN + tn) * 64 : zw);                 \
    }
    // One stage of products.  The operand pairs of the STEPS = KU * MT (k-step, M-tile) steps are fetched from
    // LDS PD steps ahead of the MFMAs that use them, through a ring of PD + 1 register pairs, and the parking
    // of the next stage's activations is spread over the last steps (by then its loads have landed): a
    // scheduling barrier after every step keeps this order in the instruction stream (left to itself the
    // compiler reuses one register pair and waits for every LDS read in turn).
#define COMPUTE_AND_PARK(a, buf, buf_store)                                                           \
    {                                                                                                 \
        constexpr int STEPS = KU * MT, PD = STEPS < 3 ? STEPS : 3;                                    \
        bf16x8 bq_[PD + 1][2];                                                                        \
        const bf16x8 *base_ = act_lds + (size_t)(buf) * STEPS * 128 + lane;                           \
        _Pragma("unroll") for (int p = 0; p < PD; ++p) { bq_[p][0] = base_[p * 128]; bq_[p][1] = base_[p * 128 + 64]; } \
        _Pragma("unroll") for (int st = 0; st < STEPS; ++st) {                                        \
            if (st + PD < STEPS) {                                                                    \
                bq_[(st + PD) % (PD + 1)][0] = base_[(st + PD) * 128];                                \
                bq_[(st + PD) % (PD + 1)][1] = base_[(st + PD) * 128 + 64];                           \
            }                                                                                         \
            const int u = st / MT, mt = st % MT;                                                      \
            _Pragma("unroll") for (int t = 0; t < TNE; ++t) {                                         \
                acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][t], bq_[st % (PD + 1)][0], acc[mt][t], 0, 0, 0); \
                acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][t], bq_[st % (PD + 1)][1], acc[mt][t], 0, 0, 0); \
            }                                                                                         \
            if (st >= STEPS - APT) PARK_TILE(buf_store, st - (STEPS - APT))                           \
            __builtin_amdgcn_sched_barrier(0);                                                        \
        }                                                                                             \
    }
    // Round r (stage r at k-steps kt .. kt + KU): request stage r + 1's activations and stage r + WD - 1's
    // weights, multiply stage r from LDS buffer r % 2 and park stage r + 1's activations in the other
    // buffer.  The barrier at the end of a round orders "every wave has read buffer b" before "buffer b is
    // overwritten" one round later, and "buffer b ^ 1 is written" before it is read in the next round.
    // prologue: stage 0 of the activations, stages 0 .. WD - 2 of the weights; stage 0 into buffer 0
    LOAD_ACT(k0)
#pragma unroll
    for (int r = 0; r < WD - 1; ++r) LOAD_W(a_[r], k0 + r * KU)
    STORE_ACT(0)
    __syncthreads();
    constexpr int PERIOD = WD % 2 ? 2 * WD : WD;      // rounds after which both ring positions repeat
    for (int kt = k0; kt < k1;) {
#pragma unroll
        for (int r = 0; r < PERIOD; ++r) {
            LOAD_ACT(kt + KU)
            LOAD_W(a_[(r + WD - 1) % WD], kt + (WD - 1) * KU)
            __builtin_amdgcn_sched_barrier(0);
            COMPUTE_AND_PARK(a_[r % WD], r & 1, (r + 1) & 1)
            __syncthreads();
            kt += KU;
            if (kt >= k1) break;
        }
    }
#undef LOAD_ACT
#undef STORE_ACT
#undef PARK_TILE
#undef LOAD_W
#undef COMPUTE_AND_PARK

    // fp32 sums of this K-slice, as whole accumulator fragments: [slice][m tile][n tile][lane]
#pragma unroll
    for (int j = 0; j < G; ++j) {
        if (grp[j] >= groups) continue;
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int ntile = grp[j] * TN + tn;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                part[(((size_t)blockIdx.y * MT + mt) * NT + ntile) * 64 + lane] = acc[mt][j * TN + tn];
        }
    }
}

// Second kernel: adds the K-slices of every accumulator fragment in slice order, applies
// rsqrt(mean(x^2) + eps) of each token when an RMSNorm is folded into the projection (PRO_NORM: the
// planes held x * gain and ssq_in the per-16-feature sums of squares of x), and runs the epilogue.
// Workgroup (x, mt): M-tile mt, the `ft` n tiles of column group x, one per wave; lane l of a wave holds features
// 16 ntile + 4 (l / 16) .. + 4 of token 16 mt + l % 16, exactly as the MFMA left them.  What it costs is latency: a
// launch, one round of loads, the stores.  So everything (up to QS slices, the epilogue's operands, the sums of
// squares) is requested before anything is used: sixteen slices where there are more than four (775M down projection 4.65 -> 4.1 us
// a launch), else four, so that 64 registers are enough and two workgroups of 1024 threads share a CU (sixteen for all: 94;
// gate/up of 44032 features at 96 rows 11.6 -> 16.9 us, of 32768 at 128 11.4 -> 16.0); and the workgroups are cut like those of the first kernel: with both
// grids a multiple of eight column groups wide, a group's slices and its epilogue meet in one XCD's L2.
template <int EPI, int PRO, int QS>
__global__ __launch_bounds__(1024) void gemm_wide_epilogue_kernel(const f32x4 *__restrict__ part, int KS, int MT, int NT,
                                                                 const float *__restrict__ ssq_in, float eps, int N, int K,
                                                                 SjdGemmEpi ep)
{
    __shared__ float rs[16];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, c = lane & 15;
    const int ft = blockDim.x >> 6, mt = blockIdx.y;
    if ((int)blockIdx.x * ft >= NT) return;                                    // (a column group added by rounding up)
    const int nt = blockIdx.x * ft + wave, ntile = min(nt, NT - 1);            // (past the end: the last tile, not written)
    const f32x4 *p = part + ((size_t)mt * NT + ntile) * 64 + lane;
    const size_t step = (size_t)MT * NT * 64;                     // from one slice to the next
    f32x4 q[QS];
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = p[(size_t)min(i, KS - 1) * step];
#pragma unroll
    for (int i = 4; i < QS; i += 4) {
        if (i >= KS) break;
#pragma unroll
        for (int j = i; j < i + 4; ++j) q[j] = p[(size_t)min(j, KS - 1) * step];
    }
    const int f_m = mt * 16 + c, f_n0 = ntile * 16 + g * 4;
    EpiPre pre;
    preload_epilogue<EPI>(ep, N, f_m, f_n0, pre);
    if (PRO == SJD_PRO_NORM) {
      if (threadIdx.x < 256) {
        // 16 threads per token add every 16th float4 of its row of partial sums, then fold
        const int tok = threadIdx.x >> 4, sl = threadIdx.x & 15;
        const int NQ = ssq_stride(K) / 4;
        const f32x4 *pp = reinterpret_cast<const f32x4 *>(ssq_in + (size_t)(mt * 16 + tok) * (NQ * 4));
        float t = 0.f;
#pragma unroll 4
        for (int i = sl; i < NQ; i += 16) { const f32x4 v = pp[i]; t += (v[0] + v[1]) + (v[2] + v[3]); }
        t += __shfl_xor(t, 8);
        t += __shfl_xor(t, 4);
        t += __shfl_xor(t, 2);
        t += __shfl_xor(t, 1);
        if (sl == 0) rs[tok] = rsqrtf(t / (float)K + eps);
      }
      __syncthreads();
    }
    f32x4 v = q[0];
#pragma unroll
    for (int i = 1; i < QS; ++i) if (i < KS) v += q[i];
    for (int y = QS; y < KS; ++y) v += p[(size_t)y * step];
    if (PRO == SJD_PRO_NORM) v *= rs[c];
    if (nt < NT) apply_epilogue<EPI>(ep, N, f_m, f_n0, v, pre);
}

// ---------------------------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------------------------
static std::mutex g_wide_mutex;
static size_t g_wide_lds[5][4][3] = {};      // dynamic LDS already enabled per (MT/2, TN, G) instantiation

// k-steps per stage: 16 (k-step, M-tile) products between two workgroup barriers whatever the row count (a
// stage of few products would spend its time in the barrier); half of that where a wave holds 3 or 4 weight
// tiles per k-step
constexpr int wide_ku(int MT, int TNE) { return MT == 2 ? (TNE >= 3 ? 4 : 8) : MT == 4 ? (TNE >= 3 ? 2 : 4) : 2; }
#define WIDE_KU wide_ku(MT, TN * G)
template <int MT, int TN, int G>
static int enable_lds_t()
{
    const size_t lds = (size_t)2 * WIDE_KU * MT * 2 * 1024;
    if (lds <= 48 * 1024) return SJD_OK;
    std::lock_guard<std::mutex> lock(g_wide_mutex);
    if (g_wide_lds[MT / 2][TN][G] < lds) {
        HIP_TRY(hipFuncSetAttribute((const void *)gemm_wide_kernel<MT, TN, G, WIDE_KU, WIDE_WAVES>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
        g_wide_lds[MT / 2][TN][G] = lds;
    }
    return SJD_OK;
}

// Dynamic LDS above the default limit has to be enabled per kernel; done when a cache handle is created,
// so that launches recorded during graph capture never touch function attributes.
int sjd_gemm_wide_setup()
{
    SJD_TRY((enable_lds_t<8, 1, 1>())); SJD_TRY((enable_lds_t<8, 1, 2>())); SJD_TRY((enable_lds_t<8, 2, 1>()));
    SJD_TRY((enable_lds_t<8, 2, 2>())); SJD_TRY((enable_lds_t<8, 3, 1>()));
    SJD_TRY((enable_lds_t<4, 1, 1>())); SJD_TRY((enable_lds_t<4, 1, 2>())); SJD_TRY((enable_lds_t<4, 2, 1>()));
    SJD_TRY((enable_lds_t<2, 1, 1>())); SJD_TRY((enable_lds_t<2, 1, 2>())); SJD_TRY((enable_lds_t<2, 2, 1>()));
    return SJD_OK;
}

// Column groups of both kernels' grids.  Workgroup i of a launch runs on XCD i % 8: with a multiple of eight column
// groups the K-slices of a group and its epilogue share an L2, so the count is rounded up (the added workgroups return
// at once) where all workgroups of the first kernel are resident together, one per CU, and there are 32 groups or more.
// Both kernels together, alone on cold weights, not rounded and rounded:
//   12848 x 640, 101 groups x 2 slices: 12.4 -> 10.6 us at 64 rows, 18.9 -> 14.5 at 128
//   30784 x 2048, 121 x 2: 33.7 -> 32.4 at 64 rows; 29504 x 4096, 116 x 2: 49.5 -> 48.5; 25664 x 512, 201 x 2: not resident, as before
//   few groups, 12 of them (O and down of 775M when they ran here): alone 8.5 -> 8.0 and 11.1 -> 10.5, but forwards 1.3 and 1.9 %
//   slower (rounded to 16, four XCDs have two groups and four have one)
static int wide_cols(int groups, int g, int ks)
{
    const int cols = (groups + WIDE_WAVES * g - 1) / (WIDE_WAVES * g), up = (cols + 7) & ~7;
    return cols >= 32 && up * ks <= 256 ? up : cols;
}

template <int MT, int TN, int G>
static int launch_wide_t(const SjdLinear *lin, const void *act, int ks, int kps, f32x4 *part, hipStream_t s)
{
    constexpr int KU = WIDE_KU;
    const size_t lds = (size_t)2 * KU * MT * 2 * 1024;
    SJD_TRY((enable_lds_t<MT, TN, G>()));
    const int groups = lin->N / 16 / TN;
    dim3 grid(wide_cols(groups, G, ks), ks);
    SJD_LAUNCH((gemm_wide_kernel<MT, TN, G, KU, WIDE_WAVES>), grid, dim3(64 * WIDE_WAVES), lds, s,
               (const bf16_t *)lin->w, act, lin->N, lin->K, kps, part);
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

template <int MT>
static int launch_wide_mt(const SjdLinear *lin, const void *act, int g, int ks, int kps, f32x4 *part, hipStream_t s)
{
    const int tn = lin->tn;
    if (tn == 1 && g == 1) return launch_wide_t<MT, 1, 1>(lin, act, ks, kps, part, s);
    if (tn == 1 && g == 2) return launch_wide_t<MT, 1, 2>(lin, act, ks, kps, part, s);
    if (tn == 2 && g == 1) return launch_wide_t<MT, 2, 1>(lin, act, ks, kps, part, s);
    if (tn == 2 && g == 2) return launch_wide_t<MT, 2, 2>(lin, act, ks, kps, part, s);
    if (tn == 3 && g == 1) return launch_wide_t<MT, 3, 1>(lin, act, ks, kps, part, s);
    return SJD_EINVAL;
}

// Workgroups and K-slices: every slice at least 8 k-steps long, and the partial sums of all slices inside
// `part_elems` floats.
void sjd_wide_plan(const SjdLinear *lin, int mt, size_t part_elems, int *g_out, int *ks_out, int *kps_out)
{
    const int KT = lin->K / 32, groups = lin->N / 16 / lin->tn;
    // two weight groups per wave: one-tile groups, and two-tile groups of a long N up to 64 rows (at more rows
    // the accumulators of four tiles per M-tile no longer fit the registers)
    int g = lin->wg > 0 ? lin->wg : (lin->tn == 1 || (lin->tn == 2 && mt <= 4 && groups >= 512) ? 2 : 1);
    if (lin->tn == 3) g = 1;
    if (g > 2) g = 2;
    const int wgx = (groups + WIDE_WAVES * g - 1) / (WIDE_WAVES * g);
    // K-slices (measured on the 7B shapes at 64 and 128 rows): about 256 workgroups where N alone gives at
    // most 128 of them; 4 slices up to 256, 2 up to 512 (more slices cost more partial-sum traffic than the
    // extra workgroups win), none above
    int ks = lin->wks > 0 ? lin->wks : wgx >= 512 ? 1 : wgx >= 256 ? 2 : wgx > 128 ? 4 : (256 + wgx - 1) / wgx;
    if (lin->wks <= 0 && lin->tn == 2 && g == 2) ks = 2;      // (measured: 86 wide workgroups x 2 beat x 3 and x 4)
    ks = std::max(1, std::min(ks, KT / 8 > 0 ? KT / 8 : 1));
    const size_t per_slice = (size_t)mt * 16 * lin->N;
    while (ks > 1 && per_slice * ks > part_elems) --ks;
    const int ku = wide_ku(mt, lin->tn * g);
    int kps = (KT + ks - 1) / ks;
    kps = (kps + ku - 1) / ku * ku;             // whole stages
    ks = (KT + kps - 1) / kps;
    *g_out = g; *ks_out = ks; *kps_out = kps;
}

// Floats the K-slices of one layer take at most, over all row counts for which it comes here.  With less room the plan
// above cuts K into fewer slices: fewer workgroups, and longer chains of fp32 sums (128 x 22016 x 4096: 3.97e-7 (2-norm) from
// 64 bits on two slices, 2.80e-7 on four).
size_t sjd_wide_part_elems(const SjdLinear *lin)
{
    size_t most = 0;
    for (int mt = 4; mt <= SJD_MTILES; mt += 2) {         // (up to 32 rows only sjd_gemm_bench comes here)
        if (sjd_span_takes(lin, mt * 16)) continue;       // (and so all row counts of this variant)
        int g, ks, kps;
        sjd_wide_plan(lin, mt, SIZE_MAX, &g, &ks, &kps);
        most = std::max(most, (size_t)mt * 16 * lin->N * ks);
    }
    return most;
}

int sjd_launch_gemm_wide(const SjdLinear *lin, const void *act, const float *ssq_in, float eps, int32_t rows,
                         const SjdGemmEpi &ep, float *part, size_t part_elems, hipStream_t s)
{
    if (rows < 1 || rows > SJD_ROWS_MAX || !part) return SJD_EINVAL;
    if (lin->tn < 1 || lin->tn > 3 || lin->N % (16 * lin->tn) || lin->K % 32) return SJD_EINVAL;
    if (ep.kind == SJD_EPI_RESID && ep.out24 && (!ep.gain_next || !ep.ssq_out)) return SJD_EINVAL;
    int mt = (rows + 15) / 16;
    mt = (mt + 1) & ~1;                          // variants for 32, 64, 96 and 128 rows
    if ((size_t)mt * 16 * lin->N > part_elems) return SJD_EINVAL;
    int g, ks, kps;
    sjd_wide_plan(lin, mt, part_elems, &g, &ks, &kps);
    f32x4 *p4 = reinterpret_cast<f32x4 *>(part);
    int rc;
    switch (mt) {
        case 2: rc = launch_wide_mt<2>(lin, act, g, ks, kps, p4, s); break;
        case 4: rc = launch_wide_mt<4>(lin, act, g, ks, kps, p4, s); break;
        case 6: rc = launch_wide_mt<6>(lin, act, g, ks, kps, p4, s); break;
        default: rc = launch_wide_mt<8>(lin, act, g, ks, kps, p4, s); break;
    }
    SJD_TRY(rc);
    const int NT = lin->N / 16;
    dim3 grid(wide_cols(NT / lin->tn, g, ks), mt);
    const dim3 block(64 * WIDE_WAVES * g * lin->tn);      // 256 .. 1024
#define LAUNCH(EPI, PRO, QS) SJD_LAUNCH((gemm_wide_epilogue_kernel<EPI, PRO, QS>), grid, block, 0, s, p4, ks, mt, NT, ssq_in, eps, lin->N, lin->K, ep)
#define GO(EPI, PRO) do { if (ks <= 4) LAUNCH(EPI, PRO, 4); else LAUNCH(EPI, PRO, 16); } while (0)
    if (ssq_in) {
        switch (ep.kind) {
            case SJD_EPI_STORE: GO(SJD_EPI_STORE, SJD_PRO_NORM); break;
            case SJD_EPI_SILU: GO(SJD_EPI_SILU, SJD_PRO_NORM); break;
            case SJD_EPI_QKV: GO(SJD_EPI_QKV, SJD_PRO_NORM); break;
            default: return SJD_EINVAL;
        }
    } else {
        switch (ep.kind) {
            case SJD_EPI_STORE: GO(SJD_EPI_STORE, SJD_PRO_A24); break;
            case SJD_EPI_RESID: GO(SJD_EPI_RESID, SJD_PRO_A24); break;
            default: return SJD_EINVAL;
        }
    }
#undef GO
#undef LAUNCH
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

// fp32 linear layers of the window forward (paper Sec. 4.1 Step 2) for the small fp32 models:
// C[M x N] = A[M x K] * W^T with plain FMA dot products.  A wave owns one output feature, or the two that its epilogue combines
// (gate and up; the rotated pair of a head), lanes split K.  These models are launch-bound: a launch is a chain of latencies
// of about 4 us whatever it computes, so what stands between two projections is done inside them.  The bf16
// weight-streaming kernel lives in sjd_gemm_bf16.hip.
#include "sjd_internal.h"

#include <algorithm>

// Sums of MR rows over the lanes of a wave: of each pair of lanes one goes on with half of the rows, so that a wave sends
// MR + log2(64 / MR) - 1 values instead of 6 MR; every sum is the tree over lane distances 32, 16 .. 1.  Returns the sum of
// row lane / (64 / MR).
template <int MR>
__device__ __forceinline__ float sum_rows(float (&a)[MR], int lane)
{
    int o = 32;
#pragma unroll
    for (int half = MR / 2; half; half /= 2, o /= 2) {
        const bool up = (lane & o) != 0;
#pragma unroll
        for (int i = 0; i < half; ++i) {
            // (values, chosen between as values: a choice of elements makes the compiler index the array by selects, 4500 of
            // them in the store variant of 32 rows)
            const float lo = a[i], hi = a[i + half];
            a[i] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, o);
        }
    }
#pragma unroll
    for (; o; o /= 2) a[0] += __shfl_xor(a[0], o);
    return a[0];
}

// NORM: A is the residual stream x; every workgroup adds the previous projection's output `add` to its rows and normalises
// them into LDS by itself (a few KB from L2), workgroup 0 leaves the sum in x_out, which is not x: others still read that.
// The sums are those of rmsnorm_kernel, in its order.  With this and the epilogues an iteration of the two-layer model is 14
// launches instead of 23 beside its verification.
template <int MR, int EPI, bool NORM>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ W, const float *__restrict__ A, int N,
                                                       int K, int all_rows, const SjdState *st, SjdGemmF32 ep)
{
    if (st && st->done) return;
    const int row0 = blockIdx.y * MR, rows = min(MR, all_rows - row0);
    A += (size_t)row0 * K;
    constexpr int NF = EPI == SJD_EPI_STORE ? 1 : 2;
    __shared__ float hs[NORM ? SJD_F32_NORM_MAX : 4];
    __shared__ float red[NORM ? MR : 1][4], inv[NORM ? MR : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), units = N / NF;
    const int unit = min((int)blockIdx.x * 4 + wave, units - 1);     // (a wave behind the last unit repeats it and writes nothing)
    const bool mine = (int)blockIdx.x * 4 + wave < units;
    // the features of this wave: f[0], and for SILU its up half, for QKV the other half of the rotated pair
    int f[2] = {unit, unit};
    int sec = 0, c0 = 0, j = 0;                   // QKV: 0 q, 1 k, 2 v; column and dim of the pair's first value
    const int half = EPI == SJD_EPI_QKV ? ep.hd / 2 : 1;      // (a power of two)
    if (EPI == SJD_EPI_SILU) f[1] = units + unit;
    if (EPI == SJD_EPI_QKV) {
        const int d2 = N / 6;
        sec = unit >= 2 * d2 ? 2 : unit >= d2 ? 1 : 0;
        const int e = unit - sec * d2;
        j = e & (half - 1); c0 = 2 * (e - j) + j;
        f[0] = sec * 2 * d2 + c0; f[1] = f[0] + half;
    }
    const float4 *w4[NF];
    float4 w[NF];
#pragma unroll
    for (int t = 0; t < NF; ++t) {
        w4[t] = reinterpret_cast<const float4 *>(W + (size_t)f[t] * K);
        w[t] = w4[t][min(lane, K / 4 - 1)];
    }
    constexpr int LPR = 64 / MR;                  // lanes that hold the sums of a row
    const int r = min(lane / LPR, rows - 1);      // the row whose values this lane finishes
    int pos = 0;
    float cs = 0.f, sn = 0.f;
    if (EPI == SJD_EPI_QKV) {
        pos = state_n(st, ep.stream) + row0 + r;
        cs = ep.cosT[(size_t)pos * half + j]; sn = ep.sinT[(size_t)pos * half + j];
    }
    if constexpr (NORM) {
        float ss[MR];
#pragma unroll
        for (int m = 0; m < MR; ++m) ss[m] = 0.f;
        for (int k0 = 0; k0 < K; k0 += 256) {
            const int k = k0 + (int)threadIdx.x, kc = min(k, K - 1);
            float v[MR];
#pragma unroll
            for (int m = 0; m < MR; ++m) v[m] = A[(size_t)min(m, rows - 1) * K + kc];
            if (ep.add) {
#pragma unroll
                for (int m = 0; m < MR; ++m) v[m] += ep.add[(size_t)(row0 + min(m, rows - 1)) * K + kc];
            }
#pragma unroll
            for (int m = 0; m < MR; ++m)
                if (m < rows && k < K) {
                    hs[m * K + k] = v[m];
                    if (blockIdx.x == 0) ep.x_out[(size_t)(row0 + m) * K + k] = v[m];
                    ss[m] += v[m] * v[m];
                }
        }
        const float t = sum_rows<MR>(ss, lane);
        if (lane % LPR == 0) red[lane / LPR][wave] = t;
        __syncthreads();
        if (threadIdx.x < MR) {
            const float q = red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3];
            inv[threadIdx.x] = rsqrtf(q / (float)K + ep.eps);
        }
        __syncthreads();
        for (int k = threadIdx.x; k < K; k += 256) {
            const float gain = ep.gain[k];
            float v[MR];
#pragma unroll
            for (int m = 0; m < MR; ++m) v[m] = hs[min(m, rows - 1) * K + k] * inv[min(m, rows - 1)] * gain;
#pragma unroll
            for (int m = 0; m < MR; ++m)
                if (m < rows) hs[m * K + k] = v[m];
        }
        __syncthreads();
    }
    float acc[NF][MR];
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
        for (int m = 0; m < MR; ++m) acc[t][m] = 0.f;
    constexpr int RC = MR < 16 ? MR : 16;
    for (int k4 = lane; k4 < K / 4; k4 += 64) {
        if (k4 >= 64) {
#pragma unroll
            for (int t = 0; t < NF; ++t) w[t] = w4[t][k4];
        }
        // The rows' values are requested together, 16 at a time (64 registers): left alone the store variants waited for each
        // row's load by itself.  Two layers of d = 1024, 4096 hidden, 8192 logits at 8, 16 and 32 rows 182, 300 and 605 us, now
        // 123, 166 and 260 (128, 512 and 1024: 64, 73 and 88, now 58, 66 and 81); all 32 at once 269, 8 at a time 273.
#pragma unroll
        for (int m0 = 0; m0 < MR; m0 += RC) {
            float4 a[RC];
#pragma unroll
            for (int m = 0; m < RC; ++m) a[m] = reinterpret_cast<const float4 *>((NORM ? hs : A) + (size_t)min(m0 + m, rows - 1) * K)[k4];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < RC; ++m)
#pragma unroll
                for (int t = 0; t < NF; ++t)
                    acc[t][m0 + m] = fmaf(w[t].x, a[m].x, fmaf(w[t].y, a[m].y, fmaf(w[t].z, a[m].z, fmaf(w[t].w, a[m].w, acc[t][m0 + m]))));
        }
    }
    float v[NF];
#pragma unroll
    for (int t = 0; t < NF; ++t) v[t] = sum_rows<MR>(acc[t], lane);
    if (!mine || lane % LPR || lane / LPR >= rows) return;
    if constexpr (EPI == SJD_EPI_STORE) {
        ep.out[(size_t)(row0 + r) * N + unit] = v[0];
    } else if constexpr (EPI == SJD_EPI_SILU) {
        const float g = v[0], u = v[1];
        ep.out[(size_t)(row0 + r) * units + unit] = g / (1.0f + expf(-g)) * u;
    } else {
        // rotate q and k (pairs j, j + hd/2) at position n + r; q -> qact, k and v -> cache row n + r
        const int d = N / 3, c1 = c0 + half;
        const float a = v[0], b = v[1];
        if (sec == 0) {
            ep.out[(size_t)(row0 + r) * d + c0] = a * cs - b * sn;
            ep.out[(size_t)(row0 + r) * d + c1] = b * cs + a * sn;
        } else if (row0 + r < ep.rows_valid) {
            float *dst = (sec == 1 ? ep.kc : ep.vc) + (size_t)pos * d;
            dst[c0] = sec == 1 ? a * cs - b * sn : a;
            dst[c1] = sec == 1 ? b * cs + a * sn : b;
        }
    }
}

// Rows in blocks of 8 over gridDim.y where the weights fit the L2 of an XCD (4 MB), from where the blocks read them again: no
// chain of sums is then longer than that of 8 rows.  An image of the two-layer model with a window of 32: 5960 us with its own rmsnorm,
// RoPE, SiLU kernels and one workgroup for all rows, 6970 with those folded in and one workgroup for all rows, 3720 so; windows of 16
// 4170, 3970, 3260; of 8 3120 and 2720.
bool sjd_f32_by8(const SjdLinear *lin, int32_t rows) { return rows <= 8 || (size_t)lin->N * lin->K <= (1 << 20); }
// the rows that a workgroup normalises by itself fit its LDS
bool sjd_f32_norm_fits(const SjdLinear *lin, int32_t rows)
{
    return sjd_f32_by8(lin, rows) && (size_t)std::min(rows, 8) * lin->K <= SJD_F32_NORM_MAX;
}

int sjd_launch_gemm_f32(const SjdLinear *lin, const float *act, int32_t rows, const SjdGemmF32 &ep, const SjdState *st, hipStream_t s)
{
    const int N = lin->N, K = lin->K;
    if (rows < 1 || rows > SJD_ROWS_F32 || K % 4) return SJD_EINVAL;
    if (ep.gain && (!ep.x_out || ep.x_out == act || !sjd_f32_norm_fits(lin, rows))) return SJD_EINVAL;
    if ((ep.kind == SJD_EPI_SILU && N % 2) || (ep.kind == SJD_EPI_QKV && (!st || N % 6 || ep.hd < 2 || (ep.hd & (ep.hd - 1)) || N / 3 % ep.hd))) return SJD_EINVAL;
    const int units = ep.kind == SJD_EPI_STORE ? N : N / 2;
    const bool by8 = sjd_f32_by8(lin, rows);
    const dim3 grid((units + 3) / 4, by8 ? (rows + 7) / 8 : 1), block(256);
    const float *W = (const float *)lin->w;
#define GO(MR, EPI, NORM) SJD_LAUNCH((gemm_f32_kernel<MR, EPI, NORM>), grid, block, 0, s, W, act, N, K, rows, st, ep)
#define ROWS(EPI) do { if (by8) GO(8, EPI, false); else if (rows <= 16) GO(16, EPI, false); else GO(32, EPI, false); } while (0)
#define KIND(EPI) do { if (ep.gain) GO(8, EPI, true); else ROWS(EPI); } while (0)
    switch (ep.kind) {
        case SJD_EPI_STORE: KIND(SJD_EPI_STORE); break;
        case SJD_EPI_SILU: KIND(SJD_EPI_SILU); break;
        case SJD_EPI_QKV: KIND(SJD_EPI_QKV); break;
        default: return SJD_EINVAL;
    }
#undef KIND
#undef ROWS
#undef GO
    HIP_TRY(hipGetLastError());
    return SJD_OK;
}

// Element-wise pieces of the window forward (paper Sec. 4.1 Step 2; the decoder itself is the
// Llama-style stack the workloads name): embedding gather for every model, and RMSNorm fused with the
// residual add for fp32 models too wide to do it inside their projections (the rest of it is done there; in bf16
// models everything is).  All of them are bandwidth-trivial (rows <= 32).
#include "sjd_internal.h"

template <typename T> struct Act;
template <> struct Act<float> {
    __device__ static float load(const float *p, size_t i) { return p[i]; }
    __device__ static void store(float *p, size_t i, float v) { p[i] = v; }
};
template <> struct Act<bf16_t> {
    __device__ static float load(const bf16_t *p, size_t i) { return bf16_to_f32(p[i]); }
};

// x[row][:] = E[id][:], from row `id_rows` on the given raw embedding rows (a prompt's ids lead); bf16 models keep x in act_off order and leave
// what the first projection reads: the hi / lo planes of x * gain (first layer's attention norm) in
// x24 and the sums of squares of x per 16 features in ssq.  Stream
// blockIdx.z takes its ids from ids.p[stream] and writes rows (stream << shift)..; one thread per 4
// consecutive features; grid (rows per stream, d / 1024, streams).
struct EmbedIds { const int32_t *p[SJD_MAX_STREAMS]; int32_t *err[SJD_MAX_STREAMS]; };
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T *E, EmbedIds ids, const float *emb_rows, int id_rows, int d, int shift,
                                                    float *x, void *x24, const bf16_t *gain, float *ssq, int vocab, int lo16)
{
    const int stream = blockIdx.z;
    const int r = blockIdx.x;
    const int j = (blockIdx.y * 256 + threadIdx.x) * 4;
    if (j >= d) return;       // (d is a multiple of 32 in bf16 models: whole groups of 4 threads leave)
    float4 v;
    // an id outside the vocabulary (the ids come from caller-supplied device memory) reads nothing: its
    // row is zero and the error flag of the handle's state is raised
    const bool raw = r >= id_rows;
    const int id = raw ? 0 : ids.p[stream][r];
    if (id < 0 || id >= vocab) {
        v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j == 0 && ids.err[stream]) *ids.err[stream] = SJD_DEVERR_TOKEN_ID;
    } else if (raw) {
        v = *reinterpret_cast<const float4 *>(emb_rows + (size_t)(r - id_rows) * d + j);
    } else if (sizeof(T) == 2) {
        const uint2 u = *reinterpret_cast<const uint2 *>(reinterpret_cast<const bf16_t *>(E) + (size_t)id * d + j);
        v = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                        __uint_as_float(u.y & 0xFFFF0000u));
    } else {
        v = *reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(E) + (size_t)id * d + j);
    }
    const int row = (stream << shift) + r;
    float *dst = sizeof(T) == 2 ? x + act_off(row, j, d / 32) : x + (size_t)row * d + j;
    *reinterpret_cast<float4 *>(dst) = v;
    if (sizeof(T) == 2) {
        const uint2 gn = *reinterpret_cast<const uint2 *>(gain + j);
        act24_store4(x24, row, j, d / 32, v.x * __uint_as_float(gn.x << 16), v.y * __uint_as_float(gn.x & 0xFFFF0000u),
                     v.z * __uint_as_float(gn.y << 16), v.w * __uint_as_float(gn.y & 0xFFFF0000u), lo16 != 0);
        float sq = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w)));
        sq += __shfl_xor(sq, 1);                      // 4 consecutive threads hold 16 consecutive features
        sq += __shfl_xor(sq, 2);
        if ((threadIdx.x & 3) == 0) ssq[(size_t)row * ssq_stride(d) + (j >> 4)] = sq;
    }
}

// x[r] += sum_p part[p][r]  (skipped when part == NULL);  h[r] = x[r] * rsqrt(mean(x[r]^2) + eps) * g
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(float *x, const float *part, int n_part, size_t part_stride,
                                                      const T *gain, int d, float eps, T *h,
                                                      const SjdState *st)
{
    if (st->done) return;
    __shared__ float red[4];
    const int r = blockIdx.x;
    float *xr = x + (size_t)r * d;
    float ss = 0.f;
    for (int j = threadIdx.x; j < d; j += 256) {
        float v = xr[j];
        for (int p = 0; p < n_part; ++p) v += part[(size_t)p * part_stride + (size_t)r * d + j];
        if (n_part) xr[j] = v;
        ss += v * v;
    }
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = red[0] + red[1] + red[2] + red[3];
    const float inv = rsqrtf(ss / (float)d + eps);
    for (int j = threadIdx.x; j < d; j += 256) Act<T>::store(h, (size_t)r * d + j, xr[j] * inv * Act<T>::load(gain, j));
}

// ---------------------------------------------------------------------------------------------
#define LAUNCH_CHECK() HIP_TRY(hipGetLastError())

int sjd_launch_embed(const sjd_model *m, const int32_t *const *ids, int32_t id_rows, const float *emb_rows,
                     int32_t rows, const SjdStreams &sm, float *x, void *x24, float *ssq, int32_t *const *err, bool lo16, hipStream_t s)
{
    if (sm.count < 1 || sm.count > SJD_MAX_STREAMS || rows < 1 || rows > (1 << sm.shift) ||
        (sm.count << sm.shift) > SJD_ROWS_MAX)
        return SJD_EINVAL;
    if (id_rows < 0 || id_rows > rows || (id_rows < rows && !emb_rows)) return SJD_EINVAL;
    if (m->cfg.dtype == 0 && sm.count != 1) return SJD_EINVAL;
    if (m->cfg.dtype == 1 && (!x24 || !ssq)) return SJD_EINVAL;
    const int d = m->cfg.d_model;
    EmbedIds e;
    for (int i = 0; i < SJD_MAX_STREAMS; ++i) {
        e.p[i] = (ids && i < sm.count) ? ids[i] : nullptr;
        e.err[i] = (err && i < sm.count) ? err[i] : nullptr;
    }
    const dim3 grid(rows, (d + 1023) / 1024, sm.count);
    if (m->cfg.dtype == 0)
        SJD_LAUNCH(embed_kernel<float>, grid, dim3(256), 0, s, (const float *)m->E, e, emb_rows, id_rows, d, sm.shift, x, x24, (const bf16_t *)nullptr, ssq, m->cfg.vocab_total, lo16 ? 1 : 0);
    else
        SJD_LAUNCH(embed_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t *)m->E, e, emb_rows, id_rows, d, sm.shift, x, x24, (const bf16_t *)m->layers[0].g1, ssq, m->cfg.vocab_total, lo16 ? 1 : 0);
    LAUNCH_CHECK();
    return SJD_OK;
}

int sjd_launch_rmsnorm(const sjd_model *m, float *x, const float *part, int32_t n_part, size_t part_stride,
                       const void *gain, int32_t rows, void *h, const SjdState *st, hipStream_t s)
{
    const int d = m->cfg.d_model;
    if (m->cfg.dtype != 0) return SJD_EINVAL;   // bf16 models normalise inside the projection kernel
    SJD_LAUNCH(rmsnorm_kernel<float>, dim3(rows), dim3(256), 0, s, x, part, n_part, part_stride,
                       (const float *)gain, d, m->cfg.rms_eps, (float *)h, st);
    LAUNCH_CHECK();
    return SJD_OK;
}

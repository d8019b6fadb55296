// Small passes shared by the 3x3x3 convolution kernels: the fixed-order reduction of split-K partial
// sums, and the one-bit-per-element ReLU masks for kernels that do not handle them themselves.
#include "common.h"
#include "conv_internal.h"

namespace k3 {

// out[i] = sum_s ws[s*count + i] in a fixed order: a block owns 64 entries; its 4 thread groups
// add the splits g, g+4, g+8, ... in increasing order and the four group sums are then combined
// as ((g0+g1)+g2)+g3.  The first countW entries go to dW, the remaining ones (bias gradient)
// to db when it is not null.
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float *__restrict__ ws, float *__restrict__ dW,
                                                             float *__restrict__ db, int64_t countW, int64_t count,
                                                             int nsplit)
{
    __shared__ float part[4][64];
    const int e = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + e;
    float s0 = 0.f, s1 = 0.f;
    if (i < count) {
        int k = g;
        for (; k + 4 < nsplit; k += 8) {   // two independent chains, merged below in a fixed order
            s0 += ws[(int64_t)k * count + i];
            s1 += ws[(int64_t)(k + 4) * count + i];
        }
        if (k < nsplit) s0 += ws[(int64_t)k * count + i];
    }
    part[g][e] = s0 + s1;
    __syncthreads();
    if (g == 0 && i < count) {
        float s = ((part[0][e] + part[1][e]) + part[2][e]) + part[3][e];
        if (i < countW) dW[i] = s;
        else if (db) db[i - countW] = s;
    }
}

__device__ __forceinline__ void add4(float4 &s, const float4 &a) { s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w; }

// Same sum for 16-byte aligned buffers whose element counts are multiples of 4: a thread adds float4
// quads, 256 / G quads x G groups of splits per block, U loads in flight for CH chains; the chains and
// then the groups are merged in a fixed order.  The last turn reads clamped places without a branch.
template <int G, int U = G == 16 ? 4 : 8, int CH = U>
__global__ __launch_bounds__(256) void reduce_partials_vec4_kernel(const float4 *__restrict__ ws, float4 *__restrict__ dW,
                                                                  float4 *__restrict__ db, int64_t quadsW, int64_t quads,
                                                                  int nsplit)
{
    constexpr int Q = 256 / G;
    __shared__ float4 part[G][Q];
    const int e = threadIdx.x % Q, g = threadIdx.x / Q;
    const int64_t i = (int64_t)blockIdx.x * Q + e;
    float4 s[CH];
#pragma unroll
    for (int j = 0; j < CH; ++j) s[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i < quads) {
        int k = g;
        for (; k + (U - 1) * G < nsplit; k += U * G) {
            float4 a[U];
#pragma unroll
            for (int j = 0; j < U; ++j) a[j] = ws[(int64_t)(k + j * G) * quads + i];
#pragma unroll
            for (int j = 0; j < U; ++j) add4(s[j % CH], a[j]);
        }
        if (k < nsplit) {
            float4 a[U - 1];
#pragma unroll
            for (int j = 0; j < U - 1; ++j) a[j] = ws[(int64_t)(k + j * G < nsplit ? k + j * G : k) * quads + i];
#pragma unroll
            for (int j = 0; j < U - 1; ++j)
                if (k + j * G < nsplit) add4(s[j % CH], a[j]);
        }
    }
#pragma unroll
    for (int n = CH / 2; n > 0; n /= 2)
#pragma unroll
        for (int j = 0; j < n; ++j) add4(s[j], s[j + n]);
    if (G > 1) {
        part[g][e] = s[0];
        __syncthreads();
        if (g > 0) return;
#pragma unroll
        for (int q = 1; q < G; ++q) add4(s[0], part[q][e]);
    }
    if (i < quads) {
        if (i < quadsW) dW[i] = s[0];
        else if (db) db[i - quadsW] = s[0];
    }
}

static bool reduce_quads(const float *ws, const float *dW, const float *db, int64_t countW, int64_t count)
{
    return count % 4 == 0 && countW % 4 == 0 && (((uintptr_t)ws | (uintptr_t)dW | (uintptr_t)db) & 15) == 0;
}

int launch_reduce_partials(const float *ws, float *dW, float *db, int64_t countW, int64_t count, int nsplit,
                           hipStream_t st)
{
    if (reduce_quads(ws, dW, db, countW, count)) {
        // A thread per quad where there are many quads with few loads each (256 -> 256 channels, 2 sets:
        // 8.6 us against 16 with sixteen groups), else as few groups as leave the chip full of blocks: a
        // wave then reads 1 KB runs.
        const int64_t quads = count / 4;
        auto run = [&](auto kernel, int q) {
            kernel<<<dim3((unsigned)((quads + q - 1) / q)), 256, 0, st>>>((const float4 *)ws, (float4 *)dW, (float4 *)db, countW / 4, quads, nsplit);
        };
        if (quads >= 65536 && nsplit <= 8) run(reduce_partials_vec4_kernel<1>, 256);
        else if (quads >= 16384) run(reduce_partials_vec4_kernel<4>, 64);
        else run(reduce_partials_vec4_kernel<16>, 16);
        K3_LAUNCH_CHECK();
        return K3_OK;
    }
    int64_t blocks = (count + 63) / 64;
    reduce_partials_kernel<<<dim3((unsigned)blocks), 256, 0, st>>>(ws, dW, db, countW, count, nsplit);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

// The same with sixteen groups and two chains for any number of sets: the order of an fp32 sum then depends
// on the number of sets alone (wgrad_ordered.hip), and on whether the alignment allows quads.
int launch_reduce_ordered(const float *ws, float *dW, float *db, int64_t countW, int64_t count, int nsplit, hipStream_t st)
{
    if (!reduce_quads(ws, dW, db, countW, count)) return launch_reduce_partials(ws, dW, db, countW, count, nsplit, st);
    reduce_partials_vec4_kernel<16, 8, 2><<<dim3((unsigned)((count / 4 + 15) / 16)), 256, 0, st>>>(
        (const float4 *)ws, (float4 *)dW, (float4 *)db, countW / 4, count / 4, nsplit);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

// ---- one-bit-per-element ReLU masks, generic passes (the MFMA kernels produce / consume the
// bits themselves; these serve the kernels that do not)
template <typename T>
__global__ __launch_bounds__(256) void relu_bits_kernel(const T *__restrict__ y, unsigned short *__restrict__ bits, int64_t nwords)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nwords; i += stride) {
        unsigned m = 0u;
#pragma unroll
        for (int e = 0; e < 16; ++e) m |= (elem<T>::ld(y + i * 16 + e) > 0.f ? 1u : 0u) << e;
        bits[i] = (unsigned short)m;
    }
}

template <typename T>
__global__ __launch_bounds__(256) void apply_relu_bits_kernel(T *__restrict__ t, const unsigned short *__restrict__ bits,
                                                             int64_t nwords)
{
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nwords; i += stride) {
        const unsigned m = bits[i];
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (!((m >> e) & 1u)) elem<T>::st(t + i * 16 + e, 0.f);
    }
}

int launch_relu_bits(int dtype, const void *y, void *bits, int64_t nwords, hipStream_t st)
{
    const int64_t want = (nwords + 255) / 256;
    const unsigned grid = (unsigned)(want < 8192 ? (want > 0 ? want : 1) : 8192);
    if (dtype == K3_F32) relu_bits_kernel<float><<<dim3(grid), 256, 0, st>>>((const float *)y, (unsigned short *)bits, nwords);
    else relu_bits_kernel<bf16_t><<<dim3(grid), 256, 0, st>>>((const bf16_t *)y, (unsigned short *)bits, nwords);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

int launch_apply_relu_bits(int dtype, void *t, const void *bits, int64_t nwords, hipStream_t st)
{
    const int64_t want = (nwords + 255) / 256;
    const unsigned grid = (unsigned)(want < 8192 ? (want > 0 ? want : 1) : 8192);
    if (dtype == K3_F32) apply_relu_bits_kernel<float><<<dim3(grid), 256, 0, st>>>((float *)t, (const unsigned short *)bits, nwords);
    else apply_relu_bits_kernel<bf16_t><<<dim3(grid), 256, 0, st>>>((bf16_t *)t, (const unsigned short *)bits, nwords);
    K3_LAUNCH_CHECK();
    return K3_OK;
}

}  // namespace k3

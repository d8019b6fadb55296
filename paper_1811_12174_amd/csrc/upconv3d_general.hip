// 2x2x2 stride-2 transposed convolution for the tensors the bf16 matrix kernels do not take -- fp32,
// and bf16 with channel counts that are no multiple of 32 -- on v_mfma_f32_16x16x4_f32: fp32 products
// and fp32 sums for any channel counts.
//
// Bound: neither memory nor the matrix core at the sizes these serve (at 2 x 20x24x28, 32 -> 16 channels
// all three passes together need 3 us for either) but the latency of one operand fetch after
// the other, so the kernels hold the next step's operands in registers while they multiply and
// spread over many short workgroups.  The thread-per-output kernels these replace walked the
// contraction with two loads per multiply-add.  Measured, before -> after (forward / backward-data /
// backward-weight with its reduction): bf16 32 -> 16 at 2 x 20x24x28: 39 / 220 / 57 -> 10 / 10 / 16 us;
// fp32 32 -> 16 at 24^3: 25 / 106 / 44 -> 7 / 9 / 20 us; fp32 64 -> 32 at 12^3: 22 / 62 / 57 -> 8 / 14 / 21 us
// (backward-weight of fp32: wgrad_ordered.hip).  Every sum keeps the order of the plain loop.
#include "common.h"
#include "conv_internal.h"
#include "quad_io.h"

namespace k3 {

template <typename T>
struct UpGeneral {
    const T *x, *dy, *w, *mask;   // x and dx: (N, D, H, W, cin); y and dy: (N, 2D, 2H, 2W, cout); w: [8][cin][cout]
    const float *bias;
    T *y, *dx;
    int64_t V;
    int D, H, W, cin, cout, nblk;   // nblk: 16-channel blocks of the output
    bool wide;                      // at least 2^31 voxels: their coordinates need 64-bit divisions
};

// first output voxel of input voxel v, i.e. that of tap (0, 0, 0)
template <typename T>
__device__ __forceinline__ int64_t up_origin(const UpGeneral<T> &p, int64_t v)
{
    if (p.wide) {
        const int64_t r = v / p.W, s = r / p.H, n = s / p.D;
        return ((n * 2 * p.D + 2 * (s - n * p.D)) * 2 * p.H + 2 * (r - s * p.H)) * (2 * (int64_t)p.W) + 2 * (v - r * p.W);
    }
    const unsigned u = (unsigned)v, r = u / (unsigned)p.W, s = r / (unsigned)p.H, n = s / (unsigned)p.D;
    return (((int64_t)n * 2 * p.D + 2 * (s - n * p.D)) * 2 * p.H + 2 * (r - s * p.H)) * (2 * (int64_t)p.W) + 2 * (u - r * p.W);
}
template <typename T>
__device__ __forceinline__ int64_t up_tap(const UpGeneral<T> &p, int tap) { return ((int64_t)(tap >> 2) * 2 * p.H + ((tap >> 1) & 1)) * (2 * (int64_t)p.W) + (tap & 1); }

// channels c .. c+3 of the `count` at p; zero beyond (QUAD: count in whole quads, 4-element aligned rows)
template <typename T, bool QUAD>
__device__ __forceinline__ f32x4 up_quad(const T *p, int c, int count, bool in)
{
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (QUAD) {
        if (in && c < count) v = buf<T>::ld4(p + c);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (in && c + j < count) v[j] = elem<T>::ld(p + c + j);
    }
    return v;
}
template <typename T, bool QUAD>
__device__ __forceinline__ void up_store(T *p, int c, int count, f32x4 v)
{
    if constexpr (QUAD) {
        if (c < count) buf<T>::st4(p + c, v);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (c + j < count) elem<T>::st(p + c + j, v[j]);
    }
}

// Forward, D[output channel][voxel]: a workgroup takes 32 voxels x 16 output channels, each wave the two
// taps of one row of the 2x2x2 block, so that its stores fill 2 neighbouring voxels.  An instruction
// multiplies four neighbouring channels, lane group kg carrying channel kg of them, and the accumulators
// start from the bias: the sums are those of the plain loop over the channels (see
// conv_general_kernel for why that order is kept).
template <typename T, bool QUAD>
__global__ __launch_bounds__(256) void up_general_fwd_kernel(UpGeneral<T> p)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int co0 = (int)(blockIdx.x % (unsigned)p.nblk) * 16;
    const int64_t v0 = (int64_t)(blockIdx.x / (unsigned)p.nblk) * 32;
    const int co = co0 + ln;
    const bool row = co < p.cout;
    const T *w = p.w + (int64_t)(2 * wv) * p.cin * p.cout + (row ? co : 0);
    const T *xp[2];
    bool in[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t v = v0 + b * 16 + ln;
        in[b] = v < p.V;
        xp[b] = p.x + (in[b] ? v : 0) * p.cin;
    }
    const int m = co0 + kg * 4;
    f32x4 acc[2][2];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const float bias = p.bias && m + r < p.cout ? p.bias[m + r] : 0.f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[t][b][r] = bias;
    }
    auto fetch = [&](int c, float (&x)[2][4], float (&a)[2][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {         // (dealt out by spread() before they are used)
            const f32x4 v = up_quad<T, QUAD>(xp[b], c + kg * 4, p.cin, in[b]);
            x[b][0] = v[0]; x[b][1] = v[1]; x[b][2] = v[2]; x[b][3] = v[3];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int ci = c + j * 4 + kg;
            const bool ok = ci < p.cin;
#pragma unroll
            for (int t = 0; t < 2; ++t) a[t][j] = ok && row ? elem<T>::ld(w + ((int64_t)t * p.cin + ci) * p.cout) : 0.f;
        }
    };
    float x[2][2][4], a[2][2][4];
    auto multiply = [&](float (&xs)[2][4], float (&as)[2][4]) __attribute__((always_inline)) {
        spread(xs[0]);
        spread(xs[1]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[t][b] = mfma_f32(as[t][j], xs[b][j], acc[t][b]);
    };
    fetch(0, x[0], a[0]);
    for (int c = 0; c < p.cin; c += 32) {     // two steps a turn: the register sets have fixed names
        if (c + 16 < p.cin) fetch(c + 16, x[1], a[1]);
        multiply(x[0], a[0]);
        if (c + 16 >= p.cin) break;
        if (c + 32 < p.cin) fetch(c + 32, x[0], a[0]);
        multiply(x[1], a[1]);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (!in[b]) continue;
        T *out = p.y + (up_origin(p, v0 + b * 16 + ln) + up_tap(p, 2 * wv)) * p.cout;
#pragma unroll
        for (int t = 0; t < 2; ++t) up_store<T, QUAD>(out + t * p.cout, m, p.cout, acc[t][b]);
    }
}

// Backward-data, D[input channel][voxel]: a wave takes 32 voxels x 16 input channels and walks the whole
// contraction, tap after tap and the output channels of a tap in order (as above), the four waves of a
// workgroup four groups of voxels.
template <typename T, bool QUAD>
__global__ __launch_bounds__(256) void up_general_dgrad_kernel(UpGeneral<T> p)
{
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int ci0 = (int)(blockIdx.x % (unsigned)p.nblk) * 16;
    const int64_t v0 = ((int64_t)(blockIdx.x / (unsigned)p.nblk) * 4 + wv) * 32;
    if (v0 >= p.V) return;
    const int ci = ci0 + ln;
    const bool row = ci < p.cin;
    const T *w = p.w + (int64_t)(row ? ci : 0) * p.cout;
    const T *gp[2];
    bool in[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int64_t v = v0 + b * 16 + ln;
        in[b] = v < p.V;
        gp[b] = p.dy + (in[b] ? up_origin(p, v) * p.cout : 0);
    }
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    // a step: 16 output channels of one tap; the next one's operands are on their way
    auto fetch = [&](int t, int c, float (&g)[2][4], float (&a)[4]) __attribute__((always_inline)) {
        const int64_t go = up_tap(p, t) * p.cout;
        const f32x4 v = up_quad<T, QUAD>(w + (int64_t)t * p.cin * p.cout, c + kg * 4, p.cout, row);
        a[0] = v[0]; a[1] = v[1]; a[2] = v[2]; a[3] = v[3];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const f32x4 u = up_quad<T, QUAD>(gp[b] + go, c + kg * 4, p.cout, in[b]);
            g[b][0] = u[0]; g[b][1] = u[1]; g[b][2] = u[2]; g[b][3] = u[3];
        }
    };
    auto multiply = [&](float (&g)[2][4], float (&a)[4]) __attribute__((always_inline)) {
        spread(a);
        spread(g[0]);
        spread(g[1]);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[b] = mfma_f32(a[j], g[b][j], acc[b]);
    };
    const int per = (p.cout + 15) / 16, steps = 8 * per;     // an even number
    int t = 0, c = 0;
    auto advance = [&]() __attribute__((always_inline)) {
        c += 16;
        if (c >= p.cout) {
            c = 0;
            t = t < 7 ? t + 1 : 7;                            // behind the last step: read again, not used
        }
    };
    float g[2][2][4], a[2][4];
    fetch(t, c, g[0], a[0]);
    advance();
    for (int s = 0; s < steps; s += 2) {                      // the register sets have fixed names
        fetch(t, c, g[1], a[1]);
        advance();
        multiply(g[0], a[0]);
        fetch(t, c, g[0], a[0]);
        advance();
        multiply(g[1], a[1]);
    }
    const int m = ci0 + kg * 4;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        if (!in[b]) continue;
        const int64_t v = v0 + b * 16 + ln;
        f32x4 s = acc[b];
        if (p.mask) s = keep_positive(s, up_quad<T, QUAD>(p.mask + v * p.cin, m, p.cin, true));
        up_store<T, QUAD>(p.dx + v * p.cin, m, p.cin, s);
    }
}

// Backward-weight, D[input channel][output channel] for each of the 8 taps: the contraction runs over
// 4 neighbouring voxels per instruction, operands come straight from memory (16 neighbouring channels per
// lane group).  The waves of a workgroup take its 16-voxel groups in turn and are added
// through LDS in a fixed order.  Blocks of input channels 0 .. 15 also sum dy: the bias gradient.
template <typename T>
__global__ __launch_bounds__(256) void up_general_wgrad_kernel(UpGeneral<T> p, float *outW, float *outB, int64_t per_split, int nsplit, int nco)
{
    constexpr int U = 4;
    __shared__ float red[4][8 * 256 + 16];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int split = (int)(blockIdx.x % (unsigned)nsplit), blk = (int)(blockIdx.x / (unsigned)nsplit);
    const int ci0 = (blk / nco) * 16, co0 = (blk % nco) * 16;
    const bool rin = ci0 + ln < p.cin, cok = co0 + ln < p.cout;
    const T *xp = p.x + (rin ? ci0 + ln : 0), *gp = p.dy + (cok ? co0 + ln : 0);
    int64_t toff[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) toff[t] = up_tap(p, 2 * t) * p.cout;
    f32x4 acc[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    float sum = 0.f;
    for (int64_t v0 = ((int64_t)split * 4 + wv) * (4 * U); v0 < p.V; v0 += (int64_t)nsplit * (16 * U)) {
        float a[U], g[U][8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t v = v0 + u * 4 + kg;
            const bool in = v < p.V;
            const int64_t vc = in ? v : 0;
            const float xv = elem<T>::ld(xp + vc * p.cin);
            const T *q = gp + up_origin(p, vc) * p.cout;
            a[u] = in && rin ? xv : 0.f;
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const float gv = elem<T>::ld(q + toff[t >> 1] + (t & 1) * p.cout);
                g[u][t] = in && cok ? gv : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = mfma_f32(a[u], g[u][t], acc[t]);
            sum += ((g[u][0] + g[u][1]) + (g[u][2] + g[u][3])) + ((g[u][4] + g[u][5]) + (g[u][6] + g[u][7]));
        }
    }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv][t * 256 + (kg * 4 + r) * 16 + ln] = acc[t][r];
    if (kg == 0) red[wv][8 * 256 + ln] = sum;
    __syncthreads();
    const int ci = ci0 + (threadIdx.x >> 4), co = co0 + (threadIdx.x & 15);
    if (ci < p.cin && co < p.cout) {
        float *o = outW + split * per_split;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int k = t * 256 + threadIdx.x;
            o[((int64_t)t * p.cin + ci) * p.cout + co] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
        }
    }
    if (outB && ci0 == 0 && threadIdx.x < 16 && co0 + threadIdx.x < p.cout) {
        const int k = 8 * 256 + threadIdx.x;
        outB[split * per_split + co0 + threadIdx.x] = ((red[0][k] + red[1][k]) + red[2][k]) + red[3][k];
    }
}

template <typename T> static bool quad_aligned(const void *p) { return ((uintptr_t)p & (4 * sizeof(T) - 1)) == 0; }

template <typename T>
static UpGeneral<T> up_general_args(int64_t N, int D, int H, int W, int cin, int cout)
{
    UpGeneral<T> p{};
    p.V = N * D * H * W;
    p.D = D; p.H = H; p.W = W; p.cin = cin; p.cout = cout;
    p.wide = p.V >= 1LL << 31;
    return p;
}

template <typename T>
static int up_fwd_t(const void *x, const void *w, const float *bias, void *y, int64_t N, int D, int H, int W, int cin, int cout, hipStream_t st)
{
    UpGeneral<T> p = up_general_args<T>(N, D, H, W, cin, cout);
    p.x = (const T *)x; p.w = (const T *)w; p.bias = bias; p.y = (T *)y;
    p.nblk = (cout + 15) / 16;
    const int64_t blocks = (p.V + 31) / 32 * p.nblk;
    if (blocks > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    const bool quad = cin % 4 == 0 && cout % 4 == 0 && quad_aligned<T>(x) && quad_aligned<T>(y);
    if (quad) up_general_fwd_kernel<T, true><<<dim3((unsigned)blocks), 256, 0, st>>>(p);
    else up_general_fwd_kernel<T, false><<<dim3((unsigned)blocks), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}
int up_general_fwd(int dtype, const void *x, const void *w, const float *bias, void *y, int64_t N, int D, int H, int W, int cin, int cout,
                   hipStream_t st)
{
    return dtype == K3_F32 ? up_fwd_t<float>(x, w, bias, y, N, D, H, W, cin, cout, st) : up_fwd_t<bf16_t>(x, w, bias, y, N, D, H, W, cin, cout, st);
}

template <typename T>
static int up_dgrad_t(const void *dy, const void *w, void *dx, const void *mask, int64_t N, int D, int H, int W, int cin, int cout,
                      hipStream_t st)
{
    UpGeneral<T> p = up_general_args<T>(N, D, H, W, cin, cout);
    p.dy = (const T *)dy; p.w = (const T *)w; p.mask = (const T *)mask; p.dx = (T *)dx;
    p.nblk = (cin + 15) / 16;
    const int64_t blocks = (p.V + 127) / 128 * p.nblk;
    if (blocks > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    const bool quad = cin % 4 == 0 && cout % 4 == 0 && quad_aligned<T>(dy) && quad_aligned<T>(w) && quad_aligned<T>(dx) && quad_aligned<T>(mask);
    if (quad) up_general_dgrad_kernel<T, true><<<dim3((unsigned)blocks), 256, 0, st>>>(p);
    else up_general_dgrad_kernel<T, false><<<dim3((unsigned)blocks), 256, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return K3_OK;
}
int up_general_dgrad(int dtype, const void *dy, const void *w, void *dx, const void *mask, int64_t N, int D, int H, int W, int cin, int cout,
                     hipStream_t st)
{
    return dtype == K3_F32 ? up_dgrad_t<float>(dy, w, dx, mask, N, D, H, W, cin, cout, st)
                           : up_dgrad_t<bf16_t>(dy, w, dx, mask, N, D, H, W, cin, cout, st);
}

int64_t up_general_max_splits(int64_t V)
{
    const int64_t s = V / 256;
    return s < 1 ? 1 : (s > 1024 ? 1024 : s);
}

// About 1024 workgroups in all (four per CU cover each other's fetches), at least 256 voxels each and no
// more sets of partial sums than ws holds; a single one writes the gradient itself.
template <typename T>
static int up_wgrad_t(const void *x, const void *dy, float *dW, float *db, float *ws, int64_t max_sets, int64_t N, int D, int H, int W,
                      int cin, int cout, hipStream_t st)
{
    UpGeneral<T> p = up_general_args<T>(N, D, H, W, cin, cout);
    p.x = (const T *)x; p.dy = (const T *)dy;
    const int64_t nco = (cout + 15) / 16, blocks = (cin + 15) / 16 * nco;
    if (blocks > 0x7fffffffLL) return K3_E_UNSUPPORTED;
    int64_t nsplit = 1024 / blocks;
    if (nsplit > up_general_max_splits(p.V)) nsplit = up_general_max_splits(p.V);
    if (nsplit > max_sets) nsplit = max_sets;
    if (nsplit < 1) nsplit = 1;
    const dim3 grid((unsigned)(nsplit * blocks));
    const int64_t countW = (int64_t)8 * cin * cout, per = countW + cout;
    const bool direct = nsplit == 1;
    up_general_wgrad_kernel<T><<<grid, 256, 0, st>>>(p, direct ? dW : ws, direct ? db : ws + countW, per, (int)nsplit, (int)nco);
    K3_LAUNCH_CHECK();
    return direct ? K3_OK : launch_reduce_partials(ws, dW, db, countW, per, (int)nsplit, st);
}
int up_general_wgrad(int dtype, const void *x, const void *dy, float *dW, float *db, float *ws, int64_t max_sets, int64_t N, int D, int H,
                     int W, int cin, int cout, hipStream_t st)
{
    return dtype == K3_F32 ? up_wgrad_ordered((const float *)x, (const float *)dy, dW, db, ws, N, D, H, W, cin, cout, st)
                           : up_wgrad_t<bf16_t>(x, dy, dW, db, ws, max_sets, N, D, H, W, cin, cout, st);
}

}  // namespace k3

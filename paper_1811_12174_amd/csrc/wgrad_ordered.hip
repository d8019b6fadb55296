// Weight gradients of fp32 tensors (3x3x3 and transposed convolution) on v_mfma_f32_16x16x4_f32, every sum in
// a fixed order that does not depend on the tiling: the voxels are cut into sets of at least 256, a set
// into 256 / cout interleaved chains (voxel s, s + chains, ... of the set), a chain is one fused multiply-add
// after the other, the chains of a set are added in order, then the sets (launch_reduce_ordered).  The
// instruction is itself a chain of four multiply-adds in lane-group order (see conv_general_kernel), so
// lane group kg takes every fourth voxel of a chain and the waves split the taps.  Other orders are as
// exact; this one is kept because it is the one results have always had, and in fp32 networks a weight
// that differs in its last bit moves ReLU signs and pooling maxima a step later (U-Net at 48^3: in one
// batch of six gradients by more than 4e-5 of their norm).
//
// Bound: neither pipe.  A step of four voxels is three matrix instructions of 32 clocks and some thirty
// address instructions a wave, and each chain's end moves its sums through the vector registers.
// Measured, thread-per-output kernels in the same order -> here: 16 -> 16 at 48^3 719 -> 38 us, 1 -> 16 there
// 135 -> 11, 64 -> 64 at 12^3 838 -> 16, 4 -> 8 at 16^3 141 -> 10, transposed 32 -> 16 at 24^3 39 -> 15, each
// before a reduction of 5 to 8 us.
#include "common.h"
#include "conv_internal.h"
#include "quad_io.h"

namespace k3 {

struct Ordered {
    const float *x1, *x2, *g, *mask;
    int c1, c2, cin, cout;
    float *ws;
    int64_t V, slab, per_split;
    int D, H, W, nsplit, chains, nco, parts;   // nco: 16-channel blocks of cout; parts: workgroups of a set and block
    FastDiv fd, fh, fw;                 // fewer than 2^31 voxels (wide: any)
    bool wide;
};

struct Coord { int d, h, w; int64_t n; };
__device__ __forceinline__ Coord coord_of(const Ordered &p, int64_t v)
{
    if (p.wide) {
        const int64_t r = v / p.W, s = r / p.H, n = s / p.D;
        return {(int)(s - n * p.D), (int)(r - s * p.H), (int)(v - r * p.W), n};
    }
    const unsigned u = (unsigned)v, r = p.fw.quot(u), s = p.fh.quot(r), n = p.fd.quot(s);
    return {(int)(s - n * p.fd.d), (int)(r - s * p.fh.d), (int)(u - r * p.fw.d), (int64_t)n};
}

// bit t: the voxel under tap t lies inside the volume
__device__ __forceinline__ unsigned taps_inside(const Ordered &p, int64_t v)
{
    const Coord c = coord_of(p, v);
    auto axis = [](int at, int size) __attribute__((always_inline)) { return (at > 0 ? 1u : 0u) | 2u | (at + 1 < size ? 4u : 0u); };
    const unsigned w = axis(c.w, p.W), h = axis(c.h, p.H), d = axis(c.d, p.D);
    const unsigned r = (h & 1u ? w : 0u) | w << 3 | (h & 4u ? w << 6 : 0u);
    return (d & 1u ? r : 0u) | r << 9 | (d & 4u ? r << 18 : 0u);
}

constexpr int ORDERED_TABLE = 10240;   // entries of a table in LDS: 40 KB leave room for three workgroups

// The walk over a set: chain s, and the first of the four voxels of the step in it (counted in the set).
// Steps behind the last one stand at voxel n: nothing is read there.
struct Walk {
    int s, i, n, chains, stride;
    bool last;     // the step ends its chain
    __device__ __forceinline__ Walk(int n_, int all) : s(0), i(0), n(n_), chains(all < n_ ? all : n_), stride(4 * all), last(4 * all >= n_) {}
    __device__ __forceinline__ void advance()
    {
        i += stride;
        if (i >= n) i = ++s < chains ? s : n;
        last = i + stride >= n;
    }
    // the first n % all chains are one voxel longer than the others
    __device__ __forceinline__ int steps(int all) const
    {
        const int len = n / all, more = n - len * all;
        return more * ((len + 4) / 4) + (chains - more) * ((len + 3) / 4);
    }
};

// a chain's end: its sum joins the set's, in the order of the chains
template <int N>
__device__ __forceinline__ void end_chain(f32x4 (&tot)[N], f32x4 (&acc)[N])
{
    asm volatile("");      // behind a branch: as selects it costs every step twelve instructions a tap
#pragma unroll
    for (int j = 0; j < N; ++j) {
        tot[j] += acc[j];
        acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

__device__ __forceinline__ int bit_mask(unsigned v, int bit) { return __builtin_amdgcn_sbfe((int)v, bit, 1); }   // -1 where it is set

// keeps a wave-uniform address in scalar registers (a descriptor made of vector ones costs a loop per load)
__device__ __forceinline__ const float *uniform(const float *p)
{
    const uint64_t v = (uint64_t)p;
    return (const float *)((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((int)v));
}

// The rows of the product are the gradient's own: row f = tap * cin + ci, and row 27 cin multiplies ones (the
// bias gradient), so that few input channels cost few instructions (4 -> 8: 7 blocks of rows where blocks
// of one tap each were 28).  A wave takes N blocks of 16 rows; at 16 channels that is a row of three
// taps, whose voxels neighbouring chains find in the CU's cache.  N = 1 and a workgroup a wave where those are too few to give every CU one.
// TABLE: which taps of a voxel lie outside is worked out once a set, in LDS.  FAST: reads through
// descriptors, an offset outside their range for what is not there (the set and its neighbours span less
// than 2 GiB, no mask); else by address.  BOTH: a block of rows may hold both sources, and every lane asks
// both, one of them in vain.
template <int N, bool TABLE, bool FAST, bool BOTH>
__global__ __launch_bounds__(N == 1 ? 64 : 640) void conv_ordered_wgrad_kernel(Ordered p)
{
    constexpr int RING = 8;     // steps in flight
    extern __shared__ unsigned table[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int kg = lane >> 4, ln = lane & 15;
    unsigned wg = blockIdx.x;
    const int part = (int)(wg % (unsigned)p.parts);
    wg /= (unsigned)p.parts;
    const int split = (int)(wg % (unsigned)p.nsplit), co0 = (int)(wg / (unsigned)p.nsplit) * 16;
    const int f0 = (part * (int)(blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(tid >> 6)) * 16 * N;   // the wave's first row
    const int64_t v0 = (int64_t)split * p.slab;
    const int n = v0 >= p.V ? 0 : (int)(v0 + p.slab < p.V ? p.slab : p.V - v0);     // (a last set may be empty)
    // bits 0 .. 26: the tap lies outside, bit 27: the voxel is none of the set
    auto outside_of = [&](int i) __attribute__((always_inline)) { return i < n ? ~taps_inside(p, v0 + i) & 0x7ffffffu : 0xfffffffu; };
    if constexpr (TABLE) {
        for (int i = tid; i < n + 4 * p.chains; i += blockDim.x) table[i] = outside_of(i);
        __syncthreads();
    }
    const int rows = 27 * p.cin;
    if (f0 > rows) return;
    const int co = co0 + ln;
    const bool cok = co < p.cout;
    const int64_t halo = ((int64_t)p.H + 1) * p.W + 1;
    const __amdgpu_buffer_rsrc_t rg = rsrc_of(FAST ? uniform(p.g + v0 * p.cout) : p.g, 0x7ffffff0);
    const int lg = cok ? (kg * p.chains * p.cout + co) * 4 : -1;
    // the lane's row in each block: its tap (27: none, bit 27 and no bit above it is ever kept), where its
    // input lies from the voxel (with descriptors: in bytes from `halo` before it), and its source
    __amdgpu_buffer_rsrc_t rx[N];
    const __amdgpu_buffer_rsrc_t ry = rsrc_of(BOTH ? uniform(p.x2 + (v0 - halo) * p.c2) : p.x1, 0x7ffffff0);
    int tap[N], step[N], also[N];
    int64_t at[N];
    bool ones[N], there[N];
    const float *src[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int f = f0 + j * 16 + ln, t = f < rows ? f / p.cin : 27, ci = f - t * p.cin;
        tap[j] = t;
        ones[j] = f == rows;
        there[j] = f < rows;
        // with descriptors a block lies in one source, that of its first row, or both are asked
        const int c0 = BOTH ? 0 : FAST ? (f0 + j * 16) % p.cin : ci;
        const bool first = c0 < p.c1;
        const int cx = first ? p.c1 : p.c2, cc = first ? ci : ci - p.c1;
        const int64_t toff = t < 27 ? ((int64_t)(t / 9 - 1) * p.H + (t / 3) % 3 - 1) * p.W + t % 3 - 1 : 0;
        src[j] = first ? p.x1 : p.x2;
        step[j] = FAST ? __builtin_amdgcn_readfirstlane(cx * 4) : cx;
        at[j] = FAST ? there[j] ? ((toff + halo + kg * p.chains) * cx + cc) * 4 : -1 : toff * cx + cc;
        also[j] = -1;
        if constexpr (BOTH) {
            if (ci >= p.c1) {
                also[j] = there[j] ? (int)(((toff + halo + kg * p.chains) * p.c2 + ci - p.c1) * 4) : -1;
                at[j] = -1;
            }
        }
        rx[j] = rsrc_of(FAST ? uniform(src[j] + (v0 - halo) * cx) : p.x1, 0x7ffffff0);
    }
    f32x4 acc[N], tot[N];
#pragma unroll
    for (int j = 0; j < N; ++j) acc[j] = tot[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float x[RING][N], g[RING];
    bool last[RING];
    auto fetch = [&](const Walk &q, float (&xr)[N], float &gr, bool &lr) __attribute__((always_inline)) {
        lr = q.last;
        const int i = q.i + kg * p.chains;
        const unsigned skip = TABLE ? table[i] : outside_of(i);
        if constexpr (FAST) {
            gr = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, lg | bit_mask(skip, 27), q.i * p.cout * 4, 0));
#pragma unroll
            for (int j = 0; j < N; ++j) {
                unsigned v = __builtin_amdgcn_raw_buffer_load_b32(rx[j], (int)at[j] | bit_mask(skip, tap[j]), q.i * step[j], 0);
                if constexpr (BOTH) v |= __builtin_amdgcn_raw_buffer_load_b32(ry, also[j] | bit_mask(skip, tap[j]), q.i * p.c2 * 4, 0);
                xr[j] = __uint_as_float(v);
            }
        } else {
            gr = 0.f;
            if (cok && !(skip >> 27)) {
                gr = p.g[(v0 + i) * p.cout + co];
                if (p.mask && !(p.mask[(v0 + i) * p.cout + co] > 0.f)) gr = 0.f;
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
                xr[j] = 0.f;
                if (there[j] && !((skip >> tap[j]) & 1u)) xr[j] = src[j][(v0 + i) * step[j] + at[j]];
            }
        }
    };
    Walk q(n, p.chains);
    const int steps = q.steps(p.chains);
#pragma unroll
    for (int r = 0; r < RING - 1; ++r) {
        fetch(q, x[r], g[r], last[r]);
        q.advance();
    }
    for (int s = 0; s < steps; s += RING) {      // (steps behind the last one multiply zeros)
#pragma unroll
        for (int r = 0; r < RING; ++r) {
            fetch(q, x[(r + RING - 1) % RING], g[(r + RING - 1) % RING], last[(r + RING - 1) % RING]);
            q.advance();
#pragma unroll
            for (int j = 0; j < N; ++j) acc[j] = mfma_f32(ones[j] ? 1.f : x[r][j], g[r], acc[j]);
            if (last[r]) end_chain(tot, acc);    // wave-uniform
        }
    }
    float *out = p.ws + (int64_t)split * p.per_split + (cok ? co : 0);
    if (!cok) return;
#pragma unroll
    for (int j = 0; j < N; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int f = f0 + j * 16 + kg * 4 + r;
            if (f <= rows) out[(int64_t)f * p.cout] = tot[j][r];
        }
}

// Transposed convolution, dW[tap][ci][co] = sum over voxels of x[v][ci] * g[the voxel under tap of v][co]: waves
// 0 and 1 take four taps each.  The bias gradient's chains run over the taps of a voxel, too: waves 2 to 5
// of the workgroups of input channels 0 .. 15 take every fourth chain and add them through LDS in order.
// FAST: where a voxel's outputs start is worked out once a set, in LDS, as bytes for a descriptor (the set's
// outputs span less than 2 GiB); else by address.
template <bool FAST>
__global__ __launch_bounds__(384) void up_ordered_wgrad_kernel(Ordered p)
{
    constexpr int RING = 4, U = 8;     // steps, and voxels of the bias gradient, in flight
    constexpr unsigned NONE = 0x80000000u;
    __shared__ float red[256][16];
    extern __shared__ unsigned table[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = lane >> 4, ln = lane & 15;
    const int split = (int)(blockIdx.x % (unsigned)p.nsplit), blk = (int)(blockIdx.x / (unsigned)p.nsplit);
    const int ci0 = (blk / p.nco) * 16, co0 = (blk % p.nco) * 16;
    const int64_t v0 = (int64_t)split * p.slab;
    const int n = v0 >= p.V ? 0 : (int)(v0 + p.slab < p.V ? p.slab : p.V - v0);
    const int co = co0 + ln;
    const bool cok = co < p.cout;
    float *out = p.ws + (int64_t)split * p.per_split;
    // first output voxel of input voxel v, and how far tap t of it is
    auto origin = [&](int64_t v) __attribute__((always_inline)) {
        const Coord c = coord_of(p, v);
        return ((c.n * 2 * p.D + 2 * c.d) * 2 * p.H + 2 * c.h) * (2 * (int64_t)p.W) + 2 * c.w;
    };
    auto under = [&](int t) __attribute__((always_inline)) { return ((int64_t)(t >> 2) * 2 * p.H + ((t >> 1) & 1)) * (2 * (int64_t)p.W) + (t & 1); };
    const int64_t o0 = n > 0 ? origin(v0) : 0;
    if constexpr (FAST) {
        for (int i = tid; i < n + U * p.chains; i += 384) table[i] = i < n ? (unsigned)((origin(v0 + i) - o0) * p.cout * 4) : NONE;
        __syncthreads();
    }
    const __amdgpu_buffer_rsrc_t rg = rsrc_of(FAST ? uniform(p.g + o0 * p.cout) : p.g, 0x7ffffff0);
    const unsigned no = cok ? 0u : NONE;
    if (wv < 2) {
        const bool rin = ci0 + ln < p.cin;
        const float *xp = p.x1 + (rin ? ci0 + ln : 0), *gp = p.g + (cok ? co : 0);
        const __amdgpu_buffer_rsrc_t rx = rsrc_of(FAST ? uniform(p.x1 + v0 * p.cin) : p.x1, 0x7ffffff0);
        const int lx = rin ? (kg * p.chains * p.cin + ci0 + ln) * 4 : -1;
        int64_t toff[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) toff[j] = under(wv * 4 + j) * p.cout;
        const int go4[4] = {__builtin_amdgcn_readfirstlane((int)toff[0] * 4), __builtin_amdgcn_readfirstlane((int)toff[1] * 4),
                            __builtin_amdgcn_readfirstlane((int)toff[2] * 4), __builtin_amdgcn_readfirstlane((int)toff[3] * 4)};
        f32x4 acc[4], tot[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = tot[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        float x[RING], g[RING][4];
        bool last[RING];
        auto fetch = [&](const Walk &q, float &xr, float (&gr)[4], bool &lr) __attribute__((always_inline)) {
            const int i = q.i + kg * p.chains;
            if constexpr (FAST) {
                const unsigned at = table[i];
                xr = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, lx | bit_mask(at, 31), q.i * p.cin * 4, 0));
                const unsigned go = (at + (unsigned)co * 4u) | no | (at & NONE);
#pragma unroll
                for (int j = 0; j < 4; ++j) gr[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, (int)go, go4[j], 0));
            } else {
                const bool in = i < n;
                const int64_t v = in ? v0 + i : 0;
                xr = in && rin ? xp[v * p.cin] : 0.f;
                const float *gv = gp + origin(v) * p.cout;
#pragma unroll
                for (int j = 0; j < 4; ++j) gr[j] = in && cok ? gv[toff[j]] : 0.f;
            }
            lr = q.last;
        };
        Walk q(n, p.chains);
        const int steps = q.steps(p.chains);
#pragma unroll
        for (int r = 0; r < RING - 1; ++r) {
            fetch(q, x[r], g[r], last[r]);
            q.advance();
        }
        for (int s = 0; s < steps; s += RING) {
#pragma unroll
            for (int r = 0; r < RING; ++r) {
                fetch(q, x[(r + RING - 1) % RING], g[(r + RING - 1) % RING], last[(r + RING - 1) % RING]);
                q.advance();
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[j] = mfma_f32(x[r], g[r][j], acc[j]);
                if (last[r]) end_chain(tot, acc);
            }
        }
        if (cok)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (ci0 + kg * 4 + r < p.cin) out[((int64_t)(wv * 4 + j) * p.cin + ci0 + kg * 4 + r) * p.cout + co] = tot[j][r];
    } else if (ci0 == 0) {
        const float *gp = p.g + (cok ? co : 0);
        const int64_t t0 = under(kg) * p.cout, t1 = under(4 + kg) * p.cout;
        const unsigned b0 = (unsigned)(t0 + co) * 4u, b1 = (unsigned)(t1 + co) * 4u;
        for (int s = wv - 2; s < (p.chains < n ? p.chains : n); s += 4) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            for (int i = s; i < n; i += U * p.chains) {
                float a[U], b[U];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int at = i + k * p.chains;
                    if constexpr (FAST) {
                        const unsigned e = table[at], hi = (e & NONE) | no;
                        a[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, (int)((e + b0) | hi), 0, 0));
                        b[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rg, (int)((e + b1) | hi), 0, 0));
                    } else {
                        const float *gv = gp + origin(at < n ? v0 + at : v0) * p.cout;
                        a[k] = at < n && cok ? gv[t0] : 0.f;
                        b[k] = at < n && cok ? gv[t1] : 0.f;
                    }
                }
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    acc = mfma_f32(1.f, a[k], acc);
                    acc = mfma_f32(1.f, b[k], acc);
                }
            }
            if (kg == 0) red[s][ln] = acc[0];                  // every row holds the sum
        }
    }
    __syncthreads();
    if (ci0 == 0 && tid < 16 && co0 + tid < p.cout) {
        float s = 0.f;
        for (int k = 0; k < (p.chains < n ? p.chains : n); ++k) s += red[k][tid];
        out[(int64_t)8 * p.cin * p.cout + co0 + tid] = s;
    }
}

static int64_t ordered_sets(int64_t V)
{
    const int64_t s = V / 256;
    return s < 1 ? 1 : s > 1024 ? 1024 : s;
}

static Ordered ordered_args(int64_t N, int64_t D, int64_t H, int64_t W, int64_t cin, int64_t cout, int taps, float *ws)
{
    Ordered p{};
    p.V = N * D * H * W;
    p.nsplit = (int)ordered_sets(p.V);
    p.slab = (p.V + p.nsplit - 1) / p.nsplit;
    p.chains = (int)(256 / (cout < 256 ? cout : 256));
    p.D = (int)D; p.H = (int)H; p.W = (int)W;
    p.cin = (int)cin; p.cout = (int)cout;
    p.nco = (int)((cout + 15) / 16);
    p.ws = ws;
    p.per_split = taps * cin * cout + cout;
    p.wide = p.V >= 1LL << 31;
    p.fd = FastDiv::of((unsigned)D); p.fh = FastDiv::of((unsigned)H); p.fw = FastDiv::of((unsigned)W);
    return p;
}

int conv_wgrad_ordered(const ConvArgs &a, float *dW, float *db, float *ws, hipStream_t st)
{
    Ordered p = ordered_args(a.N, a.D, a.H, a.W, a.c1 + a.c2, a.cout, 27, ws);
    p.x1 = (const float *)a.x; p.x2 = (const float *)a.x2;
    p.c1 = (int)a.c1; p.c2 = (int)a.c2;
    p.g = (const float *)a.dy; p.mask = (const float *)a.ymask;
    const int64_t c = p.cin > p.cout ? p.cin : p.cout, entries = p.slab + 4 * p.chains;
    const bool both = p.c2 > 0 && (p.c1 % 16 || p.c2 % 16);
    const bool fast = !p.mask && (entries + 2 * (((int64_t)p.H + 1) * p.W + 1)) * c * 4 < 0x7ffffff0LL;
    const bool table = entries <= ORDERED_TABLE;
    const int64_t blocks = (27 * (int64_t)p.cin + 16) / 16, sets = (int64_t)p.nsplit * p.nco;    // blocks of rows, the one of ones among them
    const int n = fast && table && sets * ((blocks + 2) / 3) < 1024 ? 1 : 3;        // a wave per SIMD and more, else single blocks
    const int64_t all = (blocks + n - 1) / n, waves = n == 1 ? 1 : all < 10 ? all : 10;
    p.parts = (int)((all + waves - 1) / waves);
    if (sets * p.parts > 0x7fffffffLL || p.slab > 0x3fffffffLL || blocks > 0x3ffffff) return K3_E_UNSUPPORTED;
    const size_t lds = table ? entries * sizeof(unsigned) : 0;
    auto run = [&](auto kernel) { kernel<<<dim3((unsigned)(sets * p.parts)), (unsigned)waves * 64, lds, st>>>(p); };
    if (n == 1 && both) run(conv_ordered_wgrad_kernel<1, true, true, true>);
    else if (n == 1) run(conv_ordered_wgrad_kernel<1, true, true, false>);
    else if (fast && table && both) run(conv_ordered_wgrad_kernel<3, true, true, true>);
    else if (fast && table) run(conv_ordered_wgrad_kernel<3, true, true, false>);
    else if (fast && !both) run(conv_ordered_wgrad_kernel<3, false, true, false>);
    else if (table) run(conv_ordered_wgrad_kernel<3, true, false, false>);
    else run(conv_ordered_wgrad_kernel<3, false, false, false>);
    K3_LAUNCH_CHECK();
    return launch_reduce_ordered(ws, dW, db, (int64_t)27 * p.cin * p.cout, p.per_split, p.nsplit, st);
}

int up_wgrad_ordered(const float *x, const float *dy, float *dW, float *db, float *ws, int64_t N, int D, int H, int W, int cin, int cout, hipStream_t st)
{
    Ordered p = ordered_args(N, D, H, W, cin, cout, 8, ws);
    p.x1 = x;
    p.g = dy;
    const int64_t grid = (cin + 15) / 16 * (int64_t)p.nco * p.nsplit;
    if (grid > 0x7fffffffLL || p.slab > 0x3fffffffLL) return K3_E_UNSUPPORTED;
    // the set's inputs, its outputs (eight a voxel, in rows that are 4 W outputs apart) and the taps of the last one
    const int64_t entries = p.slab + 8 * p.chains, span = (8 * p.slab + 8 * (int64_t)p.H * p.W + 16 * (int64_t)p.W) * 4;
    const bool fast = entries <= ORDERED_TABLE && span * cout < 0x7ffffff0LL && entries * cin * 4 < 0x7ffffff0LL;
    if (fast) up_ordered_wgrad_kernel<true><<<dim3((unsigned)grid), 384, entries * sizeof(unsigned), st>>>(p);
    else up_ordered_wgrad_kernel<false><<<dim3((unsigned)grid), 384, 0, st>>>(p);
    K3_LAUNCH_CHECK();
    return launch_reduce_ordered(ws, dW, db, (int64_t)8 * cin * cout, p.per_split, p.nsplit, st);
}

}  // namespace k3

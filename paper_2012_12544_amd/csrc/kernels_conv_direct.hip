// Direct (vector-ALU) convolution kernels: the arithmetic path of fp32 stages, whose 1e-4
// parity bound needs true fp32 products, and of the few bf16 shapes the MFMA kernels do not
// take (channel counts that are not a multiple of 8).  One thread per output element, fp32
// accumulation in the order (r, s, ci).
#include "dev_common.h"
#include "kernels.h"

namespace bapipe {
namespace {

constexpr int TPB = 256;

// first step r >= 0 for which x + r is a multiple of m
__device__ __forceinline__ int first_tap(int x, int m)
{
    const int q = m == 1 ? 0 : x % m;
    return q > 0 ? m - q : -q;
}

// What bounds it at the sizes of an fp32 stage (tens of thousands of outputs) is the latency of a thread's loads: V
// channels come in one load, and four such loads of each operand are requested before the first product (16 channels,
// 3x3, 32x32 images of four: 24 us with one channel at a time, 5.7 us so).  A tap outside the image reads the nearest pixel
// inside and its sum is not taken, so that no branch stands between the loads of one tap and the next.  In the gradient of
// a strided convolution a pixel only walks the taps that meet an output; walking all and dropping the rest took the backward
// pass of 66 channels, 3x3 / 2, eight 56x56 images from 896 us (taps tested and skipped, one channel at a time) to 1770;
// it is 338 so, and the forward pass 113 after 357 and 380, now that whole groups of channels need no test.
template <class T, int V>
__global__ void k_conv_gather(const T *__restrict__ in, const T *__restrict__ wt,
                              const float *__restrict__ bias, T *out, const T *__restrict__ gate,
                              int accum, int relu, int is_grad, GatherConv g)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)g.N * g.Ho * g.Wo * g.Co;
    if (i >= total) return;
    int ko = (int)(i % g.Co);
    size_t t = i / g.Co;
    int ow = (int)(t % g.Wo);
    t /= g.Wo;
    int oh = (int)(t % g.Ho);
    int n = (int)(t / g.Ho);
    float acc = bias ? bias[ko] : 0.0f;
    const int hn = oh * g.s_out - g.pad_h, wn = ow * g.s_out - g.pad_w;
    // unsigned, for a tap index plus a stride may pass the range of int
    const unsigned r0 = first_tap(hn, g.s_in), s0 = first_tap(wn, g.s_in), step = g.s_in;
    const int ih0 = (int)(hn + r0) / g.s_in, iw0 = (int)(wn + s0) / g.s_in;        // exact
    constexpr int STEP = 4 * V;
    int ih = ih0;
    for (unsigned r = r0; r < (unsigned)g.R; r += step, ++ih) {
        const bool hok = (unsigned)ih < (unsigned)g.Hi;
        const T *row = in + ((size_t)n * g.Hi + (hok ? ih : 0)) * g.Wi * g.Ci;
        const T *wp = wt + (((size_t)ko * g.R + r) * g.S + s0) * g.Ci;
        int iw = iw0;
        for (unsigned s = s0; s < (unsigned)g.S; s += step, ++iw, wp += (size_t)step * g.Ci) {
            const bool ok = hok && (unsigned)iw < (unsigned)g.Wi;
            const T *ip = row + (size_t)(ok ? iw : 0) * g.Ci;
            float sum = acc;
            int c = 0;
            for (; c + STEP <= g.Ci; c += STEP) {
                vec_t<T, V> a[4], b[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = *reinterpret_cast<const vec_t<T, V> *>(ip + c + u * V);
                    b[u] = *reinterpret_cast<const vec_t<T, V> *>(wp + c + u * V);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int j = 0; j < V; ++j) sum = fmaf(to_f32(a[u].e[j]), to_f32(b[u].e[j]), sum);
            }
            if (c < g.Ci) {                              // one to three loads of V channels are left
                vec_t<T, V> a[3], b[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const int cc = c + u * V < g.Ci ? c + u * V : c;
                    a[u] = *reinterpret_cast<const vec_t<T, V> *>(ip + cc);
                    b[u] = *reinterpret_cast<const vec_t<T, V> *>(wp + cc);
                }
#pragma unroll
                for (int u = 0; u < 3; ++u)
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const float t = fmaf(to_f32(a[u].e[j]), to_f32(b[u].e[j]), sum);
                        sum = c + u * V < g.Ci ? t : sum;
                    }
            }
            acc = ok ? sum : acc;
        }
    }
    if (relu) acc = fmaxf(acc, 0.0f);
    if (is_grad) {
        T old = from_f32<T>(0.0f), gt = old;
        if (accum) old = out[i];
        if (gate) gt = gate[i];
        out[i] = grad_out<T>(acc, accum != 0, old, gate != nullptr, gt);
    } else {
        out[i] = from_f32<T>(acc);
    }
}

// The same for a small filter and s_in = 1, out of LDS.  What bounds k_conv_gather at these sizes is the chain of a thread's loads,
// a round of 16 channels per tap, each of them a trip to an L2 that another unit has just written to, and then the L1, for the
// lanes of a wave read as many filter rows as there are output channels.  A block keeps the whole filter in LDS, rows padded to an odd
// number of 16 bytes, and takes tiles of `tw` neighbouring outputs of an image row, whose input it brings in at once: one round of
// loads a tile.  Products are added in the same order, and taps outside the image not at all.  (us, forward: 16->16 channels,
// 3x3, four 32x32 images 6.9 -> 5.1, 3->16 7.1 -> 4.4; 32->32, 16 of 64x64 311 -> 59, 3->32 63 -> 20; 8->8, one 16x16 6.8 -> 4.4.)
// A tile costs a block two barriers and a round of loads whatever is in it, so more tiles than the chip holds blocks must be worth it: 48
// outputs and 4000 products (us, k_conv_gather / here, 1x1 from 16384 rows: 64->64 39.6 / 25.0, 64->16 11.7 / 21.5, 30->64 15.0 / 22.4; 3x3, 2048 images:
// 8->16 at 4x4 22.4 / 17.3, 8->4 at 14x14 64.7 / 57.8, 3->4 there 28.6 / 43.9, 16->4 at 8x8 29.5 / 33.0).  Up to 1024 tiles it is the number of rounds in the
// other kernel's chain that counts (1x1 from 64 rows: 64->4, four, 3.9 / 3.3, 16->4, one, 2.2 / 3.0; 3x3 3->4 at 4x4, 256 images, nine, 5.3 / 4.1),
// and that a filter of 4-byte loads is not fetched for a quarter of a block's threads (150->64, 512 rows 7.8 / 8.9; 150->16 7.5 / 6.0).
constexpr int TILE_FILTER = 10240, TILE_COUT = 64;             // floats of the filter, output channels
constexpr int TILE_INPUT = 4096;                               // floats of a tile's input
template <int V>
__global__ __launch_bounds__(TPB) void k_conv_tile(const float *__restrict__ in, const float *__restrict__ wt, const float *__restrict__ bias,
                                                   float *out, const float *__restrict__ gate, int accum, int relu, int is_grad,
                                                   GatherConv g, int tw, int segments, int tiles, int pitch)
{
    extern __shared__ __align__(16) float lds[];
    typedef vec_t<float, V> vec;
    float *x = lds, *w = lds + TILE_INPUT;
    const int tid = threadIdx.x, K = g.R * g.S * g.Ci, row = ((tw - 1) * g.s_out + g.S) * g.Ci;
    for (int e = tid; e < g.Co * K / V; e += TPB) {
        const int ko = e / (K / V), k = (e - ko * (K / V)) * V;
        *reinterpret_cast<vec *>(w + ko * pitch + k) = *reinterpret_cast<const vec *>(wt + (size_t)e * V);
    }
    const int col = tid / g.Co, ko = tid - col * g.Co;
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int ow0 = tile % segments * tw, nh = tile / segments, n = nh / g.Ho, oh = nh - n * g.Ho;
        const int hn = oh * g.s_out - g.pad_h, w0 = ow0 * g.s_out - g.pad_w;
        for (int e = tid; e < g.R * row / V; e += TPB) {
            const int r = e / (row / V), c = (e - r * (row / V)) * V, iw = w0 + c / g.Ci, ih = hn + r;
            if ((unsigned)ih < (unsigned)g.Hi && (unsigned)iw < (unsigned)g.Wi)
                *reinterpret_cast<vec *>(x + r * row + c) =
                    *reinterpret_cast<const vec *>(in + (((size_t)n * g.Hi + ih) * g.Wi + w0) * g.Ci + c);
        }
        __syncthreads();
        const int ow = ow0 + col;
        if (col < tw && ow < g.Wo) {
            float acc = bias ? bias[ko] : 0.0f;
            const int wn = ow * g.s_out - g.pad_w;
            const int r0 = hn < 0 ? -hn : 0, r1 = g.Hi - hn < g.R ? g.Hi - hn : g.R;
            const int s0 = wn < 0 ? -wn : 0, s1 = g.Wi - wn < g.S ? g.Wi - wn : g.S, len = (s1 - s0) * g.Ci;
            for (int r = r0; r < r1; ++r) {
                const float *a = x + r * row + (col * g.s_out + s0) * g.Ci, *b = w + ko * pitch + (r * g.S + s0) * g.Ci;
                int c = 0;
                for (; c + 6 * V <= len; c += 6 * V) {
                    vec va[6], vb[6];
#pragma unroll
                    for (int u = 0; u < 6; ++u) {
                        va[u] = *reinterpret_cast<const vec *>(a + c + u * V);
                        vb[u] = *reinterpret_cast<const vec *>(b + c + u * V);
                    }
#pragma unroll
                    for (int u = 0; u < 6; ++u)
#pragma unroll
                        for (int j = 0; j < V; ++j) acc = fmaf(va[u].e[j], vb[u].e[j], acc);
                }
                for (; c < len; c += V) {
                    const vec va = *reinterpret_cast<const vec *>(a + c), vb = *reinterpret_cast<const vec *>(b + c);
#pragma unroll
                    for (int j = 0; j < V; ++j) acc = fmaf(va.e[j], vb.e[j], acc);
                }
            }
            if (relu) acc = fmaxf(acc, 0.0f);
            const size_t i = ((size_t)nh * g.Wo + ow) * g.Co + ko;
            if (is_grad) acc = grad_out<float>(acc, accum != 0, accum ? out[i] : 0.0f, gate != nullptr, gate ? gate[i] : 0.0f);
            out[i] = acc;
        }
        __syncthreads();
    }
}

// part[chunk][k][r][s][c] = sum over the chunk's output rows (n,p) and all q of
//   dy[n,p,q,k] * x[n, p*stride+r-pad, q*stride+s-pad, c] ;  chunk = blockIdx.y
// The K elements behind the filter's (bias != 0) are the sums of dy alone.  As two launches of their own behind this one they
// took as long as the rest of a small layer's weight gradient (16 channels, 3x3, four 32x32 images: 8.4 + 2.7 us, and 5.7 + 2.1).
// A wide filter has few chunks, so these sums are long (512->512 3x3, four 28x28 images: 448 pixels a chunk): eights are added
// in float and the eights in double (against 64 bits, normal gradients: 5.9e-8 there, 3.7e-7 one by one in float, 8.5e-8 by
// column sums; all of it in double the smallest stage's mini-batch takes 229 us instead of 218).
template <class T>
__device__ __forceinline__ void wgrad_partial(const T *__restrict__ x, const T *__restrict__ dy, float *__restrict__ part, const ConvShape &c,
                                              int rows_per_chunk, int bias, int bx, int chunk)
{
    size_t i = (size_t)bx * TPB + threadIdx.x;
    const size_t weights = (size_t)c.K * c.R * c.S * c.C, total = weights + (bias ? c.K : 0);
    if (i >= total) return;
    int row0 = chunk * rows_per_chunk, row1 = row0 + rows_per_chunk;
    if (row1 > c.N * c.P) row1 = c.N * c.P;
    float acc = 0.0f;
    if (i >= weights) {
        const T *d = dy + (i - weights);
        const size_t at = (size_t)row0 * c.Q, end = (size_t)row1 * c.Q;      // the chunk's pixels are consecutive
        double sum = 0.0;
        for (size_t p = at; p < end; p += 8) {
            float a[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) a[u] = p + u < end ? to_f32(d[(p + u) * c.K]) : 0.0f;
            sum += (double)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
        }
        part[(size_t)chunk * total + i] = (float)sum;
        return;
    }
    int ci = (int)(i % c.C);
    size_t t = i / c.C;
    int s = (int)(t % c.S);
    t /= c.S;
    int r = (int)(t % c.R);
    int k = (int)(t / c.R);
    for (int row = row0; row < row1; ++row) {
        int n = row / c.P, p = row % c.P;
        int ih = p * c.stride + r - c.pad;
        if (ih < 0 || ih >= c.H) continue;
        const T *dr = dy + ((size_t)n * c.P + p) * c.Q * c.K + k;
        const T *xr = x + ((size_t)n * c.H + ih) * c.W * c.C + ci;
        // output columns whose input column lies in the image; eight of them are requested at once (16 channels, 32x32:
        // 15 -> 8.4 us a launch)
        const int off = s - c.pad;
        const unsigned stride = c.stride;                // a distance plus a stride may pass the range of int
        const int q0 = off < 0 ? (int)((-off + stride - 1) / stride) : 0;
        const int qe = c.W - off > 0 ? (int)((c.W - off + stride - 1) / stride) : 0, q1 = qe < c.Q ? qe : c.Q;
        for (int q = q0; q < q1; q += 8) {
            float a[8], b[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int qq = q + u < q1 ? q + u : q;
                a[u] = to_f32(dr[(size_t)qq * c.K]);
                b[u] = to_f32(xr[(size_t)(qq * c.stride + off) * c.C]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (q + u < q1) acc = fmaf(a[u], b[u], acc);
        }
    }
    part[(size_t)chunk * total + i] = acc;
}

template <class T>
__global__ void k_conv_wgrad_partial(const T *__restrict__ x, const T *__restrict__ dy,
                                     float *__restrict__ part, ConvShape c, int rows_per_chunk, int bias)
{
    wgrad_partial(x, dy, part, c, rows_per_chunk, bias, blockIdx.x, blockIdx.y);
}

// The same of few channels, out of LDS.  k_conv_wgrad_partial loads two values per product and is bound by the L1 that they come from.
// Here a block has the rows of dy and x that a row of outputs meets in LDS, and a thread adds up 4 x V weights of one tap: 4 + V
// values for 4 * V products, each sum in the same order.  (us: 32->32 channels, 3x3, 16 of 64x64 198 -> 42, 3->32 98 -> 13;
// 16->16, four 32x32 images 8.1 either way, and below that, where the two rounds of loads are all there is, the other is faster: 3->16 5.7
// against 5.8, whole mini-batch of 8->8, one 16x16, 165 us against 172.  A thread has 4 x V times the work of the other kernel's, so few rows leave
// the chip idle: a wave and a half for every unit at the least (us with the reductions, other / here, one 64x64 image 8->8 (2816 threads) 8.6 / 12.8, 16->16 (10240)
// 11.0 / 14.0, four (40960) 24.6 / 18.7; 4->64, one (13312) 11.9 / 13.2, one 128x128 (26624) 25.1 / 20.6; 16->16 there (20480) 20.8 / 21.5).)
constexpr int TILE_ROWS = 10240;                               // floats of the rows in LDS
constexpr long long TILE_PRODUCTS = 32768;                     // fewest products of a row of outputs
constexpr long long TILE_THREADS = 24576;                      // fewest threads with weights or sums of their own
template <int V>
__global__ __launch_bounds__(TPB) void k_conv_wgrad_tile(const float *__restrict__ x, const float *__restrict__ dy, float *__restrict__ part,
                                                         ConvShape c, int rows_per_chunk, int bias)
{
    extern __shared__ __align__(16) float lds[];
    typedef vec_t<float, V> vec;
    typedef vec_t<float, 4> vec4;
    float *g = lds, *in = lds + c.Q * c.K;                     // [Q][K], [R][W][C]
    const int tid = threadIdx.x, items = c.K / 4 * c.R * c.S * (c.C / V), item = blockIdx.x * TPB + tid;
    const size_t weights = (size_t)c.K * c.R * c.S * c.C, total = weights + (bias ? c.K : 0);
    const int c0 = item % (c.C / V) * V, tap = item / (c.C / V), s = tap % c.S, r = tap / c.S % c.R, k0 = tap / c.S / c.R * 4;
    const int off = s - c.pad;
    const int q0 = off < 0 ? (-off + c.stride - 1) / c.stride : 0;
    const int qe = c.W > off ? (c.W - off + c.stride - 1) / c.stride : 0, q1 = qe < c.Q ? qe : c.Q;
    const int kb = item - items;                               // >= 0: the sum of dy's column kb
    const bool column = bias && kb >= 0 && kb < c.K;
    float acc[4][V] = {};
    double sum = 0.0;
    const int row0 = blockIdx.y * rows_per_chunk, last = row0 + rows_per_chunk, row1 = last < c.N * c.P ? last : c.N * c.P;
    for (int row = row0; row < row1; ++row) {
        const int n = row / c.P, p = row - n * c.P, h0 = p * c.stride - c.pad;
        if (row > row0) __syncthreads();
        for (int e = tid; e < c.Q * c.K / 4; e += TPB)
            *reinterpret_cast<vec4 *>(g + e * 4) = *reinterpret_cast<const vec4 *>(dy + (size_t)row * c.Q * c.K + e * 4);
        const int line = c.W * c.C;
        for (int e = tid; e < c.R * line / V; e += TPB) {
            const int rr = e / (line / V), at = (e - rr * (line / V)) * V, ih = h0 + rr;
            if ((unsigned)ih < (unsigned)c.H)
                *reinterpret_cast<vec *>(in + rr * line + at) = *reinterpret_cast<const vec *>(x + ((size_t)n * c.H + ih) * line + at);
        }
        __syncthreads();
        if (item < items && (unsigned)(h0 + r) < (unsigned)c.H) {
            const float *a = g + k0, *b = in + r * line + off * c.C + c0;
#pragma unroll 4
            for (int q = q0; q < q1; ++q) {
                const vec4 va = *reinterpret_cast<const vec4 *>(a + q * c.K);
                const vec vb = *reinterpret_cast<const vec *>(b + q * c.stride * c.C);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < V; ++j) acc[i][j] = fmaf(va.e[i], vb.e[j], acc[i][j]);
            }
        }
        if (column)
            for (int q = 0; q < c.Q; q += 8) {
                float a[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) a[u] = q + u < c.Q ? g[(q + u) * c.K + kb] : 0.0f;
                sum += (double)(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])));
            }
    }
    float *dst = part + (size_t)blockIdx.y * total;
    if (column) dst[weights + kb] = (float)sum;
    if (item >= items) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        vec v;
#pragma unroll
        for (int j = 0; j < V; ++j) v.e[j] = acc[i][j];
        *reinterpret_cast<vec *>(dst + (((size_t)(k0 + i) * c.R + r) * c.S + s) * c.C + c0) = v;
    }
}

// dw[i] += sum_chunk part[chunk][i], the elements from `weights` on to db.  LANES threads per element walk the chunks, eight loads requested at once, and their
// sums are added in lane order: a fixed order (bit-reproducible), and chains of chunks / LANES loads (128 chunks of 2304
// elements: 30 us with one lane, 2.7 with 16).  Up to 16 chunks, of which there are that few where the elements alone fill
// the chip, one lane takes them all, for lanes without a chunk are not free (backward pass of a 4096 -> 4096 linear layer,
// one chunk, 3674 -> 3224 us).
constexpr int RED_LANES = 16;
template <int LANES>
__device__ __forceinline__ void wgrad_reduce(const float *__restrict__ part, float *dw, float *db, size_t weights, size_t total, int chunks, int bx)
{
    constexpr int EL = TPB / LANES;
    const int el = threadIdx.x % EL, ln = threadIdx.x / EL;
    const size_t i = (size_t)bx * EL + el;
    double acc = 0.0;
    if (i < total)
        for (int k = ln; k < chunks; k += 8 * LANES) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int kk = k + u * LANES;
                v[u] = kk < chunks ? part[(size_t)kk * total + i] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
    if constexpr (LANES == 1) {
        if (i < total) *(i < weights ? dw + i : db + (i - weights)) += (float)acc;
    } else {
        __shared__ double red[LANES][EL];
        red[ln][el] = acc;
        __syncthreads();
        if (ln == 0 && i < total) {
            double t = 0.0;
#pragma unroll
            for (int l = 0; l < LANES; ++l) t += red[l][el];
            *(i < weights ? dw + i : db + (i - weights)) += (float)t;
        }
    }
}

template <int LANES> __global__ void k_wgrad_reduce(const float *__restrict__ part, float *dw, float *db,
                                                      size_t weights, size_t total, int chunks)
{
    wgrad_reduce<LANES>(part, dw, db, weights, total, chunks, blockIdx.x);
}

// Several small layers' in one launch each (one by one they are 4 to 8 us and a gap, twice a layer: smallest stage, two layers, 175 us a
// mini-batch -> 148): the same sums, the workspace side by side.
constexpr int DIRECT_GROUP = 8;
struct direct_args {
    const float *x, *dy;
    float *part, *dw, *db;
    ConvShape c;
    int rpc, chunks, blocks;                       // rows of a chunk, chunks, blocks of a chunk
    unsigned weights, total;
};
struct direct_group {
    direct_args a[DIRECT_GROUP];
    int n;
};
__global__ __launch_bounds__(TPB) void k_conv_wgrad_partial_group(direct_group in)
{
    int id = blockIdx.x, i = 0;
    while (i + 1 < in.n && id >= in.a[i].blocks * in.a[i].chunks) { id -= in.a[i].blocks * in.a[i].chunks; ++i; }
    const direct_args &j = in.a[i];
    wgrad_partial(j.x, j.dy, j.part, j.c, j.rpc, 1, id % j.blocks, id / j.blocks);
}
__device__ __forceinline__ int direct_sums(unsigned total) { return (int)((total + TPB / RED_LANES - 1) / (TPB / RED_LANES)); }
__global__ __launch_bounds__(TPB) void k_wgrad_reduce_group(direct_group in)
{
    int id = blockIdx.x, i = 0;
    while (i + 1 < in.n && id >= direct_sums(in.a[i].total)) id -= direct_sums(in.a[i++].total);
    const direct_args &j = in.a[i];
    wgrad_reduce<RED_LANES>(j.part, j.dw, j.db, j.weights, j.total, j.chunks, id);
}

constexpr size_t DIRECT_PARTS = (size_t)16 << 20;              // floats of partial sums (64 MiB)
inline size_t direct_wgrad_weights(const ConvShape &c) { return (size_t)c.K * c.R * c.S * c.C; }
inline int direct_wgrad_chunks(const ConvShape &c)
{
    const size_t weights = direct_wgrad_weights(c);
    int rows = c.N * c.P;
    size_t cap = DIRECT_PARTS / (weights ? weights : 1);
    int chunks = rows < 1024 ? rows : 1024;
    if ((size_t)chunks > cap) chunks = (int)cap;
    return chunks < 1 ? 1 : chunks;
}
// The bias gradient rides along where that leaves the filter's sums their chunks (not for 2048->4096, or
// 8->2048 from 911 image rows).
inline size_t direct_wgrad_elements(const ConvShape &c)
{
    const size_t w = direct_wgrad_weights(c);
    return direct_wgrad_chunks(c) * (w + c.K) <= DIRECT_PARTS ? w + c.K : w;
}

// paddings and sides that cannot pass the range of int when they are added
inline bool plain(int side, int pad) { return side > 0 && side < (1 << 20) && pad > -(1 << 20) && pad < (1 << 20); }
// outputs of an image row that a tile of k_conv_tile takes
inline int tile_columns(const GatherConv &g)
{
    int tw = TPB / g.Co;
    while (tw > 1 && g.R * ((tw - 1) * g.s_out + g.S) * g.Ci > TILE_INPUT) --tw;
    return tw < g.Wo ? tw : g.Wo;
}
inline bool tile_takes(const GatherConv &g, bool vec)
{
    if (!(g.s_in == 1 && g.s_out >= 1 && g.s_out <= 16 && g.R <= 16 && g.S <= 16 && g.Co <= TILE_COUT && g.Ci <= TILE_FILTER && plain(g.Hi, g.pad_h) &&
          plain(g.Wi, g.pad_w)))
        return false;
    const int K = g.R * g.S * g.Ci;
    if (!(g.Co * (K + 4) <= TILE_FILTER && K <= TILE_INPUT && (long long)g.N * g.Ho * g.Wo < (1ll << 31))) return false;
    const int tw = tile_columns(g), outputs = tw * g.Co;
    const long long tiles = (long long)g.N * g.Ho * ((g.Wo + tw - 1) / tw);
    if (!vec && outputs < TPB / 2 && g.Co * K > 4096) return false;
    return (outputs >= 48 && outputs * K >= 4000) || (tiles <= 1024 && g.R * g.S * ((g.Ci + 15) / 16) >= 4);
}
// weights (4 x V) and column sums that a chunk of rows has for the threads of k_conv_wgrad_tile
inline int wgrad_tile_items(const ConvShape &c, bool along) { return c.K / 4 * c.R * c.S * (c.C % 4 == 0 ? c.C / 4 : c.C) + (along ? c.K : 0); }
inline bool wgrad_tile_takes(const ConvShape &c, int chunks, bool along)
{
    return c.K % 4 == 0 && c.R <= 16 && c.S <= 16 && c.stride >= 1 && c.stride <= 16 && plain(c.H, c.pad) && plain(c.W, c.pad) && c.Q < (1 << 20) &&
           (long long)c.K * c.C <= 64 * 64 && (long long)c.Q * c.K + (long long)c.R * c.W * c.C <= TILE_ROWS &&
           (long long)c.K * c.C * c.R * c.S * c.Q >= TILE_PRODUCTS && (long long)chunks * wgrad_tile_items(c, along) >= TILE_THREADS;
}

}  // namespace

hipError_t conv_gather_direct(int dt, const void *in, const void *wt, const float *bias, void *out,
                              int relu, GradEpi epi, const GatherConv &g, hipStream_t s)
{
    size_t total = (size_t)g.N * g.Ho * g.Wo * g.Co;
    if (total == 0) return hipSuccess;
    unsigned nb = (unsigned)((total + TPB - 1) / TPB);
    int is_grad = (epi.gate != nullptr || epi.accum) ? 1 : 0;
    // whole 16-byte groups of four floats need a channel count that is a multiple of four and aligned operands
    const bool vec = dt == DT_F32 && g.Ci % 4 == 0 && ((uintptr_t)in | (uintptr_t)wt) % 16 == 0;
    const int K = g.R * g.S * g.Ci;
    if (dt == DT_F32 && tile_takes(g, vec)) {
        const int V = vec ? 4 : 1, pitch = V == 4 ? (K / 4 | 1) * 4 : K | 1, tw = tile_columns(g);
        const int segments = (g.Wo + tw - 1) / tw, tiles = g.N * g.Ho * segments;
        const size_t smem = (size_t)(TILE_INPUT + g.Co * pitch) * sizeof(float);
        const dim3 grid(tiles < 2048 ? tiles : 2048);
        if (V == 4)
            hipLaunchKernelGGL(k_conv_tile<4>, grid, dim3(TPB), smem, s, (const float *)in, (const float *)wt, bias, (float *)out,
                               (const float *)epi.gate, epi.accum, relu, is_grad, g, tw, segments, tiles, pitch);
        else
            hipLaunchKernelGGL(k_conv_tile<1>, grid, dim3(TPB), smem, s, (const float *)in, (const float *)wt, bias, (float *)out,
                               (const float *)epi.gate, epi.accum, relu, is_grad, g, tw, segments, tiles, pitch);
        return hipGetLastError();
    }
#define GATHER_DIRECT(T_, V_)                                                                                        \
    hipLaunchKernelGGL((k_conv_gather<T_, V_>), dim3(nb), dim3(TPB), 0, s, (const T_ *)in, (const T_ *)wt, bias,      \
                       (T_ *)out, (const T_ *)epi.gate, epi.accum, relu, is_grad, g)
    if (vec) GATHER_DIRECT(float, 4);
    else if (dt == DT_F32) GATHER_DIRECT(float, 1);
    else GATHER_DIRECT(bf16_t, 1);
#undef GATHER_DIRECT
    return hipGetLastError();
}

size_t conv_wgrad_direct_workspace(const ConvShape &c)
{
    return (size_t)direct_wgrad_chunks(c) * direct_wgrad_elements(c) * sizeof(float);
}

hipError_t conv_wgrad_direct(int dt, const void *x, const void *dy, float *dw, float *db, void *workspace,
                             const ConvShape &c, hipStream_t s)
{
    const size_t weights = direct_wgrad_weights(c);
    if (weights == 0 || c.N * c.P == 0) return hipSuccess;
    const bool along = db && direct_wgrad_elements(c) > weights;
    const size_t total = weights + (along ? c.K : 0);
    unsigned nb = (unsigned)((total + TPB - 1) / TPB);
    int chunks = direct_wgrad_chunks(c);
    int rpc = (c.N * c.P + chunks - 1) / chunks;
    chunks = (c.N * c.P + rpc - 1) / rpc;
    float *part = (float *)workspace;
    if (dt == DT_F32 && wgrad_tile_takes(c, chunks, along) && ((uintptr_t)x | (uintptr_t)dy) % 16 == 0) {
        const int V = c.C % 4 == 0 ? 4 : 1, items = wgrad_tile_items(c, along);
        const size_t smem = (size_t)(c.Q * c.K + c.R * c.W * c.C) * sizeof(float);
        const dim3 grid((items + TPB - 1) / TPB, chunks);
        if (V == 4)
            hipLaunchKernelGGL(k_conv_wgrad_tile<4>, grid, dim3(TPB), smem, s, (const float *)x, (const float *)dy, part, c, rpc, (int)along);
        else
            hipLaunchKernelGGL(k_conv_wgrad_tile<1>, grid, dim3(TPB), smem, s, (const float *)x, (const float *)dy, part, c, rpc, (int)along);
    } else if (dt == DT_F32)
        hipLaunchKernelGGL((k_conv_wgrad_partial<float>), dim3(nb, chunks), dim3(TPB), 0, s,
                           (const float *)x, (const float *)dy, part, c, rpc, (int)along);
    else
        hipLaunchKernelGGL((k_conv_wgrad_partial<bf16_t>), dim3(nb, chunks), dim3(TPB), 0, s,
                           (const bf16_t *)x, (const bf16_t *)dy, part, c, rpc, (int)along);
    if (chunks <= RED_LANES) {
        hipLaunchKernelGGL(k_wgrad_reduce<1>, dim3(nb), dim3(TPB), 0, s, part, dw, db, weights, total, chunks);
    } else {                                                       // a million elements at most
        constexpr int EL = TPB / RED_LANES;
        hipLaunchKernelGGL(k_wgrad_reduce<RED_LANES>, dim3((unsigned)((total + EL - 1) / EL)), dim3(TPB), 0, s, part, dw, db, weights, total, chunks);
    }
    const hipError_t e = hipGetLastError();
    return db && !along && e == hipSuccess ? colsum_accumulate(dt, dy, c.N * c.P * c.Q, c.K, db, workspace, s) : e;
}

// Small ones that run on k_conv_wgrad_partial with their bias sums and sixteen lanes to add their chunks
bool conv_wgrad_direct_groups(const ConvShape &c)
{
    const size_t weights = direct_wgrad_weights(c), total = direct_wgrad_elements(c);
    if (weights == 0 || (long long)c.N * c.P == 0 || total == weights || total > (1u << 20)) return false;
    int chunks = direct_wgrad_chunks(c);
    const int rpc = (c.N * c.P + chunks - 1) / chunks;
    chunks = (c.N * c.P + rpc - 1) / rpc;
    return chunks > RED_LANES && chunks * ((total + TPB - 1) / TPB) <= 4096 && !wgrad_tile_takes(c, chunks, true);
}

hipError_t conv_wgrad_direct_jobs(const WgradJob *jobs, int n, void *workspace, size_t workspace_bytes, hipStream_t s)
{
    direct_group g;
    g.n = 0;
    size_t used = 0;
    unsigned blocks = 0, sums = 0;
    auto flush = [&]() {
        if (g.n > 1) {
            hipLaunchKernelGGL(k_conv_wgrad_partial_group, dim3(blocks), dim3(TPB), 0, s, g);
            hipLaunchKernelGGL(k_wgrad_reduce_group, dim3(sums), dim3(TPB), 0, s, g);
        } else if (g.n) {
            const direct_args &j = g.a[0];
            const hipError_t e = conv_wgrad_direct(DT_F32, j.x, j.dy, j.dw, j.db, workspace, j.c, s);
            if (e != hipSuccess) return e;
        }
        g.n = 0;
        used = 0;
        blocks = sums = 0;
        return hipGetLastError();
    };
    for (int i = 0; i < n; ++i) {
        const WgradJob &j = jobs[i];
        if (!j.db || j.x2 || !conv_wgrad_direct_groups(j.c)) return hipErrorInvalidValue;
        const size_t own = (conv_wgrad_direct_workspace(j.c) + 255) / 256 * 256;
        if (g.n == DIRECT_GROUP || (g.n && used + own > workspace_bytes)) {
            const hipError_t e = flush();
            if (e != hipSuccess) return e;
        }
        direct_args &a = g.a[g.n++];
        const int want = direct_wgrad_chunks(j.c);
        a = direct_args{(const float *)j.x, (const float *)j.dy, (float *)((char *)workspace + used), j.dw, j.db, j.c, 0, 0, 0,
                        (unsigned)direct_wgrad_weights(j.c), (unsigned)direct_wgrad_elements(j.c)};
        a.rpc = (j.c.N * j.c.P + want - 1) / want;
        a.chunks = (j.c.N * j.c.P + a.rpc - 1) / a.rpc;
        a.blocks = (int)((a.total + TPB - 1) / TPB);
        used += own;
        blocks += (unsigned)(a.blocks * a.chunks);
        sums += (a.total + TPB / RED_LANES - 1) / (TPB / RED_LANES);
    }
    return flush();
}

}  // namespace bapipe

// HBM-bound kernels of a stage: ReLU, 2x2 max-pool, residual add, training-mode batch-norm,
// softmax cross-entropy, SGD update, bias-gradient column sums and boundary layout changes.
// All activations are NHWC, so the channel index is the fastest one: threads own V = 16/sizeof(T)
// consecutive channels (one 16-byte access) and neighbouring threads neighbouring channel
// groups, which keeps every wavefront's HBM access contiguous.
#include "dev_common.h"
#include "kernels.h"
#include <type_traits>

namespace bapipe {
namespace {

constexpr int TPB = 256;

inline unsigned blocks_for(size_t n, int per_block = TPB)
{
    size_t b = (n + per_block - 1) / per_block;
    return (unsigned)(b == 0 ? 1 : b);
}

template <class T> constexpr int vec_width() { return 16 / (int)sizeof(T); }

inline bool aligned16(const void *p) { return (((uintptr_t)p) & 15u) == 0; }

// ------------------------------------------------------------------ flat element-wise
template <class T, int V>
__global__ void k_relu_fwd(const T *__restrict__ x, T *__restrict__ y, size_t nvec)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= nvec) return;
    vec_t<T, V> a = reinterpret_cast<const vec_t<T, V> *>(x)[i], r;
#pragma unroll
    for (int j = 0; j < V; ++j) r.e[j] = from_f32<T>(fmaxf(to_f32(a.e[j]), 0.0f));
    reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
}

template <class T, int V>
__global__ void k_add_fwd(const T *__restrict__ a, const T *__restrict__ b, T *__restrict__ y, int relu,
                          size_t nvec)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= nvec) return;
    vec_t<T, V> va = reinterpret_cast<const vec_t<T, V> *>(a)[i];
    vec_t<T, V> vb = reinterpret_cast<const vec_t<T, V> *>(b)[i], r;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        float v = to_f32(va.e[j]) + to_f32(vb.e[j]);
        if (relu) v = fmaxf(v, 0.0f);
        r.e[j] = from_f32<T>(v);
    }
    reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
}

// dx (+)= dy, gated.  With own_gate the kernel is a stand-alone ReLU backward: the value is
// first zeroed where own_gate <= 0 (own_gate = that ReLU's output).
template <class T, int V>
__global__ void k_grad_copy(const T *__restrict__ dy, const T *__restrict__ own_gate, T *dx,
                            const T *__restrict__ gate, int accum, size_t nvec)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= nvec) return;
    vec_t<T, V> g = reinterpret_cast<const vec_t<T, V> *>(dy)[i];
    vec_t<T, V> og, old, gt, r;
    if (own_gate) og = reinterpret_cast<const vec_t<T, V> *>(own_gate)[i];
    if (accum) old = reinterpret_cast<const vec_t<T, V> *>(dx)[i];
    if (gate) gt = reinterpret_cast<const vec_t<T, V> *>(gate)[i];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        float v = to_f32(g.e[j]);
        if (own_gate && !(to_f32(og.e[j]) > 0.0f)) v = 0.0f;
        r.e[j] = grad_out<T>(v, accum != 0, old.e[j], gate != nullptr, gt.e[j]);
    }
    reinterpret_cast<vec_t<T, V> *>(dx)[i] = r;
}

// ------------------------------------------------------------------ 2x2 stride-2 max-pool
// Maximum and its place in the window of one output position, V channels
template <class T, int V>
__device__ __forceinline__ void pool_max(const vec_t<T, V> *xv, size_t base, int W, int CV, vec_t<T, V> &r, vec_t<uint8_t, V> &ri)
{
    vec_t<T, V> a[4];
    a[0] = xv[base];
    a[1] = xv[base + CV];
    a[2] = xv[base + (size_t)W * CV];
    a[3] = xv[base + (size_t)W * CV + CV];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        float best = to_f32(a[0].e[j]);
        int bi = 0;
#pragma unroll
        for (int k = 1; k < 4; ++k) {
            float v = to_f32(a[k].e[j]);
            if (v > best) {                       // strictly greater: the first maximum wins
                best = v;
                bi = k;
            }
        }
        r.e[j] = from_f32<T>(best);
        ri.e[j] = (uint8_t)bi;
    }
}

// The gradient of one output position, V channels, to the four inputs of its window.  The last column or row of an odd size is in no
// window: the positions next to it store its zeros (a launch that filled dx with them first took 2.5 us and the gap behind it).
template <class T, int V>
__device__ __forceinline__ void pool_spread(const vec_t<T, V> &g, const vec_t<uint8_t, V> &ix, const vec_t<T, V> &gt, bool gated, vec_t<T, V> *dxv,
                                            int accum, size_t base, int H, int W, int CV, int p, int q)
{
    const size_t off[4] = {0, (size_t)CV, (size_t)W * CV, (size_t)W * CV + CV};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        vec_t<T, V> old, r;
        if (accum) old = dxv[base + off[k]];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float v = (ix.e[j] == k) ? to_f32(g.e[j]) : 0.0f;
            r.e[j] = grad_out<T>(v, accum != 0, old.e[j], gated, gt.e[j]);
        }
        dxv[base + off[k]] = r;
    }
    if (accum) return;
    const vec_t<T, V> zero = {};
    const bool right = (W & 1) && 2 * q + 3 == W, below = (H & 1) && 2 * p + 3 == H;
    if (right) {
        dxv[base + 2 * off[1]] = zero;
        dxv[base + off[2] + 2 * off[1]] = zero;
    }
    if (below) {
        dxv[base + 2 * off[2]] = zero;
        dxv[base + 2 * off[2] + off[1]] = zero;
    }
    if (right && below) dxv[base + 2 * off[2] + 2 * off[1]] = zero;
}

template <class T, int V>
__global__ void k_pool_fwd(const T *__restrict__ x, T *__restrict__ y, uint8_t *__restrict__ idx, int N,
                           int H, int W, int CV)
{
    const int Ho = H / 2, Wo = W / 2;
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)N * Ho * Wo * CV;
    if (i >= total) return;
    int cv = (int)(i % CV);
    size_t t = i / CV;
    int q = (int)(t % Wo);
    t /= Wo;
    int p = (int)(t % Ho);
    int n = (int)(t / Ho);
    vec_t<T, V> r;
    vec_t<uint8_t, V> ri;
    pool_max(reinterpret_cast<const vec_t<T, V> *>(x), (((size_t)n * H + 2 * p) * W + 2 * q) * CV + cv, W, CV, r, ri);
    reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
    reinterpret_cast<vec_t<uint8_t, V> *>(idx)[i] = ri;
}

template <class T, int V>
__global__ void k_pool_bwd(const T *__restrict__ dy, const uint8_t *__restrict__ idx, T *dx,
                           const T *__restrict__ gate, int accum, int N, int H, int W, int CV)
{
    const int Ho = H / 2, Wo = W / 2;
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)N * Ho * Wo * CV;
    if (i >= total) return;
    int cv = (int)(i % CV);
    size_t t = i / CV;
    int q = (int)(t % Wo);
    t /= Wo;
    int p = (int)(t % Ho);
    int n = (int)(t / Ho);
    vec_t<T, V> g = reinterpret_cast<const vec_t<T, V> *>(dy)[i];
    vec_t<uint8_t, V> ix = reinterpret_cast<const vec_t<uint8_t, V> *>(idx)[i];
    vec_t<T, V> gt;
    if (gate) gt = reinterpret_cast<const vec_t<T, V> *>(gate)[i];
    pool_spread(g, ix, gt, gate != nullptr, reinterpret_cast<vec_t<T, V> *>(dx), accum, (((size_t)n * H + 2 * p) * W + 2 * q) * CV + cv, H, W,
                CV, p, q);
}

// The same at the end of a stage whose neighbours keep their tensors in NCHW: the pooled values leave, and their gradient comes, in that
// layout through LDS, 64 channels x PX positions of one sample a block, instead of in a launch of its own (mini-batches on one stream:
// float, 16 channels, four 32x32 images 194 -> 177 us; VGG stage 1 of five 90x90 images 394 -> 374).  grid: (position tiles, channel
// tiles, samples)
template <int V> struct pool_tile {
    static constexpr int CG = 64 / V, PX = TPB / CG;
};
template <class T, int V>
__global__ __launch_bounds__(TPB) void k_pool_fwd_nchw(const T *__restrict__ x, T *__restrict__ y, uint8_t *__restrict__ idx, T *__restrict__ y2,
                                                       int H, int W, int C)
{
    constexpr int CG = pool_tile<V>::CG, PX = pool_tile<V>::PX;
    __shared__ T tile[64][PX + 1];
    const int Ho = H / 2, Wo = W / 2, outs = Ho * Wo, CV = C / V;
    const int cl = threadIdx.x % CG, px = threadIdx.x / CG, cv = blockIdx.y * CG + cl, o0 = blockIdx.x * PX, o = o0 + px;
    const size_t n = blockIdx.z;
    if (o < outs && cv < CV) {
        vec_t<T, V> r;
        vec_t<uint8_t, V> ri;
        pool_max(reinterpret_cast<const vec_t<T, V> *>(x), ((n * H + 2 * (o / Wo)) * W + 2 * (o % Wo)) * CV + cv, W, CV, r, ri);
        const size_t i = (n * outs + o) * CV + cv;
        reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
        reinterpret_cast<vec_t<uint8_t, V> *>(idx)[i] = ri;
#pragma unroll
        for (int j = 0; j < V; ++j) tile[cl * V + j][px] = r.e[j];
    }
    __syncthreads();
#pragma unroll 4
    for (int e = threadIdx.x; e < 64 * PX; e += TPB) {
        const int c = blockIdx.y * 64 + e / PX, at = o0 + e % PX;
        if (c < C && at < outs) y2[(n * C + c) * outs + at] = tile[e / PX][e % PX];
    }
}

template <class T, int V>
__global__ __launch_bounds__(TPB) void k_pool_bwd_nchw(const T *__restrict__ dy, const uint8_t *__restrict__ idx, T *dx,
                                                       const T *__restrict__ gate, int accum, int H, int W, int C)
{
    constexpr int CG = pool_tile<V>::CG, PX = pool_tile<V>::PX;
    __shared__ T tile[64][PX + 1];
    const int Ho = H / 2, Wo = W / 2, outs = Ho * Wo, CV = C / V;
    const int cl = threadIdx.x % CG, px = threadIdx.x / CG, cv = blockIdx.y * CG + cl, o0 = blockIdx.x * PX, o = o0 + px;
    const size_t n = blockIdx.z, i = (n * outs + o) * CV + cv;
    const bool here = o < outs && cv < CV;
    vec_t<uint8_t, V> ix;
    vec_t<T, V> g, gt;
    if (here) ix = reinterpret_cast<const vec_t<uint8_t, V> *>(idx)[i];
    if (here && gate) gt = reinterpret_cast<const vec_t<T, V> *>(gate)[i];
#pragma unroll 4
    for (int e = threadIdx.x; e < 64 * PX; e += TPB) {
        const int c = blockIdx.y * 64 + e / PX, at = o0 + e % PX;
        if (c < C && at < outs) tile[e / PX][e % PX] = dy[(n * C + c) * outs + at];
    }
    __syncthreads();
    if (!here) return;
#pragma unroll
    for (int j = 0; j < V; ++j) g.e[j] = tile[cl * V + j][px];
    const int p = o / Wo, q = o % Wo;
    pool_spread(g, ix, gt, gate != nullptr, reinterpret_cast<vec_t<T, V> *>(dx), accum, ((n * H + 2 * p) * W + 2 * q) * CV + cv, H, W, CV, p, q);
}

// ------------------------------------------------------------------ windowed pooling (any window / stride / pad)
struct PoolWin {
    int N, H, W, CV, Ho, Wo, kh, kw, stride, pad;
};

// Max over the in-image part of each window, first maximum in row-major window order; the index
// stored is dh*kw + dw of the winner inside the (padded) window.
template <class T, int V>
__global__ void k_poolw_fwd(const T *__restrict__ x, T *__restrict__ y, uint8_t *__restrict__ idx, PoolWin g)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)g.N * g.Ho * g.Wo * g.CV;
    if (i >= total) return;
    int cv = (int)(i % g.CV);
    size_t t = i / g.CV;
    int q = (int)(t % g.Wo);
    t /= g.Wo;
    int p = (int)(t % g.Ho);
    int n = (int)(t / g.Ho);
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    float best[V];
    int bi[V];
#pragma unroll
    for (int j = 0; j < V; ++j) { best[j] = 0.0f; bi[j] = -1; }
    for (int dh = 0; dh < g.kh; ++dh) {
        const int ih = p * g.stride + dh - g.pad;
        if (ih < 0 || ih >= g.H) continue;
        for (int dw = 0; dw < g.kw; ++dw) {
            const int iw = q * g.stride + dw - g.pad;
            if (iw < 0 || iw >= g.W) continue;
            vec_t<T, V> a = xv[(((size_t)n * g.H + ih) * g.W + iw) * g.CV + cv];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                float v = to_f32(a.e[j]);
                if (bi[j] < 0 || v > best[j]) { best[j] = v; bi[j] = dh * g.kw + dw; }
            }
        }
    }
    vec_t<T, V> r;
    vec_t<uint8_t, V> ri;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        r.e[j] = from_f32<T>(best[j]);
        ri.e[j] = (uint8_t)(bi[j] < 0 ? 0 : bi[j]);
    }
    reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
    reinterpret_cast<vec_t<uint8_t, V> *>(idx)[i] = ri;
}

// Windows of any size and stride.  One thread per INPUT position: it visits the windows that contain the position (in (p,q)
// order, so the sum is reproducible) and adds the gradient of those whose arg-max it is.
// `gate`, indexed like dy, holds the pooled forward values: a window whose maximum is not
// positive passes nothing (its winner was zeroed by the producer's ReLU).
template <class T, int V>
__global__ void k_poolw_bwd(const T *__restrict__ dy, const uint8_t *__restrict__ idx, T *dx,
                            const T *__restrict__ gate, int accum, PoolWin g)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)g.N * g.H * g.W * g.CV;
    if (i >= total) return;
    int cv = (int)(i % g.CV);
    size_t t = i / g.CV;
    int w = (int)(t % g.W);
    t /= g.W;
    int h = (int)(t % g.H);
    int n = (int)(t / g.H);
    const int hp = h + g.pad, wp = w + g.pad;
    int p0 = hp - g.kh + 1, q0 = wp - g.kw + 1;
    p0 = p0 <= 0 ? 0 : (p0 + g.stride - 1) / g.stride;
    q0 = q0 <= 0 ? 0 : (q0 + g.stride - 1) / g.stride;
    int p1 = hp / g.stride, q1 = wp / g.stride;
    p1 = p1 < g.Ho - 1 ? p1 : g.Ho - 1;
    q1 = q1 < g.Wo - 1 ? q1 : g.Wo - 1;
    float acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = 0.0f;
    for (int p = p0; p <= p1; ++p)
        for (int q = q0; q <= q1; ++q) {
            const size_t o = (((size_t)n * g.Ho + p) * g.Wo + q) * g.CV + cv;
            const int want = (hp - p * g.stride) * g.kw + (wp - q * g.stride);
            vec_t<uint8_t, V> ix = reinterpret_cast<const vec_t<uint8_t, V> *>(idx)[o];
            vec_t<T, V> gv = reinterpret_cast<const vec_t<T, V> *>(dy)[o], gt;
            if (gate) gt = reinterpret_cast<const vec_t<T, V> *>(gate)[o];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                bool take = ix.e[j] == want;
                if (gate) take = take && to_f32(gt.e[j]) > 0.0f;
                acc[j] += take ? to_f32(gv.e[j]) : 0.0f;
            }
        }
    vec_t<T, V> *dxv = reinterpret_cast<vec_t<T, V> *>(dx);
    vec_t<T, V> old, r;
    if (accum) old = dxv[i];
#pragma unroll
    for (int j = 0; j < V; ++j) r.e[j] = grad_out<T>(acc[j], accum != 0, old.e[j], false, old.e[j]);
    dxv[i] = r;
}

// Windows of 3 or 4 at stride 2: the 2 x 2 positions 2P .. 2P + 1, 2Q .. 2Q + 1 of the padded image meet only the
// windows P - 1, P by Q - 1, Q.  One thread takes the four positions: four windows, requested together, where four threads
// request nine, one after the other.  Same sums in the same order.  Bound by HBM (bf16, with the gate, us, position by position ->
// so: 3x3, 32 images of 112x112x64 41.0 -> 27.1, 3.5 TB/s; 10 of 56x56x64 7.3 -> 5.9; 4x4, 16 of 112x112x64 25.6 -> 16.9).
// Windows of 2 do not overlap and are one request a position already (16 of 112x112x64 padded by 1, with the gate: 15.0 against
// 15.4, and added to what is stored 16.3 against 18.9).
template <class T, int V>
__global__ void k_poolw_bwd_cells(const T *__restrict__ dy, const uint8_t *__restrict__ idx, T *dx,
                                  const T *__restrict__ gate, int accum, PoolWin g, unsigned cells_h, unsigned cells_w, unsigned total)
{
    const unsigned i = blockIdx.x * TPB + threadIdx.x;
    if (i >= total) return;
    const unsigned cell = i / (unsigned)g.CV, row = cell / cells_w;
    const int cv = (int)(i % (unsigned)g.CV), Q = (int)(cell % cells_w), P = (int)(row % cells_h), n = (int)(row / cells_h);
    const int h0 = 2 * P - g.pad, w0 = 2 * Q - g.pad;
    vec_t<uint8_t, V> ix[2][2];
    vec_t<T, V> gv[2][2], gt[2][2], old[2][2];
    bool in[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int p = P - 1 + u, q = Q - 1 + v;
            in[u][v] = p >= 0 && p < g.Ho && q >= 0 && q < g.Wo;
            const size_t o = in[u][v] ? (((size_t)n * g.Ho + p) * g.Wo + q) * g.CV + cv : 0;
            ix[u][v] = reinterpret_cast<const vec_t<uint8_t, V> *>(idx)[o];
            gv[u][v] = reinterpret_cast<const vec_t<T, V> *>(dy)[o];
            if (gate) gt[u][v] = reinterpret_cast<const vec_t<T, V> *>(gate)[o];
        }
    vec_t<T, V> *dxv = reinterpret_cast<vec_t<T, V> *>(dx);
    auto inside = [&](int a, int b) { return h0 + a >= 0 && h0 + a < g.H && w0 + b >= 0 && w0 + b < g.W; };
    auto at = [&](int a, int b) { return (((size_t)n * g.H + (h0 + a)) * g.W + (w0 + b)) * g.CV + cv; };
    if (accum) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                old[a][b] = dxv[inside(a, b) ? at(a, b) : 0];
    }
    float acc[2][2][V];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int j = 0; j < V; ++j) acc[a][b][j] = 0.0f;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            float d[V];
#pragma unroll
            for (int j = 0; j < V; ++j) {
                bool take = in[u][v];
                if (gate) take = take && to_f32(gt[u][v].e[j]) > 0.0f;
                d[j] = take ? to_f32(gv[u][v].e[j]) : 0.0f;
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const int dh = 2 * (1 - u) + a, dw = 2 * (1 - v) + b, want = dh * g.kw + dw;
                    if (dh >= g.kh || dw >= g.kw) continue;
#pragma unroll
                    for (int j = 0; j < V; ++j) acc[a][b][j] += ix[u][v].e[j] == want ? d[j] : 0.0f;
                }
        }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (!inside(a, b)) continue;
            vec_t<T, V> r;
#pragma unroll
            for (int j = 0; j < V; ++j) r.e[j] = grad_out<T>(acc[a][b][j], accum != 0, old[a][b].e[j], false, old[a][b].e[j]);
            dxv[at(a, b)] = r;
        }
}

// Mean over kh x kw windows at stride (kh, kw), no padding.
template <class T, int V>
__global__ void k_avgpool_fwd(const T *__restrict__ x, T *__restrict__ y, PoolWin g)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)g.N * g.Ho * g.Wo * g.CV;
    if (i >= total) return;
    int cv = (int)(i % g.CV);
    size_t t = i / g.CV;
    int q = (int)(t % g.Wo);
    t /= g.Wo;
    int p = (int)(t % g.Ho);
    int n = (int)(t / g.Ho);
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    float acc[V];
#pragma unroll
    for (int j = 0; j < V; ++j) acc[j] = 0.0f;
    // few threads, each with a long chain of loads (a 7x7 window of 2048 channels and 32 samples is 8192 threads): eight
    // positions are requested at a time, then four, then one: 10.9 us there one by one, 8.9 in batches of eight that were
    // filled up with the last position, 4.6 so (fp32: 8.5, 8.5, 3.9).  Filling up cost where windows are small (2x2, 64
    // channels, 16 images of 112x112: 6.3, 6.7, 4.8 us).
    const vec_t<T, V> *at = xv + (((size_t)n * g.H + p * g.kh) * g.W + q * g.kw) * g.CV + cv;
    int left = g.kh * g.kw, column = 0;
    auto take = [&](auto count) {
        constexpr int B = decltype(count)::value;
        vec_t<T, V> a[B];
#pragma unroll
        for (int u = 0; u < B; ++u) {
            a[u] = *at;
            at += g.CV;
            if (++column == g.kw) {
                column = 0;
                at += (size_t)(g.W - g.kw) * g.CV;
            }
        }
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
            for (int j = 0; j < V; ++j) acc[j] += to_f32(a[u].e[j]);
        left -= B;
    };
    while (left >= 8) take(std::integral_constant<int, 8>());
    if (left >= 4) take(std::integral_constant<int, 4>());
    while (left > 0) take(std::integral_constant<int, 1>());
    const float cnt = (float)(g.kh * g.kw);
    vec_t<T, V> r;
#pragma unroll
    for (int j = 0; j < V; ++j) r.e[j] = from_f32<T>(acc[j] / cnt);
    reinterpret_cast<vec_t<T, V> *>(y)[i] = r;
}

// dx = dy / (kh*kw) for every input of a window, zero outside all windows; gate indexed like dx.
template <class T, int V>
__global__ void k_avgpool_bwd(const T *__restrict__ dy, T *dx, const T *__restrict__ gate, int accum, PoolWin g)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    size_t total = (size_t)g.N * g.H * g.W * g.CV;
    if (i >= total) return;
    int cv = (int)(i % g.CV);
    size_t t = i / g.CV;
    int w = (int)(t % g.W);
    t /= g.W;
    int h = (int)(t % g.H);
    int n = (int)(t / g.H);
    const int p = h / g.kh, q = w / g.kw;
    const bool inside = p < g.Ho && q < g.Wo;
    vec_t<T, V> gv, gt, old, r;
    if (inside) gv = reinterpret_cast<const vec_t<T, V> *>(dy)[(((size_t)n * g.Ho + p) * g.Wo + q) * g.CV + cv];
    if (gate) gt = reinterpret_cast<const vec_t<T, V> *>(gate)[i];
    vec_t<T, V> *dxv = reinterpret_cast<vec_t<T, V> *>(dx);
    if (accum) old = dxv[i];
    const float cnt = (float)(g.kh * g.kw);
#pragma unroll
    for (int j = 0; j < V; ++j) {
        float v = inside ? to_f32(gv.e[j]) / cnt : 0.0f;
        r.e[j] = grad_out<T>(v, accum != 0, old.e[j], gate != nullptr, gt.e[j]);
    }
    dxv[i] = r;
}

// ------------------------------------------------------------------ column reductions
// A [rows][C] matrix is cut into `chunks` row ranges; block (bx, chunk) owns up to TPB channel
// groups... each block reduces its rows for CGB channel groups with RY row lanes, the lanes are
// combined through LDS, and one partial per (chunk, channel, quantity) goes to the workspace.
// A second tiny kernel adds the partials in double.  Fixed partition => bit-reproducible.
struct ColPlan {
    int CV, CGB, RY, chunks, rows_per_chunk, gx;
};

inline ColPlan col_plan(int rows, int C, int V)
{
    ColPlan p;
    p.CV = C / V;
    p.CGB = p.CV < TPB ? p.CV : TPB;
    p.RY = TPB / p.CGB;
    p.gx = (p.CV + p.CGB - 1) / p.CGB;
    int want = (rows + p.RY * 16 - 1) / (p.RY * 16);      // 16 rows per thread: fewer, longer partial blocks measured faster than 8 or 4
    int cap = 1024 / p.gx;
    if (cap < 1) cap = 1;
    p.chunks = want < 1 ? 1 : (want > cap ? cap : want);
    p.rows_per_chunk = (rows + p.chunks - 1) / p.chunks;
    p.chunks = (rows + p.rows_per_chunk - 1) / p.rows_per_chunk;
    if (p.chunks < 1) p.chunks = 1;
    return p;
}

inline int col_vec(int dt, int C, const void *a, const void *b = nullptr, const void *c = nullptr)
{
    int V = dt == DT_F32 ? 4 : 8;
    bool ok = (C % V == 0) && aligned16(a) && aligned16(b) && aligned16(c);
    return ok ? V : 1;
}

// NQ quantities per element computed by functor F(row, channel-vector index, out[NQ][V])
template <class T, int V, int NQ, class F>
__device__ __forceinline__ void col_partial_body(F f, int rows, ColPlan p, float *__restrict__ part, int C)
{
    __shared__ float red[NQ * V * TPB];
    const int cx = threadIdx.x % p.CGB, ry = threadIdx.x / p.CGB;
    const int cg = blockIdx.x * p.CGB + cx;
    const int chunk = blockIdx.y;
    float acc[NQ][V];
#pragma unroll
    for (int qn = 0; qn < NQ; ++qn)
#pragma unroll
        for (int j = 0; j < V; ++j) acc[qn][j] = 0.0f;
    const bool active = ry < p.RY && cg < p.CV;
    if (active) {
        int r0 = chunk * p.rows_per_chunk, r1 = r0 + p.rows_per_chunk;
        if (r1 > rows) r1 = rows;
        // four rows per trip, all loads first (row index clamped, contribution masked): the trip costs one
        // memory round trip instead of four
        for (int r = r0 + ry; r < r1; r += 4 * p.RY) {
            float v[4][NQ][V];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int rr = r + u * p.RY;
                f(rr < r1 ? rr : r1 - 1, cg, v[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float keep = r + u * p.RY < r1 ? 1.0f : 0.0f;
#pragma unroll
                for (int qn = 0; qn < NQ; ++qn)
#pragma unroll
                    for (int j = 0; j < V; ++j) acc[qn][j] += keep * v[u][qn][j];
            }
        }
    }
#pragma unroll
    for (int qn = 0; qn < NQ; ++qn)
#pragma unroll
        for (int j = 0; j < V; ++j) red[(qn * V + j) * TPB + threadIdx.x] = acc[qn][j];
    __syncthreads();
    // All threads add up, one value of a channel group at a time.  A thread for each group, 16 sums of RY values each, left the block's
    // last microseconds to few lanes (256 channels at 56x56, 32 samples, sums of the backward pass 23.3 -> 20.1 us; ResNet stem 4840 -> 4790).
    for (int e = threadIdx.x; e < NQ * V * p.CGB; e += TPB) {
        const int v = e / p.CGB, gx = e - v * p.CGB, g = blockIdx.x * p.CGB + gx;
        if (g >= p.CV) continue;
        float s = 0.0f;
#pragma unroll 8
        for (int k = 0; k < p.RY; ++k) s += red[v * TPB + k * p.CGB + gx];
        part[((size_t)(v / V) * p.chunks + chunk) * C + g * V + v % V] = s;
    }
}

template <class T, int V>
__global__ void k_colsum_partial(const T *__restrict__ a, int rows, int C, ColPlan p, float *part)
{
    const vec_t<T, V> *av = reinterpret_cast<const vec_t<T, V> *>(a);
    auto f = [&](int r, int cg, float(&v)[1][V]) {
        vec_t<T, V> x = av[(size_t)r * p.CV + cg];
#pragma unroll
        for (int j = 0; j < V; ++j) v[0][j] = to_f32(x.e[j]);
    };
    col_partial_body<T, V, 1>(f, rows, p, part, C);
}

// Final pass over the per-chunk partials: a block owns 4 channels, its lanes (256 per channel, 64 where there are no more
// chunks) walk the chunks, eight of them requested at once, and are combined by wave butterflies and then wave by wave
// through LDS: a fixed order, so the result does not depend on scheduling.  Returns true in the lane that holds the totals.
// These launches are a chain of latencies (a megabyte or so of partials, no arithmetic): the trips per lane and the length
// of the last serial sum are what they take.  64 lanes per channel and a serial sum over all of them took 15.6 us for 1568
// chunks of 256 channels and 11 us for 128 channels, against 7.4 and 6.0 now.  Wide tensors have few chunks and many blocks,
// and waves without a chunk cost them (batch-norm of 2560 rows of 16384 floats, all passes: forward 91.7 us with 256 lanes
// per channel, 81.3 with 64; backward 171 and 158).  Neighbouring groups of four channels share cache lines of the partials,
// so they are numbered to run on one XCD.
constexpr int FIN_CH = 4, FIN_AHEAD = 8;
template <int NQ, int NT>
__device__ __forceinline__ bool col_final_sums(const float *__restrict__ part, int chunks, int C, int &c,
                                               double (&tot)[NQ])
{
    constexpr int LANES = NT / FIN_CH, WAVES = NT / 64;
    __shared__ double red[WAVES][NQ][FIN_CH];
    const int cc = threadIdx.x % FIN_CH, cl = threadIdx.x / FIN_CH;
    c = xcd_remap(blockIdx.x, gridDim.x) * FIN_CH + cc;
    double s[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) s[q] = 0.0;
    if (c < C)
        for (int k = cl; k < chunks; k += FIN_AHEAD * LANES) {
            float v[FIN_AHEAD][NQ];
#pragma unroll
            for (int u = 0; u < FIN_AHEAD; ++u) {
                const int kk = k + u * LANES;
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[u][q] = kk < chunks ? part[((size_t)q * chunks + kk) * C + c] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < FIN_AHEAD; ++u)
#pragma unroll
                for (int q = 0; q < NQ; ++q) s[q] += (double)v[u][q];
        }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
        for (int o = FIN_CH; o < 64; o <<= 1) s[q] += __shfl_xor(s[q], o, 64);
        if ((threadIdx.x & 63) < FIN_CH) red[threadIdx.x >> 6][q][cc] = s[q];
    }
    __syncthreads();
    if (cl != 0 || c >= C) return false;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) t += red[k][q][cc];
        tot[q] = t;
    }
    return true;
}

#define LAUNCH_FINAL(kernel, chunks, C, s, ...)                                                              \
    do {                                                                                                     \
        if ((chunks) > 64)                                                                                   \
            hipLaunchKernelGGL((kernel<1024>), dim3(final_blocks(C)), dim3(1024), 0, s, __VA_ARGS__);        \
        else                                                                                                 \
            hipLaunchKernelGGL((kernel<256>), dim3(final_blocks(C)), dim3(256), 0, s, __VA_ARGS__);          \
    } while (0)

inline unsigned final_blocks(int C) { return (unsigned)((C + FIN_CH - 1) / FIN_CH); }

template <int NT>
__global__ __launch_bounds__(NT) void k_colsum_final(const float *__restrict__ part, int chunks, int C, float *out)
{
    int c;
    double t[1];
    if (col_final_sums<1, NT>(part, chunks, C, c, t)) out[c] += (float)t[0];
}

// ------------------------------------------------------------------ batch-norm
template <class T, int V>
__global__ void k_bn_stat_partial(const T *__restrict__ x, int rows, int C, ColPlan p, float *part)
{
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    auto f = [&](int r, int cg, float(&v)[2][V]) {
        vec_t<T, V> a = xv[(size_t)r * p.CV + cg];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float t = to_f32(a.e[j]);
            v[0][j] = t;
            v[1][j] = t * t;
        }
    };
    col_partial_body<T, V, 2>(f, rows, p, part, C);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_bn_stat_final(const float *__restrict__ part, int chunks, int C, int rows, float eps,
                                float *stats)
{
    int c;
    double t[2];
    if (!col_final_sums<2, NT>(part, chunks, C, c, t)) return;
    double m = (double)rows, mu = t[0] / m, var = t[1] / m - mu * mu;
    if (var < 0.0) var = 0.0;
    stats[c] = (float)mu;
    stats[C + c] = (float)(1.0 / sqrt(var + (double)eps));
}

// Normalisation pass.  A thread keeps ONE channel group for its whole life (its V means, inverse
// deviations, gammas and betas sit in registers) and walks down the rows, so that per 16 bytes
// of activations there is one 16-byte load and one 16-byte store and nothing else.  Two rows per
// thread: these launches last a few microseconds, and many short blocks ramp up and drain faster
// than fewer long ones (8 rows per thread cost the ResNet stage 4 %).
constexpr int BN_ROWS_PER_THREAD = 2;

template <class T, int V>
__global__ void k_bn_apply(const T *__restrict__ x, const float *__restrict__ gamma,
                           const float *__restrict__ beta, const float *__restrict__ stats,
                           T *__restrict__ y, int relu, int rows, int C, ColPlan p,
                           const T *__restrict__ res, int relu_sum, T *__restrict__ y2)
{
    // res: the other input of a residual ADD that only this layer's output feeds - y = [relu](q(bn(x)) + res),
    // the normalised value rounded to storage first, as the stand-alone ADD would have read it
    // y2, if any, receives the same values: the stage's output beside its stashed copy
    const int cx = threadIdx.x % p.CGB, ry = threadIdx.x / p.CGB;
    const int cg = blockIdx.x * p.CGB + cx;
    if (ry >= p.RY || cg >= p.CV) return;
    float mu[V], inv[V], ga[V], be[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = stats[cg * V + j];
        inv[j] = stats[C + cg * V + j];
        ga[j] = gamma[cg * V + j];
        be[j] = beta[cg * V + j];
    }
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    vec_t<T, V> *yv = reinterpret_cast<vec_t<T, V> *>(y);
    const int r0 = blockIdx.y * (p.RY * BN_ROWS_PER_THREAD);
    int r1 = r0 + p.RY * BN_ROWS_PER_THREAD;
    if (r1 > rows) r1 = rows;
    vec_t<T, V> a[BN_ROWS_PER_THREAD], b[BN_ROWS_PER_THREAD];
#pragma unroll
    for (int u = 0; u < BN_ROWS_PER_THREAD; ++u) {            // all loads of the thread first
        const int r = r0 + ry + u * p.RY;
        a[u] = xv[(size_t)(r < r1 ? r : r1 - 1) * p.CV + cg];
        if (res) b[u] = reinterpret_cast<const vec_t<T, V> *>(res)[(size_t)(r < r1 ? r : r1 - 1) * p.CV + cg];
    }
#pragma unroll
    for (int u = 0; u < BN_ROWS_PER_THREAD; ++u) {
        const int r = r0 + ry + u * p.RY;
        if (r >= r1) break;
        vec_t<T, V> o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            float v = ga[j] * xh + be[j];
            if (relu) v = fmaxf(v, 0.0f);
            if (res) {
                v = round_to<T>(v) + to_f32(b[u].e[j]);
                if (relu_sum) v = fmaxf(v, 0.0f);
            }
            o.e[j] = from_f32<T>(v);
        }
        yv[(size_t)r * p.CV + cg] = o;
        if (y2) reinterpret_cast<vec_t<T, V> *>(y2)[(size_t)r * p.CV + cg] = o;
    }
}

template <class T, int V>
__global__ void k_bn_bwd_partial(const T *__restrict__ x, const T *__restrict__ dy,
                                 const float *__restrict__ stats, int rows, int C, ColPlan p, float *part)
{
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    const vec_t<T, V> *gv = reinterpret_cast<const vec_t<T, V> *>(dy);
    int cg0 = blockIdx.x * p.CGB + threadIdx.x % p.CGB;
    if (cg0 >= p.CV) cg0 = p.CV - 1;
    float mu[V], inv[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = stats[cg0 * V + j];
        inv[j] = stats[C + cg0 * V + j];
    }
    auto f = [&](int r, int cg, float(&v)[2][V]) {
        vec_t<T, V> a = xv[(size_t)r * p.CV + cg];
        vec_t<T, V> g = gv[(size_t)r * p.CV + cg];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float gg = to_f32(g.e[j]);
            float xh = (to_f32(a.e[j]) - mu[j]) * inv[j];
            v[0][j] = gg;
            v[1][j] = gg * xh;
        }
    };
    col_partial_body<T, V, 2>(f, rows, p, part, C);
}

// sums[c] = (sum dy, sum dy*xhat) of this micro-batch; dbeta/dgamma accumulate over micro-batches
template <int NT>
__global__ __launch_bounds__(NT) void k_bn_bwd_final(const float *__restrict__ part, int chunks, int C, float *sums,
                               float *dgamma, float *dbeta)
{
    int c;
    double t[2];
    if (!col_final_sums<2, NT>(part, chunks, C, c, t)) return;
    sums[c] = (float)t[0];
    sums[C + c] = (float)t[1];
    dbeta[c] += (float)t[0];
    dgamma[c] += (float)t[1];
}

template <class T, int V>
__global__ void k_bn_bwd_apply(const T *__restrict__ x, const T *__restrict__ dy,
                               const float *__restrict__ gamma, const float *__restrict__ stats,
                               const float *__restrict__ sums, T *dx, const T *__restrict__ gate,
                               int accum, float inv_m, int rows, int C, ColPlan p)
{
    const int cx = threadIdx.x % p.CGB, ry = threadIdx.x / p.CGB;
    const int cg = blockIdx.x * p.CGB + cx;
    if (ry >= p.RY || cg >= p.CV) return;
    float mu[V], inv[V], gi[V], m1[V], m2[V];          // mean, 1/std, gamma/std, sum(dy)/m, sum(dy*xhat)/m
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = stats[cg * V + j];
        inv[j] = stats[C + cg * V + j];
        gi[j] = gamma[cg * V + j] * inv[j];
        m1[j] = sums[cg * V + j] * inv_m;
        m2[j] = sums[C + cg * V + j] * inv_m;
    }
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    const vec_t<T, V> *gv = reinterpret_cast<const vec_t<T, V> *>(dy);
    const vec_t<T, V> *tv = reinterpret_cast<const vec_t<T, V> *>(gate);
    vec_t<T, V> *dv = reinterpret_cast<vec_t<T, V> *>(dx);
    const int r0 = blockIdx.y * (p.RY * BN_ROWS_PER_THREAD);
    int r1 = r0 + p.RY * BN_ROWS_PER_THREAD;
    if (r1 > rows) r1 = rows;
    vec_t<T, V> a[BN_ROWS_PER_THREAD], g[BN_ROWS_PER_THREAD], old[BN_ROWS_PER_THREAD], gt[BN_ROWS_PER_THREAD];
    // All loads of the thread first: dx may be one of the tensors read, so the compiler does not move a row's loads ahead of the
    // store of the row before (100352 rows of 64 channels 13.5 -> 12.6 us, 25088 of 256 11.5 -> 10.6, of 512 with the gate
    // 19.9 -> 19.7; four rows a thread 12.9, 10.8 and 21.2).
#pragma unroll
    for (int u = 0; u < BN_ROWS_PER_THREAD; ++u) {
        const int r = r0 + ry + u * p.RY;
        const size_t i = (size_t)(r < r1 ? r : r1 - 1) * p.CV + cg;
        a[u] = xv[i];
        g[u] = gv[i];
        if (accum) old[u] = dv[i];
        if (gate) gt[u] = tv[i];
    }
#pragma unroll
    for (int u = 0; u < BN_ROWS_PER_THREAD; ++u) {
        const int r = r0 + ry + u * p.RY;
        if (r >= r1) break;
        vec_t<T, V> o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            float v = gi[j] * (to_f32(g[u].e[j]) - m1[j] - xh * m2[j]);
            o.e[j] = grad_out<T>(v, accum != 0, old[u].e[j], gate != nullptr, gt[u].e[j]);
        }
        dv[(size_t)r * p.CV + cg] = o;
    }
}

// ------------------------------------------------------------------ batch-norm passes that add the partial sums themselves
// Where there are few chunks of partial sums a launch of its own to add them is mostly launch: a block of these passes owns
// 64 channels of some rows, requests its rows, adds its channels' partials meanwhile (eight lanes a channel, in double, in the
// same order in every block) and goes on.  The first row block of a slice leaves the statistics / the parameter gradients.
constexpr int BI_NT = 512, BI_CH = 64, BI_LANES = BI_NT / BI_CH, BI_AHEAD = 8;
struct slice_lds {
    double red[BI_LANES][2][BI_CH], tot[2][BI_CH];
    float a[BI_CH], b[BI_CH];
};
__device__ __forceinline__ void slice_sums(const float *__restrict__ part, int chunks, int C, int c0, slice_lds &l)
{
    const int ch = threadIdx.x % BI_CH, ln = threadIdx.x / BI_CH, c = c0 + ch < C ? c0 + ch : C - 1;
    double s[2] = {0.0, 0.0};
    for (int k = ln; k < chunks; k += BI_AHEAD * BI_LANES) {
        float v[BI_AHEAD][2];
#pragma unroll
        for (int u = 0; u < BI_AHEAD; ++u) {
            const int kk = k + u * BI_LANES;
#pragma unroll
            for (int q = 0; q < 2; ++q) v[u][q] = kk < chunks ? part[((size_t)q * chunks + kk) * C + c] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < BI_AHEAD; ++u)
#pragma unroll
            for (int q = 0; q < 2; ++q) s[q] += (double)v[u][q];
    }
    l.red[ln][0][ch] = s[0];
    l.red[ln][1][ch] = s[1];
    __syncthreads();
    if (threadIdx.x < 2 * BI_CH) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < BI_LANES; ++k) t += l.red[k][threadIdx.x / BI_CH][ch];
        l.tot[threadIdx.x / BI_CH][ch] = t;
    }
    __syncthreads();
}

template <class T, int V, int U>
__global__ __launch_bounds__(BI_NT) void k_bn_apply_sums(const T *__restrict__ x, const float *__restrict__ gamma,
                                                         const float *__restrict__ beta, const float *__restrict__ part, int chunks,
                                                         float eps, float *__restrict__ stats, T *__restrict__ y, int relu, int rows,
                                                         int C, const T *__restrict__ res, int relu_sum, T *__restrict__ y2)
{
    constexpr int CGS = BI_CH / V, RY = BI_NT / CGS;
    __shared__ slice_lds l;
    const int cx = threadIdx.x % CGS, ry = threadIdx.x / CGS, CV = C / V, c0 = blockIdx.x * BI_CH, cg = c0 / V + cx;
    const int r0 = blockIdx.y * (RY * U) + ry, cgl = cg < CV ? cg : CV - 1;
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x), *bv = reinterpret_cast<const vec_t<T, V> *>(res);
    vec_t<T, V> a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * RY < rows ? r0 + u * RY : rows - 1;
        a[u] = xv[(size_t)r * CV + cgl];
        if (res) b[u] = bv[(size_t)r * CV + cgl];
    }
    slice_sums(part, chunks, C, c0, l);
    if (threadIdx.x < BI_CH) {
        const int c = c0 + threadIdx.x;
        const double m = (double)rows, mu = l.tot[0][threadIdx.x] / m;
        double var = l.tot[1][threadIdx.x] / m - mu * mu;
        if (var < 0.0) var = 0.0;
        const float fm = (float)mu, fi = (float)(1.0 / sqrt(var + (double)eps));
        l.a[threadIdx.x] = fm;
        l.b[threadIdx.x] = fi;
        if (blockIdx.y == 0 && c < C) {
            stats[c] = fm;
            stats[C + c] = fi;
        }
    }
    __syncthreads();
    if (cg >= CV) return;
    float mu[V], inv[V], ga[V], be[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = l.a[cx * V + j];
        inv[j] = l.b[cx * V + j];
        ga[j] = gamma[cg * V + j];
        be[j] = beta[cg * V + j];
    }
    vec_t<T, V> *yv = reinterpret_cast<vec_t<T, V> *>(y);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * RY;
        if (r >= rows) break;
        vec_t<T, V> o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            float v = ga[j] * xh + be[j];
            if (relu) v = fmaxf(v, 0.0f);
            if (res) {                                   // residual ADD behind this layer, see k_bn_apply
                v = round_to<T>(v) + to_f32(b[u].e[j]);
                if (relu_sum) v = fmaxf(v, 0.0f);
            }
            o.e[j] = from_f32<T>(v);
        }
        yv[(size_t)r * CV + cg] = o;
        if (y2) reinterpret_cast<vec_t<T, V> *>(y2)[(size_t)r * CV + cg] = o;
    }
}

template <class T, int V, int U>
__global__ __launch_bounds__(BI_NT) void k_bn_bwd_apply_sums(const T *__restrict__ x, const T *__restrict__ dy,
                                                             const float *__restrict__ gamma, const float *__restrict__ stats,
                                                             const float *__restrict__ part, int chunks, T *dx,
                                                             const T *__restrict__ gate, int accum, float *dgamma, float *dbeta,
                                                             float inv_m, int rows, int C)
{
    constexpr int CGS = BI_CH / V, RY = BI_NT / CGS;
    __shared__ slice_lds l;
    const int cx = threadIdx.x % CGS, ry = threadIdx.x / CGS, CV = C / V, c0 = blockIdx.x * BI_CH, cg = c0 / V + cx;
    const int r0 = blockIdx.y * (RY * U) + ry, cgl = cg < CV ? cg : CV - 1;
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x), *gv = reinterpret_cast<const vec_t<T, V> *>(dy);
    const vec_t<T, V> *tv = reinterpret_cast<const vec_t<T, V> *>(gate);
    vec_t<T, V> *dv = reinterpret_cast<vec_t<T, V> *>(dx);
    vec_t<T, V> a[U], g[U], old[U], gt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t i = (size_t)(r0 + u * RY < rows ? r0 + u * RY : rows - 1) * CV + cgl;
        a[u] = xv[i];
        g[u] = gv[i];
        if (accum) old[u] = dv[i];
        if (gate) gt[u] = tv[i];
    }
    slice_sums(part, chunks, C, c0, l);
    if (blockIdx.y == 0 && threadIdx.x < BI_CH && c0 + threadIdx.x < C) {
        dbeta[c0 + threadIdx.x] += (float)l.tot[0][threadIdx.x];
        dgamma[c0 + threadIdx.x] += (float)l.tot[1][threadIdx.x];
    }
    if (cg >= CV) return;
    float mu[V], inv[V], gi[V], m1[V], m2[V];          // mean, 1/std, gamma/std, sum(dy)/m, sum(dy*xhat)/m
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = stats[cg * V + j];
        inv[j] = stats[C + cg * V + j];
        gi[j] = gamma[cg * V + j] * inv[j];
        m1[j] = (float)l.tot[0][cx * V + j] * inv_m;
        m2[j] = (float)l.tot[1][cx * V + j] * inv_m;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int r = r0 + u * RY;
        if (r >= rows) break;
        vec_t<T, V> o;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            float v = gi[j] * (to_f32(g[u].e[j]) - m1[j] - xh * m2[j]);
            o.e[j] = grad_out<T>(v, accum != 0, old[u].e[j], gate != nullptr, gt[u].e[j]);
        }
        dv[(size_t)r * CV + cg] = o;
    }
}

// ------------------------------------------------------------------ batch-norm in one launch
// For tensors of up to 2048 rows one block owns ONE group of V = 4 channels over ALL rows: every thread keeps its R rows in registers, the block
// reduces the statistics (wave butterflies, then the 16 wave results added in double in wave
// order: fixed order, bit-reproducible), and the same registers are normalised and stored.  The
// activations are read once, nothing goes through a workspace and there is no second launch.
// Neighbouring blocks read and write neighbouring pieces of the same cache lines, so they are numbered to run on one XCD,
// whose L2 then fetches and completes a line once instead of eight caches a piece each (1568 rows of 2048 channels:
// forward 23 -> 12 us, backward 28 -> 14; 784 rows of 1024: 11.8 -> 7.1 and 11.9 -> 7.7).
constexpr int OP_NT = 1024, OP_WAVES = OP_NT / 64;

// Makes the compiler forget what it knows about a register-resident vector (so that values derived
// from it before a reduction are recomputed after it instead of being kept alive in registers).
template <class T, int V>
__device__ __forceinline__ void forget(vec_t<T, V> &a)
{
    static_assert(sizeof(a) % 4 == 0, "whole dwords");
    uint32_t *w = reinterpret_cast<uint32_t *>(&a);
#pragma unroll
    for (int i = 0; i < (int)sizeof(a) / 4; ++i) asm volatile("" : "+v"(w[i]));
}

template <int NQV>
__device__ __forceinline__ void block_sums(float (&v)[NQV], float (*wpart)[NQV], double *tot)
{
#pragma unroll
    for (int q = 0; q < NQV; ++q) v[q] = wave_sum(v[q]);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int q = 0; q < NQV; ++q) wpart[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < NQV) {
        double t = 0.0;
        for (int w = 0; w < OP_WAVES; ++w) t += (double)wpart[w][threadIdx.x];
        tot[threadIdx.x] = t;
    }
    __syncthreads();
}

template <class T, int V, int R>
__global__ __launch_bounds__(OP_NT) void k_bn_fwd_onepass(const T *__restrict__ x, const float *__restrict__ gamma,
                                                          const float *__restrict__ beta, float eps,
                                                          T *__restrict__ y, float *__restrict__ stats, int relu,
                                                          int rows, int C, const T *__restrict__ res, int relu_sum,
                                                          T *__restrict__ y2)
{
    __shared__ float wpart[OP_WAVES][2 * V];
    __shared__ double tot[2 * V];
    __shared__ float mi[2 * V];
    const int CV = C / V, cg = xcd_remap(blockIdx.x, gridDim.x);
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    vec_t<T, V> *yv = reinterpret_cast<vec_t<T, V> *>(y);
    vec_t<T, V> a[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int r = threadIdx.x + u * OP_NT;
        a[u] = xv[(size_t)(r < rows ? r : rows - 1) * CV + cg];
    }
    float acc[2 * V];
#pragma unroll
    for (int j = 0; j < 2 * V; ++j) acc[j] = 0.0f;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const bool in = threadIdx.x + u * OP_NT < rows;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float t = in ? to_f32(a[u].e[j]) : 0.0f;
            acc[j] += t;
            acc[V + j] += t * t;
        }
    }
    block_sums<2 * V>(acc, wpart, tot);
    if (threadIdx.x < V) {
        const double m = (double)rows, mu = tot[threadIdx.x] / m;
        double var = tot[V + threadIdx.x] / m - mu * mu;
        if (var < 0.0) var = 0.0;
        const float fm = (float)mu, fi = (float)(1.0 / sqrt(var + (double)eps));
        mi[threadIdx.x] = fm;
        mi[V + threadIdx.x] = fi;
        stats[cg * V + threadIdx.x] = fm;
        stats[C + cg * V + threadIdx.x] = fi;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < R; ++u) forget(a[u]);
    float mu[V], inv[V], ga[V], be[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = mi[j];
        inv[j] = mi[V + j];
        ga[j] = gamma[cg * V + j];
        be[j] = beta[cg * V + j];
    }
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int r = threadIdx.x + u * OP_NT;
        if (r >= rows) break;
        vec_t<T, V> o, b;
        if (res) b = reinterpret_cast<const vec_t<T, V> *>(res)[(size_t)r * CV + cg];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            float v = ga[j] * xh + be[j];
            if (relu) v = fmaxf(v, 0.0f);
            if (res) {                                   // residual ADD behind this layer, see k_bn_apply
                v = round_to<T>(v) + to_f32(b.e[j]);
                if (relu_sum) v = fmaxf(v, 0.0f);
            }
            o.e[j] = from_f32<T>(v);
        }
        yv[(size_t)r * CV + cg] = o;
        if (y2) reinterpret_cast<vec_t<T, V> *>(y2)[(size_t)r * CV + cg] = o;
    }
}

template <class T, int V, int R>
__global__ __launch_bounds__(OP_NT) void k_bn_bwd_onepass(const T *__restrict__ x, const T *__restrict__ dy,
                                                          const float *__restrict__ gamma,
                                                          const float *__restrict__ stats, T *dx,
                                                          const T *__restrict__ gate, int accum, float *dgamma,
                                                          float *dbeta, float inv_m, int rows, int C)
{
    __shared__ float wpart[OP_WAVES][2 * V];
    __shared__ double tot[2 * V];
    const int CV = C / V, cg = xcd_remap(blockIdx.x, gridDim.x);
    const vec_t<T, V> *xv = reinterpret_cast<const vec_t<T, V> *>(x);
    const vec_t<T, V> *gv = reinterpret_cast<const vec_t<T, V> *>(dy);
    vec_t<T, V> a[R], g[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const int r = threadIdx.x + u * OP_NT;
        const size_t i = (size_t)(r < rows ? r : rows - 1) * CV + cg;
        a[u] = xv[i];
        g[u] = gv[i];
    }
    float mu[V], inv[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        mu[j] = stats[cg * V + j];
        inv[j] = stats[C + cg * V + j];
    }
    float acc[2 * V];
#pragma unroll
    for (int j = 0; j < 2 * V; ++j) acc[j] = 0.0f;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        const bool in = threadIdx.x + u * OP_NT < rows;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const float gg = in ? to_f32(g[u].e[j]) : 0.0f;
            const float xh = (to_f32(a[u].e[j]) - mu[j]) * inv[j];
            acc[j] += gg;
            acc[V + j] += gg * xh;
        }
    }
    block_sums<2 * V>(acc, wpart, tot);
    if (threadIdx.x < V) {
        dbeta[cg * V + threadIdx.x] += (float)tot[threadIdx.x];
        dgamma[cg * V + threadIdx.x] += (float)tot[V + threadIdx.x];
    }
    if (!dx) return;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        forget(a[u]);
        forget(g[u]);
    }
    float gi[V], m1[V], m2[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        gi[j] = gamma[cg * V + j] * inv[j];
        m1[j] = (float)tot[j] * inv_m;
        m2[j] = (float)tot[V + j] * inv_m;
    }
    const vec_t<T, V> *tv = reinterpret_cast<const vec_t<T, V> *>(gate);
    vec_t<T, V> *dv = reinterpret_cast<vec_t<T, V> *>(dx);
    constexpr int G = R < 2 ? R : 2;
#pragma unroll
    for (int h = 0; h < R / G; ++h) {
        vec_t<T, V> old[G], gt[G];
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int r = threadIdx.x + (h * G + u) * OP_NT;
            const size_t i = (size_t)(r < rows ? r : rows - 1) * CV + cg;
            if (accum) old[u] = dv[i];
            if (gate) gt[u] = tv[i];
        }
#pragma unroll
        for (int u = 0; u < G; ++u) {
            const int r = threadIdx.x + (h * G + u) * OP_NT;
            if (r < rows) {
                vec_t<T, V> o;
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    float xh = (to_f32(a[h * G + u].e[j]) - mu[j]) * inv[j];
                    float v = gi[j] * (to_f32(g[h * G + u].e[j]) - m1[j] - xh * m2[j]);
                    o.e[j] = grad_out<T>(v, accum != 0, old[u].e[j], gate != nullptr, gt[u].e[j]);
                }
                dv[(size_t)r * CV + cg] = o;
            }
        }
    }
}

// ------------------------------------------------------------------ LSTM cell
__device__ __forceinline__ float sigmoidf(float v) { return 1.0f / (1.0f + expf(-v)); }

template <class T>
__global__ void k_lstm_cell_fwd(const T *__restrict__ P, const float *__restrict__ gh, int S,
                                float *__restrict__ gates, float *__restrict__ cells, T *__restrict__ h,
                                T *__restrict__ hs, int N, int Tn, int H, int t)
{
    const size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= (size_t)N * H) return;
    const int n = (int)(i / H), j = (int)(i % H);
    const size_t row = (size_t)n * Tn + t;
    float a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        a[q] = to_f32(P[row * 4 * H + (size_t)q * H + j]);
        float rsum = 0.0f;
        for (int sp = 0; sp < S; ++sp) rsum += gh[((size_t)sp * N + n) * 4 * H + (size_t)q * H + j];
        a[q] += rsum;
    }
    const float ig = sigmoidf(a[0]), fg = sigmoidf(a[1]), gg = tanhf(a[2]), og = sigmoidf(a[3]);
    const float cprev = t > 0 ? cells[(row - 1) * H + j] : 0.0f;
    const float c = fg * cprev + ig * gg;
    float *gt = gates + row * 4 * H + j;
    gt[0] = ig;
    gt[H] = fg;
    gt[2 * (size_t)H] = gg;
    gt[3 * (size_t)H] = og;
    cells[row * H + j] = c;
    const T hv = from_f32<T>(og * tanhf(c));
    h[row * H + j] = hv;
    if (t + 1 < Tn) hs[(row + 1) * H + j] = hv;
    if (t == 0) hs[row * H + j] = from_f32<T>(0.0f);
}

template <class T>
__global__ void k_lstm_cell_bwd(const T *__restrict__ dy, const float *__restrict__ r, int S,
                                const float *__restrict__ gates, const float *__restrict__ cells,
                                float *__restrict__ dcn, T *__restrict__ D, int N, int Tn, int H, int t)
{
    const size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= (size_t)N * H) return;
    const int n = (int)(i / H), j = (int)(i % H);
    const size_t row = (size_t)n * Tn + t;
    float dh = to_f32(dy[row * H + j]);
    float rsum = 0.0f;
    for (int sp = 0; sp < S; ++sp) rsum += r[((size_t)sp * N + n) * H + j];
    dh += rsum;
    const float *gt = gates + row * 4 * H + j;
    const float ig = gt[0], fg = gt[H], gg = gt[2 * (size_t)H], og = gt[3 * (size_t)H];
    const float th = tanhf(cells[row * H + j]);
    const float cprev = t > 0 ? cells[(row - 1) * H + j] : 0.0f;
    const float carry = t + 1 < Tn ? dcn[i] : 0.0f;
    const float dc = dh * og * (1.0f - th * th) + carry;
    T *d = D + row * 4 * H + j;
    d[0] = from_f32<T>(dc * gg * ig * (1.0f - ig));
    d[H] = from_f32<T>(dc * cprev * fg * (1.0f - fg));
    d[2 * (size_t)H] = from_f32<T>(dc * ig * (1.0f - gg * gg));
    d[3 * (size_t)H] = from_f32<T>(dh * th * og * (1.0f - og));
    dcn[i] = dc * fg;
}

// ------------------------------------------------------------------ softmax cross-entropy
// A row of up to N * TPB classes stays in registers between its maximum, its sum and its store (1000 classes, 64 rows: 5.0 ->
// 3.7 us); wider rows (N = 0) are read three times.  p2, if any, receives the same values: the output beside the stashed copy.
template <class T, int N>
__global__ void k_softmax_fwd(const T *__restrict__ z, float *__restrict__ p, float *__restrict__ p2, int K)
{
    __shared__ float sh[2][TPB / 64];
    const size_t row = (size_t)blockIdx.x * K;
    const T *zr = z + row;
    float v[N ? N : 1];
    float mx = -INFINITY;
    if constexpr (N > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int k = threadIdx.x + j * TPB;
            v[j] = k < K ? to_f32(zr[k]) : -INFINITY;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) mx = fmaxf(mx, v[j]);
    } else {
        for (int k = threadIdx.x; k < K; k += TPB) mx = fmaxf(mx, to_f32(zr[k]));
    }
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) sh[0][threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = sh[0][0];
    for (int i = 1; i < TPB / 64; ++i) mx = fmaxf(mx, sh[0][i]);
    float s = 0.0f;
    if constexpr (N > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (threadIdx.x + j * TPB >= K) break;
            v[j] = expf(v[j] - mx);
            s += v[j];
        }
    } else {
        for (int k = threadIdx.x; k < K; k += TPB) s += expf(to_f32(zr[k]) - mx);
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[1][threadIdx.x >> 6] = s;
    __syncthreads();
    float t = 0.0f;
    for (int i = 0; i < TPB / 64; ++i) t += sh[1][i];
    const float inv = 1.0f / t;
    auto store = [&](int k, float e) {
        p[row + k] = e * inv;
        if (p2) p2[row + k] = e * inv;
    };
    if constexpr (N > 0) {
#pragma unroll
        for (int j = 0; j < N; ++j)
            if (threadIdx.x + j * TPB < K) store(threadIdx.x + j * TPB, v[j]);
    } else {
        for (int k = threadIdx.x; k < K; k += TPB) store(k, expf(to_f32(zr[k]) - mx));
    }
}

// Blocks 0 .. rows - 1: a row of dz.  One more: loss = -scale * sum_n log p[n, label_n] (labels outside [0,K) contribute 0).
// As two launches the second cost 4.6 us of launch (64 rows of 1000 classes).
template <class T>
__global__ void k_xent(const float *__restrict__ p, const int32_t *__restrict__ labels, float scale,
                       T *__restrict__ dz, float *loss, int rows, int K)
{
    const int n = blockIdx.x;
    if (n < rows) {
        const int lab = labels[n];
        for (int k = threadIdx.x; k < K; k += TPB) {
            float v = scale * (p[(size_t)n * K + k] - (k == lab ? 1.0f : 0.0f));
            dz[(size_t)n * K + k] = from_f32<T>(v);
        }
        return;
    }
    __shared__ float sh[TPB / 64];
    float s = 0.0f;
    for (int r = threadIdx.x; r < rows; r += TPB) {
        int lab = labels[r];
        if (lab >= 0 && lab < K) s -= logf(fmaxf(p[(size_t)r * K + lab], 1e-37f));
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int i = 0; i < TPB / 64; ++i) t += sh[i];
        loss[0] = scale * t;
    }
}

// ------------------------------------------------------------------ parameters
__global__ void k_sgd(float *__restrict__ w, float *__restrict__ g, float lr, size_t n)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    w[i] -= lr * g[i];
    g[i] = 0.0f;
}

// Element (row, col) of a matrix of `rows` rows kept in panels of 32 columns, [col / 32][row][32] (GatherConv::wt_panels)
__device__ __forceinline__ size_t panel_at(int row, int col, int rows) { return ((size_t)(col >> 5) * rows + row) * 32 + (col & 31); }

// The whole update of a weight matrix [K][R*S][C]: w -= lr g, g = 0, the working copy, the transposed (flipped) copy of
// the input gradient (see k_dgrad_filter) and the bias, in one pass on 64 x 64 tiles of one tap through LDS; V channels a
// thread and access.  HBM-bound for the big linear layers: as an update and a transposing pass that read the masters
// again VGG-16's first linear layer took 310 + 193 us, 400 us here; for a convolution layer it is one launch of a few
// microseconds instead of three.
template <class T, int V>
__device__ __forceinline__ void sgd_tile(float (&tile)[64][65], float *__restrict__ w, float *__restrict__ g, float lr, T *__restrict__ work, T *__restrict__ wt, int K,
                                         int RS, int C, float *__restrict__ b, float *__restrict__ db, bool work_panels, bool wt_panels, int bx,
                                         int by, int tap)
{
    constexpr int LANES = 64 / V, ROWS = TPB / LANES, TRIPS = 64 / ROWS;
    const int c0 = bx * 64, k0 = by * 64, tap_t = RS - 1 - tap;
    const int tx = threadIdx.x % LANES, ty = threadIdx.x / LANES;
    vec_t<float, V> wv[TRIPS], gv[TRIPS];
#pragma unroll
    for (int i = 0; i < TRIPS; ++i) {
        const int k = k0 + ty + ROWS * i, c = c0 + V * tx;
        if (k < K && c < C) {
            const size_t at = ((size_t)k * RS + tap) * C + c;
            wv[i] = *reinterpret_cast<const vec_t<float, V> *>(w + at);
            gv[i] = *reinterpret_cast<const vec_t<float, V> *>(g + at);
        }
    }
    const vec_t<float, V> zero = {};
#pragma unroll
    for (int i = 0; i < TRIPS; ++i) {
        const int k = k0 + ty + ROWS * i, c = c0 + V * tx;
        if (k < K && c < C) {
            const size_t at = ((size_t)k * RS + tap) * C + c;
            vec_t<T, V> o;
#pragma unroll
            for (int j = 0; j < V; ++j) {
                wv[i].e[j] -= lr * gv[i].e[j];
                o.e[j] = from_f32<T>(wv[i].e[j]);
                tile[ty + ROWS * i][V * tx + j] = wv[i].e[j];
            }
            *reinterpret_cast<vec_t<float, V> *>(w + at) = wv[i];
            *reinterpret_cast<vec_t<float, V> *>(g + at) = zero;
            *reinterpret_cast<vec_t<T, V> *>(work + (work_panels ? panel_at(k, c, K) : at)) = o;
        }
    }
    if (b && bx == 0 && tap == 0 && threadIdx.x < 64 && k0 + (int)threadIdx.x < K) {
        const int k = k0 + threadIdx.x;
        b[k] -= lr * db[k];
        db[k] = 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TRIPS; ++i) {
        const int c = c0 + ty + ROWS * i, k = k0 + V * tx;
        if (c < C && k < K) {
            vec_t<T, V> o;
#pragma unroll
            for (int j = 0; j < V; ++j) o.e[j] = from_f32<T>(tile[V * tx + j][ty + ROWS * i]);
            *reinterpret_cast<vec_t<T, V> *>(wt + (wt_panels ? panel_at(c, k, C) : ((size_t)c * RS + tap_t) * K + k)) = o;
        }
    }
}

template <class T, int V>
__global__ __launch_bounds__(TPB) void k_sgd_matrix(float *__restrict__ w, float *__restrict__ g, float lr, T *__restrict__ work,
                                                    T *__restrict__ wt, int K, int RS, int C, float *__restrict__ b,
                                                    float *__restrict__ db, bool work_panels, bool wt_panels)
{
    __shared__ float tile[64][65];
    sgd_tile<T, V>(tile, w, g, lr, work, wt, K, RS, C, b, db, work_panels, wt_panels, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The updates of a stage's small layers in one launch: matrices (64 x 64 tiles of a tap as above) and plain vectors (K = 0, C elements).
// One by one each was 2 to 6 us and the gap in front of it, nine of them for a bottleneck.
constexpr int SGD_GROUP = 16;
struct sgd_args {
    SgdJob job;
    unsigned blocks;
    bool vec;
};
struct sgd_group {
    sgd_args a[SGD_GROUP];
    int n;
};
template <class T> __global__ __launch_bounds__(TPB) void k_sgd_group(sgd_group in, float lr)
{
    __shared__ float tile[64][65];
    unsigned id = blockIdx.x;
    int i = 0;
    while (i + 1 < in.n && id >= in.a[i].blocks) id -= in.a[i++].blocks;
    const SgdJob &j = in.a[i].job;
    if (j.K == 0) {
        const int at = (int)id * TPB + (int)threadIdx.x;
        if (at < j.C) {
            j.w[at] -= lr * j.g[at];
            j.g[at] = 0.0f;
        }
        return;
    }
    const int tiles_c = (j.C + 63) / 64, tiles_k = (j.K + 63) / 64, t = (int)id / tiles_c;
    auto run = [&](auto width) {
        sgd_tile<T, decltype(width)::value>(tile, j.w, j.g, lr, (T *)j.work, (T *)j.wt, j.K, j.RS, j.C, j.b, j.db, j.work_panels, j.wt_panels,
                                            (int)id % tiles_c, t % tiles_k, t / tiles_k);
    };
    if (in.a[i].vec) run(std::integral_constant<int, 4>());
    else run(std::integral_constant<int, 1>());
}

// C > 0: the matrix has rows of C elements and its copy is kept in panels
template <class T> __global__ void k_recast(const float *__restrict__ w, T *__restrict__ work, size_t n, int C)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i < n) work[C ? panel_at((int)(i / C), (int)(i % C), (int)(n / C)) : i] = from_f32<T>(w[i]);
}

// wt[c][r][s][k] = w[k][R-1-r][S-1-s][c] in storage type: per tap a K x C -> C x K transpose, done
// on 64 x 64 tiles through LDS so that both the fp32 reads (along c) and the writes (along k) are
// contiguous.  grid: (C tiles, K tiles, R*S)
template <class T>
__global__ void k_dgrad_filter(const float *__restrict__ w, T *__restrict__ wt, int K, int R, int S, int C, bool panels)
{
    __shared__ float tile[64][65];
    const int c0 = blockIdx.x * 64, k0 = blockIdx.y * 64;
    const int tap = blockIdx.z, r = tap / S, q = tap - r * S;
    const int src_tap = (R - 1 - r) * S + (S - 1 - q);
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;          // 64 x 4
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int k = k0 + ty + 4 * i, c = c0 + tx;
        tile[ty + 4 * i][tx] = (k < K && c < C) ? w[((size_t)k * R * S + src_tap) * C + c] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int c = c0 + ty + 4 * i, k = k0 + tx;
        if (c < C && k < K) wt[panels ? panel_at(c, k, C) : ((size_t)c * R * S + tap) * K + k] = from_f32<T>(tile[tx][ty + 4 * i]);
    }
}

__global__ void k_fill(float *p, float v, size_t n)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i < n) p[i] = v;
}

// ------------------------------------------------------------------ layout changes
// NCHW (C channels) -> NHWC with Cp >= C physical channels, the extra ones zero
template <class T>
__global__ void k_nchw_to_nhwc(const T *__restrict__ src, T *dst, const T *__restrict__ gate, int accum,
                               int N, int C, int H, int W, int Cp)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;       // index into dst (NHWC)
    size_t total = (size_t)N * Cp * H * W;
    if (i >= total) return;
    int c = (int)(i % Cp);
    size_t t = i / Cp;
    int w = (int)(t % W);
    t /= W;
    int h = (int)(t % H);
    int n = (int)(t / H);
    T v = from_f32<T>(0.0f);
    if (c < C) v = src[(((size_t)n * C + c) * H + h) * W + w];
    if (gate || accum) {
        T old = v, gt = v;
        if (accum) old = dst[i];
        if (gate) gt = gate[i];
        v = grad_out<T>(to_f32(v), accum != 0, old, gate != nullptr, gt);
    }
    dst[i] = v;
}

// NHWC with Cp physical channels -> NCHW with the first C of them
template <class T>
__global__ void k_nhwc_to_nchw(const T *__restrict__ src, T *__restrict__ dst, int N, int C, int H, int W,
                               int Cp)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;       // index into dst (NCHW)
    size_t total = (size_t)N * C * H * W;
    if (i >= total) return;
    int w = (int)(i % W);
    size_t t = i / W;
    int h = (int)(t % H);
    t /= H;
    int c = (int)(t % C);
    int n = (int)(t / C);
    dst[i] = src[(((size_t)n * H + h) * W + w) * Cp + c];
}

// rows x Cs -> rows x Cd (zero fill when Cd > Cs, truncate when Cd < Cs)
template <class T>
__global__ void k_repad(const T *__restrict__ src, T *__restrict__ dst, size_t rows, int Cs, int Cd)
{
    size_t i = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= rows * Cd) return;
    int c = (int)(i % Cd);
    size_t r = i / Cd;
    dst[i] = c < Cs ? src[r * Cs + c] : from_f32<T>(0.0f);
}

// the common case (RGB input padded to 8 bf16 channels): one thread builds one 16-byte pixel
template <int CS>
__global__ void k_repad_to8(const uint16_t *__restrict__ src, uint4 *__restrict__ dst, size_t rows)
{
    size_t r = (size_t)blockIdx.x * TPB + threadIdx.x;
    if (r >= rows) return;
    uint16_t v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) v[c] = c < CS ? src[r * CS + c] : (uint16_t)0;
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16);
    o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16);
    o.w = v[6] | ((uint32_t)v[7] << 16);
    dst[r] = o;
}

#define DISPATCH_T(dt, ...)                        \
    do {                                           \
        if ((dt) == DT_F32) {                      \
            using T = float;                       \
            __VA_ARGS__                            \
        } else {                                   \
            using T = bf16_t;                      \
            __VA_ARGS__                            \
        }                                          \
    } while (0)

#define DISPATCH_TV(dt, vec, ...)                  \
    do {                                           \
        if ((dt) == DT_F32) {                      \
            using T = float;                       \
            if (vec) {                             \
                constexpr int V = 4;               \
                __VA_ARGS__                        \
            } else {                               \
                constexpr int V = 1;               \
                __VA_ARGS__                        \
            }                                      \
        } else {                                   \
            using T = bf16_t;                      \
            if (vec) {                             \
                constexpr int V = 8;               \
                __VA_ARGS__                        \
            } else {                               \
                constexpr int V = 1;               \
                __VA_ARGS__                        \
            }                                      \
        }                                          \
    } while (0)

inline bool flat_vec(int dt, size_t n, const void *a, const void *b = nullptr, const void *c = nullptr,
                     const void *d = nullptr)
{
    size_t V = dt == DT_F32 ? 4 : 8;
    return n % V == 0 && aligned16(a) && aligned16(b) && aligned16(c) && aligned16(d);
}

}  // namespace

// ====================================================================== launchers
hipError_t relu_fwd(int dt, const void *x, void *y, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    bool vec = flat_vec(dt, n, x, y);
    DISPATCH_TV(dt, vec, {
        size_t nv = n / V;
        hipLaunchKernelGGL((k_relu_fwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)x, (T *)y, nv);
    });
    return hipGetLastError();
}

hipError_t relu_bwd(int dt, const void *y, const void *dy, void *dx, GradEpi epi, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    bool vec = flat_vec(dt, n, y, dy, dx, epi.gate);
    DISPATCH_TV(dt, vec, {
        size_t nv = n / V;
        hipLaunchKernelGGL((k_grad_copy<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)dy,
                           (const T *)y, (T *)dx, (const T *)epi.gate, epi.accum, nv);
    });
    return hipGetLastError();
}

hipError_t grad_copy(int dt, const void *dy, void *dx, GradEpi epi, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    bool vec = flat_vec(dt, n, dy, dx, epi.gate);
    DISPATCH_TV(dt, vec, {
        size_t nv = n / V;
        hipLaunchKernelGGL((k_grad_copy<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)dy,
                           (const T *)nullptr, (T *)dx, (const T *)epi.gate, epi.accum, nv);
    });
    return hipGetLastError();
}

hipError_t add_fwd(int dt, const void *a, const void *b, void *y, int relu, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    bool vec = flat_vec(dt, n, a, b, y);
    DISPATCH_TV(dt, vec, {
        size_t nv = n / V;
        hipLaunchKernelGGL((k_add_fwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)a,
                           (const T *)b, (T *)y, relu, nv);
    });
    return hipGetLastError();
}

static bool pool_vec(int dt, int C, const void *a, const void *b, const void *c, const uint8_t *idx)
{
    return C % (dt == DT_F32 ? 4 : 8) == 0 && aligned16(a) && aligned16(b) && aligned16(c) && (uintptr_t)idx % 8 == 0;
}

// Whether the pool of these sizes and places can take or leave the pooled tensor in NCHW as well, and should.  A block has lanes for 64
// channels: of fewer than 12 most idle, which is worth the launch that it saves only for few positions (1x1 convolution and pool, two
// micro-batches, us, conversion by itself -> here: float, 4 / 8 channels, 32768 positions 128 -> 123 and 142 -> 135, 65536 182 -> 183 and
// 190 -> 189, 131072 272 -> 285 and 293 -> 295; bf16, 8 channels, 16384 83 -> 81, 65536 144 -> 152, 401408 516 -> 568; 12 float and 16 bf16
// channels are faster here at all of these sizes, 439 -> 433 and 745 -> 736 at the largest).
static bool pool_nchw(int dt, const void *pooled, int N, int H, int W, int C, bool vec)
{
    return vec && N <= 65535 && C <= 64 * 65535 && (uintptr_t)pooled % dt_size(dt) == 0 && (C >= 12 || (size_t)N * (H / 2) * (W / 2) <= 32768);
}

hipError_t maxpool2x2_fwd(int dt, const void *x, void *y, uint8_t *idx, int N, int H, int W, int C,
                          hipStream_t s, void *y_nchw, bool *stored)
{
    size_t outs = (size_t)N * (H / 2) * (W / 2) * C;
    if (outs == 0) return hipSuccess;
    const bool vec = pool_vec(dt, C, x, y, nullptr, idx);
    if (y_nchw && pool_nchw(dt, y_nchw, N, H, W, C, vec)) {
        *stored = true;
        DISPATCH_T(dt, {
            constexpr int V = vec_width<T>();
            const int px = pool_tile<V>::PX;
            hipLaunchKernelGGL((k_pool_fwd_nchw<T, V>), dim3((unsigned)(((H / 2) * (W / 2) + px - 1) / px), (unsigned)((C + 63) / 64), (unsigned)N),
                               dim3(TPB), 0, s, (const T *)x, (T *)y, idx, (T *)y_nchw, H, W, C);
        });
        return hipGetLastError();
    }
    DISPATCH_TV(dt, vec, {
        size_t nv = outs / V;
        hipLaunchKernelGGL((k_pool_fwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)x, (T *)y,
                           idx, N, H, W, C / V);
    });
    return hipGetLastError();
}

bool maxpool2x2_bwd_takes_nchw(int dt, const void *dy, const uint8_t *idx, const void *dx, const void *gate, int N, int H, int W, int C)
{
    return H >= 2 && W >= 2 && pool_nchw(dt, dy, N, H, W, C, pool_vec(dt, C, dx, gate, nullptr, idx));
}

hipError_t maxpool2x2_bwd(int dt, const void *dy, const uint8_t *idx, void *dx, GradEpi epi, int N, int H,
                          int W, int C, hipStream_t s, bool nchw)
{
    const size_t outs = (size_t)N * (H / 2) * (W / 2) * C, bytes = (size_t)N * H * W * C * dt_size(dt);
    if (((H | W) & 1) && !epi.accum && bytes % 4) return hipErrorInvalidValue;      // what the fill below cannot cover, with windows or without
    if (outs == 0) {                     // no window at all
        if (epi.accum || bytes == 0) return hipSuccess;
        hipLaunchKernelGGL(k_fill, dim3(blocks_for(bytes / 4)), dim3(TPB), 0, s, (float *)dx, 0.0f, bytes / 4);
        return hipGetLastError();
    }
    if (nchw) {
        if (!maxpool2x2_bwd_takes_nchw(dt, dy, idx, dx, epi.gate, N, H, W, C)) return hipErrorInvalidValue;
        DISPATCH_T(dt, {
            constexpr int V = vec_width<T>();
            const int px = pool_tile<V>::PX;
            hipLaunchKernelGGL((k_pool_bwd_nchw<T, V>), dim3((unsigned)(((H / 2) * (W / 2) + px - 1) / px), (unsigned)((C + 63) / 64), (unsigned)N),
                               dim3(TPB), 0, s, (const T *)dy, idx, (T *)dx, (const T *)epi.gate, epi.accum, H, W, C);
        });
        return hipGetLastError();
    }
    const bool vec = pool_vec(dt, C, dy, dx, epi.gate, idx);
    DISPATCH_TV(dt, vec, {
        size_t nv = outs / V;
        hipLaunchKernelGGL((k_pool_bwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)dy, idx,
                           (T *)dx, (const T *)epi.gate, epi.accum, N, H, W, C / V);
    });
    return hipGetLastError();
}

static PoolWin pool_win(int N, int H, int W, int C, int V, int kh, int kw, int stride, int pad)
{
    PoolWin g{N, H, W, C / V, (H + 2 * pad - kh) / stride + 1, (W + 2 * pad - kw) / stride + 1, kh, kw, stride, pad};
    return g;
}

hipError_t maxpool_fwd(int dt, const void *x, void *y, uint8_t *idx, int N, int H, int W, int C, int kh,
                       int kw, int stride, int pad, hipStream_t s, void *y_nchw, bool *stored)
{
    if (kh < 1 || kw < 1 || kh * kw > 255 || stride < 1 || pad < 0 || pad >= kh || pad >= kw ||
        H + 2 * pad < kh || W + 2 * pad < kw)
        return hipErrorInvalidValue;
    if (kh == 2 && kw == 2 && stride == 2 && pad == 0) return maxpool2x2_fwd(dt, x, y, idx, N, H, W, C, s, y_nchw, stored);
    int Vw = dt == DT_F32 ? 4 : 8;
    bool vec = (C % Vw == 0) && aligned16(x) && aligned16(y) && ((uintptr_t)idx % 8 == 0);
    DISPATCH_TV(dt, vec, {
        PoolWin g = pool_win(N, H, W, C, V, kh, kw, stride, pad);
        size_t nv = (size_t)N * g.Ho * g.Wo * g.CV;
        if (nv == 0) return hipSuccess;
        hipLaunchKernelGGL((k_poolw_fwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)x, (T *)y, idx, g);
    });
    return hipGetLastError();
}

hipError_t maxpool_bwd(int dt, const void *dy, const uint8_t *idx, void *dx, GradEpi epi, int N, int H, int W,
                       int C, int kh, int kw, int stride, int pad, hipStream_t s)
{
    if (kh < 1 || kw < 1 || kh * kw > 255 || stride < 1 || pad < 0 || pad >= kh || pad >= kw ||
        H + 2 * pad < kh || W + 2 * pad < kw)
        return hipErrorInvalidValue;
    if (kh == 2 && kw == 2 && stride == 2 && pad == 0) return maxpool2x2_bwd(dt, dy, idx, dx, epi, N, H, W, C, s);
    int Vw = dt == DT_F32 ? 4 : 8;
    bool vec = (C % Vw == 0) && aligned16(dy) && aligned16(dx) && aligned16(epi.gate) && ((uintptr_t)idx % 8 == 0);
    DISPATCH_TV(dt, vec, {
        PoolWin g = pool_win(N, H, W, C, V, kh, kw, stride, pad);
        size_t nv = (size_t)N * H * W * g.CV;
        if (nv == 0) return hipSuccess;
        const size_t cells_h = (size_t)(H - 1 + pad) / 2 + 1, cells_w = (size_t)(W - 1 + pad) / 2 + 1, cells = N * cells_h * cells_w * g.CV;
        if (stride == 2 && kh >= 3 && kw >= 3 && kh <= 4 && kw <= 4 && cells < ((size_t)1 << 31)) {
            hipLaunchKernelGGL((k_poolw_bwd_cells<T, V>), dim3(blocks_for(cells)), dim3(TPB), 0, s, (const T *)dy, idx, (T *)dx,
                               (const T *)epi.gate, epi.accum, g, (unsigned)cells_h, (unsigned)cells_w, (unsigned)cells);
            return hipGetLastError();
        }
        hipLaunchKernelGGL((k_poolw_bwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)dy, idx, (T *)dx,
                           (const T *)epi.gate, epi.accum, g);
    });
    return hipGetLastError();
}

hipError_t avgpool_fwd(int dt, const void *x, void *y, int N, int H, int W, int C, int kh, int kw, hipStream_t s)
{
    if (kh < 1 || kw < 1 || kh > H || kw > W) return hipErrorInvalidValue;
    int Vw = dt == DT_F32 ? 4 : 8;
    bool vec = (C % Vw == 0) && aligned16(x) && aligned16(y);
    DISPATCH_TV(dt, vec, {
        PoolWin g{N, H, W, C / V, H / kh, W / kw, kh, kw, 0, 0};
        size_t nv = (size_t)N * g.Ho * g.Wo * g.CV;
        if (nv == 0) return hipSuccess;
        hipLaunchKernelGGL((k_avgpool_fwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)x, (T *)y, g);
    });
    return hipGetLastError();
}

hipError_t avgpool_bwd(int dt, const void *dy, void *dx, GradEpi epi, int N, int H, int W, int C, int kh, int kw,
                       hipStream_t s)
{
    if (kh < 1 || kw < 1 || kh > H || kw > W) return hipErrorInvalidValue;
    int Vw = dt == DT_F32 ? 4 : 8;
    bool vec = (C % Vw == 0) && aligned16(dy) && aligned16(dx) && aligned16(epi.gate);
    DISPATCH_TV(dt, vec, {
        PoolWin g{N, H, W, C / V, H / kh, W / kw, kh, kw, 0, 0};
        size_t nv = (size_t)N * H * W * g.CV;
        if (nv == 0) return hipSuccess;
        hipLaunchKernelGGL((k_avgpool_bwd<T, V>), dim3(blocks_for(nv)), dim3(TPB), 0, s, (const T *)dy, (T *)dx,
                           (const T *)epi.gate, epi.accum, g);
    });
    return hipGetLastError();
}

size_t colsum_workspace(int rows, int C)
{
    ColPlan p = col_plan(rows, C, 1);           // V = 1 gives the largest chunk count bound
    ColPlan p8 = col_plan(rows, C, (C % 8 == 0) ? 8 : 1);
    ColPlan p4 = col_plan(rows, C, (C % 4 == 0) ? 4 : 1);
    int chunks = p.chunks > p8.chunks ? p.chunks : p8.chunks;
    chunks = chunks > p4.chunks ? chunks : p4.chunks;
    return (size_t)2 * chunks * C * sizeof(float) + 4 * (size_t)C * sizeof(float);
}

size_t bn_workspace(int rows, int C) { return colsum_workspace(rows, C); }

hipError_t colsum_accumulate(int dt, const void *a, int rows, int C, float *out, void *workspace,
                             hipStream_t s)
{
    if (rows <= 0 || C <= 0) return hipSuccess;
    int Vsel = col_vec(dt, C, a);
    float *part = (float *)workspace;
    DISPATCH_TV(dt, Vsel > 1, {
        ColPlan p = col_plan(rows, C, V);
        hipLaunchKernelGGL((k_colsum_partial<T, V>), dim3(p.gx, p.chunks), dim3(TPB), 0, s, (const T *)a, rows,
                           C, p, part);
        LAUNCH_FINAL(k_colsum_final, p.chunks, C, s, part, p.chunks, C, out);
    });
    return hipGetLastError();
}

// The one-launch kernels pay for their strided 8-byte loads (measured: 3x slower than the three
// coalesced launches at 6272 rows), so they are used only where launch latency is all there is:
// 16-byte aligned tensors of at most OP_R rows per thread and at least 32 channel groups.
constexpr int OP_R = 2;
static bool bn_onepass(int Vsel, int rows, int C) { return Vsel > 1 && rows <= OP_R * OP_NT && C / 4 >= 32; }

// channels per block of the one-launch kernels: 8 bytes of bf16 / 16 bytes of float per row
constexpr int OP_V = 4;
#define BN_FWD_OP(T_, R_)                                                                                        \
    hipLaunchKernelGGL((k_bn_fwd_onepass<T_, OP_V, R_>), dim3(C / OP_V), dim3(OP_NT), 0, s, (const T_ *)x, gamma, \
                       beta, eps, (T_ *)y, stats, relu, rows, C, (const T_ *)res, relu_sum, (T_ *)y2)
#define BN_BWD_OP(T_, R_)                                                                                        \
    hipLaunchKernelGGL((k_bn_bwd_onepass<T_, OP_V, R_>), dim3(C / OP_V), dim3(OP_NT), 0, s, (const T_ *)x,        \
                       (const T_ *)dy, gamma, stats, (T_ *)dx, (const T_ *)epi.gate, epi.accum, dgamma, dbeta,    \
                       1.0f / (float)rows, rows, C)

// rows per thread: four loads at a time where that leaves the chip full
static dim3 sums_grid(int rows, int C, int V, int *u)
{
    const int per = BI_NT / (BI_CH / V), slices = (C + BI_CH - 1) / BI_CH;
    auto blocks = [&](int uu) { return (long long)slices * ((rows + per * uu - 1) / (per * uu)); };
    *u = blocks(4) >= 512 ? 4 : blocks(2) >= 512 ? 2 : 1;
    return dim3((unsigned)slices, (unsigned)((rows + per * *u - 1) / (per * *u)));
}

// The statistics' final pass and the normalisation, over `chunks` partial sums at the front of the workspace
static hipError_t bn_fwd_rest(int dt, const void *x, const float *gamma, const float *beta, float eps, void *y, float *stats,
                              int relu, int rows, int C, const float *part, int chunks, int Vsel, hipStream_t s, const void *res,
                              int relu_sum, void *y2)
{
    if (Vsel > 1 && chunks <= kBnSumChunks) {
        int u;
        const dim3 grid = sums_grid(rows, C, Vsel, &u);
#define BN_FWD_SUMS(T_, V_, U_)                                                                                          \
    hipLaunchKernelGGL((k_bn_apply_sums<T_, V_, U_>), grid, dim3(BI_NT), 0, s, (const T_ *)x, gamma, beta, part, chunks, \
                       eps, stats, (T_ *)y, relu, rows, C, (const T_ *)res, relu_sum, (T_ *)y2)
#define BN_U(LAUNCH, T_, V_) do { if (u == 4) LAUNCH(T_, V_, 4); else if (u == 2) LAUNCH(T_, V_, 2); else LAUNCH(T_, V_, 1); } while (0)
        if (dt == DT_F32) BN_U(BN_FWD_SUMS, float, 4);
        else BN_U(BN_FWD_SUMS, bf16_t, 8);
        return hipGetLastError();
    }
    LAUNCH_FINAL(k_bn_stat_final, chunks, C, s, part, chunks, C, rows, eps, stats);
    DISPATCH_TV(dt, Vsel > 1, {
        ColPlan p = col_plan(rows, C, V);
        const int rpb = p.RY * BN_ROWS_PER_THREAD;
        hipLaunchKernelGGL((k_bn_apply<T, V>), dim3(p.gx, (rows + rpb - 1) / rpb), dim3(TPB), 0, s, (const T *)x,
                           gamma, beta, stats, (T *)y, relu, rows, C, p, (const T *)res, relu_sum, (T *)y2);
    });
    return hipGetLastError();
}

hipError_t bn_fwd(int dt, const void *x, const float *gamma, const float *beta, float eps, void *y,
                  float *stats, int relu, int rows, int C, void *workspace, hipStream_t s, int pre_chunks,
                  const void *res, int relu_sum, void *y2)
{
    if (rows <= 0 || C <= 0) return hipSuccess;
    if (res && relu) return hipErrorInvalidValue;          // the layer's own ReLU and a residual behind it exclude each other
    int Vsel = col_vec(dt, C, x, y, res);
    if (!aligned16(y2)) Vsel = 1;
    float *part = (float *)workspace;
    if (pre_chunks > 0)                   // statistics partials came with x: final pass and normalisation only
        return bn_fwd_rest(dt, x, gamma, beta, eps, y, stats, relu, rows, C, part, pre_chunks, Vsel, s, res, relu_sum, y2);
    if (bn_onepass(Vsel, rows, C)) {
        if (dt == DT_F32) BN_FWD_OP(float, OP_R);
        else BN_FWD_OP(bf16_t, OP_R);
        return hipGetLastError();
    }
    int chunks = 0;
    DISPATCH_TV(dt, Vsel > 1, {
        ColPlan p = col_plan(rows, C, V);
        chunks = p.chunks;
        hipLaunchKernelGGL((k_bn_stat_partial<T, V>), dim3(p.gx, p.chunks), dim3(TPB), 0, s, (const T *)x,
                           rows, C, p, part);
    });
    return bn_fwd_rest(dt, x, gamma, beta, eps, y, stats, relu, rows, C, part, chunks, Vsel, s, res, relu_sum, y2);
}

// The sums' final pass (the parameter gradients) and, if anybody reads it, dx
static hipError_t bn_bwd_rest(int dt, const void *x, const void *dy, const float *gamma, const float *stats, void *dx, float *dgamma,
                              float *dbeta, GradEpi epi, int rows, int C, float *part, int chunks, int Vsel, hipStream_t s)
{
    if (dx && Vsel > 1 && chunks <= kBnSumChunks) {
        int u;
        const dim3 grid = sums_grid(rows, C, Vsel, &u);
#define BN_BWD_SUMS(T_, V_, U_)                                                                                           \
    hipLaunchKernelGGL((k_bn_bwd_apply_sums<T_, V_, U_>), grid, dim3(BI_NT), 0, s, (const T_ *)x, (const T_ *)dy, gamma, stats, \
                       part, chunks, (T_ *)dx, (const T_ *)epi.gate, epi.accum, dgamma, dbeta, 1.0f / (float)rows, rows, C)
        if (dt == DT_F32) BN_U(BN_BWD_SUMS, float, 4);
        else BN_U(BN_BWD_SUMS, bf16_t, 8);
        return hipGetLastError();
    }
    float *sums = part + (size_t)2 * chunks * C;
    LAUNCH_FINAL(k_bn_bwd_final, chunks, C, s, part, chunks, C, sums, dgamma, dbeta);
    if (dx) {
        DISPATCH_TV(dt, Vsel > 1, {
            ColPlan p = col_plan(rows, C, V);
            const int rpb = p.RY * BN_ROWS_PER_THREAD;
            hipLaunchKernelGGL((k_bn_bwd_apply<T, V>), dim3(p.gx, (rows + rpb - 1) / rpb), dim3(TPB), 0, s,
                               (const T *)x, (const T *)dy, gamma, stats, sums, (T *)dx, (const T *)epi.gate,
                               epi.accum, 1.0f / (float)rows, rows, C, p);
        });
    }
    return hipGetLastError();
}

hipError_t bn_bwd(int dt, const void *x, const void *dy, const float *gamma, const float *stats, void *dx,
                  float *dgamma, float *dbeta, GradEpi epi, int rows, int C, void *workspace,
                  hipStream_t s, int pre_chunks)
{
    if (rows <= 0 || C <= 0) return hipSuccess;
    int Vsel = col_vec(dt, C, x, dy, dx);
    if (!aligned16(epi.gate)) Vsel = 1;
    float *part = (float *)workspace;
    if (pre_chunks > 0)                   // the sums over dy came with dy: final pass and the dx pass only
        return bn_bwd_rest(dt, x, dy, gamma, stats, dx, dgamma, dbeta, epi, rows, C, part, pre_chunks, Vsel, s);
    if (bn_onepass(Vsel, rows, C)) {
        if (dt == DT_F32) BN_BWD_OP(float, OP_R);
        else BN_BWD_OP(bf16_t, OP_R);
        return hipGetLastError();
    }
    int chunks = 0;
    DISPATCH_TV(dt, Vsel > 1, {
        ColPlan p = col_plan(rows, C, V);
        chunks = p.chunks;
        hipLaunchKernelGGL((k_bn_bwd_partial<T, V>), dim3(p.gx, p.chunks), dim3(TPB), 0, s, (const T *)x,
                           (const T *)dy, stats, rows, C, p, part);
    });
    return bn_bwd_rest(dt, x, dy, gamma, stats, dx, dgamma, dbeta, epi, rows, C, part, chunks, Vsel, s);
}

hipError_t lstm_cell_fwd(int dt, const void *P, const float *gh, int S, float *gates, float *cells, void *h,
                         void *hs, int N, int Tn, int H, int t, hipStream_t s)
{
    if (N <= 0 || H <= 0 || t < 0 || t >= Tn || S < 0 || (t == 0 && S != 0)) return hipErrorInvalidValue;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_lstm_cell_fwd<T>), dim3(blocks_for((size_t)N * H)), dim3(TPB), 0, s, (const T *)P, gh, S,
                           gates, cells, (T *)h, (T *)hs, N, Tn, H, t);
    });
    return hipGetLastError();
}

hipError_t lstm_cell_bwd(int dt, const void *dy, const float *r, int S, const float *gates, const float *cells,
                         float *dcn, void *D, int N, int Tn, int H, int t, hipStream_t s)
{
    if (N <= 0 || H <= 0 || t < 0 || t >= Tn || S < 0 || (t == Tn - 1 && S != 0)) return hipErrorInvalidValue;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_lstm_cell_bwd<T>), dim3(blocks_for((size_t)N * H)), dim3(TPB), 0, s, (const T *)dy, r, S,
                           gates, cells, dcn, (T *)D, N, Tn, H, t);
    });
    return hipGetLastError();
}

hipError_t softmax_fwd(int dt, const void *z, float *p, int rows, int K, hipStream_t s, float *p2)
{
    if (rows <= 0) return hipSuccess;
    DISPATCH_T(dt, {
        if (K <= 4 * TPB)
            hipLaunchKernelGGL((k_softmax_fwd<T, 4>), dim3(rows), dim3(TPB), 0, s, (const T *)z, p, p2, K);
        else
            hipLaunchKernelGGL((k_softmax_fwd<T, 0>), dim3(rows), dim3(TPB), 0, s, (const T *)z, p, p2, K);
    });
    return hipGetLastError();
}

hipError_t xent_bwd(int dt, const float *p, const int32_t *labels, float scale, void *dz, float *loss,
                    int rows, int K, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_xent<T>), dim3(rows + 1), dim3(TPB), 0, s, p, labels, scale, (T *)dz, loss, rows, K);
    });
    return hipGetLastError();
}

static bool sgd_vec(int dt, const SgdJob &j)
{
    // four values per access where rows of both copies and their starts allow it
    const size_t es = dt_size(dt);
    return j.C % 4 == 0 && j.K % 4 == 0 && aligned16(j.w) && aligned16(j.g) && (uintptr_t)j.work % (4 * es) == 0 && (uintptr_t)j.wt % (4 * es) == 0;
}

static hipError_t sgd_alone(int dt, const SgdJob &j, float lr, hipStream_t s)
{
    if (j.K == 0) {
        hipLaunchKernelGGL(k_sgd, dim3(blocks_for(j.C)), dim3(TPB), 0, s, j.w, j.g, lr, (size_t)j.C);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((j.C + 63) / 64), (unsigned)((j.K + 63) / 64), (unsigned)j.RS);
    DISPATCH_T(dt, {
        if (sgd_vec(dt, j))
            hipLaunchKernelGGL((k_sgd_matrix<T, 4>), grid, dim3(TPB), 0, s, j.w, j.g, lr, (T *)j.work, (T *)j.wt, j.K, j.RS, j.C, j.b, j.db,
                               j.work_panels, j.wt_panels);
        else
            hipLaunchKernelGGL((k_sgd_matrix<T, 1>), grid, dim3(TPB), 0, s, j.w, j.g, lr, (T *)j.work, (T *)j.wt, j.K, j.RS, j.C, j.b, j.db,
                               j.work_panels, j.wt_panels);
    });
    return hipGetLastError();
}

hipError_t sgd_update(int dt, const SgdJob *jobs, int n, float lr, hipStream_t s)
{
    sgd_group group;
    group.n = 0;
    unsigned blocks = 0;
    hipError_t e = hipSuccess;
    auto flush = [&]() {
        if (group.n == 1) e = sgd_alone(dt, group.a[0].job, lr, s);
        else if (group.n > 1) {
            DISPATCH_T(dt, { hipLaunchKernelGGL((k_sgd_group<T>), dim3(blocks), dim3(TPB), 0, s, group, lr); });
            e = hipGetLastError();
        }
        group.n = 0;
        blocks = 0;
        return e;
    };
    for (int i = 0; i < n; ++i) {
        const SgdJob &j = jobs[i];
        if ((j.work_panels && (j.RS != 1 || j.C % 32)) || (j.wt_panels && (j.RS != 1 || j.K % 32))) return hipErrorInvalidValue;
        const size_t own = j.K == 0 ? ((size_t)j.C + TPB - 1) / TPB : (size_t)((j.C + 63) / 64) * ((j.K + 63) / 64) * j.RS;
        if (own == 0) continue;
        // Two rounds of the chip are no launch's length: a larger matrix gains nothing by company (two LSTM layers of 1024, four matrices of
        // 1024 tiles, 6200 us a mini-batch by themselves, 6234 together)
        if (own > 512) {
            if ((e = sgd_alone(dt, j, lr, s)) != hipSuccess) return e;
            continue;
        }
        group.a[group.n++] = sgd_args{j, (unsigned)own, j.K && sgd_vec(dt, j)};
        blocks += (unsigned)own;
        if (group.n == SGD_GROUP && flush() != hipSuccess) return e;
    }
    return flush();
}

hipError_t recast(int dt, const float *w, void *work, size_t n, hipStream_t s, int panels_of)
{
    if (n == 0) return hipSuccess;
    if (panels_of % 32 || (panels_of && n % panels_of)) return hipErrorInvalidValue;
    DISPATCH_T(dt, { hipLaunchKernelGGL((k_recast<T>), dim3(blocks_for(n)), dim3(TPB), 0, s, w, (T *)work, n, panels_of); });
    return hipGetLastError();
}

hipError_t make_dgrad_filter(int dt, const float *w, void *wt, int K, int R, int S, int C, hipStream_t s, bool panels)
{
    size_t n = (size_t)K * R * S * C;
    if (n == 0) return hipSuccess;
    if (panels && (R * S != 1 || K % 32)) return hipErrorInvalidValue;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_dgrad_filter<T>), dim3((unsigned)((C + 63) / 64), (unsigned)((K + 63) / 64), (unsigned)(R * S)),
                           dim3(256), 0, s, w, (T *)wt, K, R, S, C, panels);
    });
    return hipGetLastError();
}

hipError_t fill_f32(float *p, float v, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill, dim3(blocks_for(n)), dim3(TPB), 0, s, p, v, n);
    return hipGetLastError();
}

hipError_t nchw_to_nhwc(int dt, const void *src, void *dst, GradEpi epi, int N, int C, int H, int W,
                        int Cp, hipStream_t s)
{
    size_t n = (size_t)N * Cp * H * W;
    if (n == 0) return hipSuccess;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_nchw_to_nhwc<T>), dim3(blocks_for(n)), dim3(TPB), 0, s, (const T *)src, (T *)dst,
                           (const T *)epi.gate, epi.accum, N, C, H, W, Cp);
    });
    return hipGetLastError();
}

hipError_t nhwc_to_nchw(int dt, const void *src, void *dst, int N, int C, int H, int W, int Cp,
                        hipStream_t s)
{
    size_t n = (size_t)N * C * H * W;
    if (n == 0) return hipSuccess;
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_nhwc_to_nchw<T>), dim3(blocks_for(n)), dim3(TPB), 0, s, (const T *)src, (T *)dst,
                           N, C, H, W, Cp);
    });
    return hipGetLastError();
}

hipError_t nhwc_repad(int dt, const void *src, void *dst, size_t rows, int Cs, int Cd, hipStream_t s)
{
    size_t n = rows * Cd;
    if (n == 0) return hipSuccess;
    if (dt == DT_BF16 && Cd == 8 && aligned16(dst) && (Cs == 3 || Cs == 1 || Cs == 4)) {
#define REPAD8(CS_) \
    hipLaunchKernelGGL((k_repad_to8<CS_>), dim3(blocks_for(rows)), dim3(TPB), 0, s, (const uint16_t *)src, (uint4 *)dst, rows)
        if (Cs == 3) REPAD8(3);
        else if (Cs == 1) REPAD8(1);
        else REPAD8(4);
#undef REPAD8
        return hipGetLastError();
    }
    DISPATCH_T(dt, {
        hipLaunchKernelGGL((k_repad<T>), dim3(blocks_for(n)), dim3(TPB), 0, s, (const T *)src, (T *)dst, rows, Cs, Cd);
    });
    return hipGetLastError();
}

hipError_t nhwc_to_nchw_u8(const uint8_t *src, uint8_t *dst, int N, int C, int H, int W, hipStream_t s)
{
    size_t n = (size_t)N * C * H * W;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL((k_nhwc_to_nchw<uint8_t>), dim3(blocks_for(n)), dim3(TPB), 0, s, src, dst, N, C, H, W, C);
    return hipGetLastError();
}

}  // namespace bapipe

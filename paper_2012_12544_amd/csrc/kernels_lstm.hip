// The recurrence of an LSTM layer in one launch per direction (bf16 stages, gfx950).
//
// What bounds it: T dependent steps, each a product with the same recurrent matrix (8 MB in bf16 at hidden 1024) for
// at most a few hundred sequences.  As two launches per step (product, cell) a step costs 13 us whatever its size,
// nearly all of it launch gaps and one block's load - multiply - store chain.  Here the matrix never moves: a block of
// eight waves keeps the rows of 32 hidden units in registers for the whole sequence (128 registers a lane at hidden
// 1024), and a step is the exchange of one small vector.  Hidden 1024, 50 steps, 64 sequences, one direction: 650 us
// before, 203 us (forward) and 211 us (backward) here; of a backward step of 4.4 us 1.9 us are the 16 MB that all
// blocks together read of the step before, 1.2 us the hand-over, 0.6 us the cell.
//
// Split.  16 sequences (the N of the MFMA) form a group, H/32 blocks work on a group, each owns 32 units: their four
// gates in forward (M = 128 rows, K = H in eight pieces, a piece a wave), their rows of W_h^T in backward (M = 32,
// K = 4H, half a gate a wave).  The waves' partial sums meet in LDS; thread i then owns one (sequence, unit) for all
// steps, so the cell state and the cell-gradient carry stay in its register.  Blocks of 16 units (twice the blocks, each
// reading the whole vector) made a backward step 6.1 us; in forward they were faster alone (213 against 240 us) and slower where a
// backward pass runs on another stream, because both launches then want all compute units (11.5 against 10.5 ms for a
// mini-batch of two layers).
//
// Exchange.  A block publishes its 16 x 32 slice with write-through stores (agent scope), waits for them, and then
// raises its own flag word to the number of steps it has finished; a wave polls the flags of the blocks whose slices it
// needs, one flag a lane, and reads the slices with loads of the same scope (a cache-wide acquire per wave and step cost
// twice the whole step: 529 us instead of 228 for 50 steps).  The slices go through a buffer of their own, laid out as
// the operand fragments that read them (1 KB per load instruction): the rows of the layer's tensors lie T * 8H bytes
// apart, all in one L2 channel, and reading them there took 4.7 us of a backward step.  Two copies of the buffer, by the
// parity of the step, are enough: a block that publishes step t+2 has seen every block of its group finish t+1, and
// with that finish reading t.
//
// Why every wait ends.  Blocks number themselves by a ticket taken when they START, so the blocks of the oldest
// unfinished group are resident or the next to start, and the chip has room for them unless other launches of this kind
// hold every slot with incomplete groups of their own: q launches at once hold at most q * (H/32 - 1) blocks that way,
// and the chip has at least 256 slots (one block per compute unit at hidden 1024), so eight launches at once are safe.
// A process runs at most as many kernels at once as it has hardware queues (four by default).  Beyond that a wait gives
// up after kWaitTicks: the group then finishes with NaN results instead of hanging.
#include "kernels.h"
#include "mfma_common.h"

namespace bapipe {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kUnits = 32, kSeqs = 16, kThreads = 512;
constexpr int kCtlWords = 64;                               // words of the ticket line and of each group's flags
constexpr unsigned kPoison = 0xFFFFFFFFu;                   // flag of a block that has given up
constexpr unsigned long long kWaitTicks = 1000000000ull;    // 10 s of the 100 MHz counter
// partial sums in LDS, [wave][row][16 sequences x 4 row groups]: the row pitch of 68 words keeps the 64 lanes of a
// wave, which read 32 units of 2 sequences, on different banks
constexpr int kPitch = 68;

__device__ __forceinline__ float sigmoid_f(float v) { return 1.0f / (1.0f + expf(-v)); }

// wait until flags[0..n) have all reached `need`; false: a block gave up, or the wait did
__device__ bool wait_flags(const unsigned *flags, int n, unsigned need, int lane)
{
    unsigned long long t0 = 0;
    for (unsigned it = 1;; ++it) {
        const unsigned v = lane < n ? __hip_atomic_load(flags + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : need;
        if (__all(v >= need)) {
            asm volatile("" ::: "memory");        // the reads of what was published stay below
            return __all(lane >= n || v != kPoison);
        }
        if ((it & 1023u) == 0) {
            const unsigned long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (now - t0 > kWaitTicks) return false;
        }
    }
}

// the block's published values are complete in memory, then its flag says so
__device__ __forceinline__ void publish(unsigned *flag, unsigned v)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// two neighbouring lanes' bf16 values leave as one 32-bit write-through store (by the even lane)
__device__ __forceinline__ void publish_pair(char *p, bf16_t v)
{
    const unsigned mine = v.v, other = __shfl_xor(mine, 1, 64);
    if (!(threadIdx.x & 1))
        __hip_atomic_store(reinterpret_cast<unsigned *>(p), mine | (other << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ bf16x8_t load_frag(const bf16_t *p) { return as_frag(*reinterpret_cast<const chunk16 *>(p)); }

// an operand fragment that another block has published: 16 bytes a lane, coherent at agent scope (sc1)
__device__ __forceinline__ bf16x8_t load_published(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return as_frag(__builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 16));
}

// byte offset of (k, sequence) in a buffer of K-step fragments: [K/32][lane = (k/8 % 4, sequence)][8]
__device__ __forceinline__ unsigned frag_at(int k, int seq)
{
    return (unsigned)(((k >> 5) * 64 + ((k >> 3) & 3) * 16 + seq) * 8 + (k & 7)) * 2u;
}

// H = 128 * KS
template <int KS>
__global__ __launch_bounds__(kThreads, 1) void k_lstm_seq_fwd(const bf16_t *__restrict__ P, const bf16_t *__restrict__ w_hh,
                                                              float *__restrict__ gates, float *__restrict__ cells,
                                                              bf16_t *__restrict__ h, bf16_t *__restrict__ hs, int N, int T,
                                                              unsigned *ctl, char *slices)
{
    // eight pieces of K where they come out as whole K-steps, else four pieces for each half of the rows
    constexpr int H = 128 * KS, GB = H / kUnits, KP = KS % 2 == 0 ? 8 : 4, MT = KP, KW = H / KP / 32;
    __shared__ float red[KP][32 * kPitch];
    __shared__ int s_ticket, s_dead;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) {
        s_ticket = (int)atomicAdd(ctl, 1u);
        s_dead = 0;
    }
    __syncthreads();
    const int grp = s_ticket / GB, blk = s_ticket % GB;
    unsigned *flags = ctl + (1 + grp) * kCtlWords;
    const int u0 = blk * kUnits, n0 = grp * kSeqs;
    const int row = lane & 15, quad = lane >> 4, kp = wave % KP;
    // row tile i of the block: gate i / 2, units 16 (i % 2) .. + 15; this wave's tile m is
    auto tile = [&](int m) { return KP == 8 ? m : 2 * m + wave / KP; };

    bf16x8_t w[MT][KW];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < KW; ++k)
            w[m][k] = load_frag(w_hh + (size_t)((tile(m) >> 1) * H + u0 + 16 * (tile(m) & 1) + row) * H + (kp * KW + k) * 32 + 8 * quad);

    // sequences past the last repeat it; nothing of theirs is stored in the layer's tensors
    constexpr unsigned SLICES = H * kSeqs * 2;
    char *const mine = slices + (size_t)grp * 2 * SLICES;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(mine, 0, 2 * SLICES, 0x00020000);
    const int sq = tid >> 5, un = tid & 31;
    const bool on = n0 + sq < N;
    const size_t r0 = (size_t)(on ? n0 + sq : N - 1) * T;
    const int u = u0 + un;
    bf16_t p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = P[r0 * 4 * H + q * H + u];
    if (on) hs[r0 * H + u] = from_f32<bf16_t>(0.0f);
    float c = 0.0f;
    bool dead = false;
    for (int t = 0; t < T; ++t) {
        float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (t > 0) {
            // the blocks whose units overlap this wave's piece of K
            constexpr int per = 32 * KW;
            const int f0 = kp * per / kUnits, f1 = ((kp + 1) * per + kUnits - 1) / kUnits;
            if (!dead && !wait_flags(flags + f0, f1 - f0, (unsigned)t, lane)) s_dead = 1;
            f32x4_t acc[MT] = {};
            bf16x8_t b[KW];
#pragma unroll
            for (int k = 0; k < KW; ++k) b[k] = load_published(xr, (t & 1) * SLICES + (unsigned)((kp * KW + k) * 64 + lane) * 16u);
#pragma unroll
            for (int k = 0; k < KW; ++k)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m][k], b[k], acc[m], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[kp][(tile(m) * 4 + r) * kPitch + lane] = acc[m][r];
            __syncthreads();
            dead = s_dead != 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = ((2 * q + (un >> 4)) * 4 + (un & 3)) * kPitch + ((un >> 2) & 3) * 16 + sq;
                s[q] = (red[0][at] + red[1][at]) + (red[2][at] + red[3][at]);
                if (KP == 8) s[q] += (red[KP - 4][at] + red[KP - 3][at]) + (red[KP - 2][at] + red[KP - 1][at]);
            }
        }
        const float ig = sigmoid_f(to_f32(p[0]) + s[0]), fg = sigmoid_f(to_f32(p[1]) + s[1]);
        const float gg = tanhf(to_f32(p[2]) + s[2]), og = sigmoid_f(to_f32(p[3]) + s[3]);
        c = fg * c + ig * gg;
        if (dead) c = __builtin_nanf("");
        const bf16_t hv = from_f32<bf16_t>(og * tanhf(c));
        const size_t r = r0 + t;
        if (t + 1 < T) {
            publish_pair(mine + ((t + 1) & 1) * SLICES + frag_at(u, sq), hv);
            publish(flags + blk, dead ? kPoison : (unsigned)(t + 1));
#pragma unroll
            for (int q = 0; q < 4; ++q) p[q] = P[(r + 1) * 4 * H + q * H + u];
        }
        if (on) {                                  // what nobody waits for
            float *gt = gates + r * 4 * H + u;
            gt[0] = ig;
            gt[H] = fg;
            gt[2 * H] = gg;
            gt[3 * H] = og;
            cells[r * H + u] = c;
            h[r * H + u] = hv;
            if (t + 1 < T) hs[(r + 1) * H + u] = hv;
        }
    }
}

template <int KS>
__global__ __launch_bounds__(kThreads, 1) void k_lstm_seq_bwd(const bf16_t *__restrict__ dy, const bf16_t *__restrict__ wt_h,
                                                                  const float *__restrict__ gates, const float *__restrict__ cells,
                                                                  bf16_t *__restrict__ D, int N, int T, unsigned *ctl, char *slices)
{
    constexpr int H = 128 * KS, GB = H / kUnits, KW = H / 64;      // KW: K-steps of a wave (half a gate)
    __shared__ float red[8][8 * kPitch];
    __shared__ int s_ticket, s_dead;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) {
        s_ticket = (int)atomicAdd(ctl, 1u);
        s_dead = 0;
    }
    __syncthreads();
    const int grp = s_ticket / GB, blk = s_ticket % GB;
    unsigned *flags = ctl + (1 + grp) * kCtlWords;
    const int u0 = blk * kUnits, n0 = grp * kSeqs;
    const int row = lane & 15, quad = lane >> 4;

    bf16x8_t w[2][KW];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int k = 0; k < KW; ++k) w[m][k] = load_frag(wt_h + (size_t)(u0 + 16 * m + row) * 4 * H + wave * (H / 2) + k * 32 + 8 * quad);

    constexpr unsigned SLICES = 4 * H * kSeqs * 2;
    char *const mine = slices + (size_t)grp * 2 * SLICES;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(mine, 0, 2 * SLICES, 0x00020000);
    const int sq = tid >> 5, un = tid & 31;
    const bool on = n0 + sq < N;
    const size_t r0 = (size_t)(on ? n0 + sq : N - 1) * T;
    const int u = u0 + un;
    float carry = 0.0f, g[4], c, cp;
    bf16_t dh0;
    auto fetch = [&](int t) {                      // what step t reads besides D_{t+1}; requested a step ahead
        const size_t r = r0 + t;
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = gates[r * 4 * H + q * H + u];
        c = cells[r * H + u];
        cp = t > 0 ? cells[(r - 1) * H + u] : 0.0f;
        dh0 = dy[r * H + u];
    };
    fetch(T - 1);
    bool dead = false;
    for (int t = T - 1; t >= 0; --t) {
        float s = 0.0f;
        if (t + 1 < T) {
            if (!dead && !wait_flags(flags + (wave & 1) * (GB / 2), GB / 2, (unsigned)(T - 1 - t), lane)) s_dead = 1;
            f32x4_t acc[2][2] = {};
            const unsigned src = ((t + 1) & 1) * SLICES + (unsigned)(wave * KW * 64 + lane) * 16u;
            bf16x8_t b[KW];
#pragma unroll
            for (int k = 0; k < KW; ++k) b[k] = load_published(xr, src + k * 1024);
#pragma unroll
            for (int k = 0; k < KW; ++k)
#pragma unroll
                for (int m = 0; m < 2; ++m) acc[m][k & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m][k], b[k], acc[m][k & 1], 0, 0, 0);
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 4; ++r) red[wave][(m * 4 + r) * kPitch + lane] = acc[m][0][r] + acc[m][1][r];
            __syncthreads();
            dead = s_dead != 0;
            const int at = ((un >> 4) * 4 + (un & 3)) * kPitch + ((un >> 2) & 3) * 16 + sq;
            s = ((red[0][at] + red[1][at]) + (red[2][at] + red[3][at])) + ((red[4][at] + red[5][at]) + (red[6][at] + red[7][at]));
        }
        const float dh = to_f32(dh0) + s, th = tanhf(c);
        float dc = dh * g[3] * (1.0f - th * th) + carry;
        if (dead) dc = __builtin_nanf("");
        const float d[4] = {dc * g[2] * g[0] * (1.0f - g[0]), dc * cp * g[1] * (1.0f - g[1]), dc * g[0] * (1.0f - g[2] * g[2]),
                            dh * th * g[3] * (1.0f - g[3])};
        carry = dc * g[1];
        bf16_t dv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) dv[q] = from_f32<bf16_t>(d[q]);
        if (t > 0) {
#pragma unroll
            for (int q = 0; q < 4; ++q) publish_pair(mine + (t & 1) * SLICES + frag_at(q * H + u, sq), dv[q]);
            publish(flags + blk, dead ? kPoison : (unsigned)(T - t));
            fetch(t - 1);
        }
        if (on) {
#pragma unroll
            for (int q = 0; q < 4; ++q) D[(r0 + t) * 4 * H + q * H + u] = dv[q];
        }
    }
}

int groups_of(int N) { return (N + kSeqs - 1) / kSeqs; }
size_t ctl_bytes(int N) { return (size_t)(1 + groups_of(N)) * kCtlWords * sizeof(unsigned); }

}  // namespace

// Up to hidden 1024 a block's rows fit its registers.  Past a thousand blocks (four rounds of the chip) the two launches
// per step are no longer mostly gaps: a mini-batch of 2 x 512 sequences of 20 steps at hidden 1024 (1024 blocks) takes
// 6.7 ms against 7.5 with them, of 2 x 256 3.7 against 4.9.
bool lstm_seq_supported(int N, int H) { return N > 0 && H % 128 == 0 && H <= 1024 && (long long)groups_of(N) * (H / kUnits) <= 1024; }

// ticket line and flags, then two copies of every group's slices (backward's, the wider ones)
size_t lstm_seq_workspace(int N, int H) { return ctl_bytes(N) + (size_t)groups_of(N) * 2 * 4 * H * kSeqs * 2; }

#define LSTM_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

hipError_t lstm_seq_fwd(const void *P, const void *w_hh, float *gates, float *cells, void *h, void *hs, int N, int T, int H,
                        void *workspace, hipStream_t s)
{
    const hipError_t e = fill_f32((float *)workspace, 0.0f, ctl_bytes(N) / sizeof(float), s);
    if (e != hipSuccess) return e;
    const dim3 grid(groups_of(N) * (H / kUnits));
    switch (H / 128) {
#define X(KS)                                                                                                             \
    case KS:                                                                                                              \
        hipLaunchKernelGGL((k_lstm_seq_fwd<KS>), grid, dim3(kThreads), 0, s, (const bf16_t *)P, (const bf16_t *)w_hh, gates, \
                           cells, (bf16_t *)h, (bf16_t *)hs, N, T, (unsigned *)workspace, (char *)workspace + ctl_bytes(N));                                \
        break;
        LSTM_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t lstm_seq_bwd(const void *dy, const void *wt_h, const float *gates, const float *cells, void *D, int N, int T, int H,
                        void *workspace, hipStream_t s)
{
    const hipError_t e = fill_f32((float *)workspace, 0.0f, ctl_bytes(N) / sizeof(float), s);
    if (e != hipSuccess) return e;
    const dim3 grid(groups_of(N) * (H / kUnits));
    switch (H / 128) {
#define X(KS)                                                                                                              \
    case KS:                                                                                                               \
        hipLaunchKernelGGL((k_lstm_seq_bwd<KS>), grid, dim3(kThreads), 0, s, (const bf16_t *)dy, (const bf16_t *)wt_h, gates, \
                           cells, (bf16_t *)D, N, T, (unsigned *)workspace, (char *)workspace + ctl_bytes(N));                                               \
        break;
        LSTM_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace bapipe

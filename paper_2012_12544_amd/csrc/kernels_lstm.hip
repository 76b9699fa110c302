// The recurrence of an LSTM layer in one launch per direction (bf16 stages, gfx950).
//
// What bounds it: T dependent steps, each a product with the same recurrent matrix (8 MB in bf16 at hidden 1024) for
// at most a few hundred sequences.  As two launches per step (product, cell) a step costs 13 us whatever its size,
// nearly all of it launch gaps and one block's load - multiply - store chain.  Here the matrix never moves: a block of
// eight waves keeps the rows of 32 hidden units in registers for the whole sequence (128 registers a lane at hidden
// 1024), and a step is the exchange of one small vector.  Hidden 1024, 50 steps, 64 sequences, one direction: 650 us
// before, 126 us (forward) and 156 us (backward) here, alone on the chip.  Of a step of 2.5 to 3.1 us most is the way of a
// slice from one unit to the others; in backward all blocks together read 16 MB of the step before, which took 1.9 us of 4.4
// before all its loads were requested first.
//
// Split.  16 sequences (the N of the MFMA) form a group, H/32 blocks work on a group, each owns 32 units: their four
// gates in forward (M = 128 rows, K = H in eight pieces, a piece a wave), their rows of W_h^T in backward (M = 32,
// K = 4H, half a gate a wave).  The waves' partial sums meet in LDS; thread i then owns one (sequence, unit) for all
// steps, so the cell state and the cell-gradient carry stay in its register.  Blocks of 16 units (twice the blocks, each
// reading the whole vector) made a backward step 6.1 us; in forward they were faster alone (213 against 240 us) and slower where a
// backward pass runs on another stream, because both launches then want all compute units (11.5 against 10.5 ms for a
// mini-batch of two layers).
//
// Exchange.  A block publishes its 16 x 32 slice with write-through stores (agent scope), and that is all: a slice starts out
// as words of kUnsent, which no published pair of values is, and a wave reads the slices it needs with loads of the same scope
// until there is no such word left in them.  (A flag word per block that is raised once its stores are complete, polled before
// the slices are read, puts two more trips through the fabric into each step: 172 / 166 us instead of 126 / 156.  Reading one
// word a lane before the whole: 131; reading again only the fragments that had not come: 136 / 174, for its branches.)
// The slices go through a buffer of their own, laid out as
// the operand fragments that read them (1 KB per load instruction): the rows of the layer's tensors lie T * 8H bytes
// apart, all in one L2 channel, and reading them there took 4.7 us of a backward step.
// Four copies of the buffer go round.  At step t (counted from the first that reads a slice), after its barrier, a block has
// seen every block's slice for step t, so every block is done reading those for step t - 1: it makes its own of them kUnsent
// again.  It will publish there for step t + 3.  A block that looks for that slice has seen this block's for step t + 2 before,
// which was stored after a wait for the words of kUnsent: it finds these or the new ones, never the old slice.
//
// Why the launch always ends, and with the right values.  Blocks number themselves by a ticket taken when they START, so
// the blocks of the oldest unfinished group are resident or the next to start, and they find room unless other launches of
// this kind hold every slot with incomplete groups of their own.  q launches at once hold at most q * (H/32 - 1) blocks that
// way; lstm_seq_supported asks for more compute units than eight launches can hold.  More of them (several processes on one
// GPU, a stream confined to a few units) can still leave groups incomplete, and nothing here can see that coming.  So every
// wait is bounded (kLstmWaitPolls), the group's other blocks leave when they see that one has given up (a word that they look
// at every 16 polls), and the first that
// did computes the group's sequences from the start by itself, with nobody to wait for and slices of its own: the same
// operations in the same order, its weights read again for every 32 units and step (hidden 1024, 50 steps: 14 ms).  What the
// others store meanwhile are the same values.
#include "kernels.h"
#include "mfma_common.h"

namespace bapipe {
namespace {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kUnits = 32, kSeqs = 16, kThreads = 512;
// words of the ticket line and of each group's line; its first says whether a block of it has given up
constexpr int kCtlWords = 64;
constexpr unsigned kUnsent = 0xFFFFFFFFu;                   // word of a slice: not yet published
constexpr int kCopies = 4;                                  // of a group's slices
// Partial sums in LDS.  Forward: [wave][unit][16 sequences x 4 gates], 16 bytes a (unit, sequence), the pitch keeps the 16
// lanes that are served together on different banks, those that write 16 sequences and those that read 16 units.  Backward:
// [wave][sequence][32 units], a lane writes the four neighbouring units that it has the sums of.  (One word at a time, 32
// accesses of either kind a thread and step instead of 8: forward, hidden 1024, 50 steps, 16 sequences 209 us instead of 177.)
constexpr int kPitch = 68, kRowPitch = 36;

__device__ __forceinline__ float sigmoid_f(float v) { return 1.0f / (1.0f + expf(-v)); }

// a block that gives up tells those that wait for it; true in the first of its group
__device__ bool first_to_give_up(unsigned *given_up, int *shared)
{
    if (threadIdx.x == 0) *shared = atomicExch(given_up, 1u) == 0;
    __syncthreads();
    return *shared != 0;
}

// the same number, which the compiler takes for another: what is derived from it is not kept from before
__device__ __forceinline__ int forget(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// barrier of a block whose waves have nothing in flight for each other but LDS accesses
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ void store_word(char *p, unsigned v)
{
    __hip_atomic_store(reinterpret_cast<unsigned *>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// two neighbouring lanes' bf16 values leave as one 32-bit write-through store (by the even lane); of two NaN one takes another
// payload than the word that stands for nothing sent
__device__ __forceinline__ void publish_pair(char *p, bf16_t v)
{
    const unsigned mine = v.v, other = __shfl_xor(mine, 1, 64), word = mine | (other << 16);
    if (!(threadIdx.x & 1)) store_word(p, word == kUnsent ? kUnsent - 1 : word);
}

__device__ __forceinline__ bf16x8_t load_frag(const bf16_t *p) { return as_frag(*reinterpret_cast<const chunk16 *>(p)); }

// an operand fragment that another block has published: 16 bytes a lane, coherent at agent scope (sc1)
__device__ __forceinline__ chunk16 load_published(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 16);
}

// KW fragments of a wave, 1 KB apart from `src` on.  WAIT: until no word of them is kUnsent; false when some still are after
// `polls` reads, or when a block of the group has given up.
template <int KW, bool WAIT>
__device__ __forceinline__ bool receive(__amdgpu_buffer_rsrc_t r, unsigned src, int lane, chunk16 (&b)[KW], unsigned polls,
                                        const unsigned *given_up)
{
    for (unsigned it = 1; !WAIT || it <= polls; ++it) {
#pragma unroll
        for (int k = 0; k < KW; ++k) b[k] = load_published(r, src + (unsigned)(k * 64 + lane) * 16u);
        if constexpr (!WAIT) return true;
        // All of them on their way before the first is looked at: left alone the compiler keeps two or three in flight, to
        // save registers that nobody else can have.
        __builtin_amdgcn_sched_barrier(0);
        unsigned most = 0;
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) most = b[k][j] > most ? b[k][j] : most;
        asm volatile("" ::: "memory");                     // read again in the next round
        if (__all(most != kUnsent)) return true;
        if (it % 16 == 0 && __hip_atomic_load(given_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) break;
    }
#pragma unroll
    for (int k = 0; k < KW; ++k) b[k] = chunk16{0u, 0u, 0u, 0u};
    return false;
}

// byte offset of (k, sequence) in a buffer of K-step fragments: [K/32][lane = (k/8 % 4, sequence)][8]
__device__ __forceinline__ unsigned frag_at(int k, int seq)
{
    return (unsigned)(((k >> 5) * 64 + ((k >> 3) & 3) * 16 + seq) * 8 + (k & 7)) * 2u;
}

// What a thread of a forward block works with, for a group of sequences and 32 units at a time.  H = 128 * KS.
template <int KS> struct SeqFwd {
    // eight pieces of K where they come out as whole K-steps, else four pieces for each half of the rows
    static constexpr int H = 128 * KS, GB = H / kUnits, KP = KS % 2 == 0 ? 8 : 4, MT = KP, KW = H / KP / 32;
    static constexpr unsigned SLICES = H * kSeqs * 2;
    const bf16_t *P, *w_hh;
    float *gates, *cells;
    bf16_t *h, *hs;
    int T;
    float (*red)[32 * kPitch];
    char *mine;
    __amdgpu_buffer_rsrc_t xr;
    int lane, wave, kp, sq, un;
    bool on;
    int ring;
    size_t r0;
    bf16x8_t w[MT][KW];
    bf16_t p[4], hv;
    float s[4], ig, fg, gg, og, c;

    __device__ __forceinline__ void place(int tid, int n0, int N, char *slice, int copies)
    {
        lane = tid & 63;
        wave = tid >> 6;
        kp = wave % KP;
        sq = tid >> 5;
        un = tid & 31;
        on = n0 + sq < N;
        // sequences past the last repeat it; nothing of theirs is stored in the layer's tensors
        r0 = (size_t)(on ? n0 + sq : N - 1) * T;
        mine = slice;
        ring = copies - 1;
        xr = __builtin_amdgcn_make_buffer_rsrc(slice, 0, copies * SLICES, 0x00020000);
        c = 0.0f;
        start();
    }
    __device__ __forceinline__ void start()
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = 0.0f;
    }
    // row tile i of 32 units: gate i / 2, units 16 (i % 2) .. + 15; this wave's tile m is
    __device__ __forceinline__ int tile(int m) const { return KP == 8 ? m : 2 * m + wave / KP; }
    __device__ __forceinline__ void load_rows(int u0)
    {
        const int row = lane & 15, quad = lane >> 4;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int k = 0; k < KW; ++k)
                w[m][k] = load_frag(w_hh + (size_t)((tile(m) >> 1) * H + u0 + 16 * (tile(m) & 1) + row) * H + (kp * KW + k) * 32 + 8 * quad);
    }
    __device__ __forceinline__ void fetch(int t, int u)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) p[q] = P[(r0 + t) * 4 * H + q * H + u];
    }
    // this wave's share of W_h h of step t - 1, to LDS
    template <bool WAIT> __device__ __forceinline__ bool multiply(int t, unsigned polls = 0, const unsigned *given_up = nullptr)
    {
        f32x4_t acc[MT] = {};
        chunk16 b[KW];
        const bool came = receive<KW, WAIT>(xr, (unsigned)(t & ring) * SLICES + (unsigned)(kp * KW) * 1024u, lane, b, polls, given_up);
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m][k], as_frag(b[k]), acc[m], 0, 0, 0);
        // row 4 quad + r of a half's tile is a unit; its four gates are four tiles apart by two
        constexpr int HALVES = MT / 4;
#pragma unroll
        for (int a = 0; a < HALVES; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int half = HALVES == 2 ? a : wave / KP, unit = 16 * half + 4 * (lane >> 4) + r;
                *reinterpret_cast<float4 *>(&red[kp][unit * kPitch + 4 * (lane & 15)]) =
                    make_float4(acc[a][r], acc[HALVES + a][r], acc[2 * HALVES + a][r], acc[3 * HALVES + a][r]);
            }
        return came;
    }
    __device__ __forceinline__ void collect()
    {
        float4 v[KP];
#pragma unroll
        for (int k = 0; k < KP; ++k) v[k] = *reinterpret_cast<const float4 *>(&red[k][un * kPitch + 4 * sq]);
        auto sum = [&](auto of) {
            float t = (of(v[0]) + of(v[1])) + (of(v[2]) + of(v[3]));
            if (KP == 8) t += (of(v[KP - 4]) + of(v[KP - 3])) + (of(v[KP - 2]) + of(v[KP - 1]));
            return t;
        };
        s[0] = sum([](const float4 &f) { return f.x; });
        s[1] = sum([](const float4 &f) { return f.y; });
        s[2] = sum([](const float4 &f) { return f.z; });
        s[3] = sum([](const float4 &f) { return f.w; });
    }
    __device__ __forceinline__ void cell()
    {
        ig = sigmoid_f(to_f32(p[0]) + s[0]);
        fg = sigmoid_f(to_f32(p[1]) + s[1]);
        gg = tanhf(to_f32(p[2]) + s[2]);
        og = sigmoid_f(to_f32(p[3]) + s[3]);
        c = fmaf(fg, c, ig * gg);                  // one rounding wherever the compiler puts this
        hv = from_f32<bf16_t>(og * tanhf(c));
    }
    __device__ __forceinline__ void send(int t, int u) { publish_pair(mine + ((t + 1) & ring) * SLICES + frag_at(u, sq), hv); }
    // what step t - 1 has read is unsent again
    __device__ __forceinline__ void clear(int t, int u)
    {
        if (!(threadIdx.x & 1)) store_word(mine + ((t - 1) & ring) * SLICES + frag_at(u, sq), kUnsent);
    }
    __device__ __forceinline__ void store(int t, int u)
    {
        if (!on) return;
        const size_t r = r0 + t;
        float *gt = gates + r * 4 * H + u;
        gt[0] = ig;
        gt[H] = fg;
        gt[2 * H] = gg;
        gt[3 * H] = og;
        cells[r * H + u] = c;
        h[r * H + u] = hv;
        if (t + 1 < T) hs[(r + 1) * H + u] = hv;
    }
};

template <int KS>
__global__ __launch_bounds__(kThreads, 1) void k_lstm_seq_fwd(const bf16_t *__restrict__ P, const bf16_t *__restrict__ w_hh,
                                                              float *__restrict__ gates, float *cells,
                                                              bf16_t *__restrict__ h, bf16_t *__restrict__ hs, int N, int T,
                                                              unsigned *ctl, char *slices, unsigned polls)
{
    using S = SeqFwd<KS>;
    constexpr int GB = S::GB;
    __shared__ __align__(16) float red[S::KP][32 * kPitch];
    __shared__ int s_ticket, s_dead, s_first;
    if (threadIdx.x == 0) {
        s_ticket = (int)atomicAdd(ctl, 1u);
        s_dead = 0;
    }
    __syncthreads();
    if ((unsigned)s_ticket >= gridDim.x) return;                // another launch has written the workspace: no group, no slices
    bool dead = false;
    {
        const int grp = s_ticket / GB, blk = s_ticket % GB;
        const unsigned *given_up = ctl + (1 + grp) * kCtlWords;
        S a{P, w_hh, gates, cells, h, hs, T, red};
        a.place(threadIdx.x, grp * kSeqs, N, slices + (size_t)grp * kCopies * S::SLICES, kCopies);
        const int u = blk * kUnits + a.un;
        a.load_rows(blk * kUnits);
        a.fetch(0, u);
        if (a.on) hs[a.r0 * S::H + u] = from_f32<bf16_t>(0.0f);
        for (int t = 0; t < T; ++t) {
            if (t > 0) {
                if (!a.template multiply<true>(t, polls, given_up)) s_dead = 1;
                __syncthreads();
                a.collect();
                dead = s_dead != 0;
                if (dead) break;
            }
            a.cell();
            if (t + 1 < T) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // clear() of the step before
                a.send(t, u);
                if (t > 1) a.clear(t, u);
                lds_barrier();
                a.fetch(t + 1, u);
            }
            a.store(t, u);                         // what nobody waits for
        }
    }
    if (!dead) return;
    const int tid = forget(threadIdx.x), grp = s_ticket / GB;
    if (!first_to_give_up(ctl + (1 + grp) * kCtlWords, &s_first)) return;
    S a{P, w_hh, gates, cells, h, hs, T, red};
    a.place(tid, grp * kSeqs, N, slices + ((size_t)(gridDim.x / GB) * kCopies + (size_t)grp * 2) * S::SLICES, 2);
    for (int t = 0; t < T; ++t) {
        for (int b = 0; b < GB; ++b) {
            const int u = b * kUnits + a.un;
            a.fetch(t, u);
            a.c = t > 0 ? cells[(a.r0 + t - 1) * S::H + u] : 0.0f;
            if (t > 0) {
                a.load_rows(b * kUnits);
                a.template multiply<false>(t);
                __syncthreads();
                a.collect();
                __syncthreads();
            }
            a.cell();
            if (t + 1 < T) a.send(t, u);
            a.store(t, u);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
}

// the same for a backward block
template <int KS> struct SeqBwd {
    static constexpr int H = 128 * KS, GB = H / kUnits, KW = H / 64;      // KW: K-steps of a wave (half a gate)
    static constexpr unsigned SLICES = 4 * H * kSeqs * 2;
    const bf16_t *dy, *wt_h;
    const float *gates, *cells;
    bf16_t *D;
    int T;
    float (*red)[kSeqs * kRowPitch];
    char *mine;
    __amdgpu_buffer_rsrc_t xr;
    int lane, wave, sq, un, n;
    bool on;
    int ring;
    size_t r0;
    bf16x8_t w[2][KW];
    float carry, g[4], c, cp, s;
    bf16_t dh0, dv[4];

    __device__ __forceinline__ void place(int tid, int n0, int N, char *slice, int copies)
    {
        lane = tid & 63;
        wave = tid >> 6;
        sq = tid >> 5;
        un = tid & 31;
        on = n0 + sq < N;
        n = on ? n0 + sq : N - 1;
        r0 = (size_t)n * T;
        mine = slice;
        ring = copies - 1;
        xr = __builtin_amdgcn_make_buffer_rsrc(slice, 0, copies * SLICES, 0x00020000);
        carry = s = 0.0f;
    }
    __device__ __forceinline__ void load_rows(int u0)
    {
        const int row = lane & 15, quad = lane >> 4;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int k = 0; k < KW; ++k) w[m][k] = load_frag(wt_h + (size_t)(u0 + 16 * m + row) * 4 * H + wave * (H / 2) + k * 32 + 8 * quad);
    }
    __device__ __forceinline__ void fetch(int t, int u)        // what step t reads besides D_{t+1}; requested a step ahead
    {
        const size_t r = r0 + t;
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = gates[r * 4 * H + q * H + u];
        c = cells[r * H + u];
        cp = t > 0 ? cells[(r - 1) * H + u] : 0.0f;
        dh0 = dy[r * H + u];
    }
    // this wave's share of W_h^T D of step t + 1, to LDS
    template <bool WAIT> __device__ __forceinline__ bool multiply(int t, unsigned polls = 0, const unsigned *given_up = nullptr)
    {
        f32x4_t acc[2][2] = {};
        chunk16 b[KW];
        const bool came = receive<KW, WAIT>(xr, (unsigned)((t + 1) & ring) * SLICES + (unsigned)(wave * KW) * 1024u, lane, b, polls, given_up);
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
            for (int m = 0; m < 2; ++m) acc[m][k & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m][k], as_frag(b[k]), acc[m][k & 1], 0, 0, 0);
#pragma unroll
        for (int m = 0; m < 2; ++m)
            *reinterpret_cast<float4 *>(&red[wave][(lane & 15) * kRowPitch + 16 * m + 4 * (lane >> 4)]) =
                make_float4(acc[m][0][0] + acc[m][1][0], acc[m][0][1] + acc[m][1][1], acc[m][0][2] + acc[m][1][2], acc[m][0][3] + acc[m][1][3]);
        return came;
    }
    __device__ __forceinline__ void collect()
    {
        const int at = sq * kRowPitch + un;
        s = ((red[0][at] + red[1][at]) + (red[2][at] + red[3][at])) + ((red[4][at] + red[5][at]) + (red[6][at] + red[7][at]));
    }
    __device__ __forceinline__ void cell()
    {
        const float dh = to_f32(dh0) + s, th = tanhf(c);
        const float dc = dh * g[3] * (1.0f - th * th) + carry;
        const float d[4] = {dc * g[2] * g[0] * (1.0f - g[0]), dc * cp * g[1] * (1.0f - g[1]), dc * g[0] * (1.0f - g[2] * g[2]),
                            dh * th * g[3] * (1.0f - g[3])};
        carry = dc * g[1];
#pragma unroll
        for (int q = 0; q < 4; ++q) dv[q] = from_f32<bf16_t>(d[q]);
    }
    __device__ __forceinline__ void send(int t, int u)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) publish_pair(mine + (t & ring) * SLICES + frag_at(q * H + u, sq), dv[q]);
    }
    // what step t + 1 has read is unsent again
    __device__ __forceinline__ void clear(int t, int u)
    {
        if (threadIdx.x & 1) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) store_word(mine + ((t + 2) & ring) * SLICES + frag_at(q * H + u, sq), kUnsent);
    }
    __device__ __forceinline__ void store(int t, int u)
    {
        if (!on) return;
#pragma unroll
        for (int q = 0; q < 4; ++q) D[(r0 + t) * 4 * H + q * H + u] = dv[q];
    }
};

// carry_of: [N][H], touched only by a block that computes a group by itself
template <int KS>
__global__ __launch_bounds__(kThreads, 1) void k_lstm_seq_bwd(const bf16_t *__restrict__ dy, const bf16_t *__restrict__ wt_h,
                                                                  const float *__restrict__ gates, const float *__restrict__ cells,
                                                                  bf16_t *__restrict__ D, float *carry_of, int N, int T,
                                                                  unsigned *ctl, char *slices, unsigned polls)
{
    using S = SeqBwd<KS>;
    constexpr int GB = S::GB;
    __shared__ __align__(16) float red[8][kSeqs * kRowPitch];
    __shared__ int s_ticket, s_dead, s_first;
    if (threadIdx.x == 0) {
        s_ticket = (int)atomicAdd(ctl, 1u);
        s_dead = 0;
    }
    __syncthreads();
    if ((unsigned)s_ticket >= gridDim.x) return;
    bool dead = false;
    {
        const int grp = s_ticket / GB, blk = s_ticket % GB;
        const unsigned *given_up = ctl + (1 + grp) * kCtlWords;
        S a{dy, wt_h, gates, cells, D, T, red};
        a.place(threadIdx.x, grp * kSeqs, N, slices + (size_t)grp * kCopies * S::SLICES, kCopies);
        const int u = blk * kUnits + a.un;
        a.load_rows(blk * kUnits);
        a.fetch(T - 1, u);
        for (int t = T - 1; t >= 0; --t) {
            if (t + 1 < T) {
                if (!a.template multiply<true>(t, polls, given_up)) s_dead = 1;
                __syncthreads();
                a.collect();
                dead = s_dead != 0;
                if (dead) break;
            }
            a.cell();
            if (t > 0) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // clear() of the step before
                a.send(t, u);
                if (t + 2 < T) a.clear(t, u);
                lds_barrier();
                a.fetch(t - 1, u);
            }
            a.store(t, u);
        }
    }
    if (!dead) return;
    const int tid = forget(threadIdx.x), grp = s_ticket / GB;
    if (!first_to_give_up(ctl + (1 + grp) * kCtlWords, &s_first)) return;
    S a{dy, wt_h, gates, cells, D, T, red};
    a.place(tid, grp * kSeqs, N, slices + ((size_t)(gridDim.x / GB) * kCopies + (size_t)grp * 2) * S::SLICES, 2);
    for (int t = T - 1; t >= 0; --t) {
        for (int b = 0; b < GB; ++b) {
            const int u = b * kUnits + a.un;
            a.fetch(t, u);
            if (t + 1 < T) {
                a.carry = carry_of[(size_t)a.n * S::H + u];
                a.load_rows(b * kUnits);
                a.template multiply<false>(t);
                __syncthreads();
                a.collect();
                __syncthreads();
            } else {
                a.carry = 0.0f;
            }
            a.cell();
            if (a.on) carry_of[(size_t)a.n * S::H + u] = a.carry;
            if (t > 0) a.send(t, u);
            a.store(t, u);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
}

// no ticket drawn, nobody has given up, nothing sent: `zeros` 16-byte words of 0, then `ones` of kUnsent
__global__ __launch_bounds__(256) void k_lstm_prepare(chunk16 *p, unsigned zeros, unsigned ones)
{
    for (unsigned i = blockIdx.x * 256u + threadIdx.x; i < zeros + ones; i += gridDim.x * 256u) {
        const unsigned v = i < zeros ? 0u : kUnsent;
        p[i] = chunk16{v, v, v, v};
    }
}

int groups_of(int N) { return (N + kSeqs - 1) / kSeqs; }
size_t ctl_bytes(int N) { return (size_t)(1 + groups_of(N)) * kCtlWords * sizeof(unsigned); }

hipError_t prepare(void *workspace, int N, size_t slices, hipStream_t s)
{
    const unsigned zeros = (unsigned)(ctl_bytes(N) / 16), ones = (unsigned)(groups_of(N) * kCopies * slices / 16), want = (zeros + ones + 1023) / 1024;
    hipLaunchKernelGGL(k_lstm_prepare, dim3(want < 1024 ? want : 1024), dim3(256), 0, s, (chunk16 *)workspace, zeros, ones);
    return hipGetLastError();
}

}  // namespace

// Up to hidden 1024 a block's rows fit its registers.  Past a thousand blocks (four rounds of the chip) the two launches
// per step are no longer mostly gaps: a mini-batch of 2 x 512 sequences of 20 steps at hidden 1024 (1024 blocks) takes
// 6.7 ms against 7.5 with them, of 2 x 256 3.7 against 4.9.  Every round of the chip (three blocks to a unit at hidden 128,
// two up to 384, then one) loads the matrix again, which a short sequence does not pay back: at hidden 1024, forward +
// backward of a layer, one launch against two per step: 512 sequences (four rounds) of 2 steps 76 + 139 us against 42 + 112,
// of 6 164 + 244 against 141 + 257; 256 (two rounds) of 2 48 + 86 against 32 + 77, of 4 66 against 73 forward.
// A single step has no product at all (16 sequences: 20 + 40 us against 12 + 32).
// The blocks wait for each other: a group has to find its blocks' slots beside up to seven more such launches (forward and
// backward passes of up to four stages), at one block per compute unit; a GPU partition of few units takes two launches a step.
bool lstm_seq_supported(int N, int T, int H, int compute_units)
{
    if (N < 1 || T < 2 || H % 128 != 0 || H > 1024 || 8 * (H / kUnits - 1) >= compute_units) return false;
    const long long blocks = (long long)groups_of(N) * (H / kUnits);
    const int per_unit = H <= 128 ? 3 : H <= 384 ? 2 : 1;
    return blocks <= 1024 && 2 * blocks <= 256ll * per_unit * T;
}

// ticket line and groups' lines, then the copies of every group's slices (backward's, the wider ones), then two of those of the
// blocks that compute a group by themselves
size_t lstm_seq_workspace(int N, int H) { return ctl_bytes(N) + (size_t)groups_of(N) * (kCopies + 2) * 4 * H * kSeqs * 2; }

#define LSTM_CASES(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

hipError_t lstm_seq_fwd(const void *P, const void *w_hh, float *gates, float *cells, void *h, void *hs, int N, int T, int H,
                        void *workspace, hipStream_t s, unsigned wait_polls)
{
    const hipError_t e = prepare(workspace, N, (size_t)H * kSeqs * 2, s);
    if (e != hipSuccess) return e;
    const dim3 grid(groups_of(N) * (H / kUnits));
    switch (H / 128) {
#define X(KS)                                                                                                             \
    case KS:                                                                                                              \
        hipLaunchKernelGGL((k_lstm_seq_fwd<KS>), grid, dim3(kThreads), 0, s, (const bf16_t *)P, (const bf16_t *)w_hh, gates, \
                           cells, (bf16_t *)h, (bf16_t *)hs, N, T, (unsigned *)workspace, (char *)workspace + ctl_bytes(N), wait_polls);      \
        break;
        LSTM_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t lstm_seq_bwd(const void *dy, const void *wt_h, const float *gates, const float *cells, float *dcn, void *D, int N, int T, int H,
                        void *workspace, hipStream_t s, unsigned wait_polls)
{
    const hipError_t e = prepare(workspace, N, (size_t)4 * H * kSeqs * 2, s);
    if (e != hipSuccess) return e;
    const dim3 grid(groups_of(N) * (H / kUnits));
    switch (H / 128) {
#define X(KS)                                                                                                              \
    case KS:                                                                                                               \
        hipLaunchKernelGGL((k_lstm_seq_bwd<KS>), grid, dim3(kThreads), 0, s, (const bf16_t *)dy, (const bf16_t *)wt_h, gates, \
                           cells, (bf16_t *)D, dcn, N, T, (unsigned *)workspace, (char *)workspace + ctl_bytes(N), wait_polls);               \
        break;
        LSTM_CASES(X)
#undef X
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace bapipe

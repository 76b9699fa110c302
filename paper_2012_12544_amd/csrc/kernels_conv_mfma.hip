// bf16 MFMA implicit-GEMM convolution for gfx950 (CDNA4): forward / dgrad ("gather" form) and
// wgrad.  fp32 accumulation in v_mfma_f32_32x32x16_bf16; operands staged through LDS.
//
// Gather form (forward and dgrad share it, see GatherConv):
//     out[pixel][ko] = sum_k  X[pixel][k] * Wt[ko][k],   k = (r, s, ki), ki fastest
// is a GEMM whose K index is contiguous in memory for both operands (NHWC activations,
// [Ko][R][S][Ki] filters), which is exactly the per-lane fragment the MFMA wants (8 consecutive
// k for one row).  A block owns BP output pixels x BC output channels; 16-byte chunks of the
// operand rows travel from HBM/L2 straight into LDS (buffer_load ... lds, no register staging)
// into a ring of three K-tiles; the XOR swizzle that makes the ds_read_b128 fragment loads
// bank-conflict free is applied on the global side, by choosing which chunk a lane fetches.
// The MFMA's A operand is the filter tile and its B operand the pixel tile, so a lane ends up
// with 4 consecutive output channels of one pixel per accumulator quad; the tile is then
// staged through LDS as [pixel][channel] to leave the kernel as 16-byte, fully coalesced rows
// (with bias / ReLU, or with the gradient epilogue: accumulate + ReLU gate of the producer).
//
// wgrad:  dw[ko][r][s][c] += sum_pixels dy[pixel][ko] * x[pixel @ tap (r,s)][c]
// contracts over pixels, which are NOT contiguous for either operand: tiles are stored in LDS
// as [pixel][channel] exactly as they come from HBM, and the fragments are fetched with the
// CDNA4 transposing LDS read (ds_read_b64_tr_b16), which hands each lane 4 consecutive
// pixels of one channel.  The pixel range is split over blocks (split-K); partial sums go to
// a workspace and a second kernel adds them in a fixed order into the fp32 accumulators.
#include "kernels.h"
#include "mfma_common.h"
#include <type_traits>

namespace bapipe {
namespace {

template <int BK> __device__ __forceinline__ int swz(int row)
{
    // 16-byte slots of 16 consecutive rows must fall into 16 different bank groups
    return BK == 32 ? ((row >> 2) & 3) : ((row >> 1) & 7);
}

// ------------------------------------------------------------------------------------------
// gather convolution
// ------------------------------------------------------------------------------------------
// The operand tiles travel HBM/L2 -> LDS without touching registers: buffer_load_dwordx4 ... lds
// writes the 64 lanes' 16-byte chunks to 64 consecutive LDS slots starting at a wave-uniform
// address, and a lane whose offset is outside the buffer gets zeros (that is the zero padding of
// the convolution and the ragged tile edges).  The XOR swizzle of the tile layout is applied by
// choosing WHICH chunk a lane fetches, since WHERE it lands is fixed by the lane id.
// STAGES tiles form a ring; tile kt+STAGES-1 is requested right after the barrier that retires
// tile kt-1, so STAGES-1 K-tiles of latency are covered while the MFMAs run.
// PHASED (gradient of a strided convolution, s_in > 1): an output pixel only meets the taps whose offset is congruent to
// its own position modulo the stride, so the output is taken apart into the grids of pixels with equal remainders;
// on each the product is an ordinary stride-1 one with the taps of that class (for 3x3 / 2: 4, 2, 2 and 1 of the 9).
// blockIdx.z is the class, the one with most taps first.  Without it three quarters of the multiply-adds meet a zero:
// 3x3 / 2 with the gate and batch-norm sums of a bottleneck, 32 samples, 512 channels, 14x14 from 7x7: 104 -> 24 us; 128
// channels, 56x56 from 28x28: 84 -> 41 us.  With the taps not innermost only for 1x1 filters, whose K is the channels of the
// one tap either way.
// PANELS: the filter is kept in panels of 32 columns (GatherConv::wt_panels).  A wave-wide load fetches whole cache lines whatever BK,
// and what a tile streams is one or two pieces of memory (25088->4096, 64 rows, 50.0 -> 45 us; 4096->4096 16.1 -> 15.1).  A variant of
// its own: layouts as arguments cost the others up to 0.7 % of a mini-batch.
template <int BP, int BC, int WP, int WC, int BK, int STAGES, int KG, bool S1, bool TAPS_INNER, bool PHASED = false, bool PANELS = false>
__global__ __launch_bounds__(WP *WC *KG * 64, WP *WC *KG >= 8 ? 1 : 2) void k_gather_mfma(
    const bf16_t *__restrict__ in, const bf16_t *__restrict__ wt, const float *__restrict__ bias,
    bf16_t *out, const bf16_t *__restrict__ gate, int accum, int relu, int is_grad, GatherGeom g,
    int tiles_c, unsigned in_bytes, unsigned wt_bytes, float *__restrict__ part, int kt_per_split, int part_tiles,
    float *__restrict__ stat_part, const bf16_t *__restrict__ bn_x, const float *__restrict__ bn_stats,
    const bf16_t *old_from, unsigned *tickets)
{
    constexpr int NW = WP * WC, NT = NW * KG * 64;      // waves of a group, threads of the block
    constexpr int CPR = BK / 8;              // 16-byte chunks per tile row
    constexpr int RPW = 64 / CPR;            // tile rows one wave-wide load covers
    constexpr int XL = BP / (RPW * NW);      // loads per wave for the pixel tile
    constexpr int WL = BC / (RPW * NW);      // loads per wave for the filter tile
    constexpr int WT_P = BP / WP, WT_C = BC / WC;
    constexpr int TP = WT_P / 32, TC = WT_C / 32;
    constexpr int KSUB = BK / 16;
    constexpr bool WHOLE = BK == 64 && NW == 4;
    constexpr int SROW = BC + 4;             // staging row (elements): 8-byte aligned, odd multiple of 8 bytes
    constexpr int STAGE_ELEMS = (BP + BC) * BK;
    static_assert(XL >= 1 && WL >= 1 && BP % (RPW * NW) == 0 && BC % (RPW * NW) == 0, "tile/thread mismatch");
    // BK = 64: a whole K-tile of fragments in registers while the next one is read (see the loop)
    static_assert(BK == 32 || (BK == 64 && S1 && TAPS_INNER && (NW & 1) == 0), "lane-to-slot maps below");

    extern __shared__ __align__(16) unsigned char smem[];
    const lds_addr_of lds_of(smem);
    // KG > 1: the groups' sums meet in front of the staging tile
    constexpr int PITCH = BC + 4;
    constexpr size_t PARK_BYTES = KG > 1 ? (size_t)KG * BP * PITCH * 4 : 0;
    constexpr size_t RING_BYTES = (size_t)KG * STAGES * STAGE_ELEMS * 2, TILE_BYTES = (size_t)BP * SROW * 2, EPI_BYTES = PARK_BYTES + TILE_BYTES + NT * 8;
    uint16_t *sO = reinterpret_cast<uint16_t *>(smem + PARK_BYTES);    // [BP][SROW] (epilogue, reuses the ring)
    float *sBias = reinterpret_cast<float *>(smem + (RING_BYTES > EPI_BYTES ? RING_BYTES : EPI_BYTES));   // [BC]
    int *sPix = reinterpret_cast<int *>(sBias + BC);                  // PHASED: [BP] output pixel of a tile row, npix past the end

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_id % NW, kg = wave_id / NW;                 // place inside the group, group
    uint16_t *ring = reinterpret_cast<uint16_t *>(smem) + kg * STAGES * STAGE_ELEMS;      // the group's [STAGES][ W tile | X tile ]
    const int wp = wave % WP, wc = wave / WP;
    // slot (row, c') a lane fills inside one wave-wide load, and the chunk column it must fetch
    const int lrow = lane / CPR;
    const int lc = (lane % CPR) ^ swz<BK>(wave * RPW + lrow);       // = c' ^ swz(row); the same for every load

    // split-K: blockIdx.y owns K-tiles [kt0, kt1) and leaves fp32 partial sums in part[split][pixel][co]
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int tile_c = bid % tiles_c, tile_p = bid / tiles_c;
    const int co0 = tile_c * BC;
    const int pix0 = tile_p * BP;                    // pixel counts fit 31 bits (checked by the launcher)
    const int npix = g.N * g.Ho * g.Wo;
    const int K = g.R * g.S * g.Ci;
    // the class of a PHASED block: output pixels (s_in i + pa, s_in j + pb) and the taps (r0 + s_in i, q0 + s_in j)
    const int sd = PHASED ? g.s_in : 1;
    int pa = 0, pb = 0, r0 = 0, q0 = 0, Rn = g.R, Sn = g.S, Hp = g.Ho, Wp = g.Wo;
    if (PHASED) {
        const int zc = (int)blockIdx.z, ch = sd < g.Ho ? sd : g.Ho, cw = sd < g.Wo ? sd : g.Wo;      // remainders that occur
        pa = (zc / cw + g.pad_h) % ch;               // class 0 (stride up to the image): the pixels that tap (0, 0) reaches
        pb = (zc % cw + g.pad_w) % cw;
        r0 = (g.pad_h % sd - pa + sd) % sd;
        q0 = (g.pad_w % sd - pb + sd) % sd;
        Rn = r0 < g.R ? (g.R - r0 + sd - 1) / sd : 0;
        Sn = q0 < g.S ? (g.S - q0 + sd - 1) / sd : 0;
        Hp = (g.Ho - pa + sd - 1) / sd;
        Wp = (g.Wo - pb + sd - 1) / sd;
    }
    const int rows = g.N * Hp * Wp;                  // output pixels of the class
    const int KT = TAPS_INNER ? (g.Ci / BK) * Rn * Sn : (Rn * Sn * g.Ci + BK - 1) / BK;
    constexpr unsigned OOB = 0x80000000u;

    __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(in), 0, (int)in_bytes, 0x00020000);
    __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(wt), 0, (int)wt_bytes, 0x00020000);

    // ---- per-lane gather state: the pixel rows this lane fetches (row = (i*NW + wave)*RPW + lrow)
    // FAST (taps innermost, at most 32 of them; stride 1): everything that depends on the lane is
    // computed once - the byte offset of the lane's chunk at tap (0,0) and a bit mask of the taps
    // that fall inside the image - so that a K-tile costs one scalar offset, one mask test and one
    // add per load.
    constexpr bool FAST = TAPS_INNER;
    static_assert(!PANELS || (FAST && !PHASED), "1x1 filters of whole K-tiles");
    static_assert(!TAPS_INNER || S1, "a strided operand takes its taps in the flattened order");
    int hb[XL], wb[XL];
    unsigned xoff[XL];                       // generic: byte offset of pixel (n, 0, 0), channel 0; FAST: see above
    unsigned tapmask[XL];
#pragma unroll
    for (int i = 0; i < XL; ++i) {
        int p = pix0 + (i * NW + wave) * RPW + lrow;
        tapmask[i] = 0;
        if (p < rows) {
            int ow = p % Wp;
            int t = p / Wp;
            int oh = t % Hp;
            int n = t / Hp;
            hb[i] = PHASED ? oh + (pa + r0 - g.pad_h) / sd : oh * g.s_out - g.pad_h;      // exact division
            wb[i] = PHASED ? ow + (pb + q0 - g.pad_w) / sd : ow * g.s_out - g.pad_w;
            xoff[i] = (unsigned)n * (unsigned)(g.Hi * g.Wi * g.Ci) * 2u;
            if (FAST) {
                for (int r = 0; r < Rn; ++r)
                    for (int q = 0; q < Sn; ++q)
                        if ((unsigned)(hb[i] + r) < (unsigned)g.Hi && (unsigned)(wb[i] + q) < (unsigned)g.Wi)
                            tapmask[i] |= 1u << (r * Sn + q);
                xoff[i] += (unsigned)((hb[i] * g.Wi + wb[i]) * g.Ci + 8 * lc) * 2u;     // may wrap; the tap offset undoes it
            }
        } else {
            hb[i] = -(1 << 28);          // fails every bounds check below
            wb[i] = 0;
            xoff[i] = 0;
        }
    }
    unsigned woff[WL];
#pragma unroll
    for (int i = 0; i < WL; ++i) {
        int co = co0 + (i * NW + wave) * RPW + lrow;
        if constexpr (PANELS) {
            woff[i] = co < g.Co ? (unsigned)((lc >> 2) * g.Co + co) * 64u + 16u * (lc & 3) : OOB;
        } else {
            woff[i] = co < g.Co ? (unsigned)co * (unsigned)K * 2u : OOB;
            if (FAST && co < g.Co) woff[i] += 16u * lc;
        }
    }
    // K order.  TAPS_INNER (Ci a multiple of BK): tile kt covers channels [cit*BK, +BK) of tap
    // (kt % RS), taps innermost, so that consecutive tiles re-read almost the same pixels (shifted
    // by one column / one row) and hit in the CU's vector L1.  Otherwise k = (r, s, ci) flattened,
    // ci fastest, and a tile may straddle taps.  Both operands use the same order.
    const int kt0 = part ? blockIdx.y * kt_per_split : 0;
    const int kt1 = part ? (kt0 + kt_per_split < KT ? kt0 + kt_per_split : KT) : KT;
    int ti = kt0 + kg;                                 // the group's next tile; it takes every KG-th
    int kk = ti * BK + 8 * lc;                        // flattened k of this lane's chunk (generic order)
    int kr = kk / (g.S * g.Ci), ks = (kk / g.Ci) % g.S, kc = kk % g.Ci;
    if (PHASED && KT == 0) kr = g.R;                   // a class without taps reads nothing
    int cb = 0;                                        // FAST: first channel of the tile (wave-uniform)
    if (TAPS_INNER) {
        const int taps = PHASED ? (KT ? Rn * Sn : 1) : g.R * g.S, tap = ti % taps;
        kr = tap / (PHASED ? (KT ? Sn : 1) : g.S);
        ks = tap % (PHASED ? (KT ? Sn : 1) : g.S);
        cb = KT ? ti / taps * BK : g.Ci;               // a class without taps reads nothing
    }

    auto issue_tile = [&](int stage) {
        uint16_t *sw = ring + stage * STAGE_ELEMS, *sx = sw + BC * BK;
        if constexpr (FAST) {
            const bool kin = KG > 1 ? ti < kt1 : cb < g.Ci;
            const unsigned bit = kin ? 1u << (kr * Sn + ks) : 0u;
            const int tap = PHASED ? (r0 + sd * kr) * g.S + q0 + sd * ks : kr * g.S + ks;
            const unsigned xo = (unsigned)((kr * g.Wi + ks) * g.Ci + cb) * 2u;
            const unsigned wo = !kin ? OOB : PANELS ? (unsigned)(cb * g.Co) * 2u : (unsigned)(tap * g.Ci + cb) * 2u;
#pragma unroll
            for (int i = 0; i < XL; ++i) {
                unsigned vo = (tapmask[i] & bit) ? xoff[i] + xo : OOB;
                dma16(xrsrc, lds_of(sx + (i * NW + wave) * RPW * BK), vo);
            }
#pragma unroll
            for (int i = 0; i < WL; ++i) {
                unsigned vo = (woff[i] + wo) | (woff[i] & OOB);       // rows past Co stay out of range
                if (!kin) vo = OOB;                                   // and so do tiles past K
                dma16(wrsrc, lds_of(sw + (i * NW + wave) * RPW * BK), vo);
            }
            return;                                   // the caller advances (kr, ks, cb) after its MFMAs
        }
        const bool kin = kr < g.R && (KG == 1 || ti < kt1);
        const unsigned koff = (unsigned)kk * 2u;
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            int hn = hb[i] + kr, wn = wb[i] + ks;
            int ih, iw;
            bool ok;
            if (S1) {
                ih = hn;
                iw = wn;
                ok = kin && (unsigned)ih < (unsigned)g.Hi && (unsigned)iw < (unsigned)g.Wi;
            } else {
                ih = hn / g.s_in;
                iw = wn / g.s_in;
                ok = kin && hn >= 0 && wn >= 0 && ih * g.s_in == hn && iw * g.s_in == wn && ih < g.Hi && iw < g.Wi;
            }
            unsigned vo = ok ? xoff[i] + (unsigned)((ih * g.Wi + iw) * g.Ci + kc) * 2u : OOB;
            dma16(xrsrc, lds_of(sx + (i * NW + wave) * RPW * BK), vo);
        }
#pragma unroll
        for (int i = 0; i < WL; ++i) {
            unsigned vo = (kin && woff[i] != OOB) ? woff[i] + koff : OOB;
            dma16(wrsrc, lds_of(sw + (i * NW + wave) * RPW * BK), vo);
        }
        // advance to the next K-tile
        ti += KG;
        kk += KG * BK;
        kc += KG * BK;
        while (kc >= g.Ci) {
            kc -= g.Ci;
            if (++ks == g.S) {
                ks = 0;
                ++kr;
            }
        }
    };
    // FAST path: step (kr, ks, cb) to the next K-tile.  Kept apart from issue_tile so that the branchy
    // scalar code does not split the block in which the MFMAs and the address arithmetic interleave.
    auto advance_tile = [&]() {
        if (FAST) {
            ti += KG;
            if (KG > 1 && Rn * Sn == 1) {
                cb += KG * BK;
                return;
            }
#pragma unroll
            for (int j = 0; j < KG; ++j)
                if (++ks == Sn) {
                    ks = 0;
                    if (++kr == Rn) {
                        kr = 0;
                        cb += BK;
                    }
                }
        }
    };

    f32x16_t acc[TC][TP];
#pragma unroll
    for (int a = 0; a < TC; ++a)
#pragma unroll
        for (int b = 0; b < TP; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // These tiles take all of a K that was split over blocks before, so that an accumulator would add more terms than a split's did.
    // Its sum is put aside and started anew every part_tiles K-tiles: sums of one sign, 3x3 512->512 from 1568 pixels, 5.0e-8 off 64
    // bits where one sum per group was 1.7e-7 and six splits 7.2e-8; 256->64 from 25088 6.1e-8, 2.9e-7 and 8.6e-8.  16 registers
    // (32 of 128 x 64) more, and up to 0.4 % of a mini-batch of small layers.
    constexpr bool PARTS = KG > 1 || BC == 64;
    constexpr int AC = PARTS ? TC : 1, AP = PARTS ? TP : 1;
    f32x16_t aside[AC][AP];
#pragma unroll
    for (int a = 0; a < AC; ++a)
#pragma unroll
        for (int b = 0; b < AP; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) aside[a][b][v] = 0.0f;
    auto put_aside = [&]() {
        if constexpr (PARTS) {
#pragma unroll
            for (int a = 0; a < TC; ++a)
#pragma unroll
                for (int b = 0; b < TP; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        aside[a][b][v] += acc[a][b][v];
                        acc[a][b][v] = 0.0f;
                    }
        }
    };

    const int frow = lane & 31, fhalf = lane >> 5;
    // operand fragments of K-sub-step ks16 of the tile in ring slot `stage`
    auto load_frags = [&](int stage, int ks16, bf16x8_t(&fa)[TC], bf16x8_t(&fb)[TP]) {
        const uint16_t *cw = ring + stage * STAGE_ELEMS, *cx = cw + BC * BK;
        const int ch = 2 * ks16 + fhalf;
#pragma unroll
        for (int a = 0; a < TC; ++a) {
            int row = wc * WT_C + a * 32 + frow;
            fa[a] = as_frag(*reinterpret_cast<const chunk16 *>(cw + row * BK + ((ch ^ swz<BK>(row)) << 3)));
        }
#pragma unroll
        for (int b = 0; b < TP; ++b) {
            int row = wp * WT_P + b * 32 + frow;
            fb[b] = as_frag(*reinterpret_cast<const chunk16 *>(cx + row * BK + ((ch ^ swz<BK>(row)) << 3)));
        }
    };
    auto mfma_all = [&](const bf16x8_t(&fa)[TC], const bf16x8_t(&fb)[TP]) {
#pragma unroll
        for (int a = 0; a < TC; ++a)
#pragma unroll
            for (int b = 0; b < TP; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    };

    // the block's bias slice goes to LDS now; it is read after the barriers of the main loop
    if (tid < BC) sBias[tid] = (bias && co0 + tid < g.Co) ? bias[co0 + tid] : 0.0f;
    if (PHASED) {
        for (int i = tid; i < BP; i += NT) {
            const int p = pix0 + i;
            sPix[i] = p < rows ? ((p / (Hp * Wp)) * g.Ho + p / Wp % Hp * sd + pa) * g.Wo + p % Wp * sd + pb : npix;
        }
    }
    const int tile_z = PHASED ? (int)blockIdx.z * ((int)gridDim.x / tiles_c) + tile_p : tile_p;      // of the statistics
    const int tiles_all = ((int)gridDim.x / tiles_c) * (PHASED ? (int)gridDim.z : 1);

    // Software pipeline.  The ring holds STAGES tiles in flight or in use; every iteration requests
    // exactly XL+WL loads per wave (tiles past the end fetch zeros nobody multiplies), so "at most
    // (STAGES-2)*(XL+WL) outstanding" means the next tile has landed.  Fragments are double-buffered
    // in registers: the LDS reads of a sub-step are issued one sub-step (one group of MFMAs) before
    // they are needed, and the barrier that publishes tile kt+1 sits between the two MFMA groups of
    // tile kt.  By then every wave holds all of tile kt in registers, so its slot is refilled at once.
    // sched_barrier pins that order: left alone the scheduler sinks the reads next to their MFMAs.
    constexpr int NLOAD = XL + WL;
    const int n_it = (kt1 - kt0 + KG - 1) / KG;
#pragma unroll
    for (int st = 0; st < STAGES; ++st) {
        issue_tile(st);
        advance_tile();
    }
    WAIT_VMCNT((STAGES - 1) * NLOAD);
    WAIT_LGKMCNT(0);       // no scalar load may be pending at loop entry, or every LDS wait in the loop becomes a full drain
    __builtin_amdgcn_s_barrier();
    if constexpr (WHOLE) {
        // Few MFMAs per wave and sub-step (two for a 64 x 32 wave tile) cannot cover the LDS latency of the next
        // sub-step's reads, and a launch of about one block per compute unit has nobody else to cover it: the tile is
        // read one whole K-tile ahead instead, so one barrier and one wait, both behind eight MFMAs, serve 64 channels.
        bf16x8_t fa[2][KSUB][TC], fb[2][KSUB][TP];
#pragma unroll
        for (int j = 0; j < KSUB; ++j) load_frags(0, j, fa[0][j], fb[0][j]);
        int rd = 0;
        int it = 0, end = 0;
        do {
            end = !PARTS || end + part_tiles > n_it ? n_it : end + part_tiles;       // part_tiles is even
            for (; it < end; it += 2) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {             // two tiles a trip: which half holds what is known when compiling
                    if (it + h >= end) break;
                    const int nx = rd + 1 == STAGES ? 0 : rd + 1;
                    WAIT_LGKMCNT(0);                      // this wave holds all of tile it + h
                    WAIT_VMCNT((STAGES - 2) * NLOAD);     // its share of the next one has landed
                    __builtin_amdgcn_s_barrier();
#pragma unroll
                    for (int j = 0; j < KSUB; ++j) load_frags(nx, j, fa[h ^ 1][j], fb[h ^ 1][j]);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_tile(rd);
#pragma unroll
                    for (int j = 0; j < KSUB; ++j) mfma_all(fa[h][j], fb[h][j]);
                    __builtin_amdgcn_sched_barrier(0);
                    advance_tile();
                    rd = nx;
                }
            }
            put_aside();
        } while (PARTS && end < n_it);
    } else {
        static_assert(KSUB % 2 == 0, "fragments of even sub-steps in one set of registers, of odd ones in the other");
        bf16x8_t fa[2][TC], fb[2][TP];
        load_frags(0, 0, fa[0], fb[0]);
        int rd = 0;
        int it = 0, end = 0;
        do {
            end = !PARTS || end + part_tiles > n_it ? n_it : end + part_tiles;
            for (; it < end; ++it) {
                const int nx = rd + 1 == STAGES ? 0 : rd + 1;
#pragma unroll
                for (int j = 0; j + 1 < KSUB; ++j) {
                    load_frags(rd, j + 1, fa[(j + 1) & 1], fb[(j + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);        // keep the reads ahead of the MFMAs that hide them
                    mfma_all(fa[j & 1], fb[j & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                WAIT_LGKMCNT(0);                              // this wave has read all of tile kt
                WAIT_VMCNT((STAGES - 2) * NLOAD);             // its share of tile kt+1 has landed
                __builtin_amdgcn_s_barrier();
                load_frags(nx, 0, fa[0], fb[0]);
                __builtin_amdgcn_sched_barrier(0);
                issue_tile(rd);                               // tile kt+STAGES into the slot just retired; its address
                mfma_all(fa[1], fb[1]);                       // arithmetic is free to mix with these MFMAs
                __builtin_amdgcn_sched_barrier(0);
                advance_tile();
                rd = nx;
            }
            put_aside();
        } while (PARTS && end < n_it);
    }
    WAIT_VMCNT(0);
    __syncthreads();

    auto &sums_of = [&]() -> auto & {
        if constexpr (PARTS) return aside;
        else return acc;
    }();
    // threads that move the finished tile in 16-byte units
    constexpr int CH8 = BC / 8;                 // 16-byte units per pixel row
    constexpr int ET = NT < BP * CH8 ? NT : BP * CH8;
    if constexpr (KG > 1) {
        // [group][pixel][channel] floats; every thread adds the groups' copies of a float4, in their order
        float *park = reinterpret_cast<float *>(smem);
#pragma unroll
        for (int a = 0; a < TC; ++a)
#pragma unroll
            for (int b = 0; b < TP; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(park + (kg * BP + wp * WT_P + b * 32 + frow) * PITCH + wc * WT_C + a * 32 + 8 * q + 4 * fhalf) =
                        make_float4(sums_of[a][b][4 * q], sums_of[a][b][4 * q + 1], sums_of[a][b][4 * q + 2], sums_of[a][b][4 * q + 3]);
        __syncthreads();
        // a float4 of the tile to the staging tile, with bias and ReLU
        auto to_tile = [&](int prow, int col, float4 v) {
            const float4 bv = *reinterpret_cast<const float4 *>(sBias + col);
            v.x += bv.x; v.y += bv.y; v.z += bv.z; v.w += bv.w;
            if (relu) v = make_float4(fmaxf(v.x, 0.0f), fmaxf(v.y, 0.0f), fmaxf(v.z, 0.0f), fmaxf(v.w, 0.0f));
            chunk8 c8;
            c8[0] = pack_bf16(v.x, v.y);
            c8[1] = pack_bf16(v.z, v.w);
            *reinterpret_cast<chunk8 *>(sO + prow * SROW + col) = c8;
        };
        // K split over blocks: part[split][pixel][co].  Where there are tickets (PANELS: linear layers) the blocks of a tile count themselves, and the one that comes
        // last adds all the sums, in the order of the splits, and goes on to the epilogue: nobody waits.  Stores and loads are of agent
        // scope, and a block counts itself when its stores are complete, so that no cache has to be written back.  It takes 2.5 us, a launch
        // that adds them 4.8 and the gap in front of it.  Without tickets the sums are left to the next launch.
        const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(part, 0, (int)((unsigned)gridDim.y * npix * g.Co * 4u), 0x00020000);
        auto part_at = [&](int split, int prow, int col) {
            const int p = pix0 + prow, co = co0 + col;
            return p < npix && co < g.Co ? ((unsigned)(split * npix + p) * g.Co + co) * 4u : OOB;
        };
        auto put_part = [&](int prow, int col, float4 v) {
            if (PANELS && tickets)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(chunk16, v), prsrc, part_at(blockIdx.y, prow, col), 0, 16);
            else if (pix0 + prow < npix && co0 + col < g.Co)
                *reinterpret_cast<float4 *>(part + ((size_t)blockIdx.y * npix + pix0 + prow) * g.Co + co0 + col) = v;
        };
        auto all_parts = [&](int prow, int col) {
            float4 t = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            for (int k = 0; k < (int)gridDim.y; k += 4) {
                chunk16 c[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) c[u] = __builtin_amdgcn_raw_buffer_load_b128(prsrc, k + u < (int)gridDim.y ? part_at(k + u, prow, col) : OOB, 0, 16);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float4 v = __builtin_bit_cast(float4, c[u]);
                    t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
                }
            }
            return t;
        };
        auto last_split = [&]() {
            if (!tickets) return false;
            int *last = reinterpret_cast<int *>(sBias + BC);                 // where a PHASED tile, whose K is whole, has its pixels
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid == 0) {
                unsigned *t = tickets + blockIdx.x;
                *last = __hip_atomic_fetch_add(t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.y - 1;
                if (*last) __hip_atomic_store(t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __syncthreads();
            return *last != 0;
        };
        constexpr int F4 = BC / 4;
        for (int i = tid; i < BP * F4; i += NT) {
            const int prow = i / F4, col = i % F4 * 4;
            float4 v = *reinterpret_cast<const float4 *>(park + prow * PITCH + col);
#pragma unroll
            for (int u = 1; u < KG; ++u) {
                const float4 w = *reinterpret_cast<const float4 *>(park + (u * BP + prow) * PITCH + col);
                v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
            }
            if (part) put_part(prow, col, v);
            else to_tile(prow, col, v);
        }
        if (part) {
            if (!PANELS || !last_split()) return;
            for (int i = tid; i < BP * F4; i += NT) to_tile(i / F4, i % F4 * 4, all_parts(i / F4, i % F4 * 4));
        }
    } else if (part) {
        // split-K: raw fp32 sums, 4 consecutive channels of one pixel per store; bias, ReLU and the
        // gradient epilogue are applied by the reduction kernel
        float *dst = part + (size_t)blockIdx.y * npix * g.Co;
#pragma unroll
        for (int a = 0; a < TC; ++a)
#pragma unroll
            for (int b = 0; b < TP; ++b) {
                const int p = pix0 + wp * WT_P + b * 32 + frow;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int co = co0 + wc * WT_C + a * 32 + 8 * q + 4 * fhalf;
                    if (p < npix && co < g.Co)
                        *reinterpret_cast<float4 *>(dst + (size_t)p * g.Co + co) =
                            make_float4(sums_of[a][b][4 * q], sums_of[a][b][4 * q + 1], sums_of[a][b][4 * q + 2], sums_of[a][b][4 * q + 3]);
                }
            }
        return;
    }

    // ---- epilogue: every wave parks its sub-tile in LDS as [pixel][channel] (bf16, bias and ReLU
    // applied), one barrier, then the block streams the tile out as 16-byte coalesced rows
    const chunk16 zero16 = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int a = 0; a < (KG == 1 ? TC : 0); ++a) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int col = wc * WT_C + a * 32 + 8 * q + 4 * fhalf;      // channel inside the tile
            const float4 bv = *reinterpret_cast<const float4 *>(sBias + col);
#pragma unroll
            for (int b = 0; b < TP; ++b) {
                const int prow = wp * WT_P + b * 32 + frow;              // pixel inside the tile
                float v0 = sums_of[a][b][4 * q] + bv.x, v1 = sums_of[a][b][4 * q + 1] + bv.y;
                float v2 = sums_of[a][b][4 * q + 2] + bv.z, v3 = sums_of[a][b][4 * q + 3] + bv.w;
                if (relu) {
                    v0 = fmaxf(v0, 0.0f);
                    v1 = fmaxf(v1, 0.0f);
                    v2 = fmaxf(v2, 0.0f);
                    v3 = fmaxf(v3, 0.0f);
                }
                chunk8 c8;
                c8[0] = pack_bf16(v0, v1);
                c8[1] = pack_bf16(v2, v3);
                *reinterpret_cast<chunk8 *>(sO + prow * SROW + col) = c8;
            }
        }
    }
    // The tile leaves in 16-byte units, UNITS per thread.  What a gradient unit needs besides its own value (gate row,
    // stored gradient, batch-norm input) is requested for a whole batch of units before the first of them is used or
    // stored - the first batch now, while the staging tile is being completed.  Requested unit by unit, behind the store
    // of the one before (which may alias), each cost a memory latency: 1x1 128->256 at 56x56, 32 samples, with the stored
    // gradient added, 53 -> 48 us; 3x3 / 2 gradient of 128 channels at 56x56 with the batch-norm sums, 44 -> 42 us.
    constexpr int UNITS = BP * CH8 / ET;        // per thread
    constexpr int BATCH = UNITS < 8 ? UNITS : 8;
    static_assert(ET % CH8 == 0 && UNITS % BATCH == 0, "a thread keeps one channel group; whole batches");
    const int c8i = tid % CH8, rg = tid / CH8, co = co0 + c8i * 8;
    auto pixel_of = [&](int it) { const int prow = rg + it * (ET / CH8); return PHASED ? sPix[prow] : pix0 + prow; };
    chunk16 gpre[BATCH] = {}, opre[BATCH] = {}, xpre[BATCH] = {};
    auto fetch = [&](chunk16(&to)[BATCH], const bf16_t *from, int it0) {
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int p = tid < ET ? pixel_of(it0 + j) : npix;
            to[j] = p < npix && co < g.Co ? *reinterpret_cast<const chunk16 *>(from + (size_t)p * g.Co + co) : zero16;
        }
    };
    auto request = [&](int it0) {
        if (gate) fetch(gpre, gate, it0);
        if (accum) fetch(opre, old_from ? old_from : out, it0);
        if (bn_x) fetch(xpre, bn_x, it0);
    };
    if (is_grad) request(0);
    // Per-channel sums over this pixel tile for a batch-norm, stat_part[q][pixel tile][channel], the layout the final pass
    // of the column reductions reads.  For one whose output gradient this is (bn_x its input, bn_stats its mean and
    // 1/std): of dy and dy*xhat, taken on the way out.
    float bs1[8], bs2[8], bmu[8], binv[8];
    if (bn_x) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            bs1[j] = bs2[j] = 0.0f;
            bmu[j] = co + j < g.Co ? bn_stats[co + j] : 0.0f;
            binv[j] = co + j < g.Co ? bn_stats[g.Co + co + j] : 0.0f;
        }
    }
    __syncthreads();
    // For one that follows: of the STORED (rounded) values and their squares, what its first pass would compute.  All
    // threads walk down the staged tile, NT / BC of them per channel (one per channel left three of four waves of a
    // 256 x 64 tile waiting for 256 rows: 1x1 and 3x3 64->64 at 56x56 and their like, 23.4 -> 22 us a launch).
    float2 *sums = reinterpret_cast<float2 *>(smem + PARK_BYTES + TILE_BYTES);        // [GROUPS][BC]
    constexpr int ST = NT / BC < BP ? NT : BP * BC;                     // threads that add them up
    constexpr int GROUPS = ST / BC, GROWS = BP / GROUPS;
    if (stat_part && !bn_x && tid < ST) {
        const int cc = tid % BC, r0 = tid / BC * GROWS;
        const int here = rows - pix0 < BP ? rows - pix0 : BP, r1 = r0 + GROWS < here ? r0 + GROWS : here;
        float2 t = make_float2(0.0f, 0.0f);
#pragma unroll 8
        for (int r = r0; r < r1; ++r) {
            const float v = __uint_as_float((uint32_t)sO[r * SROW + cc] << 16);
            t.x += v;
            t.y += v * v;
        }
        sums[tid] = t;
    }
#pragma unroll
    for (int it0 = 0; it0 < UNITS; it0 += BATCH) {
        if (it0 && is_grad) request(it0);
#pragma unroll
        for (int j0 = 0; j0 < BATCH; ++j0) {
            const int p = tid < ET ? pixel_of(it0 + j0) : npix;
            if (p < npix && co < g.Co) {
                const uint16_t *src = sO + (rg + (it0 + j0) * (ET / CH8)) * SROW + c8i * 8;
                const chunk8 lo = *reinterpret_cast<const chunk8 *>(src), hi = *reinterpret_cast<const chunk8 *>(src + 4);
                chunk16 r = {lo[0], lo[1], hi[0], hi[1]};
                if (is_grad) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) r[j] = grad_epilogue_pair(r[j], opre[j0][j], gpre[j0][j], accum != 0, gate != nullptr);
                }
                *reinterpret_cast<chunk16 *>(out + (size_t)p * g.Co + co) = r;
                if (bn_x) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float gj = __uint_as_float((j & 1) ? (r[j >> 1] & 0xFFFF0000u) : (r[j >> 1] << 16));
                        const float xj = __uint_as_float((j & 1) ? (xpre[j0][j >> 1] & 0xFFFF0000u) : (xpre[j0][j >> 1] << 16));
                        bs1[j] += gj;
                        bs2[j] += gj * ((xj - bmu[j]) * binv[j]);
                    }
                }
            }
        }
    }
    if (!stat_part) return;
    float *red = reinterpret_cast<float *>(smem);                          // [RG][2][BC]; what was parked and staged is free now
    constexpr int RG = ET / CH8;                                           // threads that share a channel group
    static_assert((size_t)RG * BC * 2 * sizeof(float) <= PARK_BYTES + TILE_BYTES && ST % BC == 0 && BP % GROUPS == 0, "sums fit their places");
    __syncthreads();
    if (bn_x) {
        if (tid < ET) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                red[(rg * 2 + 0) * BC + c8i * 8 + j] = bs1[j];
                red[(rg * 2 + 1) * BC + c8i * 8 + j] = bs2[j];
            }
        }
        __syncthreads();
    }
    if (tid < BC && co0 + tid < g.Co) {
        float2 t = make_float2(0.0f, 0.0f);
        if (bn_x) {
            // eights in float, the eights in double: one after the other, the 64 of a 64 x 64 tile of wave groups left dgamma of
            // 784 rows 1.2e-7 off 64 bits (7.7e-8 so; 8.6e-8 where one launch reads such a tensor whole)
            static_assert(RG % 8 == 0, "whole eights");
            double tx = 0.0, ty = 0.0;
#pragma unroll 2
            for (int k = 0; k < RG; k += 8) {
                float e[8], f[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    e[u] = red[((k + u) * 2 + 0) * BC + tid];
                    f[u] = red[((k + u) * 2 + 1) * BC + tid];
                }
                tx += (double)(((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7])));
                ty += (double)(((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])));
            }
            t = make_float2((float)tx, (float)ty);
        } else {
#pragma unroll
            for (int k = 0; k < GROUPS; ++k) {
                t.x += sums[k * BC + tid].x;
                t.y += sums[k * BC + tid].y;
            }
        }
        stat_part[(size_t)tile_z * g.Co + co0 + tid] = t.x;
        stat_part[((size_t)tiles_all + tile_z) * g.Co + co0 + tid] = t.y;
    }
}

// out[p][co] = epilogue( sum_split part[split][p][co] + bias[co] ), 8 channels per thread
__global__ void k_gather_splitk_reduce(const float *__restrict__ part, int splits, size_t total, int Co,
                                       const float *__restrict__ bias, bf16_t *out,
                                       const bf16_t *__restrict__ gate, int accum, int relu, int is_grad,
                                       const bf16_t *old_from)
{
    size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i >= total) return;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = 0.0f;
    for (int k = 0; k < splits; ++k) {
        float4 a = *reinterpret_cast<const float4 *>(part + (size_t)k * total + i);
        float4 b = *reinterpret_cast<const float4 *>(part + (size_t)k * total + i + 4);
        v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
        v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
    }
    const int co = (int)(i % Co);
    vec_t<bf16_t, 8> old, gt, r;
    if (is_grad && accum) old = *reinterpret_cast<const vec_t<bf16_t, 8> *>((old_from ? old_from : out) + i);
    if (is_grad && gate) gt = *reinterpret_cast<const vec_t<bf16_t, 8> *>(gate + i);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float x = v[j] + (bias ? bias[co + j] : 0.0f);
        if (relu) x = fmaxf(x, 0.0f);
        r.e[j] = is_grad ? grad_out<bf16_t>(x, accum != 0, old.e[j], gate != nullptr, gt.e[j]) : from_f32<bf16_t>(x);
    }
    *reinterpret_cast<vec_t<bf16_t, 8> *>(out + i) = r;
}

struct GatherPlan {
    int bp, bc, bk, kg, splits, kt_per_split, part_tiles;
    int classes;             // 1, or the classes of a PHASED launch
    int busy;                // classes that have taps
    long long class_pix;     // output pixels of the largest class
};

// output pixels of the largest class
long long class_pixels(const GatherConv &g) { return (long long)g.N * ((g.Ho + g.s_in - 1) / g.s_in) * ((g.Wo + g.s_in - 1) / g.s_in); }

// The taps-innermost order of K needs whole K-tiles of channels and a 32-bit tap mask; for a 1x1 filter there is one tap and
// any K will do.  Of its classes one has the tap and the others only their epilogue (a projection shortcut's gradient, 56x56
// of 256 channels, 32 samples: 27 us, as a dense product into the workspace and a pass that spread it 16 + 23).
// A class is a step of the grid's z axis (65536 at most): s_in^2 of them, fewer where the image is smaller than the stride.
// More of them than the chip holds blocks have to fill a quarter of a tile each, or their epilogues take longer than the
// products with zeros (backward of 1x1 / 100, 64 channels, one 100x100 image: 67 us as 10000 classes, 13 without; 1x1 / 20:
// 9.0 us as 400 classes, 13.4 without).
int gather_classes(const GatherConv &g)
{
    if (g.s_in == 1 || g.s_in > 65535 || g.s_out != 1 || g.pad_h < 0 || g.pad_w < 0) return 1;
    if (!(g.R == 1 && g.S == 1) && (g.Ci % 32 != 0 || g.R * g.S > 32)) return 1;
    const long long n = (long long)(g.s_in < g.Ho ? g.s_in : g.Ho) * (g.s_in < g.Wo ? g.s_in : g.Wo);
    return n <= 1024 || (n <= 65535 && class_pixels(g) >= 16) ? (int)n : 1;
}

// Tile shape and split-K factor.  K is split only when there are very few output tiles (the linear
// layers: one pixel tile).
GatherPlan gather_plan(const GatherConv &g)
{
    GatherPlan p;
    const long long npix = (long long)g.N * g.Ho * g.Wo;
    p.classes = gather_classes(g);
    p.busy = (g.R < g.s_in ? g.R : g.s_in) * (g.S < g.s_in ? g.S : g.s_in);
    if (p.busy > p.classes) p.busy = p.classes;
    p.class_pix = p.classes == 1 ? npix : class_pixels(g);
    p.bp = p.class_pix <= 64 ? 64 : 256;
    p.bc = g.Co <= 64 ? 64 : 128;
    if (p.bp == 64) p.bc = 128;
    auto tiles_of = [&](int bp) { return p.busy * ((p.class_pix + bp - 1) / bp) * ((g.Co + p.bc - 1) / p.bc); };
    // Up to 400 tiles of 256 x 128 are one round of the chip (two blocks a unit); 256 x 256 would leave units without one, and
    // twice as many of 128 x 128 come to a round and a half and fetch more (3x3 512->256 at 28x28, 64 samples, 392 tiles: 163 us
    // against 134; 4096->1024 from 6000 rows, 192: 77 against 70; 294 tiles, 256->128 at 56x56: 62 against 64).  Of fewer than
    // about 200 alone on the chip the smaller tiles fill more of it, beside other streams only of fewer than 128 (mini-batches of
    // three 3x3 512->512 layers at 14x14, us, 256 x 128 against 128 x 128: one stream 132 tiles 3695 / 3500, 160 3956 / 3785,
    // 184 4170 / 4062, 196 4253 / 4198, 248 4649 / 4920, of 256->256 at 28x28 210 tiles 2699 / 2705; three streams 120 tiles
    // 3372 / 2740, 132 2779 / 3000, 144 2938 / 3192, 160 3180 / 3553).
    const long long least = g.beside ? 128 : 192;
    const bool few = p.bp == 256 && p.bc == 128 && tiles_of(256) < 400 && tiles_of(256) >= least;
    if (!few && p.bp == 256 && p.bc == 128 && tiles_of(256) < 400) p.bp = 128;
    // small products (the bottleneck blocks of ResNet: under ~8 GMAC) are bound by the latency of a block's
    // load - multiply - store chain, not by throughput: many 64-pixel blocks and no split of K were the
    // fastest choice on every such shape measured (e.g. 1x1 1024->256 at 14x14: 11.5 us against 22.2)
    // So are products up to twice that whose 64-pixel tiles fit two blocks per unit (3x3 512->512 at 14x14, 32 samples:
    // 47.6 -> 36.8 us; the LSTM's input gradient, 3200 x 1024 x 4096: 59 -> 43), if they do not fetch much more that way.  A
    // 3x3 filter re-reads the tile's pixels, and filters up to 12 MB stay in the L2s; of larger 1x1 filters every row of
    // tiles streams its own copy (4096->4096, 900 rows, two blocks per unit: 46.0 us against 63.6; 25088->4096, 128 rows, K
    // split over half as many tiles: 54 against 73), so there it takes one block per unit and no split (6144->3072, 600
    // rows: 58.6 -> 46.9; 4096->4096, 512 rows: 43.6 -> 39.9).
    const double macs = (double)npix * g.Co * g.R * g.S * g.Ci / p.classes;
    const bool cheap = g.R * g.S > 1 || (double)g.Co * g.Ci * 2 <= 12e6 || (tiles_of(64) > 128 && tiles_of(64) <= 256);
    if (p.bc == 128 && npix > 64 && (macs < 8e9 || (macs < 16e9 && tiles_of(64) <= 512 && cheap))) p.bp = 64;
    // plenty of 256-pixel tiles and whole 256-channel tiles: one 8-wave block per CU owns 256 x 256, which
    // halves the L2 -> LDS traffic of two independent 256 x 128 blocks (3 % on the 512-channel 28x28 layers)
    if (!few && p.bp == 256 && p.bc == 128 && g.Co % 256 == 0) p.bc = 256;
    // Few tiles: a block's chain of K-steps is what takes the time, and splitting K over blocks costs a second launch (and
    // leaves no statistics for a batch-norm).  K is split over the wave groups of a block instead, on the smallest tiles that
    // come to one block per unit (us, KG = 1 with its reduction before -> now: 32 x 32, 1024->256 from 784 pixels 10.7 -> 6.2,
    // 3x3 256->256 12.9 -> 10.5, 4096->4096 for 8 rows 12.2 -> 9.2; 32 x 64, 2048->512 from 1000 14.6 -> 8.9; 64 x 64, 2048->512
    // from 1568 18.9 -> 11.5, 3x3 512->512 27.9 -> 21.8).  More tiles than that hide each other's latencies better (64 x 64,
    // 3x3 256->512 from 3136 pixels, 392 tiles: 25.5 against 17.9).  Not for a large filter, which every row of tiles would
    // fetch again; one row of 64 takes it in as many splits as make a block per unit (25088->4096, 64 rows: 47.2 -> 38.5).
    const long long K = (long long)g.R * g.S * g.Ci;
    auto count = [&](int bp, int bc) { return ((npix + bp - 1) / bp) * ((g.Co + bc - 1) / bc); };
    const bool large = 2.0 * g.Co * K > 40e6, k64 = g.Ci % 64 == 0 && g.R * g.S <= 32;
    // Few rows of a 1x1 filter of 15 to 20 M weights, maps of single pixels: 64 x 64 tiles, and as many blocks share a tile's K as make a block
    // per unit.  Filters in panels, 33 / 64 rows, that the caches do not hold, us, as one launch of the tiles below -> so: 9216->2048, eight shares
    // and the launch that adds them, 18.6 / 23.0 -> 15.7 / 16.0; 6144->3072, five, 16.1 / 18.0 -> 14.4 / 15.5; 4096->4096, four, which the
    // last of them adds, 14.7 / 14.3 -> 12.8 / 13.6; 3072->5120, three, 13.2 / 14.6 -> 12.3 / 12.9; two: 3072->6144 15.0 / 15.2 -> 13.8 / 14.8,
    // 2560->6144 13.2 / 13.6 -> 12.8 / 14.1, 2048->8192 13.0 / 13.1 -> 12.4 / 13.2.  Of fewer weights a share would be too short
    // (2048->2048, four of 512, 7.8 -> 11).  Of filters in rows a launch adds the shares; mini-batches of four (LSTM: two) micro-batches, either
    // direction: 1x1 / 2 of 1x1 maps, 33 / 64 rows, 4096->4096 277 / 276 -> 258 / 262, 2048->8192 277 / 285 -> 260 / 268, 9216->2048 313 / 322 ->
    // 293 / 309; LSTM of 2048, one step, 713 / 744 -> 705 / 711, of 1984, 50 rows, 689 -> 665; its dependent steps the same either way.
    // A gradient of classes of pixels (s_in > 1, more than one pixel) keeps the kernel that knows them.
    const bool flat = (g.s_in == 1 || (g.Ho == 1 && g.Wo == 1)) && g.Hi == 1 && g.Wi == 1 && g.R * g.S == 1 && !g.by_norm && 2.0 * g.Co * K > 30e6;
    p.kg = 1;
    if (flat && npix > 32 && npix <= 64 && k64 && count(64, 64) <= 128) {
        p.kg = 2;
    } else if (g.s_in == 1 && large && npix > 32) {
        if (npix <= 64 && k64 && count(64, 64) <= 128) p.kg = 2;
    } else if (g.s_in == 1 && K >= 512 && count(32, 32) <= 256) {
        p.kg = 8;
        p.bp = p.bc = 32;
    } else if (g.s_in == 1 && K >= 512 && count(32, 64) <= 256) {
        p.kg = 4;
        p.bp = 32;
        p.bc = 64;
    } else if (g.s_in == 1 && K >= 256 && count(64, 64) <= 256) {
        p.kg = 2;
    }
    if (p.kg == 2) p.bp = p.bc = 64;
    // Tiles of eight waves, one block to a unit, with K-tiles of 64 channels.  A row of 64 channels is a whole cache line: of 32
    // it is half of one, which costs the vector L1 the same request (rows 1 KB apart from the L2s: 75 against 139 bytes per ns
    // and unit).  256 x 256 (us, BK = 32 -> so; 3x3 512->512 at 28x28, 64 samples, 236 -> 227, 256->512 132 -> 128, 512->256,
    // 196 tiles, 147 as 392 of 256 x 128 -> 123); 256 x 128 where those come to one block a unit at most: 512->512 at 14x14, 64
    // samples, 196 tiles, 82 -> 70, 52 samples 74 -> 66, 40 (124 tiles, 248 of 64 x 128) 47 against 64; 128 x 256 the same.  Beside other streams
    // the units that few large tiles leave idle are not lost: mini-batches of three 3x3 layers on three streams, us, 256 x 256
    // against 256 x 128: 512->512 at 14x14, 40 samples (124 halves) 2999 / 2845, 64 (196) 4496 / 4709, 256->256 at 28x28, 32
    // (98 pixel tiles, 98 halves x 2) 2088 / 2171.  K below 1024 is bound by the epilogue, which a lone block does not overlap
    // (residual block with 1x1 filters of 128 to 256 channels, three streams, 3477 -> 3540); other widths keep two blocks of four waves.
    const long long halves = count(256, 128);
    // Fewer than 144 halves, or rows of pixels that mostly end outside the image, are faster on the smaller tiles (3x3 128->2048 at
    // 13x17, 9 samples, 128 halves: 18.4 us against 25.0 as 128 x 256; 4096->4096 from 900 rows 52.3 / 58.6, 1500 rows 75.6 / 63.9;
    // 1x1 1024->2048 from 3136 pixels 32.2 / 23.0; 25088<-4096 from 64 rows, 196 tiles, 51.6 / 59.8).
    const bool whole = 8 * npix >= 7 * 256 * ((npix + 255) / 256);
    const bool eight = p.kg == 1 && g.s_in == 1 && k64 && K >= 1024 && p.bc >= 128 && halves >= 144 && whole && (g.Co % 256 == 0 || halves <= 256);
    p.bk = 32;
    if (eight) {
        p.bk = 64;
        p.bp = p.bc = 256;
        if (g.Co % 256 || halves <= (g.beside ? 180 : 256)) {
            if (g.Co % 256 == 0 && halves < least) p.bp = 128;
            else p.bc = 128;
        }
    }
    // Up to 64 channels the tile is 128 x 64, four blocks (37 KB of LDS each) to a unit, not 256 x 64: half the fragments a wave waits for and twice
    // the blocks that hide it (7x7 / 2 of the stem, 224x224, 32 images 54.7 -> 44.2 us; 64->64 from 401408 pixels 1x1 32.0 ->
    // 24.0, from 40500 3x3 13.8 -> 12.3, from 387200 61.4 -> 56.0, from 100352 20.2 -> 20.6).
    if (p.bc == 64 && p.bp == 256) p.bp = 128;
    const long long tiles = tiles_of(p.bp);
    // K-tiles of 64 channels, read a whole tile ahead, for 64-pixel tiles that come to at most two blocks per compute
    // unit (that kernel's LDS and registers allow no more): 3x3 256->256 and 1x1 1024->256 at 14x14, 32 samples, 196
    // blocks, together 21.8 -> 18.1 us a launch; VGG-16's first linear layer 54.5 -> 48 us forward, 63.8 -> 52 gradient.
    // With more blocks than that the four smaller ones that fit a unit hide the latencies better (1x1 512->256 at 56x56,
    // 3136 blocks: 53 us against 81).  Does not depend on `beside`: K is summed in another order.
    if ((p.kg == 2 && k64) || (p.kg == 1 && p.bp == 64 && tiles <= 512 && k64 && (g.s_in == 1 || p.classes > 1))) p.bk = 64;
    const int BK = p.bk;
    const int KT = g.Ci % BK == 0 ? (g.Ci / BK) * g.R * g.S : (g.R * g.S * g.Ci + BK - 1) / BK;
    long long want = p.kg > 1 ? (large || (flat && p.kg == 2) ? 256 / tiles : 1) : tiles >= 128 || eight ? 1 : (512 + tiles - 1) / tiles;
    long long most = KT * BK / 512;                 // at least 512 of K per split
    if (want > most) want = most;
    if (want > 32) want = 32;
    if (want < 1 || p.classes > 1) want = 1;
    p.kt_per_split = (int)((KT + want - 1) / want);
    p.splits = (KT + p.kt_per_split - 1) / p.kt_per_split;
    // equal parts of at most 384 of K
    const int in_group = (p.kt_per_split + p.kg - 1) / p.kg, parts = (in_group * BK + 383) / 384;
    p.part_tiles = parts > 1 ? ((in_group + parts - 1) / parts + 1) / 2 * 2 : in_group + 1;
    return p;
}

template <int BP, int BC, int WP, int WC, int BK, int STAGES, int KG = 1>
hipError_t launch_gather(const void *in, const void *wt, const float *bias, void *out, int relu, GradEpi epi,
                         const GatherConv &g, const GatherPlan &plan, void *workspace, unsigned *tickets, hipStream_t s, bool raw = false,
                         float *stat_part = nullptr, const void *bn_x = nullptr, const float *bn_stats = nullptr)
{
    constexpr int NT = WP * WC * KG * 64;
    constexpr size_t main_bytes = (size_t)KG * STAGES * (BP + BC) * BK * 2;
    // the groups' sums, staging tile, per-thread sums
    constexpr size_t epi_bytes = (KG > 1 ? (size_t)KG * BP * (BC + 4) * 4 : 0) + (size_t)BP * (BC + 4) * 2 + NT * 8;
    constexpr size_t smem_flat = (main_bytes > epi_bytes ? main_bytes : epi_bytes) + BC * sizeof(float) + sizeof(int);
    const bool phased = plan.classes > 1;
    // Of a kernel that does not look at the grid's z axis every class would store all tiles
    if (phased && (KG > 1 || (BK == 64 && BP != 64))) return hipErrorInvalidValue;
    constexpr size_t smem_phased = smem_flat + BP * sizeof(int);
    const size_t smem = phased ? smem_phased : smem_flat;
    static_assert(smem_phased <= (NT >= 512 || STAGES > 4 ? 160 : 80) * 1024, "two blocks of 4 waves (one of 8, or with a deep ring) must fit the 160 KB LDS of a CU");
    const long long npix = (long long)g.N * g.Ho * g.Wo;
    const int tiles_p = (int)((plan.class_pix + BP - 1) / BP), tiles_c = (g.Co + BC - 1) / BC;
    const int is_grad = (epi.gate != nullptr || epi.accum) ? 1 : 0;
    const unsigned in_bytes = (unsigned)((size_t)g.N * g.Hi * g.Wi * g.Ci * 2);
    const unsigned wt_bytes = (unsigned)((size_t)g.Co * g.R * g.S * g.Ci * 2);
    float *part = (plan.splits > 1 || raw) ? (float *)workspace : nullptr;      // raw: the fp32 partials are the result
    // One block of wave groups, which has its tile in rows, adds up to four sums faster than a launch would start; of eight the launch,
    // whose blocks share them, is the faster way, and so it is where a thread has its sums in pieces of 16 bytes (64 rows, us: 12544<-2048,
    // four splits of 64 x 128, 16.0 and 4.9 by launch, 25.2)
    if (raw || KG == 1 || plan.splits > 4 || !g.wt_panels) tickets = nullptr;
    else if (plan.splits > 1 && (!tickets || tiles_p * tiles_c > kGatherTickets)) return hipErrorInvalidValue;
    dim3 grid((unsigned)(tiles_p * tiles_c), (unsigned)plan.splits, (unsigned)plan.classes);
#define GATHER_LAUNCH(S1_, TI_, ...)                                                                                   \
    do {                                                                                                          \
        auto kfn = k_gather_mfma<BP, BC, WP, WC, BK, STAGES, KG, S1_, TI_, __VA_ARGS__>;                              \
        static bool attr_set = false;                                                                             \
        if (!attr_set && smem > 64 * 1024) {                                                                      \
            hipError_t e = hipFuncSetAttribute((const void *)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); \
            if (e != hipSuccess) return e;                                                                        \
            attr_set = true;                                                                                      \
        }                                                                                                         \
        hipLaunchKernelGGL(kfn, grid, dim3(NT), smem, s, (const bf16_t *)in, (const bf16_t *)wt, bias,          \
                           (bf16_t *)out, (const bf16_t *)epi.gate, epi.accum, relu, is_grad, (GatherGeom)g, tiles_c, in_bytes, \
                           wt_bytes, part, plan.kt_per_split, plan.part_tiles, stat_part, (const bf16_t *)bn_x, bn_stats,         \
                           (const bf16_t *)epi.accum_from, tickets);                                             \
    } while (0)
    const bool taps_inner = g.Ci % BK == 0 && g.R * g.S <= 32;      // the stride-1 variant keeps a 32-bit tap mask
    if (g.wt_panels) {
        if (taps_inner && !phased && g.s_in == 1) GATHER_LAUNCH(true, true, false, true);
        else return hipErrorInvalidValue;
    } else if constexpr (STAGES > 4) {
        return hipErrorInvalidValue;                                // only filters in panels take the deep ring
    } else if constexpr (KG > 1) {                                  // stride-1 operands
        if (taps_inner) GATHER_LAUNCH(true, true, false);
        else if constexpr (BK == 32) GATHER_LAUNCH(true, false, false);
    } else if constexpr (BK == 64) {
        if constexpr (BP == 64) {
            if (phased) GATHER_LAUNCH(true, true, true);
            else GATHER_LAUNCH(true, true, false);
        } else GATHER_LAUNCH(true, true, false);                    // one class
    } else if (phased) {
        if (taps_inner) GATHER_LAUNCH(true, true, true);
        else GATHER_LAUNCH(true, false, true);
    } else if (g.s_in == 1) {
        if (taps_inner) GATHER_LAUNCH(true, true, false);
        else GATHER_LAUNCH(true, false, false);
    } else {
        GATHER_LAUNCH(false, false, false);
    }
#undef GATHER_LAUNCH
    if (part && !raw && !tickets) {
        const size_t total = (size_t)npix * g.Co;
        hipLaunchKernelGGL(k_gather_splitk_reduce, dim3((unsigned)((total / 8 + 255) / 256)), dim3(256), 0, s, part,
                           plan.splits, total, g.Co, bias, (bf16_t *)out, (const bf16_t *)epi.gate, epi.accum, relu,
                           is_grad, (const bf16_t *)epi.accum_from);
    }
    return hipGetLastError();
}

hipError_t launch_plan(const void *in, const void *wt, const float *bias, void *out, int relu, GradEpi epi, const GatherConv &g,
                       const GatherPlan &p, void *workspace, unsigned *tickets, hipStream_t s, bool raw = false, float *stat_part = nullptr,
                       const void *bn_x = nullptr, const float *bn_stats = nullptr)
{
#define TILE(...) return launch_gather<__VA_ARGS__>(in, wt, bias, out, relu, epi, g, p, workspace, tickets, s, raw, stat_part, bn_x, bn_stats)
    if (p.kg == 8) TILE(32, 32, 1, 1, 32, 4, 8);
    if (p.kg == 4) TILE(32, 64, 1, 2, 32, 4, 4);
    if (p.kg == 2 && p.bk == 64) TILE(64, 64, 2, 2, 64, 3, 2);
    if (p.kg == 2) TILE(64, 64, 2, 2, 32, 4, 2);
    // A filter that is streamed from memory, by blocks that have a unit to themselves: five K-tiles on their way instead of two
    // (25088<-4096, 64 rows, in panels, 41.2 -> 39.4 us; from rows of 8 KB, two on their way and every block from a K-tile of its own, 43.8)
    if (p.bk == 64 && p.bp == 64 && g.wt_panels && p.class_pix <= 64 && (g.Co + 127) / 128 * p.splits <= 256) TILE(64, 128, 1, 4, 64, 6);
    if (p.bk == 64 && p.bp == 64) TILE(64, 128, 1, 4, 64, 3);
    if (p.bk == 64 && p.bc == 256 && p.bp == 128) TILE(128, 256, 2, 4, 64, 3);
    if (p.bk == 64 && p.bc == 256) TILE(256, 256, 2, 4, 64, 2);
    if (p.bk == 64) TILE(256, 128, 4, 2, 64, 3);
    if (p.bp == 64) TILE(64, 128, 1, 4, 32, 3);
    if (p.bc == 64) TILE(128, 64, 4, 1, 32, 3);
    if (p.bc == 256) TILE(256, 256, 2, 4, 32, 3);
    if (p.bp == 128) TILE(128, 128, 2, 2, 32, 3);
    TILE(256, 128, 2, 2, 32, 3);
#undef TILE
}

// ------------------------------------------------------------------------------------------
// wgrad
// ------------------------------------------------------------------------------------------
// The GEMM's N index is the flattened (r, s, c) filter position n = (r*S + s)*C + c, so a tile
// of BCI columns covers one tap (or part of it) when C >= BCI and several taps when C is small.
// grid: the blocks of one product after another (job_of); those of a product, renumbered over the XCDs, by split of the pixels and by
// (ko tile, n tile) in it, the second product of a pair behind the first.  Same HBM -> LDS ring as the gather
// kernel: STAGES tiles of 32 pixels, requests issued STAGES-1 tiles ahead, hand-placed vmcnt waits.
// KG > 1: the block is KG groups of waves, each with a ring and a full set of sums of its own, that take the steps in turn;
// their sums meet in LDS at the end.  A lone block's chain of steps is KG times shorter that way, and nothing is written and
// read again for it, as the partial sums of KG times as many splits would be.
// LDS bytes of a block: the rings, or what KG groups park at the end
template <int BKO, int BCI, int STAGES, int KG>
constexpr size_t kWgradLds = KG > 1 && (size_t)KG * (BKO * (BCI + 4) + BKO) * 4 > (size_t)KG * STAGES * 32 * (BKO + BCI) * 2
                                 ? (size_t)KG * (BKO * (BCI + 4) + BKO) * 4
                                 : (size_t)KG * STAGES * 32 * (BKO + BCI) * 2;

// One product of a launch, or two of one shape with the same dy.
struct WgradArgs {
    const bf16_t *x, *x2, *dy;
    float *part, *part2, *bpart;
    size_t split_stride;
    ConvShape c;
    int tiles, tiles_n, splits, blocks;          // tiles of a split, blocks of the product
    int pix_per_split, part_tiles, add_to_dst;
    unsigned x_bytes, dy_bytes;
};
struct WgradPair : WgradArgs {};
// Products of one launch: small ones fill a fraction of the chip each, and a launch apiece lets them wait for each other (three
// of a bottleneck of 256 channels at 14x14, four samples, 64 to 144 blocks each: mini-batch 868 -> 774 us; four of the first VGG stage, 90x90, five
// samples, 252 blocks each and their reductions: 481 -> 390).  Ones that give every unit a block gain nothing and do not wait for
// others (ResNet's end 2792 -> 2827).  Those that wait anyway, for the hand-over to a stream of their own, go out together whatever
// their blocks: ones of 256 and more by themselves, conv4 block of ResNet 1392 us against 1361, its conv3 block and stem the same.
constexpr int WG_GROUP = 6;
template <class Args> struct Group {
    Args a[WG_GROUP];
    int n;
};
typedef Group<WgradArgs> WgradGroup;

// The product that a block of a launch belongs to, and the block's number in it.  A launch of one has it at hand: looking it up costs
// a chain of scalar loads, 0.5 us of a short launch.
template <class Args> __device__ __forceinline__ const Args &job_of(const Group<Args> &g, int &id)
{
    int job = 0;
    while (job + 1 < g.n && id >= g.a[job].blocks) id -= g.a[job++].blocks;
    return g.a[job];
}
template <class Args> __device__ __forceinline__ const Args &job_of(const Args &a, int &) { return a; }

template <int BKO, int BCI, int WKO, int WCI, int STAGES, int KG, class In>
__global__ __launch_bounds__(WKO *WCI *KG * 64, KG == 1 ? 2 : 1) void k_wgrad_mfma(In in)
{
    int id = blockIdx.x;
    const WgradArgs &job_args = job_of(in, id);
    const ConvShape c = job_args.c;
    const bf16_t *dy = job_args.dy;
    const size_t split_stride = job_args.split_stride;
    const int tiles = job_args.tiles, tiles_n = job_args.tiles_n, splits = job_args.splits, pix_per_split = job_args.pix_per_split;
    const int part_tiles = job_args.part_tiles, add_to_dst = job_args.add_to_dst;
    const unsigned x_bytes = job_args.x_bytes, dy_bytes = job_args.dy_bytes;
    constexpr int BKP = 32;
    constexpr int NW = WKO * WCI;                        // waves of a group
    constexpr int STEP = KG * BKP;                       // pixels from one tile of a group to its next
    constexpr int CPA = BKO / 8, CPB = BCI / 8;          // 16-byte chunks per tile row
    constexpr int AL = (BKP * CPA / 64) / NW, BL = (BKP * CPB / 64) / NW;   // wave-wide loads per wave and tile
    constexpr int WT_KO = BKO / WKO, WT_CI = BCI / WCI;
    constexpr int TA = WT_KO / 32, TB = WT_CI / 32;
    constexpr int STAGE_ELEMS = BKP * (BKO + BCI);
    constexpr unsigned OOB = 0x80000000u;
    static_assert(AL >= 1 && BL >= 1 && (BKP * CPA / 64) % NW == 0 && (BKP * CPB / 64) % NW == 0, "tile/thread mismatch");

    extern __shared__ __align__(16) unsigned char smem[];
    const lds_addr_of lds_of(smem);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave = wave_id % NW, kg = wave_id / NW;            // place inside the group, group
    const int wk = wave % WKO, wi = wave / WKO;
    uint16_t *ring = reinterpret_cast<uint16_t *>(smem) + kg * STAGES * STAGE_ELEMS;      // the group's [STAGES][ A tile | B tile ]
    // The tiles of one pixel split read the same dy and x rows: number the blocks so that a split's tiles run on
    // one XCD (one L2) - consecutive block ids go round the eight XCDs, so each XCD gets a contiguous range of
    // (split, tile) positions.  With a single split (or few blocks) this is the identity up to a permutation.
    const int pos = xcd_remap(id, job_args.blocks);
    const int nth = pos / tiles, bx = pos - nth * tiles;
    // The second product of a pair: another x, the same dy.  Launches that have none do not ask (1x1 512->2048 from 1568 rows 13.2 -> 12.8 us,
    // 1024->256 from 6272 15.3 -> 15.0).
    const bool second = std::is_same<In, WgradPair>::value && nth >= splits;
    const int by = second ? nth - splits : nth;
    const bf16_t *x = second ? job_args.x2 : job_args.x;
    float *part = second ? job_args.part2 : job_args.part, *bpart = second ? nullptr : job_args.bpart;
    const int tn = bx % tiles_n, tko = bx / tiles_n;
    const int ko0 = tko * BKO, n0 = tn * BCI;
    const int Ntot = c.R * c.S * c.C;
    const int npix = c.N * c.P * c.Q;
    const int p_begin = by * pix_per_split;
    const int p_end = p_begin + pix_per_split < npix ? p_begin + pix_per_split : npix;
    const int KT = (p_end - p_begin + KG * BKP - 1) / (KG * BKP);      // tiles of a group, which takes every KG-th
    const int p_first = p_begin + kg * BKP;

    __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(x), 0, (int)x_bytes, 0x00020000);
    __amdgpu_buffer_rsrc_t grsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(dy), 0, (int)dy_bytes, 0x00020000);

    // ---- A (dy) loads: lane fills slot (row, c') of wave-load q = i*NW + wave and fetches chunk c.
    // All addresses are kept as running byte offsets: a tile step adds a constant, so the loop body
    // has no multiplications.
    int ap[AL];                  // pixel of the lane's row in the current tile (huge if its chunk is past K)
    unsigned aoff[AL];           // byte offset of its chunk
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int slot = (i * NW + wave) * 64 + lane;
        const int row = slot / CPA, cs = slot % CPA;
        const int ch = ((((cs >> 1) ^ wg_swz<BKO>(row)) << 1) | (cs & 1));
        const bool kin = ko0 + ch * 8 < c.K;
        ap[i] = kin ? p_first + row : (1 << 30);
        aoff[i] = ((unsigned)(p_first + row) * (unsigned)c.K + (unsigned)(ko0 + ch * 8)) * 2u;
    }
    // ---- B (x) loads: filter position of the lane's chunk column (fixed) and its pixel (advancing):
    // bp = output pixel index, (ph, pw) = stride * (output row, column), boff = byte offset of the
    // input element under the lane's tap.  Moving one output column / row / image forward changes
    // boff by a constant each.
    int bp[BL], ph[BL], pw[BL], br[BL], bs[BL];
    unsigned boff[BL];
    const int Qs = c.Q * c.stride, Ps = c.P * c.stride;
    const bool one_pixel = c.P == 1 && c.Q == 1;
    const unsigned sample_bytes = (unsigned)(c.H * c.W * c.C) * 2u;
    const unsigned colstep = (unsigned)(c.stride * c.C) * 2u;
    const unsigned rowstep = (unsigned)(c.stride * (c.W - c.Q) * c.C) * 2u;                 // extra, on top of Q columns
    const unsigned imgstep = (unsigned)((c.H - c.P * c.stride) * c.W * c.C) * 2u;           // extra, on top of P rows
    const int rows_on = STEP / c.Q, cols_on = STEP % c.Q;
    const unsigned tilestep = (unsigned)STEP * colstep + (unsigned)rows_on * rowstep;
#pragma unroll
    for (int i = 0; i < BL; ++i) {
        const int slot = (i * NW + wave) * 64 + lane;
        const int row = slot / CPB, cs = slot % CPB;
        const int ch = ((((cs >> 1) ^ wg_swz<BCI>(row)) << 1) | (cs & 1));
        const int n = n0 + ch * 8;
        const int tap = n / c.C, ci = n % c.C;
        br[i] = tap / c.S - c.pad;
        bs[i] = tap % c.S - c.pad;
        const int p0 = p_first + row;
        bp[i] = n < Ntot ? p0 : (1 << 30);
        const int q = p0 % c.Q, t = p0 / c.Q;
        const int pr = t % c.P, img = t / c.P;
        ph[i] = pr * c.stride;
        pw[i] = q * c.stride;
        boff[i] = (unsigned)(((img * c.H + ph[i] + br[i]) * c.W + pw[i] + bs[i]) * c.C + ci) * 2u;   // may wrap at the borders
    }

    auto issue_tile = [&](int stage) {
        uint16_t *sa = ring + stage * STAGE_ELEMS, *sb = sa + BKP * BKO;
#pragma unroll
        for (int i = 0; i < AL; ++i) {
            unsigned vo = ap[i] < p_end ? aoff[i] : OOB;
            dma16(grsrc, lds_of(sa + (i * NW + wave) * 512), vo);
        }
#pragma unroll
        for (int i = 0; i < BL; ++i) {
            const bool ok = bp[i] < p_end && (unsigned)(ph[i] + br[i]) < (unsigned)c.H && (unsigned)(pw[i] + bs[i]) < (unsigned)c.W;
            unsigned vo = ok ? boff[i] : OOB;
            dma16(xrsrc, lds_of(sb + (i * NW + wave) * 512), vo);
        }
    };
    // step the per-lane pixel state to the next tile (kept out of issue_tile: its loops would split
    // the block in which the loads' address arithmetic interleaves with the MFMAs)
    auto advance_tile = [&]() {
#pragma unroll
        for (int i = 0; i < AL; ++i) {
            ap[i] += STEP;
            aoff[i] += (unsigned)(STEP * c.K) * 2u;
        }
#pragma unroll
        for (int i = 0; i < BL; ++i) {
            bp[i] += STEP;
            if (one_pixel) {                     // linear layers: every "pixel" is the next sample
                boff[i] += STEP * sample_bytes;
                continue;
            }
            // STEP pixels on = rows_on whole rows and cols_on columns, plus a row where the columns wrap
            pw[i] += cols_on * c.stride;
            ph[i] += rows_on * c.stride;
            boff[i] += tilestep;
            if (pw[i] >= Qs) {
                pw[i] -= Qs;
                boff[i] += rowstep;
                ph[i] += c.stride;
            }
            while (ph[i] >= Ps) {                // at most once from STEP pixels an image
                ph[i] -= Ps;
                boff[i] += imgstep;
            }
        }
    };

    f32x16_t acc[TA][TB];
#pragma unroll
    for (int a = 0; a < TA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.0f;

    // bias gradient = column sums of dy: the waves holding the dy fragments of filter-column tile 0
    // add up their fragment values on the side (lane -> output channel, 8 pixels per step)
    const bool do_bias = bpart != nullptr && tn == 0 && wi == 0;
    float bsum[TA];
#pragma unroll
    for (int a = 0; a < TA; ++a) bsum[a] = 0.0f;
    // Groups of waves: a product takes fewer splits, so a group's sum has more terms than a split's had.  It is put aside and started
    // anew every part_tiles tiles: 320x2880 from 3136 rows, one split, 1.08e-7 off 64 bits (normal operands) where one sum was
    // 2.3e-7 and seven splits of 448 rows 1.24e-7; 16 registers of 128 more and 0.2 % of a mini-batch.
    constexpr bool PARTS = KG > 1 || std::is_same<In, WgradPair>::value;
    constexpr int FA = PARTS ? TA : 1, FB = PARTS ? TB : 1;
    // Tiles of a pair take all of the rows: their parts are added up in double.
    using side_t = typename std::conditional<KG == 1, double, float>::type;
    side_t aside[FA][FB][16], baside[FA];
#pragma unroll
    for (int a = 0; a < FA; ++a) {
        baside[a] = 0;
#pragma unroll
        for (int b = 0; b < FB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) aside[a][b][v] = 0;
    }
    auto fold = [&]() {
        if constexpr (PARTS) {
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                baside[a] += bsum[a];
                bsum[a] = 0.0f;
#pragma unroll
                for (int b = 0; b < TB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        aside[a][b][v] += acc[a][b][v];
                        acc[a][b][v] = 0.0f;
                    }
            }
        }
    };

    auto load_frags = [&](int stage, int k0, bf16x8_t(&fa)[TA], bf16x8_t(&fb)[TB]) {
        const uint16_t *sa = ring + stage * STAGE_ELEMS, *sb = sa + BKP * BKO;
#pragma unroll
        for (int a = 0; a < TA; ++a) fa[a] = tr_frag<BKO>(sa, wk * WT_KO + a * 32, k0, lane);
#pragma unroll
        for (int b = 0; b < TB; ++b) fb[b] = tr_frag<BCI>(sb, wi * WT_CI + b * 32, k0, lane);
    };
    auto add_bias = [&](const bf16x8_t(&fa)[TA]) {
        if (do_bias) {
#pragma unroll
            for (int a = 0; a < TA; ++a) bsum[a] = frag_sum(fa[a], bsum[a]);
        }
    };
    auto mfma_all = [&](const bf16x8_t(&fa)[TA], const bf16x8_t(&fb)[TB]) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[a], fb[b], acc[a][b], 0, 0, 0);
    };

    // Same software pipeline as the gather kernel: STAGES tiles in the ring, fragments double-buffered
    // in registers, the barrier that publishes tile kt+1 between the two MFMA groups of tile kt.
    constexpr int NLOAD = AL + BL;
#pragma unroll
    for (int st = 0; st < STAGES; ++st) {
        issue_tile(st);
        advance_tile();
    }
    WAIT_VMCNT((STAGES - 1) * NLOAD);
    WAIT_LGKMCNT(0);
    __builtin_amdgcn_s_barrier();
    // Of large wave tiles the transposing reads of the next sub-step (two an operand fragment, 12 for 128 x 64) go out between
    // the MFMAs, not in front of them: 512x4608 from 50176 rows 237 -> 232 us, 2304x512 132 -> 128.  (Tiles of few MFMAs, and the
    // gather kernel's plain reads, half as many, are better off in front: 128x1152 from 10125 rows 15.9 us against 16.8.)
    constexpr int NM = TA * TB, RPM = (2 * (TA + TB) + NM - 1) / NM;      // MFMAs of a sub-step, reads behind each
    constexpr bool MIXED = NM >= 8;
    bf16x8_t fa0[TA], fb0[TB], fa1[TA], fb1[TB];
    load_frags(0, 0, fa0, fb0);
    int rd = 0, kt = 0, end = 0;
    do {
        end = !PARTS || end + part_tiles > KT ? KT : end + part_tiles;
        for (; kt < end; ++kt) {
            const int nx = rd + 1 == STAGES ? 0 : rd + 1;
            if constexpr (MIXED) {
                add_bias(fa0);
                __builtin_amdgcn_sched_barrier(0);
                load_frags(rd, 16, fa1, fb1);
                mfma_all(fa0, fb0);
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                add_bias(fa1);
            } else {
                load_frags(rd, 16, fa1, fb1);
                __builtin_amdgcn_sched_barrier(0);
                add_bias(fa0);
                mfma_all(fa0, fb0);
                __builtin_amdgcn_sched_barrier(0);
            }
            WAIT_LGKMCNT(0);
            WAIT_VMCNT((STAGES - 2) * NLOAD);
            __builtin_amdgcn_s_barrier();
            if constexpr (MIXED) {
                __builtin_amdgcn_sched_barrier(0);
                load_frags(nx, 0, fa0, fb0);
                issue_tile(rd);
                mfma_all(fa1, fb1);
#pragma unroll
                for (int i = 0; i < NM; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);        // address arithmetic of the loads
                    __builtin_amdgcn_sched_group_barrier(0x100, RPM, 0);
                }
            } else {
                load_frags(nx, 0, fa0, fb0);
                __builtin_amdgcn_sched_barrier(0);
                issue_tile(rd);
                add_bias(fa1);
                mfma_all(fa1, fb1);
            }
            __builtin_amdgcn_sched_barrier(0);
            advance_tile();
            rd = nx;
        }
        fold();
    } while (PARTS && end < KT);
    WAIT_VMCNT(0);
    if constexpr (PARTS && KG == 1) {
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[a][b][v] = (float)aside[a][b][v];
    }

    if constexpr (KG > 1) {
        // Every group parks its sums in LDS ([row][column] floats over its own ring and the next ones), then all threads
        // add the KG copies of a float4 in the groups' order and write it.
        constexpr int PITCH = BCI + 4;
        static_assert((size_t)KG * (BKO * PITCH + BKO) * 4 <= kWgradLds<BKO, BCI, STAGES, KG>, "the sums fit");
        float *sums = reinterpret_cast<float *>(smem), *sbias = sums + KG * BKO * PITCH;
        const int col = lane & 31, half = lane >> 5;
        __syncthreads();                                      // every wave has left its ring
#pragma unroll
        for (int a = 0; a < TA; ++a)
#pragma unroll
            for (int b = 0; b < TB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    sums[(kg * BKO + wk * WT_KO + a * 32 + 8 * (v >> 2) + 4 * half + (v & 3)) * PITCH + wi * WT_CI + b * 32 + col] = aside[a][b][v];
        if (do_bias) {
#pragma unroll
            for (int a = 0; a < TA; ++a) {
                const float t = baside[a] + __shfl_xor(baside[a], 32, 64);
                if (half == 0) sbias[kg * BKO + wk * WT_KO + a * 32 + col] = t;
            }
        }
        __syncthreads();
        float *dst = part + (size_t)by * split_stride;
        constexpr int NT = NW * KG * 64, F4 = BCI / 4, IT = BKO * F4 / NT;
        static_assert(IT >= 1 && BKO * F4 % NT == 0, "whole rounds of the block");
        float4 o[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int at = it * NT + tid, ko = ko0 + at / F4, n = n0 + at % F4 * 4;
            o[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (add_to_dst && ko < c.K && n < Ntot) o[it] = *reinterpret_cast<const float4 *>(dst + (size_t)ko * Ntot + n);
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int at = it * NT + tid, row = at / F4, c4 = at % F4 * 4, ko = ko0 + row, n = n0 + c4;
            float4 t = *reinterpret_cast<const float4 *>(sums + row * PITCH + c4);
#pragma unroll
            for (int g = 1; g < KG; ++g) {
                const float4 v = *reinterpret_cast<const float4 *>(sums + (g * BKO + row) * PITCH + c4);
                t.x += v.x; t.y += v.y; t.z += v.z; t.w += v.w;
            }
            if (ko < c.K && n < Ntot)
                *reinterpret_cast<float4 *>(dst + (size_t)ko * Ntot + n) = make_float4(t.x + o[it].x, t.y + o[it].y, t.z + o[it].z, t.w + o[it].w);
        }
        if (bpart != nullptr && tn == 0 && tid < BKO && ko0 + tid < c.K) {
            float *bdst = bpart + (size_t)by * split_stride + ko0 + tid, t = sbias[tid];
#pragma unroll
            for (int g = 1; g < KG; ++g) t += sbias[g * BKO + tid];
            *bdst = add_to_dst ? *bdst + t : t;
        }
        return;
    }
    // partial[split][ko][n]
    float *dst = part + (size_t)by * split_stride;
    const int col = lane & 31, half = lane >> 5;
    if (do_bias) {
        float *bdst = bpart + (size_t)by * split_stride;
#pragma unroll
        for (int a = 0; a < TA; ++a) {
            float t;
            if constexpr (PARTS) t = (float)(baside[a] + __shfl_xor(baside[a], 32, 64));
            else t = bsum[a] + __shfl_xor(bsum[a], 32, 64);
            const int ko = ko0 + wk * WT_KO + a * 32 + col;
            if (half == 0 && ko < c.K) bdst[ko] = add_to_dst ? bdst[ko] + t : t;
        }
    }
    // The accumulators leave through LDS: each wave parks one 32-row slice of its sub-tile in a region
    // of its own ([32][WT_CI] floats; the ring is free by now) and reads it back as float4 so that 16
    // lanes cover 256 contiguous bytes of one dw row.  Straight from the registers a row segment would
    // be 32 separate 4-byte read-modify-writes.
    __syncthreads();                                          // every wave has left the ring
    float *stg = reinterpret_cast<float *>(smem) + wave * (32 * WT_CI);
    constexpr int F4R = WT_CI / 4;                            // float4 per staged row
    constexpr int RPI = 64 / F4R;                             // rows one wave-wide access covers
#pragma unroll
    for (int a = 0; a < TA; ++a) {
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) stg[(8 * (v >> 2) + 4 * half + (v & 3)) * WT_CI + b * 32 + col] = acc[a][b][v];
        WAIT_LGKMCNT(0);
        __builtin_amdgcn_wave_barrier();
        // all reads of the slice first, then all writes: one round trip to memory per slice, not one per row group
        constexpr int IT = 32 / RPI;
        float4 t[IT], o[IT];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int row = it * RPI + lane / F4R, c4 = (lane % F4R) * 4;
            const int ko = ko0 + wk * WT_KO + a * 32 + row, n = n0 + wi * WT_CI + c4;
            t[it] = *reinterpret_cast<const float4 *>(stg + row * WT_CI + c4);
            o[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (add_to_dst && ko < c.K && n < Ntot) o[it] = *reinterpret_cast<const float4 *>(dst + (size_t)ko * Ntot + n);
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int row = it * RPI + lane / F4R, c4 = (lane % F4R) * 4;
            const int ko = ko0 + wk * WT_KO + a * 32 + row, n = n0 + wi * WT_CI + c4;
            if (ko < c.K && n < Ntot)
                *reinterpret_cast<float4 *>(dst + (size_t)ko * Ntot + n) =
                    make_float4(t[it].x + o[it].x, t[it].y + o[it].y, t[it].z + o[it].z, t[it].w + o[it].w);
        }
        WAIT_LGKMCNT(0);
        __builtin_amdgcn_wave_barrier();
    }
}

// dw[i] += sum_k part[k][i].  A block owns 64 float4 columns; its 4 split-lanes walk the partials
// with stride 4 and are combined through LDS in lane order (the result does not depend on timing), in double: the layers of
// most rows have up to 256 partials (64x64 from 100352 rows, normal operands, 8.9e-8 off 64 bits; in float 1.7e-7).
// Entries past total_w are the bias partials and go to db.  total_w and total are multiples of 4
// (channel counts are multiples of 8).
struct SplitkArgs {                              // tests/launch_recorder.c reads it
    const float *part;
    float *dw, *db;
    size_t total_w, total;
    int splits, blocks;
};
typedef Group<SplitkArgs> SplitkGroup;
template <class In> __global__ void k_splitk_reduce(In in)
{
    int id = blockIdx.x;
    const SplitkArgs &job = job_of(in, id);
    const float *__restrict__ part = job.part;
    float *dw = job.dw, *db = job.db;
    const size_t total_w = job.total_w, total = job.total;
    const int splits = job.splits;
    __shared__ double red[4][4][64];
    const int col = threadIdx.x & 63, sl = threadIdx.x >> 6;
    const size_t i = ((size_t)id * 64 + col) * 4;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < total) {
#pragma unroll 4
        for (int k = sl; k < splits; k += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(part + (size_t)k * total + i);
            acc[0] += v.x; acc[1] += v.y; acc[2] += v.z; acc[3] += v.w;
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[sl][q][col] = acc[q];
    __syncthreads();
    if (sl == 0 && i < total) {
        float *out = i < total_w ? dw + i : db + (i - total_w);
        float4 d = *reinterpret_cast<float4 *>(out);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = ((red[0][q][col] + red[1][q][col]) + red[2][q][col]) + red[3][q][col];
        d.x += (float)acc[0]; d.y += (float)acc[1]; d.z += (float)acc[2]; d.w += (float)acc[3];
        *reinterpret_cast<float4 *>(out) = d;
    }
}

struct WgradPlan {
    int bko, bci, kg, tiles_ko, tiles_n, splits, pix_per_split;
    int part_tiles;          // wave groups: tiles of 32 pixels that a group adds up before it puts the sum aside
    bool pair;
};

// beside: kernels of other streams run beside the launch.  Only the tile may depend on it, not the splits: every sum stays the
// same, in the same order.
// pair: of two such products that share dy, if the plan says that they can be one (`pair`).
WgradPlan wgrad_plan(const ConvShape &c, bool beside, bool pair = false)
{
    WgradPlan p;
    p.pair = false;
    const int Ntot = c.R * c.S * c.C;
    const long long npix = (long long)c.N * c.P * c.Q;
    auto tiles_of = [&](int bko, int bci) { return (long long)((c.K + bko - 1) / bko) * ((Ntot + bci - 1) / bci); };
    // A product of up to 14 GMAC is bound by the chain of steps of one block, and by what it fetches per step, not by the
    // matrix cores: 64-column tiles whose steps two groups of four waves take in turn.  64 x 64 up to 3 GMAC and for narrow
    // layers, 128 x 64 above (with the reduction of the partial sums, us, KG = 1 before -> now: 256x1024 from 784 rows 15.0 ->
    // 7.9, 256x2304 16.9 -> 8.8, from 6272 rows 30.5 -> 26.2; 2048x512 from 1568 22.4 -> 12.2; 64x576 from 40500 22.9 -> 17.4,
    // from 320000 63 -> 58; 512x4608 from 3136 38.1 -> 35; 4096x1024 from 3200 56.6 -> 45.4; 512x2304 from 6272 37.6 -> 34.4).
    // Larger products (256x2304 from 25088 rows: 53.7 against 54.1, from 100352 148 against 173), and those of more tiles
    // than the chip holds at once (4096x4096 from 1024 rows: 53 against 74; 25088x4096 from 128: 171 against 210), where the
    // operands and the sums themselves are what moves, take wider tiles.
    const double macs = (double)npix * c.K * Ntot;
    const bool narrow = c.K <= 64 || Ntot <= 64;
    p.kg = 2;
    p.bci = 64;
    p.part_tiles = 0;
    if (tiles_of(64, 64) <= 1024 && (c.K <= 64 || macs < 3e9)) {
        p.bko = 64;
    } else if (tiles_of(128, 64) <= 512 && (narrow || macs < 14e9)) {
        p.bko = 128;
    } else {
        p.kg = 1;
        p.bci = 128;
        p.bko = c.K > 128 && macs >= 8e9 && npix > 128 ? 256 : 128;
        // One block of eight waves and 256 x 256 per unit fetches two thirds of what two of 256 x 128 do.  Where its tiles are
        // whole and the pixels make a block per unit out of them (with the reduction: 512x4608 from 50176 rows 254 -> 231 us,
        // 512x2304 139 -> 122, from 12544 rows 83 -> 75; 25088x4096 from 1024 rows, 1568 tiles, 316 -> 331).  Beside other kernels a
        // short launch keeps the smaller blocks, which share a unit with theirs (mini-batches of three 3x3 512->512 layers, three
        // streams, us, 256 x 128 against 256 x 256: 12544 rows 3560 / 3715, 15680 4350 / 4400, 18816 5215 / 5170, 21952 5950 / 5890,
        // 25088 6690 / 6630, 25600 6425 / 6200, 31360 7615 / 7170, 50176 12250 / 11650).
        const long long whole = tiles_of(256, 256);
        if (p.bko == 256 && c.K % 256 == 0 && Ntot % 256 == 0 && whole <= 128 && whole * ((npix + 1023) / 1024) >= 224 &&
            !(beside && npix < 25000))
            p.bci = 256;
    }
    // Both products of a pair as tiles of 256 x 128, eight waves each, where that is about a block per unit: half the operand
    // bytes of 128 x 64 (4096x1024 from 3200 rows, twice: 72 us against 85; from 1024 34 / 41; rings of five or six stages no faster).  Other
    // pairs are two products that share launches, as any do (2048x512 from 3200 rows 31 us, one by one 42).  A block has all of the rows: its sums
    // are put aside as often as those of the smaller tiles, and added up in double (1024 hidden units, sums of one sign, off 64 bits, weights and
    // bias: 3200 rows 3.9e-8 and 2.2e-8, one by one 4.9e-8 and 3.4e-8, added up in float 6.2e-8 and 4.4e-8, at 67 us; 12800 rows 2.9e-8 and
    // 2.2e-8, one by one 1.5e-7 and 3.5e-8, in float 1.1e-7 and 8.1e-8).
    if (pair && c.R * c.S == 1 && c.K % 256 == 0 && c.C % 128 == 0 && npix >= 1024 && 2 * tiles_of(256, 128) >= 192 && 2 * tiles_of(256, 128) <= 256) {
        p.pair = true;
        p.kg = 1;
        p.bko = 256;
        p.bci = 128;
        p.tiles_ko = c.K / 256;
        p.tiles_n = c.C / 128;
        p.splits = 1;
        p.pix_per_split = (int)((npix + 31) / 32 * 32);
        const int halves = (int)((npix + 63) / 64), parts = (halves + 11) / 12;
        p.part_tiles = (halves + parts - 1) / parts;
        return p;
    }
    p.tiles_ko = (c.K + p.bko - 1) / p.bko;
    p.tiles_n = (Ntot + p.bci - 1) / p.bci;
    const long long tiles = (long long)p.tiles_ko * p.tiles_n;
    if (p.kg == 2) {
        // us, fitted to 60 shapes of 10 to 100 000 tile steps: a step of 64 pixels of a unit's only block and of one of several
        // that share it; a second launch and the partial sums, written and read
        double best = 1e30;
        long long want = 1;
        const double alone = p.bko == 64 ? 0.36 : 0.45, shared = p.bko == 64 ? 0.30 : 0.36;
        for (long long sp = 1; sp <= 256; ++sp) {
            if (sp > 1 && (npix < 64 * sp || tiles * sp > 2048 || (double)sp * c.K * (Ntot + 1) * 4 > 32e6)) break;
            const long long per_unit = (tiles * sp + 255) / 256;
            const double cost = (double)per_unit * (double)((npix + 64 * sp - 1) / (64 * sp)) * (per_unit == 1 ? alone : shared) +
                                (sp > 1 ? 3.5 + (double)sp * c.K * Ntot * 2e-6 : 0.0);
            if (cost < best) {
                best = cost;
                want = sp;
            }
        }
        // Where larger products of a map take units of 128 pixels, these are no less exact below that line: parts of 4 tiles, and at least
        // four splits of 2048 pixels and more, of which wide layers would take two or three (sums of one sign, off 64 bits, units, as any other
        // product, so: 64->64 at 16x16, 2 samples 4.3e-8, 6.0e-8, 4.0e-8; 256->256, 8 3.9e-8, 5.3e-8, 2.9e-8, and 26.6 us, 15.3, 18.6).
        const bool units = wgrad3x3_units(c);
        if (units && tiles >= 128 && npix >= 2048 && want < 4) want = 4;
        const long long pps = ((npix + want - 1) / want + 63) / 64 * 64;
        p.pix_per_split = (int)pps;
        p.splits = npix > 0 ? (int)((npix + pps - 1) / pps) : 1;
        // equal parts of at most 12 tiles, 384 pixels
        const int most = units ? 4 : 12, tiles_g = (int)(pps / 64), parts = (tiles_g + most - 1) / most;
        p.part_tiles = parts ? (tiles_g + parts - 1) / parts : 1;
        return p;
    }
    // Split count: the chip holds 512 blocks at once (256 CUs x 2), and a launch whose block count is
    // just above a multiple of that leaves most CUs idle during the last blocks.  Take the split count
    // that minimises (time relative to perfectly filled rounds) + (relative cost of the partials: every
    // split writes and re-reads a full fp32 copy of dw, about 500/npix of the MFMA time each); at least
    // 512 pixels per split.
    long long max_by_work = (npix + 511) / 512;
    if (max_by_work > 256) max_by_work = 256;
    if (max_by_work < 1) max_by_work = 1;
    const long long slots = p.bci == 256 ? 256 : 512;      // half as many tiles, so the same split count
    long long want = 1;
    double best = 1e30;
    for (long long sp = 1; sp <= max_by_work; ++sp) {
        const long long blocks = tiles * sp, rounds = (blocks + slots - 1) / slots;
        const double cost = (double)(rounds * slots) / (double)blocks + 500.0 * (double)sp / (double)npix;
        if (cost < best) {
            best = cost;
            want = sp;
        }
    }
    long long pps = (npix + want - 1) / want;
    pps = (pps + 31) / 32 * 32;
    if (pps < 32) pps = 32;
    p.pix_per_split = (int)pps;
    p.splits = (int)((npix + pps - 1) / pps);
    if (p.splits < 1) p.splits = 1;
    return p;
}

}  // namespace

bool conv_gather_mfma_supported(const GatherConv &g)
{
    // byte offsets into the operands are 32-bit (buffer addressing)
    return g.Ci % 8 == 0 && g.Co % 8 == 0 && g.Ci >= 8 && g.s_in >= 1 && g.s_out >= 1 &&
           (long long)g.N * g.Hi * g.Wi * g.Ci * 2 < (1ll << 31) && (long long)g.Co * g.R * g.S * g.Ci * 2 < (1ll << 31) &&
           (long long)g.N * g.Ho * g.Wo < (1ll << 31) - 512;
}

size_t conv_gather_mfma_workspace(const GatherConv &g)
{
    if (conv3x3_halo_supported(g) || conv3x3_c8_supported(g)) return 0;
    GatherPlan p = gather_plan(g);
    return p.splits > 1 ? (size_t)p.splits * g.N * g.Ho * g.Wo * g.Co * sizeof(float) : 0;
}

int conv_gather_mfma_stat_chunks(const GatherConv &g)
{
    if (!conv_gather_mfma_supported(g) || conv3x3_halo_supported(g) || conv3x3_c8_supported(g)) return 0;
    const GatherPlan p = gather_plan(g);
    if (p.splits != 1) return 0;
    return (int)(p.classes * ((p.class_pix + p.bp - 1) / p.bp));
}

hipError_t conv_gather_mfma(const void *in, const void *wt, const float *bias, void *out, int relu,
                            GradEpi epi, const GatherConv &g, void *workspace, unsigned *tickets, hipStream_t s, float *stat_part,
                            const void *bn_x, const float *bn_stats)
{
    if (!conv_gather_mfma_supported(g) || (g.wt_panels && (g.R * g.S != 1 || g.s_in != 1 || g.Ci % 32))) return hipErrorInvalidValue;
    if (stat_part && conv_gather_mfma_stat_chunks(g) == 0) return hipErrorInvalidValue;
    if (bn_x && (!stat_part || !bn_stats || !(epi.gate || epi.accum))) return hipErrorInvalidValue;   // gradient epilogue only
    if ((long long)g.N * g.Ho * g.Wo == 0) return hipSuccess;
    if (epi.accum_from && (!epi.accum || conv3x3_halo_supported(g))) return hipErrorInvalidValue;   // gather kernel only
    if (conv3x3_halo_supported(g)) return conv3x3_halo_mfma(in, wt, bias, out, relu, epi, g, s);
    if (!epi.gate && !epi.accum && conv3x3_c8_supported(g)) return conv3x3_c8_mfma(in, wt, bias, out, relu, g, s);
    return launch_plan(in, wt, bias, out, relu, epi, g, gather_plan(g), workspace, tickets, s, false, stat_part, bn_x, bn_stats);
}

size_t conv_gather_mfma_raw_workspace(const GatherConv &g)
{
    return (size_t)gather_plan(g).splits * g.N * g.Ho * g.Wo * g.Co * sizeof(float);
}

hipError_t conv_gather_mfma_raw(const void *in, const void *wt, const GatherConv &g, float *part, int *splits,
                                hipStream_t s)
{
    if (!conv_gather_mfma_supported(g) || !part || !splits || g.Co % 4 != 0) return hipErrorInvalidValue;
    const GatherPlan p = gather_plan(g);
    *splits = p.splits;
    if ((long long)g.N * g.Ho * g.Wo == 0) return hipSuccess;
    const GradEpi none{nullptr, 0};
    return launch_plan(in, wt, nullptr, nullptr, 0, none, g, p, part, nullptr, s, true);
}

bool conv_wgrad_mfma_supported(const ConvShape &c)
{
    // 32-bit byte offsets into both operands (buffer addressing)
    return c.C % 8 == 0 && c.K % 8 == 0 && c.C >= 8 && c.K >= 8 &&
           (long long)c.N * c.H * c.W * c.C * 2 < (1ll << 31) && (long long)c.N * c.P * c.Q * c.K * 2 < (1ll << 31);
}

size_t conv_wgrad_mfma_workspace(const ConvShape &c)
{
    if (wgrad3x3_halo_supported(c)) return wgrad3x3_halo_workspace(c);
    if (wgrad3x3_c8_supported(c)) return wgrad3x3_c8_workspace(c);
    WgradPlan p = wgrad_plan(c, false);
    return p.splits == 1 ? 0 : (size_t)p.splits * ((size_t)c.K * c.R * c.S * c.C + c.K) * sizeof(float);
}

// products of one tile shape that wait for their launch, and the partial sums that wait for theirs
namespace {
struct WgradBatch {
    WgradGroup g;
    SplitkGroup r;
    int bko = 0, bci = 0, kg = 0;
};

hipError_t launch_batch(WgradBatch &b, hipStream_t s)
{
    if (b.g.n == 0) return hipSuccess;
    unsigned blocks = 0, sums = 0;
    for (int i = 0; i < b.g.n; ++i) blocks += (unsigned)b.g.a[i].blocks;
    for (int i = 0; i < b.r.n; ++i) sums += (unsigned)b.r.a[i].blocks;
#define WG_LAUNCH(BKO_, BCI_, WKO_, WCI_, KG_, IN_, in_)                                                   \
    do {                                                                                                   \
        constexpr size_t smem = kWgradLds<BKO_, BCI_, 3, KG_>;                                             \
        auto kfn = k_wgrad_mfma<BKO_, BCI_, WKO_, WCI_, 3, KG_, IN_>;                                      \
        static bool attr_set = false;                                                                      \
        if (!attr_set && smem > 64 * 1024) {                                                               \
            hipError_t e = hipFuncSetAttribute((const void *)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem); \
            if (e != hipSuccess) return e;                                                                 \
            attr_set = true;                                                                               \
        }                                                                                                  \
        hipLaunchKernelGGL(kfn, dim3(blocks), dim3(WKO_ * WCI_ * KG_ * 64), smem, s, in_);                 \
    } while (0)
    const WgradArgs &one = b.g.a[0];
    const WgradPair two{one};
    if (b.g.n > 1 && b.bko == 64)                          // products with wave groups
        WG_LAUNCH(64, 64, 2, 2, 2, WgradGroup, b.g);
    else if (b.g.n > 1)
        WG_LAUNCH(128, 64, 2, 2, 2, WgradGroup, b.g);
    else if (one.x2)                                       // the tile that is only taken for pairs
        WG_LAUNCH(256, 128, 4, 2, 1, WgradPair, two);
    else if (b.kg == 2 && b.bko == 64)
        WG_LAUNCH(64, 64, 2, 2, 2, WgradArgs, one);
    else if (b.kg == 2)
        WG_LAUNCH(128, 64, 2, 2, 2, WgradArgs, one);
    else if (b.bci == 256)
        WG_LAUNCH(256, 256, 2, 4, 1, WgradArgs, one);
    else if (b.bko == 256)
        WG_LAUNCH(256, 128, 2, 2, 1, WgradArgs, one);
    else
        WG_LAUNCH(128, 128, 2, 2, 1, WgradArgs, one);
#undef WG_LAUNCH
    if (b.r.n > 1) hipLaunchKernelGGL(k_splitk_reduce<SplitkGroup>, dim3(sums), dim3(256), 0, s, b.r);
    else if (b.r.n) hipLaunchKernelGGL(k_splitk_reduce<SplitkArgs>, dim3(sums), dim3(256), 0, s, b.r.a[0]);
    b.g.n = b.r.n = 0;
    return hipGetLastError();
}
}  // namespace

bool conv_wgrad_mfma_groups(const ConvShape &c)
{
    if (!conv_wgrad_mfma_supported(c) || wgrad3x3_halo_supported(c) || wgrad3x3_c8_supported(c)) return false;
    const WgradPlan p = wgrad_plan(c, false);
    return p.kg == 2 && (long long)p.tiles_ko * p.tiles_n * p.splits < 256;
}

hipError_t conv_wgrad_mfma_jobs(const WgradJob *jobs, int n, void *workspace, size_t workspace_bytes, hipStream_t s, bool beside)
{
    WgradBatch batch[2] = {};                               // of 64 and of 128 output channels a tile
    size_t used = 0;
    auto launch_all = [&]() {
        for (WgradBatch &b : batch) {
            const hipError_t e = launch_batch(b, s);
            if (e != hipSuccess) return e;
        }
        used = 0;
        return hipSuccess;
    };
    auto add = [&](const WgradJob &j, bool pair) {
        ConvShape c = j.c;
        if (!conv_wgrad_mfma_supported(c)) return hipErrorInvalidValue;
        if ((long long)c.N * c.P * c.Q == 0) return hipSuccess;
        // A 1x1 filter at stride 1 contracts over a plain list of rows: as images of one pixel a tile step is one constant
        // add.  (The step over image rows costs a lane up to 32 trips where a row is one pixel, as in a sequence: the LSTM's
        // weight gradients, 3200 rows, 4096 x 1024, 99 -> 38 us.)
        if (c.R == 1 && c.S == 1 && c.stride == 1 && c.pad == 0) {
            c.N *= c.P * c.Q;
            c.H = c.W = c.P = c.Q = 1;
        }
        hipError_t e = hipSuccess;
        if (wgrad3x3_halo_supported(c) || wgrad3x3_c8_supported(c)) {
            if ((e = launch_all()) != hipSuccess) return e;
            e = wgrad3x3_halo_supported(c) ? wgrad3x3_halo_mfma(j.x, j.dy, j.dw, j.db, workspace, c, s)
                                           : wgrad3x3_c8_mfma(j.x, j.dy, j.dw, j.db, workspace, c, s);
            return e;
        }
        const WgradPlan p = wgrad_plan(c, beside, pair);
        const int direct = p.splits == 1;
        const size_t total_w = (size_t)c.K * c.R * c.S * c.C, total = total_w + (j.db ? c.K : 0);
        const size_t want = direct ? 0 : ((size_t)p.splits * total * sizeof(float) + 255) / 256 * 256;
        WgradBatch &b = batch[p.bko != 64];
        // a product without wave groups fills the chip by itself
        if ((p.kg == 1 || used + want > workspace_bytes || b.g.n == WG_GROUP) && (e = launch_all()) != hipSuccess) return e;
        float *part = direct ? j.dw : (float *)((char *)workspace + used);
        used += want;
        b.bko = p.bko;
        b.bci = p.bci;
        b.kg = p.kg;
        const int tiles = p.tiles_ko * p.tiles_n;
        b.g.a[b.g.n++] = {(const bf16_t *)j.x, pair ? (const bf16_t *)j.x2 : nullptr, (const bf16_t *)j.dy, part, j.dw2,
                          !j.db ? nullptr : (direct ? j.db : part + total_w), total, c, tiles, p.tiles_n, p.splits,
                          tiles * p.splits * (pair ? 2 : 1), p.pix_per_split, p.part_tiles, direct,
                          (unsigned)((size_t)c.N * c.H * c.W * c.C * 2), (unsigned)((size_t)c.N * c.P * c.Q * c.K * 2)};
        if (!direct) b.r.a[b.r.n++] = {part, j.dw, j.db, total_w, total, p.splits, (int)((total / 4 + 63) / 64)};
        return p.kg == 1 ? launch_all() : hipSuccess;
    };
    for (int k = 0; k < n; ++k) {
        const WgradJob &j = jobs[k];
        const bool pair = j.x2 && wgrad_plan(j.c, beside, true).pair;
        hipError_t e = add(j, pair);
        if (e == hipSuccess && j.x2 && !pair) e = add({j.x2, j.dy, j.dw2, nullptr, j.c}, false);
        if (e != hipSuccess) return e;
    }
    return launch_all();
}

hipError_t conv_wgrad_mfma(const void *x, const void *dy, float *dw, float *db, void *workspace,
                           const ConvShape &c, hipStream_t s, bool beside)
{
    const WgradJob job{x, dy, dw, db, c};
    return conv_wgrad_mfma_jobs(&job, 1, workspace, ~(size_t)0, s, beside);      // one product fits: not asked, a plan is a microsecond of the host
}

}  // namespace bapipe

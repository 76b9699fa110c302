// Host-callable launchers of the stage's HIP kernels.  Internal to the library: the public
// interface is include/bapipe_stage.h.  All tensors are NHWC in HBM; `dtype` selects the
// storage type (0 = float, 1 = bf16) of activations, activation gradients and working
// weights; master weights, weight gradients, statistics and losses are always float.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace bapipe {

enum { DT_F32 = 0, DT_BF16 = 1 };
inline size_t dt_size(int dt) { return dt == DT_F32 ? 4 : 2; }

// out[n,oh,ow,ko] = sum_{r,s,ki} in[n,ih,iw,ki] * wt[ko][r][s][ki]  (+ bias[ko]),
// ih = (oh*s_out + r - pad_h) / s_in when divisible and inside [0,Hi), same for iw.
//   forward conv : in = x,  s_out = stride, s_in = 1,      pad = pad,       wt = w [K][R][S][C]
//   dgrad        : in = dy, s_out = 1,      s_in = stride, pad = R-1-pad,   wt = flipped,
//                  channel-transposed copy [C][R][S][K]
// GatherGeom is what k_gather_mfma reads and is handed; the rest is for the plan and the launcher.
struct GatherGeom {
    int N, Hi, Wi, Ci, Ho, Wo, Co, R, S, s_out, s_in, pad_h, pad_w;
    // Kernels of other streams run beside this launch.  Alone on the chip a launch wants every compute unit busy; beside others,
    // units it leaves idle are not lost, and fewer, larger blocks (less operand traffic per FLOP) are the better neighbour.
    // Only the pixel tile may depend on it: every output element is still one sum over K in the same order.
    int beside = 0;
    // The output is the input of a batch-norm, or the gradient of one's output: kernels that leave it the sums it needs are preferred.
    int by_norm = 0;
};
struct GatherConv : GatherGeom {
    // wt is kept in panels of 32 columns, [Ci / 32][Co][32] (1x1 filters, Ci a multiple of 32): neighbouring rows of a K-tile are one
    // piece of memory.  No tile and no share of K depends on it; who adds the shares and the depth of the operand ring do.
    int wt_panels = 0;
};

// Forward-convolution geometry (x: N,H,W,C ; y: N,P,Q,K ; filter R x S).
struct ConvShape {
    int N, H, W, C, P, Q, K, R, S, stride, pad;
};

// Epilogue options of kernels that write an activation gradient (see grad_out()).
struct GradEpi {
    const void *gate;  // forward values deciding the producer's fused-ReLU mask, or NULL
    int accum;         // add to what is already stored
    // With accum: the stored value is read from here (same layout as the destination) instead of from the
    // destination itself - the other contribution to a gradient with two sources, taken where it already lies
    // instead of being copied first.  Honoured by the MFMA gather convolution; NULL everywhere else.
    const void *accum_from = nullptr;
};

// ---- direct (CUDA-core style) convolution: fp32 stages and shapes the MFMA path skips
hipError_t conv_gather_direct(int dt, const void *in, const void *wt, const float *bias, void *out,
                              int relu, GradEpi epi, const GatherConv &g, hipStream_t s);
size_t conv_wgrad_direct_workspace(const ConvShape &c);
// dw += dy^T x over all pixels; db (may be null) += column sums of dy, with a workspace that also holds colsum_workspace
hipError_t conv_wgrad_direct(int dt, const void *x, const void *dy, float *dw, float *db, void *workspace,
                             const ConvShape &c, hipStream_t s);

// ---- bf16 MFMA implicit-GEMM convolution (kernels_conv_mfma.hip)
bool conv_gather_mfma_supported(const GatherConv &g);
size_t conv_gather_mfma_workspace(const GatherConv &g);      // split-K partials (0 if K is not split)
// bn_x / bn_stats (optional, gradient epilogue, with stat_part): the output is the gradient of a batch-norm's
// output; stat_part then receives the per-tile sums of dy and dy*xhat (xhat from bn_x and the saved mean, 1/std)
// stat_part (optional): the kernel also leaves, per pixel tile, the per-channel sum and sum of squares of
// the values it stores - [2][chunks][Co] floats with chunks = conv_gather_mfma_stat_chunks(g) - which is what
// bn_fwd would otherwise compute in a pass of its own; only where that function returns a non-zero count
int conv_gather_mfma_stat_chunks(const GatherConv &g);
// tickets: kGatherTickets words that are zero, and zero again behind every launch; launches that may run at once need words of their own
constexpr int kGatherTickets = 128;
hipError_t conv_gather_mfma(const void *in, const void *wt, const float *bias, void *out, int relu,
                            GradEpi epi, const GatherConv &g, void *workspace, unsigned *tickets, hipStream_t s,
                            float *stat_part = nullptr, const void *bn_x = nullptr, const float *bn_stats = nullptr);
// 3x3 / stride 1 / pad 1 with the input halo of a 16x16 output patch resident in LDS
// (kernels_conv_halo.hip); conv_gather_mfma routes to it when it applies
bool conv3x3_halo_supported(const GatherConv &g);
hipError_t conv3x3_halo_mfma(const void *in, const void *wt, const float *bias, void *out, int relu,
                             GradEpi epi, const GatherConv &g, hipStream_t s);
// forward of a 3x3 / stride 1 / pad 1 conv whose input has 8 channels in memory (the padded RGB stage input)
bool conv3x3_c8_supported(const GatherConv &g);
hipError_t conv3x3_c8_mfma(const void *in, const void *wt, const float *bias, void *out, int relu,
                           const GatherConv &g, hipStream_t s);
// same convolution with a 2x2 stride-2 max-pool fused into the epilogue: writes the pooled output
// [N][H/2][W/2][Co] and the arg-max indices (one byte each, same layout); the conv output is not stored
bool conv3x3_halo_pool_supported(const GatherConv &g);
hipError_t conv3x3_halo_pool_mfma(const void *in, const void *wt, const float *bias, int relu, void *pool_out,
                                  uint8_t *pool_idx, const GatherConv &g, hipStream_t s);
// The same implicit GEMM leaving raw fp32 sums: part[split][pixel][co], *splits partial results the
// caller adds up (no bias, no epilogue, no rounding).  Used for the recurrent products of the LSTM.
size_t conv_gather_mfma_raw_workspace(const GatherConv &g);
hipError_t conv_gather_mfma_raw(const void *in, const void *wt, const GatherConv &g, float *part, int *splits,
                                hipStream_t s);
bool wgrad3x3_units(const ConvShape &c);          // whether the map comes apart into units of 8x16 pixels, as both of these need it
bool wgrad3x3_halo_supported(const ConvShape &c);
size_t wgrad3x3_halo_workspace(const ConvShape &c);
hipError_t wgrad3x3_halo_mfma(const void *x, const void *dy, float *dw, float *db, void *workspace,
                              const ConvShape &c, hipStream_t s);
// weight gradient of a 3x3 / stride 1 / pad 1 conv whose input has 8 channels in memory (the padded RGB stage input)
bool wgrad3x3_c8_supported(const ConvShape &c);
size_t wgrad3x3_c8_workspace(const ConvShape &c);
hipError_t wgrad3x3_c8_mfma(const void *x, const void *dy, float *dw, float *db, void *workspace, const ConvShape &c,
                            hipStream_t s);
bool conv_wgrad_mfma_supported(const ConvShape &c);
size_t conv_wgrad_mfma_workspace(const ConvShape &c);
// dw += dy^T x over all pixels; db (may be null) += column sums of dy
// beside: kernels of other streams run beside the launch (as in GatherConv; the sums do not depend on it)
hipError_t conv_wgrad_mfma(const void *x, const void *dy, float *dw, float *db, void *workspace,
                           const ConvShape &c, hipStream_t s, bool beside = false);

// Several of them, in as few launches as their tiles and the workspace allow: the same sums as one by one.  Each by itself must fit
// the workspace.
// x2, dw2: another product of the same shape with the same dy, dw2 += dy^T x2; where both are tiles of one launch, their sums are those of
// that launch
struct WgradJob {
    const void *x, *dy;
    float *dw, *db;
    ConvShape c;
    const void *x2 = nullptr;
    float *dw2 = nullptr;
};
// the same for small float layers with a bias, for which the first function says yes
bool conv_wgrad_direct_groups(const ConvShape &c);
hipError_t conv_wgrad_direct_jobs(const WgradJob *jobs, int n, void *workspace, size_t workspace_bytes, hipStream_t s);
bool conv_wgrad_mfma_groups(const ConvShape &c);      // whether it fills so little of the chip that it should wait for others
hipError_t conv_wgrad_mfma_jobs(const WgradJob *jobs, int n, void *workspace, size_t workspace_bytes, hipStream_t s, bool beside);

// ---- column sums over a [rows][C] matrix: out[c] += sum_r a[r][c]  (bias gradient)
size_t colsum_workspace(int rows, int C);
hipError_t colsum_accumulate(int dt, const void *a, int rows, int C, float *out, void *workspace,
                             hipStream_t s);

// ---- element-wise / pooling / normalisation
hipError_t relu_fwd(int dt, const void *x, void *y, size_t n, hipStream_t s);
hipError_t relu_bwd(int dt, const void *y, const void *dy, void *dx, GradEpi epi, size_t n, hipStream_t s);
// y_nchw: a second destination of y, in NCHW; *stored says whether it was taken
hipError_t maxpool2x2_fwd(int dt, const void *x, void *y, uint8_t *idx, int N, int H, int W, int C,
                          hipStream_t s, void *y_nchw = nullptr, bool *stored = nullptr);
// gate (if any) is indexed like dy (the pooled tensor), not like dx.  nchw: dy is in that layout, where the other function says yes
hipError_t maxpool2x2_bwd(int dt, const void *dy, const uint8_t *idx, void *dx, GradEpi epi_pooled_gate,
                          int N, int H, int W, int C, hipStream_t s, bool nchw = false);
bool maxpool2x2_bwd_takes_nchw(int dt, const void *dy, const uint8_t *idx, const void *dx, const void *gate, int N, int H, int W, int C);
// any window / stride / padding (kh*kw <= 255): idx = dh*kw + dw of the first maximum inside the
// padded window; backward adds the gradients of all windows that chose an input (fixed order)
hipError_t maxpool_fwd(int dt, const void *x, void *y, uint8_t *idx, int N, int H, int W, int C, int kh,
                       int kw, int stride, int pad, hipStream_t s, void *y_nchw = nullptr, bool *stored = nullptr);
hipError_t maxpool_bwd(int dt, const void *dy, const uint8_t *idx, void *dx, GradEpi epi_pooled_gate, int N,
                       int H, int W, int C, int kh, int kw, int stride, int pad, hipStream_t s);
// mean over kh x kw windows at stride (kh, kw), no padding; gate (if any) indexed like dx
hipError_t avgpool_fwd(int dt, const void *x, void *y, int N, int H, int W, int C, int kh, int kw, hipStream_t s);
hipError_t avgpool_bwd(int dt, const void *dy, void *dx, GradEpi epi, int N, int H, int W, int C, int kh, int kw,
                       hipStream_t s);
hipError_t add_fwd(int dt, const void *a, const void *b, void *y, int relu, size_t n, hipStream_t s);
// dx (+)= dy with the epilogue of grad_out
hipError_t grad_copy(int dt, const void *dy, void *dx, GradEpi epi, size_t n, hipStream_t s);

// ---- LSTM cell, one time step t over all N sequences (gate order i, f, g, o; H = hidden size)
// P: input projection incl. bias [N][T][4H] (storage type); gh: S partial recurrent sums [S][N][4H]
// (S = 0 at t = 0); writes gates [N][T][4H] and cells [N][T][H] (float), h [N][T][H] and the
// one-step-delayed copy hs (hs[:, t+1] = h[:, t], hs[:, 0] = 0) in the storage type.
hipError_t lstm_cell_fwd(int dt, const void *P, const float *gh, int S, float *gates, float *cells, void *h,
                         void *hs, int N, int T, int H, int t, hipStream_t s);
// dy: gradient of h [N][T][H]; r: S partial sums of W_h^T D_{t+1} [S][N][H] (S = 0 at t = T-1);
// dcn [N][H] carries dc_{t+1}*f_{t+1} between steps; writes D[:, t] (pre-activation gradients,
// [N][T][4H], storage type).
hipError_t lstm_cell_bwd(int dt, const void *dy, const float *r, int S, const float *gates, const float *cells,
                         float *dcn, void *D, int N, int T, int H, int t, hipStream_t s);

// ---- the whole recurrence of an LSTM layer in one launch per direction, bf16 (kernels_lstm.hip); arguments as above,
// w_hh [4H][H] and wt_h [H][4H] are the recurrent matrix and its transpose in the storage type.  A block that has polled for
// another one's step wait_polls times gives up, and its group of sequences is computed by one block alone: the results are
// the same bit for bit, whatever the limit.
constexpr unsigned kLstmWaitPolls = 1u << 14;      // each a read of the slices that a wave needs, 0.5 to 1.5 us
bool lstm_seq_supported(int N, int T, int H, int compute_units);
size_t lstm_seq_workspace(int N, int H);
hipError_t lstm_seq_fwd(const void *P, const void *w_hh, float *gates, float *cells, void *h, void *hs, int N, int T, int H,
                        void *workspace, hipStream_t s, unsigned wait_polls = kLstmWaitPolls);
hipError_t lstm_seq_bwd(const void *dy, const void *wt_h, const float *gates, const float *cells, float *dcn, void *D, int N, int T, int H,
                        void *workspace, hipStream_t s, unsigned wait_polls = kLstmWaitPolls);

size_t bn_workspace(int rows, int C);
// Up to so many chunks of partial sums the normalisation and gradient passes add them up themselves.  Two launches against one,
// us: 1568 rows of 512 channels, 25 chunks, 6.9 / 4.0 forward and 7.1 / 4.4 backward; 6272 rows, 98 chunks, 256 channels 6.8 /
// 6.8 and 512 7.1 / 11.3.
constexpr int kBnSumChunks = 64;
// whether a batch-norm is better off with the partial sums of a neighbouring kernel than in one launch that reads its input whole
inline bool bn_takes_partials(int rows, int chunks) { return rows > 2048 || chunks <= kBnSumChunks; }
// stats: [2][C] floats (mean, invstd)
// pre_chunks > 0: the workspace already holds [2][pre_chunks][C] partial sums of x and x^2 (left there by
// the kernel that produced x) and the first pass over x is skipped
// res: the other input of a residual ADD fed only by this layer - y = [relu_sum](round(bn(x)) + res) in one pass
// y2: a second destination for y
hipError_t bn_fwd(int dt, const void *x, const float *gamma, const float *beta, float eps, void *y,
                  float *stats, int relu, int rows, int C, void *workspace, hipStream_t s, int pre_chunks = 0,
                  const void *res = nullptr, int relu_sum = 0, void *y2 = nullptr);
// pre_chunks > 0: the workspace already holds [2][pre_chunks][C] partial sums of dy and dy*xhat
hipError_t bn_bwd(int dt, const void *x, const void *dy, const float *gamma, const float *stats,
                  void *dx, float *dgamma, float *dbeta, GradEpi epi, int rows, int C,
                  void *workspace, hipStream_t s, int pre_chunks = 0);

// p = softmax(z) rows of K classes (float out), p2: a second destination
hipError_t softmax_fwd(int dt, const void *z, float *p, int rows, int K, hipStream_t s, float *p2 = nullptr);
// dz = scale*(p - onehot), loss[0] = -scale*sum_n log p[n,label]
hipError_t xent_bwd(int dt, const float *p, const int32_t *labels, float scale, void *dz, float *loss,
                    int rows, int K, hipStream_t s);

// ---- parameters
// w <- w - lr*g ; g <- 0 of a plain vector (K = 0, C elements), or of a weight matrix [K][RS][C] with its working copy and transposed
// copy (see recast and make_dgrad_filter), and of its bias b / db [K] (may be NULL)
struct SgdJob {
    float *w, *g;
    void *work, *wt;
    float *b, *db;
    int K, RS, C;
    bool work_panels, wt_panels;
};
// the updates of a stage, small ones together
hipError_t sgd_update(int dt, const SgdJob *jobs, int n, float lr, hipStream_t s);
// panels_of: columns of the matrix whose copy is kept in panels (GatherConv::wt_panels), 0: as it is
hipError_t recast(int dt, const float *w, void *work, size_t n, hipStream_t s, int panels_of = 0);
// wt[c][R-1-r][S-1-s][k] = work(w[k][r][s][c])   (dgrad filter)
hipError_t make_dgrad_filter(int dt, const float *w, void *wt, int K, int R, int S, int C, hipStream_t s, bool panels = false);
hipError_t fill_f32(float *p, float v, size_t n, hipStream_t s);

// ---- boundary layout conversion NCHW <-> NHWC (same storage type); optional ReLU gate.
// The NHWC side has Cp >= C physical channels (zero padded); nhwc_repad changes the channel
// count of an NHWC tensor (zero fill or truncation).
hipError_t nchw_to_nhwc(int dt, const void *src, void *dst, GradEpi epi, int N, int C, int H, int W,
                        int Cp, hipStream_t s);
hipError_t nhwc_to_nchw(int dt, const void *src, void *dst, int N, int C, int H, int W, int Cp,
                        hipStream_t s);
hipError_t nhwc_repad(int dt, const void *src, void *dst, size_t rows, int Cs, int Cd, hipStream_t s);
hipError_t nhwc_to_nchw_u8(const uint8_t *src, uint8_t *dst, int N, int C, int H, int W, hipStream_t s);

}  // namespace bapipe

// Internal declarations shared by the host orchestration (api.cpp) and the
// kernel files.  Activations live channel-last, [B][H][W][Cp] with the channel
// count rounded up to a multiple of 8 (padding channels hold zeros); FC-side
// activations are [B][ld] row-major.  The input of a first convolution over at
// most 4 channels is instead kept with 4 channels per pixel and its zero border
// (see Gather).  All kernels target gfx950 only.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace asgd {

enum DType { kF32 = 0, kBF16 = 1 };
inline size_t dtype_size(int dt) { return dt == kBF16 ? 2 : 4; }

// n / d for 0 <= n < 2^31 by multiply-high and shift.
struct FastDiv {
    uint32_t d, mul, sh;
};
FastDiv make_fastdiv(uint32_t d);

constexpr int kPushCopies = 4;   // replicas' copies that one push can write besides the parameters

// What happens to one accumulator element C[m][n] on its way to memory.
// The same routine serves the GEMM kernels and the split-K reduction.
struct Epilogue {
    void *out = nullptr;   // OutT [M][ld] (mode 0) or fp32 canonical conv filter gradient (mode 1)
    long ld = 0;
    int out_f32 = 0;       // 1: out is fp32 whatever the compute type
    const void *bias = nullptr;  // compute type, [bias_n]; added first to columns n < bias_n
    int bias_n = 0;
    int relu = 0;
    int drop = 0;          // dropout after ReLU: keep iff hash(m*drop_F+n) >= drop_thr
    uint64_t drop_key = 0;
    uint32_t drop_thr = 0;
    int drop_F = 0;
    float drop_scale = 1.f;
    const void *mask_src = nullptr;  // compute type, [M][mask_ld]: v = mask_src > 0 ? v*mask_scale : 0
    long mask_ld = 0;
    float mask_scale = 1.f;
    int mode = 0;          // 1: rows are cout, columns are (ky,kx,ci_padded) -> [cout][cin][kh][kw]
                           // 2: columns are (ky, kx*cw_rwc+ci) over window rows of cw_cinp elements -> the same
    int cw_cout = 0, cw_cin = 0, cw_cinp = 0, cw_kh = 0, cw_kw = 0;
    int cw_rwc = 4;        // mode 2: channels per stored pixel (column j of a window row is kx * cw_rwc + ci)
    // Push inside the gradient kernel (mode 0, no split-K): C[m][n] is the gradient g of parameter upd_w[m*ld + n]; the kernel
    // applies t = g + wd*w, v = mu*v - lr*t, w += v to upd_w / upd_v and writes the new parameters to upd_copies copies in the
    // compute type.  out (if any) receives g, upd_acc (if any) upd_acc + g, or g if upd_acc_first.  All [M][ld], rows and column
    // groups of 8 aligned to 16 bytes.
    float *upd_w = nullptr, *upd_v = nullptr, *upd_acc = nullptr;
    void *upd_copy[kPushCopies] = {};
    int upd_copies = 0, upd_acc_first = 0, upd_slim = 0;   // upd_slim: in fc_push where it takes the layer
    float upd_lr = 0.f, upd_mu = 0.f, upd_wd = 0.f;
};

// Gather description for an implicit-GEMM operand taken from a channel-last
// tensor x[N][H][W][C].  GEMM rows (direct form) enumerate (n, oy, ox) on a
// grid Ho x Wo; the K index enumerates (ky, kx, c).  The element is
// x[n][(oy*sm + ky - pad)/ds][(ox*sm + kx - pad)/ds][c] when both divisions
// are exact and in range, else 0.  Forward conv: sm = stride, ds = 1.
// Data gradient: sm = 1, ds = stride, pad = k-1-pad with a flipped filter.
struct Gather {
    const void *x = nullptr;
    int N = 0, H = 0, W = 0, C = 0;
    int Ho = 0, Wo = 0;
    int kh = 0, kw = 0, sm = 1, ds = 1, pad = 0;
    size_t bytes = 0;      // size of the tensor in bytes (at most 1 GiB); pieces outside it read as zeros
    // Byte strides between image rows and between pixels; 0 = dense (W*C and C elements).  Window-row form of a
    // convolution over few input channels: the tensor is stored with its zero border, 4 channels per pixel, and
    // described as kw = 1, pad = 0, C = one padded window row (kw*4 elements rounded up to 16 bytes), so that
    // the K index is (ky, kx*4 + c) and a whole window row is one contiguous run.
    size_t rowb = 0, pix = 0;
};

struct GemmPlan {
    int splits = 1;          // split-K factor
    int bm = 128, bn = 128;  // rows of a tile (filter gradients: 32, 64 or 128), columns (convolutions: 32 or 128)
    size_t ws_floats = 0;    // fp32 scratch needed when splits > 1
    bool stream = false;     // fc_split: weights by non-temporal loads
};

// The partial sums of a split GEMM, to be added up by `blocks` workgroups of 256 threads: in a launch of their own, or beside something
// else that neither waits for them nor writes their place.  later (where a routine has it): filled instead of launching the reduction
// (blocks stays 0 where the sums were whole).  On one stream a reduction of its own is 4 to 8 us in a chain of small kernels.
struct Reduction {
    const float *ws = nullptr; Epilogue ep;
    int splits = 0, M = 0, N = 0;
    int lanes = 1;                          // that share eight outputs (1, 8, 32, 256); 0: filters by runs of the canonical layout, with
    int npos = 0, cb = 0, chunks = 0;       // window positions, channels of a workgroup, and workgroups per output channel
    unsigned blocks = 0;
};

// us that the workgroups of a launch keep the 256 CUs busy, where per_cu of them fit a CU and r on one CU take t(r) us.
template <class F> double rounds_us(long workgroups, int per_cu, F t)
{
    const long round = 256L * per_cu, rest = workgroups % round;
    return (double)(workgroups / round) * t(per_cu) + (rest ? t((int)((rest + 255) / 256)) : 0.0);
}

// us that the filter gradient of a fully-connected layer takes while it leaves more than half of the CUs idle (0 if it does not).
double lone_fc_wgrad_us(int dtype, long out, long in, long batch);

// Stride-1 convolutions over equal grids (forward, and the data gradient as a convolution with flipped filters): K steps
// of 16 channels per chunk (0: the convolution does not run this way), chunks, tile shape, patch loads per thread and chunk,
// and the size of a group's packed filters.  Packed element (n, pos, c): blocks of 32 output columns, then chunks, window positions and K steps, each K
// step 64 lanes x 8 channels in the order the matrix cores take them (see direct_index).
struct DirectPlan {
    int ks = 0, nchunks = 0, tile = 0, npl = 0;
    size_t nblk_elems = 0, pack_elems = 0;
};
// All groups of a layer run in one launch: a and ep of the first group (N columns each), the groups' packed filters one after the other.
DirectPlan plan_direct(int dtype, const Gather &a, int N, int groups);   // none where the general engine is the faster one
// whether the general engine in K splits (plan_conv) is faster than plan d
bool split_is_faster(int dtype, const Gather &a, int N, int groups, const DirectPlan &d, size_t partials);
int conv_direct(int dtype, const Gather &a, const void *wpack, int N, int groups, const Epilogue &ep, const DirectPlan &plan, hipStream_t s);

// Filter gradients of stride-1 convolutions over equal grids in 16-bit data (conv_wgrad.hip): tile shape (-1: does not run
// this way), pixel ranges.  All groups of a layer run in one launch: dy [pixels][ldy]
// with M channels per group one after the other, x the gather of the first group.
struct WgradPlan {
    int tile = -1, splits = 0;
    size_t ws_floats = 0;    // fp32 scratch
};
WgradPlan plan_wgrad(int dtype, int M, int groups, const Gather &x, size_t max_ws_floats);
int conv_wgrad(const void *dy, long ldy, int M, int groups, const Gather &x, const Epilogue &ep, const WgradPlan &plan, float *ws, Reduction *later, hipStream_t s);
// C = ep(sum over splits of ws[split][M][N]), added in a fixed order: launched, or left to the caller in *later
int splitk_reduce(int dtype, const float *ws, int splits, const Epilogue &ep, int M, int N, Reduction *later, hipStream_t s);
int launch_reduction(int dtype, const Reduction &r, hipStream_t s);

// Every operand must fit in 1 GiB.
// C[M][N] = A[M][K] * B[N][K]^T; A gathered (direct), B plain K-contiguous.
GemmPlan plan_gemm(long M, long N, long K, int dtype, int max_splits);
// partials: floats that partial sums may take
GemmPlan plan_conv(long M, long N, long K, int dtype, int zoom, size_t partials, double *us);
GemmPlan plan_filter_grad(long M, long N, long K, int dtype, size_t partials);
int gemm_gather_plain(int dtype, const Gather &a, const void *b, long ldb, int N, const Epilogue &ep,
                      const GemmPlan &plan, float *ws, hipStream_t s);
// A plain [M][lda], B plain [b_rows][ldb], both K-contiguous; columns n >= b_rows of C are computed as zeros.
int gemm_plain_plain(int dtype, const void *a, long lda, int M, const void *b, long ldb, int N, int b_rows, int K,
                     const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s);
// A plain [M][lda] K-contiguous; B stored [K][ldb] (rows n contiguous).
int gemm_plain_trans(int dtype, const void *a, long lda, int M, const void *bt, long ldb, int N, int K,
                     const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s);
// A stored [K][lda] (rows m contiguous), B stored [K][ldb].
int gemm_trans_trans(int dtype, const void *at, long lda, int M, const void *bt, long ldb, int N, int K,
                     const Epilogue &ep, const GemmPlan &plan, float *ws, hipStream_t s);
// Partial sums ws[split][M][N] of A[M][K], M up to 64, times fully-connected weights in 16-bit data, [N][K] (rows past b_rows count as zeros) or
// trans [K][N] (fc_split.hip)
int fc_split(bool trans, const void *a, long lda, int M, const void *b, long ldb, int N, int b_rows, int K, int splits, bool stream, float *ws, hipStream_t s);
// Whether it is to read them by non-temporal loads: bytes of a net's 16-bit parameters, of its workspace, replicas whose passes run beside each other
bool fc_split_streams(size_t weights, size_t workspace, int replicas);
// Small fully-connected products (the kernel for them takes both): the weight gradient of layer w (stored or pushed as we says) and the
// data gradient of layer d in one launch.  They may be one layer's; not where the push rewrites the weights that d reads.
struct FcGrads { const void *dy, *x, *w; long ld_dy, ld_x; int batch, in, out; };   // output gradients, inputs, weights [out][in]
bool fc_pair_applies(const FcGrads &w, const FcGrads &d);
int fc_pair(int dtype, const FcGrads &w, const FcGrads &d, const Epilogue &we, const Epilogue &de, hipStream_t s);
// Logits (as gemm_plain_plain) and softmax cross-entropy (as launch_softmax_ce; dz [M][ep.ld]) in one launch: up to 16 classes
bool fc_softmax_applies(long M, long N, long K);
int fc_softmax(int dtype, const void *a, long lda, int M, const void *b, long ldb, int N, int classes, int K, const Epilogue &ep, const int32_t *labels, void *dz,
               float *row_loss, hipStream_t s);
// The push of a fully-connected layer's weights in their gradient kernel (fc_push.hip): operands as in gemm_trans_trans
// Whether the pushes of a pass are better off there than in the general kernel: parameters of the net, operations of its convolutions' gradients, images,
// whether the pass stays on one stream for its size, whether other replicas' passes run beside it.
bool fc_push_pays(size_t params, double conv_flops, long batch, bool one_stream, bool others);
bool fc_push_applies(int dtype, int M, int N, int K, const Epilogue &ep);
int fc_push(const void *at, long lda, int M, const void *bt, long ldb, int N, int K, const Epilogue &ep, hipStream_t s);
// Filter gradient: A stored [K = B*Ho*Wo][lda] (rows = cout), B gathered with the
// reduction index enumerating (n, oy, ox) and rows enumerating (ky, kx, c).
int gemm_trans_gather(int dtype, const void *at, long lda, int M, const Gather &b, const Epilogue &ep,
                      const GemmPlan &plan, float *ws, Reduction *later, hipStream_t s);
// fp32 scratch (in floats) the filter gradient of a first convolution in window-row form wants in plan.ws_floats to
// run as one persistent kernel with a partial result per workgroup; 0 where that kernel does not apply
size_t rows_wgrad_ws_floats(int dtype, int M, const Gather &b);

// ---- streaming kernels (kernels_stream.hip) --------------------------------
// Whether an update over n parameters reads its `arrays` fp32 vectors (parameters and state; the gradient, read once, is non-temporal in any case)
// by non-temporal loads: where these and the copy of copy_es bytes a parameter that it writes are larger than 384 MiB, one and a half times
// the memory-side cache.  Up to there some of a vector is still in the cache at the next pass, beyond it ordinary loads only push out what is
// needed elsewhere.  us, ordinary / non-temporal, the same vectors again / after a copy of 1 GiB: momentum 24 M 70 / 80, 76 / 85; 40 M 126 / 129,
// 123 / 134; 50 M 175 / 166, 159 / 171; 62 M 225 / 206, 200 / 211; with a bf16 copy 28 M 89 / 98, 97 / 105; 40 M 145 / 135, 141 / 144; 62 M 256 / 211, 228 / 227;
// with an fp32 copy 28 M 96 / 100, 108 / 112; 36 M 154 / 126, 139 / 143; Adagrad as momentum; Adadelta 24 M 98 / 118, 114 / 122; 36 M 184 / 176, 169 / 180; 50 M
// 265 / 244, 243 / 249.  Passes with the update behind the gradient: 25.7 M 233 / 243, 38 M 299 / 300, 58.8 M 469 / 432.
bool beyond_cache(size_t n, int arrays, size_t copy_es);
int launch_update(float *w, float *v, const float *g, size_t n, float lr, float mu, float wd,
                  int *version_counter, hipStream_t s);
// the update, and the updated parameters written to `copy` (fp32 or bf16) in the same pass; n parameters of a vector of total
int launch_update_snapshot(float *w, float *v, const float *g, size_t n, size_t total, float lr, float mu, float wd, void *copy,
                           int dst_dtype, hipStream_t s);
// The update of up to 8 ranges [off, off + cnt) of the parameter vector in one launch, with what a replay does beside it in the same
// pass: the gradient added to acc (or written there if acc_first), the new parameters written to copies in fp32 or
// bf16, the version counter advanced and a log record (update, worker, counter) per fetch.  All bases 16-byte aligned.
struct PushRanges {
    float *w, *v; const float *g; float *acc;
    float lr, mu, wd;
    int acc_first, n, ncopies, nlogs;
    void *copy[2 * kPushCopies];
    unsigned f32mask;                       // bit c: copy c is fp32
    int *counter;
    int32_t *log[kPushCopies]; int log_update[kPushCopies], log_worker[kPushCopies];
    size_t off[8], cnt[8]; unsigned blk[9]; // blk filled by the launch
};
int launch_push_ranges(PushRanges &p, hipStream_t s);
// Adagrad / Adadelta server updates (one pass, in place)
int launch_adagrad(float *w, float *h, const float *g, size_t n, float lr, float eps, float wd, hipStream_t s);
int launch_adadelta(float *w, float *a, float *b, const float *g, size_t n, float rho, float eps, float wd, hipStream_t s);
// acc = g (first) or acc + g
int launch_accumulate(float *acc, const float *g, size_t n, bool first, hipStream_t s);
int launch_snapshot(const float *src, void *dst, size_t n, int dst_dtype, const int *version_counter,
                    int32_t *log_slot, int log_update, int log_worker, hipStream_t s);
// Filter packing for all convolution layers of a net in one launch.  Per layer: canonical filters
// [cout][cin][k][k] -> forward pack wf [coutp][k][k][cinp] and, if wd is given, the flipped data-gradient pack
// wd [cinp][k][k][coutp]; or (rw = channels per stored pixel > 0) the window-row pack wf [coutp][k][KW], element (ky, kx*rw + ci), zeros elsewhere.
// fks / dks > 0: that pack is in the order of conv_direct instead.
struct PackJob {
    const void *w; void *wf; void *wd;
    int cout, cin, k, coutp, cinp, rw, KW;
    int fks, fch, dks, dch;   // K steps per chunk and chunks of wf / wd where they are packed for conv_direct (0: rows)
    int cinw;             // filled by launch_head: input channels of wf with the padding of its last chunk
    unsigned start, nf;   // filled by launch_head
};
struct PackJobs { PackJob j[12]; int n; unsigned total; };
// Input staging: images [B][C][H][W] (compute type) -> channel-last [B][H][W][Cp] with zero padding channels (pc = 0), or
// into the interior of a bordered [B][H+2*pad][Wp][pc] tensor (pc = 1..4 channels per pixel; the border is not written).
struct StageJob {
    const void *src; void *dst;   // src == nullptr: nothing to stage
    int B, C, H, W, Cp, pad, Wp, pc;
    unsigned total; FastDiv dHW, dH, dWq;   // filled by launch_head
};
// the head of a forward pass: the filters of up to 12 layers packed and the images staged, in one launch where it can be
int launch_head(int dtype, PackJobs &jobs, const StageJob &st, hipStream_t s);
// nonneg: x holds no negative values (below is a ReLU); a matter of speed only
int launch_pool_fwd(int dtype, const void *x, int nonneg, void *y, uint8_t *arg, int B, int H, int W, int Cp, int k, int stride,
                    hipStream_t s);
// dx[pixel] = sum of dy over the windows whose recorded maximum is this pixel; times [x > 0] if relu
int launch_pool_bwd(int dtype, const void *dy, const uint8_t *arg, const void *x, int relu, void *dx, int B, int H,
                    int W, int Cp, int k, int stride, float *bands, const Reduction *beside, hipStream_t s);
// bands != nullptr: the kernel also leaves the column sums of dx in bands[Cp][pool_bwd_bands(...)] (stage 1 of a
// bias gradient); only for shapes where pool_bwd_bands is not 0.  beside != nullptr, for the same shapes: partial sums added up in the same launch
long pool_bwd_bands(int dtype, int B, int H, int W, int Cp, int k, int stride);
// cross-channel response normalisation on channel-last tensors: y = a * (bias + alpha * window sum of a^2)^(-beta);
// backward writes da (times [a > 0], the ReLU of the convolution below, if relu) from a and dy; size odd, <= 9
int launch_lrn_fwd(int dtype, const void *a, void *y, size_t pixels, int Cp, int size, float alpha, float beta, float bias, hipStream_t s);
int launch_lrn_bwd(int dtype, const void *a, const void *dy, int relu, void *da, size_t pixels, int Cp, int size, float alpha, float beta,
                   float bias, hipStream_t s);
// Normalisation and a pool of window k, stride 2, on top of it in one pass each: forward a -> pooled y and positions; backward
// writes da, times [a > 0], from the gradient dy at the pool's output, and leaves the column sums of da in
// bands[Cp][lrn_pool_bands(...)].  lrn_pool_bands is 0 where the pair does not run this way: where the kernels do not
// take it, or (not if always) where separate ones are faster.  Separate ones need more workspace.  forked: the
// weight gradients run on the side stream.
long lrn_pool_bands(int dtype, int B, int H, int W, int Cp, int k, int stride, bool forked, bool always);
int launch_lrn_pool_fwd(int dtype, const void *a, void *y, uint8_t *arg, int B, int H, int W, int Cp, int size, float alpha, float beta, float bias, int k,
                        hipStream_t s);
int launch_lrn_pool_bwd(int dtype, const void *a, const void *dy, const uint8_t *arg, void *da, int B, int H, int W, int Cp, int size, float alpha,
                        float beta, float bias, int k, float *bands, hipStream_t s);
// A pool of window k, stride 2, under a fully-connected layer: forward straight into flat [B][C*Ho*Wo] in (c,h,w) order (and the
// positions, channel-last); backward from dflat, masked where relu by flat > 0, into dx, with the column sums of dx in
// bands[Cp][pool_flat_bands(...)].  pool_flat_bands is 0 as lrn_pool_bands is.
long pool_flat_bands(int dtype, int B, int H, int W, int C, int Cp, int k, int stride, bool forked, bool always);
int launch_pool_flat_fwd(int dtype, const void *x, int nonneg, void *flat, uint8_t *arg, int B, int H, int W, int C, int Cp, int k, hipStream_t s);
int launch_pool_flat_bwd(int dtype, const void *dflat, const void *flat, int relu, const uint8_t *arg, void *dx, int B, int H, int W, int C, int Cp, int k,
                         float *bands, hipStream_t s);
// channel-last [B][H][W][Cp] -> [B][C*H*W] in (c,h,w) order, and back (zero padding channels; optional ReLU mask)
int launch_flatten(int dtype, const void *x, void *flat, int B, int H, int W, int C, int Cp, hipStream_t s);
int launch_unflatten(int dtype, const void *dflat, const void *x_for_mask, int relu, void *dx, int B, int H, int W,
                     int C, int Cp, hipStream_t s);
// db[n] = sum_m dy[m][n], n < N, fp32, fixed summation order, in two stages: launch_colsum_partial sums bands of
// rows into ws (colsum_ws_floats floats, not shared with another pending job) and appends a job;
// launch_colsum_finish adds the bands of all pending jobs (up to 12) in one launch.
// ws[band][ld] (bf16: in that type), or ws[column][nblk] if colmajor; sums are divided by div
struct ColsumJob { const float *ws; float *db; long ld; int nblk, N; unsigned start_block; int colmajor, bf16; float div; };
struct ColsumJobs { ColsumJob j[12]; int n; };
int launch_colsum_partial(int dtype, const void *dy, long ld, long M, int N, float *db, float *ws, ColsumJobs &jobs, hipStream_t s);
// the same with the first stage put off: colsum_partial_defer appends the tensor to s1 (and its second stage to jobs),
// launch_colsum_stage1 sums the bands of all appended tensors (up to 12) in one launch
struct ColsumS1Job { const void *dy; float *ws; long ld, M, rows_per_block; int chunks, cpb, rl, gx, gy; unsigned start_block; };
struct ColsumS1Jobs { ColsumS1Job j[12]; int n; };
int colsum_partial_defer(int dtype, const void *dy, long ld, long M, int N, float *db, float *ws, ColsumS1Jobs &s1, ColsumJobs &jobs);
int launch_colsum_stage1(int dtype, ColsumS1Jobs &s1, hipStream_t s);
// beside != nullptr: partial sums added up in the same launch
int launch_colsum_finish(int dtype, ColsumJobs &jobs, const Reduction *beside, hipStream_t s);
size_t colsum_ws_floats(int dtype, long M, long ld);
// softmax cross-entropy over fp32 logits [B][ld]: the loss of every row, whose mean loss_job appends to the bias sums' second
// stage, and dz (compute type, [B][ld], zero padding columns)
int launch_softmax_ce(int dtype, const float *z, long ld, const int32_t *labels, int B, int C, void *dz, float *row_loss, hipStream_t s);
void loss_job(const float *row_loss, int B, float *loss, ColsumJobs &jobs);
int launch_fill_zero(void *p, size_t bytes, hipStream_t s);
// debug exports (canonical layouts)
int launch_export_nhwc(int dtype, const void *x, float *dst, int B, int H, int W, int C, int Cp, hipStream_t s);
int launch_export_rows(int dtype, int src_f32, const void *x, long ld, float *dst, int B, int F, hipStream_t s);
int launch_export_argmax(const uint8_t *arg, uint8_t *dst, int B, int H, int W, int C, int Cp, hipStream_t s);
int launch_dropout_mask(uint8_t *dst, size_t count, uint64_t key, uint32_t thr, hipStream_t s);

// host-side key of the dropout generator for one (seed, step, worker, layer)
uint64_t dropout_key(uint64_t seed, uint64_t step, uint32_t worker, uint32_t layer);

}  // namespace asgd

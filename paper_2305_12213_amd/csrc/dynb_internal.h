// Internal declarations shared by the library's translation units (not part of the ABI).
#ifndef DYNB_INTERNAL_H
#define DYNB_INTERNAL_H

#include <cstddef>
#include <cstdint>

#include "../../include/dynb.h"

namespace dynb {

// Records a thread-local message and returns `code`.
int fail(int code, const char* fmt, ...);

constexpr int COL_PAD = 64;   // leading dimensions are padded to a multiple of this ...
constexpr int NARROW_PITCH = 32;   // ... except images of at most so many channels, whose rows are this wide

inline int64_t round_up(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Row segments of the K workers, passed to kernels by value.
// off[k]: first row of worker k in the caller's batch, off[K] = sum(b).
struct Segs {
  int K;
  int off[DYNB_MAX_WORKERS + 1];
};

struct Lambdas {
  int K;
  float w[DYNB_MAX_WORKERS];
};

// A list of index ranges [off, off + len) of the flat parameter vector, passed to kernels by
// value: one launch serves all the small tensors (biases, padding) of a model.
constexpr int MAX_RANGES = 48;
struct Ranges {
  int n;
  int64_t off[MAX_RANGES];
  int64_t len[MAX_RANGES];
};

// Kernel classes for the timing aid.
enum KClass {
  KC_GEMM_FWD = 0,
  KC_GEMM_DGRAD,
  KC_GEMM_WGRAD,
  KC_PACK,
  KC_SOFTMAX,
  KC_BIAS_GRAD,
  KC_FINALIZE,
  KC_AGGREGATE,
  KC_UPDATE,
  KC_WEIGHT_CAST,
  KC_CONV_AUX,
  KC_NORM,
  KC_GEMM_WGRAD_SMALL,   // bf16 weight gradients that run on the 128 x 128-tile kernels
  KC_GEMM_SMALL,         // bf16 forward / input-gradient products on 128 x 128 tiles
  KC_GEMM_WGRAD_64,      // bf16 weight gradients on the 64 x 64-tile kernel
  KC_GEMM_64,            // bf16 forward / input-gradient products on the 64 x 64-tile kernel
  KC_GEMM_128X64,        // ... on 128 x 64 tiles
  KC_COUNT
};

// Brackets one launch with events when timing is on.  flops/bytes are the algorithmic
// work of the launch (accumulated per class).
struct Timed {
  Timed(KClass cls, void* stream, double flops, double bytes);
  ~Timed();
  int cls;             // -1: timing is off
  void* stream;
  void* start;         // hipEvent_t, owned until the destructor queues the pair
  void* stop;
};

enum { MODE_FWD = 0, MODE_DGRAD = 1, MODE_WGRAD = 2 };

// C'[i][j] = sum_k A[i][k] * B[j][k]; both operands are k-contiguous with 16-byte aligned
// rows.  Meaning of (i, j) and of the outputs depends on `mode`:
//   FWD   : i = batch row, j = output feature.  v = acc + bias[j], optional ReLU;
//           C[i*ldc + j] = T(v) if C; Cf[i*ldcf + j] = v if Cf.
//   DGRAD : i = batch row, j = input feature.  v = mask[i*ldmask + j] > 0 ? acc : 0 (mask
//           optional); C[i*ldc + j] = T(v).  With `addend` (bf16 only: the gradient that reaches
//           the same tensor over a residual branch) acc is first rounded to T and
//           addend[i*ldadd + j] added, then the mask is applied.
//   WGRAD : one group per worker g; i = output feature, j = input feature;
//           Cf[g*group_stride + j*ldcf + i] = acc.  A = dy and B = the input as they are,
//           ROW-MAJOR [batch rows][lda / ldb]; the reduction runs over worker g's rows
//           [off[g], off[g+1]).
struct GemmArgs {
  const void* A; int64_t lda; int M;   // rows of A  (i)
  const void* B; int64_t ldb; int N;   // rows of B  (j)
  int K;                               // reduction length (FWD/DGRAD), multiple of 8
  int mode;
  const float* bias; int relu;
  void* C; int64_t ldc;
  float* Cf; int64_t ldcf;
  const void* mask; int64_t ldmask;
  const void* addend; int64_t ldadd;   // DGRAD, bf16: see above
  int64_t group_stride;
  int groups_per_block;                // WGRAD, bf16 kernel: workers streamed by one workgroup
  // WGRAD, unsplit (bf16: optional): also write the bias gradient bias_grad[g*group_stride + i] =
  // sum over worker g's rows of A[row][i].  Grouped launches (fp32, bf16 on 64 x 64 tiles) with `agg`: its
  // weighted aggregate too, to bias_agg[i] (others: left to the pass over the small tensors).
  float* bias_grad;
  float* bias_agg;
  // Implicit-GEMM gather of operand A for a 3x3 convolution with zero padding 1 (bf16 only).
  // conv == 0: A is a plain matrix.  conv == 1 (forward): row i is output pixel (n, y, x) of a
  // row_h x row_w grid and reduction index k = (kh*3 + kw)*cp + c reads channel c of source
  // pixel (y*stride + kh - 1, x*stride + kw - 1).  conv == 2 (input gradient): row i is input
  // pixel (n, y, x) and k reads channel c of output pixel ((y + 1 - kh)/stride,
  // (x + 1 - kw)/stride) when both divisions are exact.  Out-of-range taps read zero.
  // A points at the source tensor [n * src_h * src_w][lda]; cp is a multiple of 8.
  int conv, src_h, src_w, row_h, row_w, stride, cp;
  // set by launch_gemm: log2(cp) when the cheap addressing applies (cp a power of two >= 32,
  // so that a 32-deep stage lies within one tap; the source pixel of a tap is the row's own
  // pixel plus an offset that is the same for all rows; source tensor below 2 GiB), else -1
  int gather_log2cp;
  double alg_flops, alg_bytes;         // algorithmic work of the launch (timing aid only)
  // WGRAD, bf16 kernel: split every worker's reduction into `split` chunks of `chunk` columns
  // (a multiple of 64).  Chunk c of worker g writes its tile to partial + (g*split + c) *
  // partial_stride (row pitch ldcf); launch_wgrad_reduce sums the chunks in a fixed order.
  // split <= 1: no split, tiles go straight to Cf.
  int split, chunk;
  float* partial;
  int64_t partial_stride;
  // WGRAD, optional: also write agg[j*ldcf + i] = sum_g lam[g] * (tile of worker g), summed in
  // ascending g (fp32) or a fixed, tile-dependent rotation of it (bf16): the weighted aggregation
  // of Eq. 2 while the per-worker tiles are still in registers.  Only
  // in the kernels that walk all workers of a tile: large bf16 layers when gemm_fuses_aggregate() says so,
  // grouped launches (fp32, bf16 on 64 x 64 tiles) always can.
  float* agg;
  float lam[DYNB_MAX_WORKERS];
  const void* zeros;   // 16 bytes of zeros in device memory (set by launch_gemm): what copies
                       // fetch for rows past a worker's last and taps outside an image
};

// Softmax cross-entropy in the launch of the last product (softmax_head.h): dz = (softmax(logits) -
// onehot(y)) / (rows of the worker), zero in columns [C, ldd), rowloss[row]; the logits are not stored.
struct HeadArgs {
  const int32_t* y;
  void* dz; int64_t ldd;
  float* rowloss;
  Segs segs;
};
// whether that product's kernel has whole rows at hand
bool head_applies(int dtype, const GemmArgs& a);
// the class that such a launch is timed in
KClass gemm_class(int dtype, const GemmArgs& a);
// (with `head`: a forward product for which head_applies)
int launch_gemm(int dtype, const GemmArgs& a, const Segs& s, void* stream, const HeadArgs* head = nullptr);
int launch_gemm_f32(const GemmArgs& a, const HeadArgs* head, void* stream);   // forward / input gradient (gemm_f32.hip)
bool gemm_f32_head_applies(const GemmArgs& a);
void launch_gemm_f32_head(const GemmArgs& a, const HeadArgs& head, unsigned tiles, void* stream);   // (its 16 x 16 tiles)
// What ends an iteration (step_end.h): loss[g] = mean of rowloss over worker g's rows; grads[g][P .. P_pad)
// = 0; out[P .. P_pad) = 0 if out.
struct StepEnd {
  const float* rowloss; float* loss;
  float* grads; int64_t P, P_pad;
  float* out;
};
// fp32 weight gradients of up to WGRAD_F32_ITEMS layers (all over the same rows) in one launch, which does
// the step's end too if `end`
constexpr int WGRAD_F32_ITEMS = 8;
int launch_wgrad_f32(const GemmArgs* a, int n, const Segs& s, const StepEnd* end, void* stream);
// whether a wave walks all workers of its tile in any case (the tiles fill the chip), and what walking them,
// to form the average, costs beside divided ones
bool wgrad_f32_walks(const GemmArgs& a, const Segs& s);
double wgrad_f32_fold_us(const GemmArgs& a, const Segs& s);
// The choice behind it: a walk over all workers of `walk_us` beside a `shares`-th of it (fold_us: the
// difference), and a pass over K results of `weights` floats.
constexpr int64_t AGGREGATE_ALONE = 65536;   // from so many on, a launch of its own (else part of the last)
double fold_us(double walk_us, int shares, int64_t weights, int K);
double average_pass_us(int64_t weights, int K);
// bf16 products with few tiles (gemm_small.hip): whether one (unsplit) counts as such, and the launch.
bool gemm_small_applies(const GemmArgs& a);
int launch_gemm_small(const GemmArgs& a, const HeadArgs* head, void* stream);   // forward / input gradient
// forward / input gradient of dense bf16 layers on larger tiles (gemm_lines.hip)
enum { LINES_256, LINES_128, LINES_128X64 };
int gemm_lines_tiles(const GemmArgs& a);
int launch_gemm_lines(const GemmArgs& a, void* stream);
// weight gradients of up to WGRAD_SMALL_ITEMS such layers (all over the same rows) in one launch, which does
// the step's end too if `end`
constexpr int WGRAD_SMALL_ITEMS = 8;
int launch_wgrad_small(const GemmArgs* a, int n, const Segs& s, const StepEnd* end, void* stream);
// whether that is faster than the 128 x 128-tile kernel (and, with `average`, a pass over its results);
// the other two as for fp32
bool wgrad_small_pays(const GemmArgs& a, const Segs& s, bool average);
bool wgrad_small_past(const GemmArgs* a, int n, int K);   // whether the results of such a launch leave past the caches
bool wgrad_small_walks(const GemmArgs& a, const Segs& s);
double wgrad_small_fold_us(const GemmArgs& a, const Segs& s);
// Whether a bf16 weight-gradient launch of launch_gemm of these dimensions can take GemmArgs::agg.
bool gemm_fuses_aggregate(int dtype, const GemmArgs& a);
// out[e] = sum_k lam.w[k] * g[k*worker_stride + e], e < n, ascending k (any alignment)
int launch_aggregate_range(const float* g, int64_t worker_stride, const Lambdas& lam, int64_t n,
                           float* out, void* stream);
// the same over every range r: out[off_r + e] from g[k*worker_stride + off_r + e]
int launch_aggregate_ranges(const float* g, int64_t worker_stride, const Lambdas& lam,
                            const Ranges& r, float* out, void* stream);

// x fp32 [rows][D] -> out T [rows][ld]
int launch_pack_rows(int dtype, const float* x, int rows, int D, void* out, int64_t ld,
                     void* stream);
// logits fp32 [rows][ldz] -> dz T [rows][ldd] (pad columns zero), rowloss[rows]
int launch_softmax_xent(int dtype, const float* logits, int64_t ldz, const int32_t* y, int C,
                        void* dz, int64_t ldd, int ld_cols, float* rowloss, const Segs& s,
                        void* stream);
// grads[g*group_stride + n] = sum over worker g's rows of dy[row][n] (bf16 [rows][ld]; ld a
// multiple of 64, zeros in the padding columns)
int launch_bias_grad_rows(const void* dy, int64_t ld, int N, float* grads, int64_t group_stride,
                          const Segs& s, void* stream);
// Reads `bytes` (a multiple of 16, 16-byte aligned) and discards them: what a launch is about to
// fetch several times over, brought into the last-level cache by one sequential pass.
int launch_touch(const void* p, int64_t bytes, void* stream);
// The step's end; with end.out (and lam, small): also out[range] = sum_k lam_k grads[k][range] for every
// range of `small`, in the same launch.
int launch_finalize(const StepEnd& end, const Segs& s, const Lambdas* lam, const Ranges* small, void* stream);
int launch_aggregate(const float* grads, const Lambdas& lam, int64_t n, float* out, void* stream);
int launch_sgd(float* params, const float* g, int64_t n, float lr, void* stream);
int launch_momentum(float* params, float* v, const float* g, int64_t n, float lr, float mu,
                    void* stream);
// One optimizer step per parameter.  kind: DYNB_OPT_*.  s1 = velocity (momentum) or first
// moment (Adam), s2 = second moment (Adam).  Adam's bias corrections are passed as
// inv_c1 = 1/(1 - beta1^t), inv_c2 = 1/(1 - beta2^t), and omb = 1 - beta, all formed in double.
struct UpdateRule {
  int kind;
  float lr, mu;
  float beta1, beta2, omb1, omb2, eps, inv_c1, inv_c2;
};
// Fills the Adam fields of r for step t (t >= 1, betas in [0, 1)).
void set_adam(UpdateRule& r, double beta1, double beta2, float eps, int64_t t);
// Where the gradient of a parameter comes from: a finished vector g (lam.K == 0), or the K
// per-worker gradients g + k*worker_stride, summed with weights lam.w[k] in ascending k
// (the weighted aggregation of Eq. 2 done on the fly).
struct GradSource {
  const float* g;
  int64_t worker_stride;
  Lambdas lam;
};

// Weights W fp32 [taps][R][C] at parameter offset `off` (a dense layer: one tap), each tap with its
// copies Wn T [R][ldn] and Wt T [C][ldt] (T = the model's storage type), tap_n / tap_t elements
// apart.  Passed to the kernel by value.
constexpr int MAX_CAST_MATS = 8;
struct CastMats {
  int n;
  int64_t off[MAX_CAST_MATS];
  int R[MAX_CAST_MATS], C[MAX_CAST_MATS], taps[MAX_CAST_MATS];
  void* Wn[MAX_CAST_MATS];
  int64_t ldn[MAX_CAST_MATS], tap_n[MAX_CAST_MATS];
  void* Wt[MAX_CAST_MATS];
  int64_t ldt[MAX_CAST_MATS], tap_t[MAX_CAST_MATS];
  int first_block[MAX_CAST_MATS + 1];   // first workgroup of each matrix (set by the launcher)
};
// Rows of a tile of `tile_columns` in such a launch over K workers' gradients (0: over their average).
int cast_tile_rows(const CastMats& mats, int tile_columns, int K);
// The copies alone, of the weights as they are.
int launch_weight_casts(int dtype, const float* params, CastMats& mats, void* stream);
// The same together with the packed input act T [rows][ld] = x fp32 [rows][D], zeros beyond (rows = 0: none),
// and zeros in the columns [pad_from, pad_ld) of T tensors [pad_rows][pad_ld].
constexpr int MAX_PADS = 4 * MAX_CAST_MATS;
struct Prepare {
  const float* x; void* act;
  int rows, D;
  int64_t ld;
  int n;
  void* pad[MAX_PADS];
  int pad_rows[MAX_PADS], pad_from[MAX_PADS], pad_ld[MAX_PADS];
};
int launch_prepare(int dtype, const float* params, CastMats& mats, const Prepare& pr, void* stream);
// One launch: the optimizer step of every matrix of `mats` fused with the refresh of its two
// copies, and the element-wise step of every range of `small`; s1/s2 point at the state of
// parameter 0 (may be null when the rule has no such state)
int launch_update_cast(int dtype, float* params, CastMats& mats, const Ranges& small,
                       const GradSource& src, const UpdateRule& rule, float* s1, float* s2,
                       void* stream);
// element-wise step of every range of r
int launch_update_ranges(float* params, const Ranges& r, const GradSource& src, const UpdateRule& rule,
                         float* s1, float* s2, void* stream);
// plain streaming Adam over n parameters (n a multiple of 4, 16-byte aligned pointers)
int launch_adam(float* params, float* m, float* v, const float* g, int64_t n,
                const UpdateRule& rule, void* stream);
// out[g*group_stride + e] = sum_{c < split} partial[(g*split + c)*partial_stride + e], e < n
int launch_wgrad_reduce(const float* partial, int split, int64_t partial_stride, int64_t n,
                        float* out, int64_t group_stride, int K, void* stream);

// ---- convolution helpers (bf16 storage) ----
int launch_gap_forward(const void* act, int64_t lda, int HW, int C, int samples, void* pooled,
                       int64_t ldp, void* stream);
int launch_gap_backward(const void* dpooled, int64_t ldp, const void* act, int64_t lda, int HW,
                        int C, int samples, int relu, void* dact, int64_t ldd, void* stream);
// Forward / input gradient of a 3x3 convolution from one halo tile in LDS (conv_direct.hip):
// takes the same description as the gathered-operand GEMM where conv_direct_applies() says so.
bool conv_direct_applies(int dtype, const GemmArgs& a);
int launch_conv_direct(const GemmArgs& a, void* stream);
// The same for 64 reduction channels with the weights resident in LDS (conv_resident.hip).
bool conv_resident_applies(int dtype, const GemmArgs& a);
int launch_conv_resident(const GemmArgs& a, void* stream);
// The same from a flat run of pixels, images of any shape (conv_flat.hip).
bool conv_flat_applies(int dtype, const GemmArgs& a);
int launch_conv_flat(const GemmArgs& a, void* stream);

// Input gradient with stride 2, all parity classes of a run of pixels together (conv_strided_grad.hip).
bool conv_strided_grad_applies(int dtype, const GemmArgs& a);
int launch_conv_strided_grad(const GemmArgs& a, void* stream);

// The rows of every worker cut into chunks of `rows` rows: first[k] = index of worker k's first
// chunk, first[K] = number of chunks (chunk c of worker k starts at off[k] + (c - first[k]) * rows).
struct RowChunks {
  int rows;
  int first[DYNB_MAX_WORKERS + 1];
};
RowChunks make_row_chunks(const Segs& s, int rows);

// Per-worker weight gradient of a 3x3 convolution straight from the row-major activations
// (bf16 in: [samples*H*W][ldi], dy: [samples*Ho*Wo][ldd]; dW[k * group_stride + (tap*Cin +
// ci)*Cout + co] and the bias gradient db[k * group_stride + co], fp32).  chunk_rows =
// conv_wgrad_chunk_rows(largest row count of the model's plan); scratch:
// conv_wgrad_scratch_floats() floats.
int conv_wgrad_chunk_rows(int64_t max_rows);
int64_t conv_wgrad_scratch_floats(int64_t max_rows, int max_workers, int Cin, int Cout);
// n layers of one geometry (and chunk_rows) at a time.
constexpr int CONV_WGRAD_ITEMS = 8;
struct ConvWgradLayer {
  const void* in; const void* dy;
  float* dW; float* db;
};
// How the first of them are worked on together.
enum { CONV_WGRAD_TAPS, CONV_WGRAD_ROWS, CONV_WGRAD_FLAT };
struct ConvWgradPlan {
  int kernel;          // CONV_WGRAD_TAPS ..
  int ci32, co32;      // 32-channel tiles on either side of a channel block
  bool paired;         // two groups of waves, which halve a chunk
  int layers;          // so many in one launch
  RowChunks ch;
  int sum_groups;      // groups of threads that divide a worker's chunks in the sum: 1, 4 or 16
};
ConvWgradPlan conv_wgrad_plan(int n, int64_t ldi, int Cin, int H, int W, int64_t ldd, int Cout, int Ho, int Wo, int stride,
                              int chunk_rows, int64_t scratch_floats, const Segs& s);
int launch_conv_wgrad(const ConvWgradLayer* layers, int n, int64_t ldi, int Cin, int H, int W, int64_t ldd,
                      int Cout, int Ho, int Wo, int stride, int chunk_rows, float* scratch,
                      int64_t scratch_floats, int64_t group_stride, const Segs& s, double flops, double bytes,
                      void* stream);

// The first convolution of a model, on images of at most three channels (conv_stem.hip): forward and
// weight gradient straight from the caller's fp32 pixels [images * H * W][Cin].
bool conv_stem_applies(int Cin);
int launch_stem_forward(const float* x, int Cin, int H, int W, int Ho, int Wo, int stride, int64_t pixels,
                        const void* w, int kf, const float* bias, int N, int relu, void* out,
                        int64_t ldo, double flops, double bytes, void* stream);
int launch_stem_wgrad(const float* x, int Cin, int H, int W, int Ho, int Wo, int stride, const void* dy,
                      int64_t ldd, int Cout, int chunk_rows, float* scratch, int64_t scratch_floats, float* dW,
                      float* db, int64_t group_stride, const Segs& s, double flops, double bytes, void* stream);

// Batch normalisation over each worker's own rows (bf16; x: T [rows][ldx], y: T [rows][ldy]):
// writes mean / rstd [k][C] (kept for the backward pass).  `scratch`: row_scratch_floats() floats
// (the partial results of the row chunks), shared by forward and backward.
constexpr int BN_CHUNK_ROWS = 256;
int64_t row_scratch_floats(int64_t max_rows, int max_workers, int C);
// With `skip` (a residual addition fused in): y = relu_sum?(T(normalised) + skip).
int launch_bn_forward(const void* x, int64_t ldx, int C, const float* gamma, const float* beta,
                      float eps, int relu, float* mean, float* rstd, float* scratch,
                      const void* skip, int64_t lds_, int relu_sum, void* y, int64_t ldy,
                      const Segs& s, void* stream);
// dgamma / dbeta[k * group_stride + c] (fp32, per worker) from dy (already masked by the layer's
// own ReLU); with need_dx also dx (T [rows][ldo]), masked by x > 0 when relu_below
int launch_bn_backward(const void* dy, int64_t ldd, const void* x, int64_t ldx, int C,
                       const float* gamma, const float* mean, const float* rstd, float* scratch,
                       float* dgamma, float* dbeta, int64_t group_stride, int need_dx,
                       int relu_below, void* dx, int64_t ldo, const Segs& s, void* stream);
// out = relu?(a + b) over `width` (padded, a multiple of 8) columns of `rows` rows
int launch_add_forward(const void* a, int64_t lda, const void* b, int64_t ldb, int64_t width,
                       int64_t rows, int relu, void* out, int64_t ldo, void* stream);
// dst = (accumulate ? dst : 0) + (relu ? src where act > 0 : src), same extent convention
int launch_grad_route(const void* src, int64_t lds_, const void* act, int64_t lda, int64_t width,
                      int64_t rows, int relu, int accumulate, void* dst, int64_t ldd, void* stream);

}  // namespace dynb

#endif

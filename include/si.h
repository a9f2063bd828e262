/*
 * si.h -- C ABI of the Streamlined-Inference hot path on MI355X (gfx950).
 *
 * Two operations of "Fast and Memory-Efficient Video Diffusion Using
 * Streamlined Inference" (arXiv 2411.01171):
 *
 *   - the Feature Slicer + Operator Grouping forward of one video-UNet
 *     transformer block (Sec. 4.1, Sec. 4.2.1, Eq. 1): the input feature is cut
 *     into windows along an axis the block's operators do not mix, every window
 *     runs through the whole operator group, and its result lands in place in
 *     a preallocated output, so that live intermediates are those of one slice;
 *   - Step Rehash's reuse-or-recompute test (Sec. 4.3, Appendix B): the
 *     similarity of a feature with its cached counterpart against a threshold,
 *     and the key-step search of Algorithm 1 over a similarity map.
 *
 * Conventions common to all entry points
 *   - Every pointer named *device* is GPU memory owned by the caller; the
 *     library never allocates or frees device memory.  Pointers named *host*
 *     are ordinary process memory.  Descriptor structs themselves live in host
 *     memory and are read before the call returns.
 *   - Work is enqueued on `stream` (a hipStream_t passed as void*; NULL = the
 *     default stream) and the call returns without waiting, unless stated.
 *   - Errors are returned as si_status; nothing aborts or throws.  All
 *     argument validation happens before the first GPU call, so every error
 *     other than SI_ERR_HIP can be provoked on a machine without a GPU.
 *   - Device base pointers must be 16-byte aligned.
 *   - State the library keeps: per device, up to two auxiliary streams
 *     (non-blocking, default priority) and three events, created the first
 *     time a forward call pipelines windows and kept until the process ends;
 *     calls that pipeline windows on the same device share them, so forward
 *     calls on one device must not overlap in time from several host threads.
 *     A small host table remembers which workspaces hold re-laid-out weights
 *     (SI_FWD_WEIGHTS_PACKED).  Nothing else outlives a call.
 */
#ifndef SI_H_
#define SI_H_

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef enum {
  SI_OK = 0,
  SI_ERR_NULL = 1,      /* a required pointer is NULL */
  SI_ERR_SHAPE = 2,     /* inconsistent or unsupported sizes */
  SI_ERR_DTYPE = 3,     /* unknown or mismatching element types */
  SI_ERR_SLICE = 4,     /* slice axis illegal for the block kind, or slice_len < 1 */
  SI_ERR_ALIGN = 5,     /* a device pointer is not 16-byte aligned */
  SI_ERR_WORKSPACE = 6, /* workspace / scratch too small */
  SI_ERR_ARG = 7,       /* other invalid argument (aliasing, NaN threshold, ...) */
  SI_ERR_HIP = 8        /* a HIP runtime call or kernel launch failed */
} si_status;

typedef enum { SI_F32 = 0, SI_BF16 = 1 } si_dtype;

/* Temporal blocks attend over the F frames of one spatial position; spatial
 * blocks attend over the H*W positions of one frame and cross-attend to the
 * context tokens; a temporal block follows every spatial one (Sec. 3). */
typedef enum { SI_BLOCK_TEMPORAL = 0, SI_BLOCK_SPATIAL = 1 } si_block_kind;

/* Slice axis (Sec. 4.1).  SI_AXIS_F: windows of frames, legal for spatial
 * blocks only (the spatial-layer slicer; both batch entries of a frame index
 * travel together).  SI_AXIS_HW: windows of flattened positions p = h*W + w,
 * legal for temporal blocks only (the temporal-layer slicer never cuts the
 * frame axis, because that would change the result). */
typedef enum { SI_AXIS_F = 2, SI_AXIS_HW = 3 } si_axis;

/* Contiguous 5-D feature [B, C, F, H, W] in device memory (W fastest). */
typedef struct {
  void* ptr;      /* device */
  int32_t dtype;  /* si_dtype */
  int64_t B, C, F, H, W;
} si_tensor5;

/* Contiguous context tokens [B, M, Cc] in device memory; spatial blocks only.
 * The same context row block serves every frame of batch entry b. */
typedef struct {
  const void* ptr; /* device */
  int32_t dtype;   /* si_dtype, must equal the feature's */
  int64_t B, M, Cc;
} si_context;

/* Parameters of one block.  All pointers are device memory in the feature's
 * element type, read-only.  Matrices are row-major [in, out]; D = heads *
 * dim_head is the inner width.  A NULL bias means zero; a NULL norm gain means
 * one and a NULL norm shift means zero.
 *
 *   GroupNorm(gn_groups, gn_eps; gn_g, gn_b [C]) per (batch, frame, group)
 *   h  = tokens w_in [C,D] + b_in [D]
 *   h += Attn(LN(h; ln1_g, ln1_b) (+ frame embedding if add_sin_pe)) wo [D,D] + bo [D]
 *        with q,k,v = a wq, a wk, a wv ([D,D] each, no bias), scale 1/sqrt(dim_head)
 *   spatial only:
 *   h += Attn(q = LN(h; ln2_g, ln2_b) wq2 [D,D]; k,v = ctx wk2, ctx wv2 [Cc,D]) wo2 [D,D] + bo2 [D]
 *   u  = LN(h; ln3_g, ln3_b) w1 [D,8D] + b1 [8D];  h += (u[:4D] * gelu_erf(u[4D:])) w2 [4D,D] + b2 [D]
 *   out = x + h w_out [D,C] + b_out [C]
 *
 * The frame embedding is the sinusoidal table PE[f,2i] = sin(f/10000^(2i/D)),
 * PE[f,2i+1] = cos(f/10000^(2i/D)), f = 0..F-1, and applies to temporal
 * blocks only. */
typedef struct {
  int32_t kind; /* si_block_kind */
  int32_t heads, dim_head, gn_groups;
  float gn_eps, ln_eps;
  int32_t add_sin_pe;
  const void *gn_g, *gn_b, *w_in, *b_in;
  const void *ln1_g, *ln1_b, *wq, *wk, *wv, *wo, *bo;
  const void *ln2_g, *ln2_b, *wq2, *wk2, *wv2, *wo2, *bo2; /* spatial only, else ignored */
  const void *ln3_g, *ln3_b, *w1, *b1, *w2, *b2;
  const void *w_out, *b_out;
} si_block_weights;

/* Bytes of device workspace si_block_forward needs for these arguments: the
 * intermediates of the slices in flight (Sec. 4.2.1: one sliced sub-feature at
 * a time; Sec. 4.2.2: up to si_windows_in_flight of them when slices are many
 * and small) plus slice-independent items (GroupNorm statistics, the
 * re-laid-out weights, the context keys/values).  An fp32 temporal block that
 * runs as one kernel over all windows re-lays out nothing and is counted with
 * one window's intermediates.  `ctx` may be NULL for temporal blocks.  Returns 0 if the arguments are invalid (the same checks
 * as si_block_forward, pointers excepted).  Host-only; touches no GPU. */
size_t si_workspace_bytes(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                          int32_t axis, int64_t slice_len);

/* Of si_workspace_bytes, the part that holds activation-derived data (slice
 * intermediates, GroupNorm statistics, context keys/values); the remainder is
 * re-laid-out weights.  Same arguments, same validity rule. */
size_t si_live_activation_bytes(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                                int32_t axis, int64_t slice_len);

/* Windows that si_block_forward keeps in flight for these arguments (Sec. 4.2.2:
 * pipelining across slices): 1, or 2 / 3 when the slices are many and small,
 * each on a stream of its own (the caller's plus library-owned ones, forked
 * after the once-per-call work and joined before the call's work on `stream`
 * ends) and with window intermediates of its own.  0 if the arguments are
 * invalid.  Host-only. */
int32_t si_windows_in_flight(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                             int32_t axis, int64_t slice_len);

/* Sliced block forward (Sec. 4.1, 4.2.1, Eq. 1).
 *
 *   x, out     [B,C,F,H,W], same shape and dtype; `out` must not overlap `x`
 *              (x is re-read for the residual).  Every element of out is written.
 *   w          block parameters (see si_block_weights); ctx: context or NULL.
 *   axis       si_axis; slice_len >= 1 in units of that axis.  Window i covers
 *              [i*slice_len, min((i+1)*slice_len, extent)); the last may be
 *              ragged.  slice_len >= extent runs the block unsliced.
 *   workspace  device memory of at least si_workspace_bytes(...) bytes, 256-byte
 *              aligned; contents on entry are ignored and on exit unspecified.
 *
 * GroupNorm statistics are taken per (batch, frame, group) over the whole
 * H*W extent before the first slice; they are the only quantity that crosses
 * position windows.  Supported: C and D multiples of 8, dim_head a multiple
 * of 8 and <= 128, C divisible by gn_groups, H*W*F*B*C < 2^40.
 * Returns SI_ERR_* on invalid arguments (nothing enqueued) or SI_ERR_HIP. */
si_status si_block_forward(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                           si_tensor5* out, int32_t axis, int64_t slice_len,
                           void* workspace, size_t workspace_bytes, void* stream);

/* si_block_forward with options.  flags:
 *   SI_FWD_WEIGHTS_PACKED  the caller vouches that `workspace` was last used by a forward call
 *                          (any entry point) with the SAME weight values, tensor shapes, context
 *                          shape, axis and slice_len, and has not been written since: the
 *                          re-laid-out weights and the frame table it still holds are used as
 *                          they are and the re-layout pass is skipped (weights are constant
 *                          across diffusion steps).  Everything activation-derived (statistics,
 *                          context keys / values) is recomputed.  What the host can see of a
 *                          broken promise is refused with SI_ERR_ARG before anything is
 *                          enqueued: a workspace pointer that no re-laying-out call of this
 *                          process used last with the same shapes, slicing, device and
 *                          parameter pointers.  Changed values behind the same pointers, or a
 *                          workspace written in between, give wrong results, not an error.
 * Unknown flag bits -> SI_ERR_ARG.  flags == 0 is si_block_forward. */
#define SI_FWD_WEIGHTS_PACKED 1u
si_status si_block_forward_ex(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                              si_tensor5* out, int32_t axis, int64_t slice_len, void* workspace,
                              size_t workspace_bytes, uint32_t flags, void* stream);

/* Scratch bytes si_rehash_check needs for n elements (partial sums). */
size_t si_rehash_scratch_bytes(int64_t n);

/* Step Rehash similarity test (Sec. 4.3.1, Appendix B: "S_ij >= gamma").
 *
 * Computes cos = <a,b> / (|a||b|) over the n elements of feat_t and feat_prev
 * (device, dtype `dtype`, any shape flattened) with float64 accumulation in a
 * fixed order, and decision = 1 (reuse the cached feature) if cos >= thresh,
 * else 0 (recompute).  The decision is taken as dot >= thresh*sqrt(na*nb) in
 * float64.  Both inputs all-zero: cos = 1; exactly one all-zero: cos = 0; a
 * non-finite sum: cos = NaN, decision 0.
 *
 *   cos_dev       device double*, may be NULL
 *   decision_dev  device int32_t*, required
 *   scratch       device, >= si_rehash_scratch_bytes(n), 16-byte aligned
 * n == 0 is legal (both all-zero).  thresh NaN -> SI_ERR_ARG. */
si_status si_rehash_check(const void* feat_t, const void* feat_prev, int64_t n, int32_t dtype,
                          float thresh, double* cos_dev, int32_t* decision_dev,
                          void* scratch, void* stream);

/* As si_rehash_check, then waits for `stream` and returns the results in host
 * memory.  result_dev: device memory of at least 16 bytes (holds cos, decision). */
si_status si_rehash_check_sync(const void* feat_t, const void* feat_prev, int64_t n, int32_t dtype,
                               float thresh, void* scratch, void* result_dev, void* stream,
                               double* cos_host, int32_t* decision_host);

/* si_rehash_check for callers that cannot allocate device memory: code under
 * HIP graph capture, tight serving loops, harnesses that forbid hipMalloc.  The
 * partial sums live in a device array inside the library
 * (SI_REHASH_STATIC_SCRATCH_BYTES per GPU, held until the process ends) instead
 * of a caller-provided scratch buffer; the call allocates nothing.  Same
 * arguments, results and error codes as si_rehash_check otherwise; n larger than
 * SI_REHASH_STATIC_MAX_N -> SI_ERR_SHAPE (nothing enqueued).  All calls on one
 * GPU share the array: calls that overlap in time on one GPU (two streams, two
 * threads) race and give wrong results; calls on one stream, or otherwise
 * ordered, are safe, and nothing has to be cleared between them.
 * si_init_device resolves the array's address on the current device ahead of
 * time (optional; otherwise the first call on a device does it), e.g. before a
 * graph capture begins.  Returns SI_OK or SI_ERR_HIP. */
#define SI_REHASH_STATIC_SCRATCH_BYTES 49152
#define SI_REHASH_STATIC_MAX_N (1LL << 33)
si_status si_init_device(void);
si_status si_rehash_check_static(const void* feat_t, const void* feat_prev, int64_t n, int32_t dtype,
                                 float thresh, double* cos_dev, int32_t* decision_dev, void* stream);

/* Anchor of the one-pass Step Rehash walk around one block: input and output
 * of the last step at which the block was computed.  x_key and y_key are
 * caller-owned device buffers of the feature's size and dtype, 16-byte
 * aligned, disjoint from each other, from x, out and the workspace; the
 * library writes them.  `valid` is host state: set it to 0 before the first
 * step (nothing cached yet); the library sets it to 1. */
typedef struct {
  void* x_key;
  void* y_key;
  int32_t valid;
} si_rehash_cache;

/* Sliced block forward under Step Rehash, decided causally (Sec. 4.3: skip a
 * block whose feature barely moved; Algorithm 1's anchoring: always compare
 * with the last computed step, never just the previous one).  The test of
 * si_rehash_check is applied to the block's INPUT: cos(x, cache->x_key) >=
 * gamma -> out := cache->y_key (the cached output is handed back; over as many
 * consecutive steps as the test keeps passing) and nothing else runs;
 * otherwise out := si_block_forward(x) bit for bit, and x, out become the new
 * anchor (two device-to-device copies).  With cache->valid == 0 the block is
 * computed unconditionally.  out->ptr may equal cache->y_key (the one overlap
 * that is allowed): the result then lives in the anchor's output buffer, a
 * reused step copies nothing and a computed step copies only x; the caller
 * must be done with it before the next call on this cache.
 *
 * The similarity sums ride on the GroupNorm statistics pass (x is read once
 * for both; the anchor input is the only extra read), then the call WAITS for
 * `stream` to learn the decision -- it is not asynchronous when
 * cache->valid != 0.  Arguments as si_block_forward (same workspace size);
 * gamma NaN -> SI_ERR_ARG.
 *   cos_host     host, may be NULL: the cosine, NaN when no test was taken
 *   reused_host  host, required: 1 = cached output handed back, 0 = computed */
si_status si_block_forward_rehash(const si_tensor5* x, const si_block_weights* w, const si_context* ctx,
                                  si_tensor5* out, int32_t axis, int64_t slice_len, void* workspace,
                                  size_t workspace_bytes, si_rehash_cache* cache, float gamma, void* stream,
                                  double* cos_host, int32_t* reused_host);

/* Parameters of one Spatial ResBlock operator group (Sec. 4.2.1: the
 * consecutive GroupNorm, Conv2D and SiLU operators of the Spatial ResBlock
 * form one spatial group).  Device pointers, dtype of the feature, 16-byte
 * aligned.  Convolution kernels in (output channel, input channel, row,
 * column) order -- w_conv1 [c_out, C, 3, 3], w_conv2 [c_out, c_out, 3, 3] --
 * applied as a cross-correlation with zero padding 1 and stride 1; w_temb
 * row-major [temb_dim, c_out]; gn2 and the biases have c_out entries.  NULL biases mean
 * zero, NULL gains / shifts mean one / zero.  w_temb is required iff
 * temb_dim > 0. */
typedef struct {
  int32_t gn_groups;
  float gn_eps;
  int32_t temb_dim; /* width of the timestep embedding, 0 = none */
  const void *gn1_g, *gn1_b, *w_conv1, *b_conv1;
  const void *w_temb, *b_temb;
  const void *gn2_g, *gn2_b, *w_conv2, *b_conv2;
  int32_t c_out;                 /* output channels; 0 or x->C: no channel change, identity skip */
  const void *w_skip, *b_skip;   /* 1x1 skip convolution [c_out, C], required iff c_out != C */
} si_resblock_weights;

/* Workspace bytes of si_resblock_forward, and the activation-derived part of
 * it (one slice's intermediates plus statistics; the rest is re-laid-out
 * kernels).  0 if the arguments are invalid.  Host-only. */
size_t si_resblock_workspace_bytes(const si_tensor5* x, const si_resblock_weights* w, int64_t slice_len);
size_t si_resblock_live_activation_bytes(const si_tensor5* x, const si_resblock_weights* w, int64_t slice_len);

/* Sliced Spatial ResBlock forward (Sec. 4.1 spatial layers slicer, Sec. 4.2.1, Eq. 1):
 *   out = skip(x) + Conv3x3(SiLU(GN2( Conv3x3(SiLU(GN1(x))) + b1 + e ))) + b2,
 *   e[b, :] = SiLU(temb[b, :]) w_temb + b_temb  broadcast over frames and positions,
 *   skip(x) = x, or w_skip x + b_skip per pixel when the block changes the channel count,
 * with GroupNorm statistics per (batch, frame, group).  The merged batch x
 * frame axis is sliced: window i covers frames [i*slice_len, min((i+1)*
 * slice_len, F)) of every batch entry, goes through the whole group on its
 * own and is written to its window of `out` (every element of out is
 * written; out must not overlap x).
 *   x          [B,C,F,H,W] bf16 (SI_ERR_DTYPE otherwise); out [B,c_out,F,H,W]; C and c_out multiples
 *              of 32 and of gn_groups, at most 64 channels per group
 *   temb       device [B, temb_dim] or NULL when temb_dim == 0
 *   workspace  device, >= si_resblock_workspace_bytes(...), 256-byte aligned
 * Returns SI_ERR_* on invalid arguments (nothing enqueued) or SI_ERR_HIP. */
si_status si_resblock_forward(const si_tensor5* x, const si_resblock_weights* w, const void* temb, si_tensor5* out,
                              int64_t slice_len, void* workspace, size_t workspace_bytes, void* stream);

/* Spatial Up/DownSample of the ResBlock group (Sec. 4.2.1 names the operators;
 * the definitions taken are those of the latent-diffusion U-Nets), sliced along
 * frames like si_resblock_forward:
 *   SI_RESAMPLE_DOWN  out = Conv3x3(x), zero padding 1, stride 2:
 *                     out[.., y, x] = b + sum w[o,c,i,j] * x[.., 2y+i-1, 2x+j-1];
 *                     out is [B,C,F,ceil(H/2),ceil(W/2)]
 *   SI_RESAMPLE_UP    out = Conv3x3(u) + b, zero padding 1, u[.., Y, X] = x[.., Y/2, X/2]
 *                     (nearest-neighbour doubling); out is [B,C,F,2H,2W]
 * x, out bf16, C a multiple of 32; w_conv [C, C, 3, 3] and b_conv (may be NULL)
 * device bf16.  Operands stay bf16 (exact), accumulation is fp32, one rounding
 * of the result.  Workspace and error behaviour as si_resblock_forward. */
typedef enum { SI_RESAMPLE_DOWN = 0, SI_RESAMPLE_UP = 1 } si_resample_kind;
size_t si_resample_workspace_bytes(const si_tensor5* x, int32_t kind, int64_t slice_len);
si_status si_resample_forward(const si_tensor5* x, int32_t kind, const void* w_conv, const void* b_conv, si_tensor5* out,
                              int64_t slice_len, void* workspace, size_t workspace_bytes, void* stream);

/* Key-step search, Algorithm 1 (Appendix B).  Host only.
 *   S      host, row-major K x K similarity map; only S[i][anchor] entries are read
 *   gamma  threshold, must satisfy gamma <= 1 and gamma <= S[i][i] where visited
 *   G_out  host, capacity K; receives the key steps in ascending order, no duplicates
 * Returns |G| (>= 1), or -1 on invalid arguments (K < 1, NULL, gamma NaN or > 1,
 * a visited diagonal entry below gamma). */
int32_t si_key_step_search(const float* S, int32_t K, float gamma, int32_t* G_out);

/* Measurement aid, not part of the product path: process-wide state, off by
 * default, not thread-safe, and never to be enabled while other threads call
 * the library.  Optional per-stage timing.  When enabled, the forward entry
 * points and si_rehash_check record a HIP event pair around every kernel
 * launch, and windows that would otherwise run two at a time on two streams
 * run one after the other on the caller's stream, so that each pair brackets
 * one kernel alone on the GPU (event overhead is added; results are the same).
 * si_stage_timing_read waits for the recorded events, adds each pair's
 * duration to its stage, writes up to `cap` entries (stage name, total
 * milliseconds, launches) and clears the record.  Returns the number of stages,
 * or -1 on a HIP error.  Not thread-safe; host pointers. */
void si_stage_timing_enable(int32_t on);
int32_t si_stage_timing_read(const char** names, double* total_ms, int64_t* launches, int32_t cap);

const char* si_status_str(int32_t status);
int32_t si_abi_version(void);

#ifdef __cplusplus
}
#endif
#endif /* SI_H_ */

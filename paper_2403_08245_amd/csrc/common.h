// Shared declarations of the libsmoe kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "smoe.h"

typedef __bf16 bf16_t;

struct smoe_ctx {
  int device;
  int num_cu;
  int stream_grid;  // blocks of the persistent kernels: one per compute unit, a multiple of 8 (one share per XCD), at most 256
  unsigned long long *clock_probe;  // device array the persistent s2s kernels report their clocks to, or NULL (smoe_set_clock_probe)
  int group_m;      // M-tiles per group of the persistent scatter2scatter kernels' tile order (4; smoe_set_tile_group)
  int tile_shape;   // persistent scatter2scatter tiles (see S2SArgs::tile_shape, smoe_set_kernel_mode)
  int kernel_mode;  // 0 auto, 1 plain tiled kernels only, 2 one block per tile (testing aid, see smoe_set_kernel_mode)
  int32_t *route_scratch;  // this device's copy of the routing kernels' static scratch array (smoe_route_noalloc)
};

#define SMOE_LAUNCH_CHECK()                                   \
  do {                                                        \
    if (hipGetLastError() != hipSuccess) return SMOE_ERR_HIP; \
  } while (0)

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
static inline size_t dtype_size(smoe_dtype d) { return d == SMOE_BF16 ? 2 : 4; }
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16_t>(bf16_t v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16_t from_f32<bf16_t>(float v) { return (bf16_t)v; }  // RNE

// point-wise non-linearities of Alg. 3 (GELU is the exact erf form)
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
  float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752440f));
  float pdf = expf(-0.5f * x * x) * 0.39894228040143267794f;
  return cdf + x * pdf;
}
__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + expf(-x)); }

// How a GEMM operand's rows are addressed through the routing arrays.
//   sorted position i -> row i (grouped) or o[i] / fan (scattered source with fan-out)
//   or o[i] (scattered destination).
struct RowMap {
  const int32_t *o;  // sorted_scattered_idxs, or nullptr when rows are already grouped
  int fan;           // divisor applied to o[i]; 1 for slot-indexed tensors
};
__device__ __forceinline__ int map_row(const RowMap &m, int i) {
  return m.o ? (m.fan > 1 ? m.o[i] / m.fan : m.o[i]) : i;
}

// ---- routing.hip
int launch_topk_gate(hipStream_t s, const float *logits, int T, int E, int k, int32_t *idx, float *gates);
int launch_attn_fwd(hipStream_t s, const void *Q, const void *K, const void *V, void *O, float *LSE, int B, int T, int G,
                    int h);
size_t attn_bwd_workspace_bytes(int B, int T, int G, int h);
// dq_apart: no part of dQ lies over O (a launch less).  dq_rows: row of dQ that each query row's gradient goes to (NULL: its own).
int launch_attn_bwd(hipStream_t s, const void *Q, const void *K, const void *V, const void *O, const void *dO,
                    const float *LSE, void *ws, void *dQ, void *dK, void *dV, int B, int T, int G, int h, bool dq_apart = false,
                    const int32_t *dq_rows = nullptr);
int launch_dense_offsets(hipStream_t s, int32_t *off, int n);
int launch_add3(hipStream_t s, const void *a, const void *b, const void *c, void *out, size_t n);
int launch_topk_gate_bwd(hipStream_t s, const int32_t *idx, const float *gates, const float *dgates, int T, int E, int k,
                         float *dlogits);
constexpr int ROUTE_MAX_E = 16384;   // the routing kernels keep one or two 4-byte counters per expert in LDS (up to 128 KB of 160)
size_t route_workspace_bytes(int Tk, int E);
// Static device scratch of smoe_route_noalloc: its size, and the address of the current device's copy.
constexpr size_t ROUTE_SCRATCH_BYTES = (size_t)1 << 20;
int route_scratch_address(int32_t **ptr);
int init_route_kernels();            // with the context's device current
int launch_route(hipStream_t s, const int32_t *expert_idxs, int Tk, int E, int32_t *sorted_e,
                 int32_t *sorted_s, int32_t *offsets, void *ws);

// ---- elementwise.hip
int launch_act_fwd(hipStream_t s, smoe_act act, const void *Hpre, void *H, int rows, int d_expert);
int launch_act_bwd(hipStream_t s, smoe_act act, const void *Hpre, const void *dH, void *dHpre, int rows, int d_expert);
// Y[t] = sum_j g[t*k+j] * Yhat[t*k+j] (+ more0[t] + more1[t], both or neither); g == nullptr means all ones.
int launch_combine(hipStream_t s, smoe_dtype dt, const void *Yhat, const float *g, void *Y, int T, int k, int d, const void *more0 = nullptr,
                   const void *more1 = nullptr);
// out[i] = g[o[i]] * in[o[i] / fan]; g == nullptr means all ones
int launch_group(hipStream_t s, smoe_dtype dt, const void *in, const int32_t *o, int fan, const float *g,
                 void *out, int Tk, int d);
// inv[o[i]] = i
int launch_invert(hipStream_t s, const int32_t *o, int32_t *inv, int Tk);
// dg[o[i]] = sum_c part[i, c] (a fixed order; ld is even), and inv[o[i]] = i unless inv is NULL: finishes the routing-weight gradient left in slabs by the fused
// backward epilogues.
int launch_dp_reduce(hipStream_t s, const float *part, int ld, const int32_t *o, float *dg, int32_t *inv, int Tk);
// dg[s] = <dY[s / kp], Yhat[s]>
int launch_rowdot(hipStream_t s, smoe_dtype dt, const void *dY, const void *Yhat, float *dg, int Tk, int kp, int d);

struct RowDots {      // dg[s] = <dY[s / kp], Yhat[s]> for s < Tk, rows of d elements (16-byte multiples)
  const void *dY = nullptr, *Yhat = nullptr;
  float *dg = nullptr;    // NULL: none
  int Tk = 0, kp = 1, d = 0;
};
// one of them, by one wavefront
template <typename T> __device__ __forceinline__ void row_dot(const RowDots &r, int s, int lane) {
  constexpr int V = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(V)));
  const T *a = (const T *)r.dY + (size_t)(s / r.kp) * r.d, *b = (const T *)r.Yhat + (size_t)s * r.d;
  float acc = 0.f;
  for (int c = lane * V; c < r.d; c += 64 * V) {
    const vec x = *reinterpret_cast<const vec *>(a + c), y = *reinterpret_cast<const vec *>(b + c);
#pragma unroll
    for (int i = 0; i < V; ++i) acc = fmaf(to_f32<T>(x[i]), to_f32<T>(y[i]), acc);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) r.dg[s] = acc;
}

// The copy launch_group makes of bf16 rows, by the inverse of the order indices: Tk / fan source rows, each read once.  In the same launch,
// where given: the row dots of dp, and a second, unweighted copy of rows of d2 elements with the same fan.
int launch_spread(hipStream_t s, const void *in, const int32_t *inv, int fan, const float *g, void *out, int Tk, int d, const RowDots &dots = RowDots{},
                  const void *in2 = nullptr, void *out2 = nullptr, int d2 = 0);

// ---- GEMM launchers (gemm_plain.hip, gemm_mfma.hip)
struct S2SArgs {      // C[out(i), :] = A[in(i), :] * op(W[e(i)])   for sorted rows i
  const void *A;      // [*, K] rows addressed through a_map
  const void *W;      // [E, d_in, d_out]
  void *C;            // [*, N] rows addressed through c_map
  RowMap a_map, c_map;
  const int32_t *offsets;  // [E+1]; persistent kernels: NULL stands for E segments of Tk / E rows each
  int E, Tk;
  int K, N;           // contraction length and output width
  int ldw;            // row stride of W[e] (= d_out)
  size_t w_stride;    // elements between experts (= d_in * d_out)
  int trans_w;        // 0: op(W) = W (K = d_in, N = d_out); 1: op(W) = W^T (K = d_out, N = d_in)
  // Optional scratch for splitting the contraction of the last, partly filled round of tiles over the
  // compute units that would otherwise idle (S2S_TAIL_WS_BYTES of device memory, or NULL: no split).
  float *tail_ws;
  int grid = 256;     // blocks of the persistent kernel (smoe_ctx::stream_grid)
  int tile_shape = 0; // persistent scatter2scatter tiles: 0 chosen by size, 1 128 x 256 only, 2 256 x 256 only (smoe_ctx::tile_shape)
  int group_m = 4;    // tiles are numbered in groups of this many M-tiles x all N-tiles (smoe_ctx::group_m)
  // Bytes of all the weights that the call may read, of all its experts and of its other product too (0: only this product's).
  // More than the last-level cache holds will not be there at the next call, and launches that read each weight about once then
  // read them past the caches.  All experts count, also where a few tokens use a part of them: the next tokens use others (4 tokens
  // on 64 experts, 157 of 402 MB read, the forward pass past the caches / through them: other tokens at every call 42.4 / 42.1 us,
  // another layer of the same size at every call 43.1 / 48.7; only the very same tokens again are dearer, 42.9 / 37.8).
  size_t call_weights = 0;
  // Optional second dense product of the same sizes in the same launch (persistent kernels, no order indices, no fused
  // activation; E = 2, both segments Tk / 2 rows): segment 1 reads A2 and W2 and writes C2, which point to where segment
  // 0's numbering would have them (run_s2s_pair in api.hip sets them).
  const void *A2 = nullptr, *W2 = nullptr;
  void *C2 = nullptr;
  // Optional fused SwiGLU of Alg. 3 (forward, expert-sorted output only): W's columns are
  // [gate | up] halves of width N / 2 and H [*, N / 2] receives silu(gate) * up; C may then be
  // NULL when the pre-activation is not kept.
  void *H;
  // Optional fused SwiGLU backward of Alg. 3 (input-gradient product of the second ParallelLinear, expert-sorted
  // out, op(W) = W^T, N = d_expert): A holds the UNWEIGHTED upstream rows, gathered through a_map, so the fp32 accumulators are
  // dH / p.  With Hpre_in [Tk, 2N] (the saved pre-activation), row_scale [Tk] (the routing weights in slot order, read through
  // the same order indices) and dp_part [Tk, 2 * ceil(N / 256)] fp32 set, the epilogue writes
  // C = dHpre [Tk, 2N] = sigma'(Hpre) * weight * acc instead of dH, and per row and 128-column slab the
  // partial dot <acc, silu(gate) * up> whose sum over the slabs is Alg. 2's dp for that row; with Hw_out and H_in
  // [Tk, N] (the saved hidden activations) also Hw = weight * H.
  // Optional [2 * grid] device array: block b leaves the shader-clock cycles and the 100 MHz real-time ticks between its
  // first and last instruction in entries 2b and 2b+1 (measurement aid: the ratio is the clock the block ran at).
  unsigned long long *clock_probe = nullptr;
  const void *Hpre_in = nullptr;
  const float *row_scale = nullptr;
  float *dp_part = nullptr;
  // The same idea for any activation (still the W2^T product on unweighted rows): with H_in [Tk, N] (the saved
  // hidden activations), row_scale and dp_part set and Hpre_in NULL, the epilogue writes C = dH = weight * acc, the
  // slabs of dp = <acc, H>, and, when Hw_out [Tk, N] is given, Hw = weight * H (the routing-weighted hidden rows
  // that let groupXTY take the unweighted sorted dY for dW2 as well).  The activation's derivative stays a row kernel.
  // With a scattered output (c_map set, Hw_out given) H and dH lie in slot order, the slabs and Hw in expert-sorted order.
  const void *H_in = nullptr;
  void *Hw_out = nullptr;
  // fp32 kernels (gemm_plain.hip): with H set the activation `act` is applied in the epilogue (C may be NULL), with Hpre_in
  // set C receives act'(Hpre) times the product; gates (fp32, slot order, through the order indices `slots`) scales its rows.
  int act = SMOE_ACT_NONE;
  const float *gates = nullptr;
  const int32_t *slots = nullptr;
};
struct DWArgs {       // dW[e] = sum_{i in segment e} A[i, :]^T B[i, :]   (rows expert-sorted, or read through the row maps)
  const void *A;      // [Tk, M]
  const void *B;      // [Tk, N]
  void *dW;           // [E, M, N]
  const int32_t *offsets;
  int E, Tk, M, N;
  // Optional scratch (S2S_TAIL_WS_BYTES of device memory, or NULL): when the output tiles of all experts fill
  // only a fraction of the chip (a dense projection run as one expert), each segment's rows are cut into chunks
  // that leave fp32 partial tiles here, added in chunk order by a second kernel.
  float *split_ws = nullptr;
  int grid = 256;     // blocks of the persistent kernel (smoe_ctx::stream_grid)
  // Optional second weight gradient of the same sizes in the same launch (persistent kernel; E = 2), as S2SArgs has it.
  const void *A2 = nullptr, *B2 = nullptr;
  void *dW2 = nullptr;
  // Optional further weight gradient over the same segments in the same launch (persistent kernel, no split): dW3 [E, M3, N3] from
  // A3 [Tk, M3] and B3 [Tk, N3].
  const void *A3 = nullptr, *B3 = nullptr;
  void *dW3 = nullptr;
  int M3 = 0, N3 = 0;
  // Persistent and fp32 kernels: rows of A, B and A3 read through the order indices (the same in all of them) instead of from
  // sorted copies.  Persistent kernel: not A beside dW3, nothing beside dW2.
  RowMap a_map{nullptr, 1}, b_map{nullptr, 1}, a3_map{nullptr, 1};
  // The order indices, needed with dW3: that launch fetches them whichever of its operands it reads through them, and also for none.
  const int32_t *order = nullptr;
  // fp32 kernels: B's rows scaled by the routing weights (fp32, slot order; needs b_map).
  const float *gates = nullptr;
};
constexpr size_t LAST_LEVEL_CACHE = (size_t)256 << 20;
static inline bool weights_pass_caches(const S2SArgs &a) {
  return (a.call_weights ? a.call_weights : (size_t)a.E * a.K * a.N * 2) > LAST_LEVEL_CACHE;
}
int launch_s2s_plain(hipStream_t s, smoe_dtype dt, const S2SArgs &a);
int launch_dw_plain(hipStream_t s, smoe_dtype dt, const DWArgs &a);
bool f32_backward_fits(const S2SArgs &x, const DWArgs &w, const RowDots &d);   // into one launch
int launch_f32_backward(hipStream_t s, const S2SArgs &x, const DWArgs &w, const RowDots &d);
bool s2s_mfma_supported(const S2SArgs &a);
bool dw_mfma_supported(const DWArgs &a);
int launch_s2s_mfma(hipStream_t s, const S2SArgs &a);
int launch_dw_mfma(hipStream_t s, const DWArgs &a);
// Per-device set-up of the kernels that need more dynamic LDS than the default limit (called by
// smoe_create with the context's device current).
int init_mfma_kernels();
int init_stream_kernels();
// persistent tile-stream kernels (gemm_stream.hip)
constexpr size_t S2S_TAIL_WS_BYTES = (size_t)256 * 256 * 256 * sizeof(float);   // 256 partial tiles of 256 x 256 fp32
bool s2s_stream_supported(const S2SArgs &a);
bool s2s_stream_swiglu_supported(const S2SArgs &a);
bool s2s_stream_swiglu_bwd_supported(const S2SArgs &a);
bool s2s_stream_dp_supported(const S2SArgs &a);
int launch_s2s_stream(hipStream_t s, const S2SArgs &a);
// Small-batch (decoding) forward products: 32-row tiles of four wavefronts, bound by the weight stream.
// Takes a.H like the persistent kernel (fused SwiGLU).
bool s2s_decode_supported(const S2SArgs &a);
int launch_s2s_decode(hipStream_t s, const S2SArgs &a);
bool dw_stream_supported(const DWArgs &a);
int launch_dw_stream(hipStream_t s, const DWArgs &a);
bool dw_stream_two_pay(const DWArgs &a);   // is a launch with dW3 shorter than one for each?
